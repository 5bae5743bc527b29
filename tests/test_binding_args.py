"""How the per-token calls marshal their arguments, without a GPU: the native module is bound to stand-ins for the
library's entry points that record what they are called with."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2603_08453_amd import binding as lc

VP, INT, SZ = ctypes.c_void_p, ctypes.c_int, ctypes.c_size_t
SIGNATURES = {
    "decode_step": (VP, VP, VP, VP, VP, INT, INT, VP, VP, VP, VP, INT, VP, SZ, VP),
    "decode_step_static": (VP, VP, VP, VP, VP, INT, INT, VP, VP, VP, VP, INT, VP),
    "retrieve": (VP, VP, INT, INT, VP, VP, VP, INT, VP, SZ, VP),
    "sparse_decode": (VP, VP, VP, VP, VP, VP, VP, INT, INT, VP, VP, VP, SZ, VP),
    "append": (VP, VP, VP, VP, VP, VP, VP, VP, SZ, VP),
}


class Stream:
    cuda_stream = 0


class FakeIndex:
    handle = None
    address = 0x1000


@pytest.fixture()
def calls():
    """name -> arguments of the last call that reached the (stand-in) library."""
    seen = {}
    keep = []
    for name, sig in SIGNATURES.items():
        def record(*a, name=name):
            seen[name] = a
            if name == "append":
                seen["flags"] = ctypes.string_at(a[6], 4) if a[6] else None
            return 0
        keep.append(ctypes.CFUNCTYPE(INT, *sig)(record))
    lc._fast().bind(*(ctypes.cast(f, VP).value for f in keep))
    yield seen
    lc._fast_mod = None                                      # (the next call binds the library again)
    lc._fast()


def tensors(B=1, H=2, G=2, T=8, cap=5):
    return dict(q=torch.zeros(B, H * G, 128, dtype=torch.bfloat16), K=torch.zeros(B, H, T, 128, dtype=torch.bfloat16),
                V=torch.zeros(B, H, T, 128, dtype=torch.bfloat16), out=torch.zeros(B, H * G, 128), ws=torch.zeros(256, dtype=torch.uint8),
                ids=torch.zeros(B, H, cap, dtype=torch.int32), counts=torch.zeros(B, H, dtype=torch.int32))


@pytest.mark.parametrize("budget,want", [(1024, 1024), (np.int64(7), 7), (True, 1), (torch.tensor(9), 9), (2 ** 40 + 3, 3),
                                         (2 ** 80 + 5, 5), (1024.9, None), ("1024", None), (None, None)])
def test_budget_of_a_retrieval_is_an_integer(calls, budget, want):
    t = tensors()
    args = (FakeIndex, t["q"], budget, t["ids"], t["counts"], t["ws"])
    if want is None:
        with pytest.raises(ctypes.ArgumentError):
            lc.lc_retrieve(*args, stream=Stream)
        assert "retrieve" not in calls
    else:
        lc.lc_retrieve(*args, stream=Stream)
        assert calls["retrieve"][2:4] == (4, want) and calls["retrieve"][7] == 5


@pytest.mark.parametrize("budget,want", [(1024, 1024), (np.int64(7), 7), (1024.9, 1024), ("1024", 1024), (2 ** 40 + 3, 3)])
def test_budget_of_a_step_is_what_int_gives(calls, budget, want):
    t = tensors()
    lc.lc_decode_step(FakeIndex, t["q"], t["K"], t["V"], budget, t["out"], t["ws"], stream=Stream)
    assert calls["decode_step"][5:7] == (4, want)
    lc.lc_decode_step_static(FakeIndex, t["q"], t["K"], t["V"], budget, t["out"], stream=Stream)
    assert calls["decode_step_static"][5:7] == (4, want)
    with pytest.raises(ValueError):
        lc.lc_decode_step(FakeIndex, t["q"], t["K"], t["V"], "many", t["out"], t["ws"], stream=Stream)


@pytest.mark.parametrize("call", ["retrieve", "decode_step", "decode_step_static", "sparse_decode", "append"])
def test_other_threads_run_while_the_library_works(call):
    """The library's entry points replaced by the C library's usleep, whose argument is the handle: 200 ms in which
    another thread has to get on."""
    import threading
    usleep = ctypes.cast(ctypes.CDLL(None).usleep, VP).value
    lc._fast().bind(*[usleep] * 5)
    try:
        class Sleep:
            handle = None
            address = 200_000
        t, ticks, done = tensors(), [0], threading.Event()
        row = torch.zeros(1, 2, 128, dtype=torch.bfloat16)

        def tick():
            while not done.wait(0.001):
                ticks[0] += 1
        thread = threading.Thread(target=tick)
        thread.start()
        before = ticks[0]
        if call == "retrieve":
            lc.lc_retrieve(Sleep, t["q"], 8, t["ids"], t["counts"], t["ws"], stream=Stream)
        elif call == "decode_step":
            lc.lc_decode_step(Sleep, t["q"], t["K"], t["V"], 8, t["out"], t["ws"], stream=Stream)
        elif call == "decode_step_static":
            lc.lc_decode_step_static(Sleep, t["q"], t["K"], t["V"], 8, t["out"], stream=Stream)
        elif call == "sparse_decode":
            lc.lc_sparse_decode(Sleep, t["q"], t["K"], t["V"], t["ids"], t["counts"], t["out"], t["ws"], stream=Stream)
        else:
            lc.lc_append(Sleep, t["K"], t["V"], row, row, [1], t["ws"], stream=Stream)
        got = ticks[0] - before
        done.set()
        thread.join()
        assert got >= 5
    finally:
        lc._fast_mod = None
        lc._fast()


def test_close_flags(calls):
    """Any sized iterable of truth values; one that an element's truth value shortens is read as it was."""
    t = tensors(B=4)
    row = torch.zeros(4, 2, 128, dtype=torch.bfloat16)

    def flags(close):
        calls.clear()
        lc.lc_append(FakeIndex, t["K"], t["V"], row, row, close, t["ws"], stream=Stream)
        return calls["flags"]

    assert flags(None) is None
    assert flags([0, 1, 0, 1]) == flags((False, True, None, "x")) == flags(np.array([0, 1, 0, 2])) == b"\0\1\0\1"
    assert flags([1]) == b"\1\0\0\0"
    with pytest.raises(TypeError):
        flags(x for x in (1, 0, 1, 0))
    with pytest.raises(TypeError):
        flags(3)

    class Shortens:
        def __bool__(self):
            del changing[1:]
            return True

    changing = [Shortens(), 0, [1], [1]]
    assert flags(changing) == b"\1\0\1\1"


def test_calls_without_the_native_module(monkeypatch):
    """ctypes marshals the per-token calls then, and says so once; here they reach the library, which refuses the
    null handle before any GPU work."""
    import sys
    import warnings
    monkeypatch.setattr(lc, "_fast_mod", None)
    monkeypatch.delattr(sys.modules[lc.__package__], "_lychee_torch", raising=False)
    monkeypatch.setitem(sys.modules, lc.__package__ + "._lychee_torch", None)

    class Closed:
        handle = None
        address = 0

    t = tensors()
    row = torch.zeros(1, 2, 128, dtype=torch.bfloat16)
    with pytest.warns(RuntimeWarning, match="ctypes marshals"):
        with pytest.raises(lc.LycheeError) as e:
            lc.lc_retrieve(Closed, t["q"], 8, t["ids"], t["counts"], t["ws"], stream=Stream)
        assert e.value.code == lc.LC_ERR_INVALID_ARG
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        for call in (lambda: lc.lc_decode_step(Closed, t["q"], t["K"], t["V"], 8, t["out"], t["ws"], stream=Stream),
                     lambda: lc.lc_decode_step_static(Closed, t["q"], t["K"], t["V"], 8, t["out"], stream=Stream),
                     lambda: lc.lc_sparse_decode(Closed, t["q"], t["K"], t["V"], t["ids"], t["counts"], t["out"], t["ws"],
                                                 stream=Stream),
                     lambda: lc.lc_append(Closed, t["K"], t["V"], row, row, [1], t["ws"], stream=Stream)):
            with pytest.raises(lc.LycheeError) as e:
                call()
            assert e.value.code == lc.LC_ERR_INVALID_ARG
