"""The decode step whose workgroups share the scoring, against the two separate calls: shares around the numbers of chunks that a pass
takes, chunk counts around the kernel's instances and its largest, several steps in a row, the caller's own number of splits, a buffer that held another
index, chunks that no workgroup's share holds, and other streams' kernels beside it.  That the scoring is shared is asserted, as the
two-kernel form gives the same."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


class _Index:
    def __init__(self, chunks, H, G, centers, budget, sink=0, seed=0, spare=0, splits=0, longest=5):
        import torch
        from paper_2603_08453_amd import binding as lc
        self.lc, self.torch, self.budget, self.H, self.G, self.B = lc, torch, budget, H, G, len(chunks)
        r = np.random.default_rng(seed + sum(chunks))
        self.bounds = [np.concatenate([[0], np.cumsum(r.integers(1, longest + 1, size=m))]).astype(np.int32) for m in chunks]
        self.lens = [int(b[-1]) for b in self.bounds]
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)
        rows, self.cap = max(self.lens) + spare, max(chunks) + spare
        self.K, self.V = self.draw(self.B, H, rows, 128), self.draw(self.B, H, rows, 128)
        self.cfg = lc.lc_config_default(levels=2, fanout=16, kmeans_iters=1, max_chunks=self.cap, max_tokens=rows, center_dtype=centers,
                                        sink_tokens=sink, decode_splits=splits)
        self.ib = torch.full((lc.lc_index_bytes(self.cfg, self.B, H),), 0xA5, dtype=torch.uint8, device="cuda")
        self.ws = torch.full((lc.lc_workspace_bytes(self.cfg, self.B, H * G, H),), 0xA5, dtype=torch.uint8, device="cuda")
        self.build()

    def draw(self, *shape):
        return self.torch.randn(shape, generator=self.gen, device="cuda").to(self.torch.bfloat16)

    def build(self):
        self.idx = self.lc.lc_build_index(self.cfg, self.K, self.lens, self.bounds, self.ib, self.ws)

    def query(self):
        return self.draw(self.B, self.H * self.G, 128)

    def shares(self):
        """Whether the step is one kernel (beyond 128 chunks: one whose workgroups share the scoring)."""
        return self.lc.lc_bench_step_is_one_kernel(self.idx, self.H * self.G, self.budget)

    def posted(self):
        """The keys that the steps have posted, with the step's number above them: the last part of the index buffer."""
        words = self.B * self.H * min(self.cap, 2560)
        assert words * 8 % 256 == 0
        return self.ib[-words * 8:].view(self.torch.int64)

    def step(self, q, out=None, lse=None):
        out = self.torch.full((self.B, self.H * self.G, 128), float("nan"), device="cuda") if out is None else out
        lse = self.torch.full((self.B, self.H * self.G), float("nan"), device="cuda") if lse is None else lse
        ids = self.torch.full((self.B, self.H, self.cap), -7, dtype=self.torch.int32, device="cuda")
        n = self.torch.full((self.B, self.H), -1, dtype=self.torch.int32, device="cuda")
        self.lc.lc_decode_step(self.idx, q, self.K, self.V, self.budget, out, self.ws, lse=lse, chunk_ids=ids, counts=n)
        return ids, n, out, lse

    def check(self, q):
        torch, lc = self.torch, self.lc
        ids, n, out, lse = self.step(q)
        want, m = torch.full_like(ids, -7), torch.full_like(n, -1)
        ref, ref_lse = torch.full_like(out, float("nan")), torch.full_like(lse, float("nan"))
        lc.lc_retrieve(self.idx, q, self.budget, want, m, self.ws)
        lc.lc_sparse_decode(self.idx, q, self.K, self.V, want, m, ref, self.ws, lse=ref_lse)
        assert torch.equal(n, m)
        for b in range(self.B):
            for h in range(self.H):
                assert torch.equal(ids[b, h, : n[b, h]], want[b, h, : m[b, h]])
        # (the same chunks; another number of splits adds up in another order)
        assert torch.allclose(out, ref, rtol=1e-4, atol=2e-5) and torch.allclose(lse, ref_lse, rtol=1e-5, atol=1e-5)


# One to 32 splits by the budget; 32 (sequence, head) pairs fill the device, two do not.  `to`: the largest group size at which the workgroups share the
# scoring (0: never).  The shares: 32 chunks and less, up to 64, 80 and 128; the instances: up to 512, 1024, 1536 and 2560 chunks.
@pytest.mark.parametrize("G,centers", [(1, 0), (4, 0), (4, 1), (7, 0), (8, 1)])
@pytest.mark.parametrize("chunks,H,budget,to", [
    ([129], 2, 300, 8), ([255, 1], 2, 512, 8), ([257], 2, 512, 8), ([511, 130], 2, 513, 8), ([513], 1, 2048, 8), ([1024, 1025], 1, 2048, 8),
    ([1535], 1, 4000, 8), ([1536, 400], 2, 4000, 8), ([1537], 2, 4000, 0), ([1537], 8, 4096, 8), ([513, 7, 400, 512], 8, 512, 8),
    ([577, 640, 641, 1], 8, 512, 8), ([1023, 1024, 0, 65], 8, 512, 8), ([1024] * 4, 8, 600, 8), ([1025] * 4, 8, 512, 0), ([2559], 8, 4096, 8),
    ([2560], 8, 4096, 8), ([2560, 2300], 8, 2048, 4), ([2561], 8, 4096, 0)])
def test_shares(chunks, H, budget, to, G, centers):
    x = _Index(chunks, H, G, centers, budget)
    assert x.shares() == (G <= to)
    for _ in range(3):
        x.check(x.query())


# The caller's own number of splits, as far as there are tokens for them: shares of four chunks and up, and more workgroups than run at the
# same time, where those that run would wait for the others (two kernels).
@pytest.mark.parametrize("G,centers", [(1, 0), (4, 1), (7, 0)])
@pytest.mark.parametrize("chunks,H,longest,splits,one", [([200], 2, 160, 256, True), ([200], 2, 60, 64, True), ([200, 190], 2, 160, 256, False),
                                                         ([513], 2, 5, 64, True), ([700], 8, 5, 256, True), ([700, 650], 8, 5, 256, False),
                                                         ([2500], 4, 5, 256, True), ([2500], 8, 5, 256, False), ([900, 100, 2], 3, 5, 3, False)])
def test_splits_of_the_callers(chunks, H, longest, splits, one, G, centers):
    x = _Index(chunks, H, G, centers, 10 ** 6, splits=splits, longest=longest)
    assert x.shares() == one
    for budget in (10 ** 6, x.lens[0] // 2, 300):
        x.budget = budget
        for _ in range(2):
            x.check(x.query())


def test_pinned_chunks_and_no_budget():
    for sink, budget in ((40, 500), (9, 0), (0, 10 ** 6)):
        x = _Index([600, 140], 2, 4, 0, budget, sink=sink)
        assert x.shares()
        x.check(x.query())


def test_a_buffer_that_held_another_index():
    """The keys that the steps on one index have posted are no keys of the index that comes into the same buffer later, by a build or an import: its first step has
    the number that they carry.  (Whether a stale key would be read is a matter of time, so the words themselves are looked at.)"""
    x = _Index([704], 4, 4, 0, 720)
    keys, blob = x.K.clone(), x.lc.lc_index_export(x.idx)
    for _ in range(3):
        assert x.shares() and not x.posted().any()
        x.check(x.query())
        assert bool((x.posted() >> 32 == 1).all())
        x.K.copy_(x.draw(*x.K.shape))
        x.build()
    x.check(x.query())
    x.K.copy_(keys)
    x.idx = x.lc.lc_index_import(x.cfg, blob, x.ib)
    assert not x.posted().any()
    x.check(x.query())


@pytest.mark.parametrize("spare", [0, 2456, 9980])
def test_keys_of_chunks_to_come_are_cleared(spare):
    """As many as a step may post, however few chunks there are."""
    x = _Index([100, 36], 8, 4, 0, 512, spare=spare)
    assert not x.posted().any()
    x.ib.fill_(0xA5)
    x.build()
    assert not x.posted().any()


def test_chunks_that_nobody_posted():
    """A captured step on an index that has grown beyond what its workgroups share out."""
    import torch
    x = _Index([130], 2, 4, 0, 256, spare=64)
    q, out, lse = x.query(), torch.empty((1, 8, 128), device="cuda"), torch.empty((1, 8), device="cuda")
    assert x.shares()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        x.lc.lc_decode_step(x.idx, q, x.K, x.V, x.budget, out, x.ws, lse=lse)
        side.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            x.lc.lc_decode_step(x.idx, q, x.K, x.V, x.budget, out, x.ws, lse=lse)
    torch.cuda.current_stream().wait_stream(side)
    for turn in range(3):
        if turn:                                             # four splits of 36 chunks: 144 of them are shared out
            for _ in range(32):
                x.lc.lc_append(x.idx, x.K, x.V, x.draw(1, 2, 128), x.draw(1, 2, 128), [1], x.ws)
        q.copy_(x.query())
        out.fill_(float("nan"))
        graph.replay()
        got, got_lse = out.clone(), lse.clone()
        _, _, ref, ref_lse = x.step(q)
        assert torch.equal(got, ref) and torch.equal(got_lse, ref_lse)
        x.check(q)


def test_an_index_that_has_grown_takes_a_captured_step_no_longer():
    """The chunks behind all shares are scored before anyone looks for them: a replay on a grown index gives what a step launched anew gives, in
    about its time (left to those that look for them in vain it took three to four times as long)."""
    import torch
    x = _Index([130], 2, 4, 0, 256, spare=320)

    def capture():
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            x.lc.lc_decode_step(x.idx, q, x.K, x.V, x.budget, out, x.ws, lse=lse)
            side.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=side):
                for _ in range(10):
                    x.lc.lc_decode_step(x.idx, q, x.K, x.V, x.budget, out, x.ws, lse=lse)
        torch.cuda.current_stream().wait_stream(side)
        return graph

    def us(graph):
        took = []
        for _ in range(10):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            a.record()
            graph.replay()
            b.record()
            torch.cuda.synchronize()
            took.append(a.elapsed_time(b) * 100)
        return min(took)

    q, out, lse = x.query(), torch.empty((1, 8, 128), device="cuda"), torch.empty((1, 8), device="cuda")
    assert x.shares()
    graph, grown = capture(), 0
    # four splits of 36 chunks, an instance that holds 512: one chunk behind them, one workgroup's 16, a turn of all four, several turns
    for more in (15, 16 + 14, 64 + 14, 65 + 14, 300):
        while grown < more:
            x.lc.lc_append(x.idx, x.K, x.V, x.draw(1, 2, 128), x.draw(1, 2, 128), [1], x.ws)
            grown += 1
        q.copy_(x.query())
        out.fill_(float("nan"))
        old = us(graph)
        got, got_lse = out.clone(), lse.clone()
        _, _, ref, ref_lse = x.step(q)
        assert torch.equal(got, ref) and torch.equal(got_lse, ref_lse)
        x.check(q)
        assert old < 1.8 * us(capture()) + 2, more


def test_steps_beside_other_streams_kernels():
    """Workgroups of a step that have no place yet, because two other streams keep the device busy: those that have one wait for their keys for a while
    and then score for themselves.  The same bits as on a quiet device."""
    import torch
    xs = [_Index([2300], 8, 4, 0, 2048, seed=1), _Index([500, 620, 41], 8, 7, 1, 1024, seed=2)]
    qs = [x.query() for x in xs]
    assert all(x.shares() for x in xs)
    alone = [x.step(q)[2:] for x, q in zip(xs, qs)]
    noise = torch.randn((4096, 4096), device="cuda")
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(3)]
    outs = [[(torch.empty_like(o), torch.empty_like(l)) for _ in range(30)] for o, l in alone]
    torch.cuda.synchronize()
    for i in range(30):
        with torch.cuda.stream(streams[2]):
            if i % 3 == 0:
                torch.mm(noise, noise)
        for x, q, out, stream in zip(xs, qs, outs, streams):
            x.lc.lc_decode_step(x.idx, q, x.K, x.V, x.budget, out[i][0], x.ws, lse=out[i][1], stream=stream)
    torch.cuda.synchronize()
    for (o, l), got in zip(alone, outs):
        assert all(torch.equal(a, o) and torch.equal(b, l) for a, b in got)
