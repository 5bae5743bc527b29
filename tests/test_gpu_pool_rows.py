"""Chunk representatives from their rows: lengths around a wavefront's batches (32 rows; two in registers, one in LDS, then none), row
strides of every kind, values that are not finite."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

LENGTHS = [1, 2, 3, 4, 5, 31, 32, 33, 36, 63, 64, 65, 95, 96, 97, 127, 128, 129, 160, 161, 300, 1000, 7]


def chunks_of(K, bounds, **config):
    """Level-0 centers and radii, [head] -> float64 arrays."""
    import torch
    from paper_2603_08453_amd import binding as lc
    H, T = K.shape[1], K.shape[2]
    cfg = lc.lc_config_default(levels=2, fanout=8, kmeans_iters=1, max_chunks=len(bounds) - 1, max_tokens=T, **config)
    ib = torch.zeros(lc.lc_index_bytes(cfg, 1, H), dtype=torch.uint8, device="cuda")
    ws = torch.zeros(lc.lc_workspace_bytes(cfg, 1, H, H), dtype=torch.uint8, device="cuda")
    idx = lc.lc_build_index(cfg, K, [int(bounds[-1])], [bounds], ib, ws)
    heads = lc.unpack_blob(lc.lc_index_export(idx))["seqs"][0]["heads"]
    return [(h[0]["center"].astype(np.float64), h[0]["radius"].astype(np.float64)) for h in heads]


def check(K, bounds, **config):
    half = config.get("center_dtype", 0) == 1
    n = np.diff(bounds)
    for h, (center, radius) in enumerate(chunks_of(K, bounds, **config)):
        x = K[0, h, : bounds[-1]].double().cpu().numpy()
        mean = np.add.reduceat(x, bounds[:-1], axis=0) / n[:, None]
        size = np.add.reduceat(np.abs(x), bounds[:-1], axis=0) / n[:, None]
        # n additions and two roundings in float32, half a unit of bfloat16 if that is what is stored
        bound = (n[:, None] + 2) * 2.0 ** -24 * size + (2.0 ** -8 * np.abs(mean) if half else 0.0)
        assert (np.abs(center - mean) <= bound).all()
        far = np.maximum.reduceat(np.linalg.norm(x - np.repeat(center, n, axis=0), axis=1), bounds[:-1])
        # the radius covers every row, and is inflated by 4e-6 and the roundings of a sum of 128 squares (16 of them in a lane)
        assert (radius >= far).all() and (radius <= far * (1 + 4e-6 + 2.0 ** -19) + 1e-30).all()


@pytest.mark.parametrize("centers", [0, 1])
@pytest.mark.parametrize("layout", ["heads", "tokens", "padded"])
def test_rows(layout, centers):
    import torch
    bounds = np.concatenate([[0], np.cumsum(LENGTHS)]).astype(np.int32)
    T, H = int(bounds[-1]), 3
    gen = torch.Generator(device="cuda")
    gen.manual_seed(centers)
    if layout == "heads":
        K = torch.randn((1, H, T, 128), generator=gen, device="cuda").to(torch.bfloat16)
    elif layout == "tokens":
        K = torch.randn((1, T, H, 128), generator=gen, device="cuda").to(torch.bfloat16).transpose(1, 2)
    else:
        K = torch.randn((1, H, T, 136), generator=gen, device="cuda").to(torch.bfloat16)[..., :128]
    check(K, bounds, center_dtype=centers)


@pytest.mark.parametrize("step", [2 ** 25 - 8, 2 ** 25])             # (the longest row stride whose batch has 31 bits of offset, and the next)
def test_rows_far_apart(step):
    import torch
    bounds = np.array([0, 1, 4, 6], dtype=np.int32)
    store = torch.zeros(6 * step, dtype=torch.bfloat16, device="cuda")
    K = store.as_strided((1, 1, 6, 128), (6 * step, 6 * step, step, 1))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    K.copy_(torch.randn((1, 1, 6, 128), generator=gen, device="cuda"))
    check(K, bounds)


def test_values_that_are_not_finite():
    import torch
    bounds = np.array([0, 40, 100, 140, 145], dtype=np.int32)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(2)
    K = torch.randn((1, 1, 145, 128), generator=gen, device="cuda").to(torch.bfloat16)
    (before, _), = chunks_of(K, bounds)
    K[0, 0, 3, 9] = float("inf")
    K[0, 0, 99, 127] = float("nan")
    K[0, 0, 141, 0], K[0, 0, 142, 0] = float("inf"), float("-inf")
    (center, radius), = chunks_of(K, bounds)
    assert center[0, 9] == np.inf and np.isnan(center[1, 127]) and np.isnan(center[3, 0])
    ok = np.ones_like(center, dtype=bool)
    ok[0, 9] = ok[1, 127] = ok[3, 0] = False
    # (the same sums in another order: 60 additions at most)
    assert np.allclose(center[ok], before[ok], rtol=0, atol=60 * 2.0 ** -24 * 5.0)
    assert radius[0] == np.inf and np.isfinite(radius[2])
