"""Export of an imported index gives the blob back bit for bit, at the sizes where the windowed word map can go
wrong: one window and several, a remainder, one level, sequences without chunks, bfloat16 chunk centers, more
sequences than the kernels keep table rows for on chip."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def random_blob(lc, rng, H, L, F, chunks, bf16):
    seqs = []
    for M in chunks:
        bounds = np.concatenate([[0], np.cumsum(rng.integers(1, 5, size=M))]).astype(np.int32)
        N = [M]
        for _ in range(1, L):
            N.append(max(1, -(-N[-1] // F)))
        heads = []
        for _h in range(H):
            levels = []
            for l in range(L):
                c = rng.standard_normal((N[l], 128), dtype=np.float32)
                if l == 0 and bf16:
                    c = (c.view(np.uint32) & np.uint32(0xFFFF0000)).view(np.float32)
                up = N[l + 1] if l + 1 < L else 1
                levels.append(dict(center=c, radius=rng.random(N[l], dtype=np.float32),
                                   parent=rng.integers(0, up, size=N[l]).astype(np.int32) if l + 1 < L
                                   else np.full(N[l], -1, dtype=np.int32),
                                   ntok=rng.integers(0, 99, size=N[l]).astype(np.int32),
                                   nchunk=rng.integers(0, 9, size=N[l]).astype(np.int32)))
            heads.append(levels)
        seqs.append(dict(T=int(bounds[-1]) + 3, bounds=bounds, heads=heads))
    return lc.pack_blob(len(chunks), H, 128, L, F, lc.LC_GEOMETRY_TOKEN_BALL, seqs,
                        center_dtype=lc.LC_CENTER_BF16 if bf16 else lc.LC_CENTER_F32)


@pytest.mark.parametrize("H,L,F,chunks,bf16", [
    (1, 1, 4, [1], False),
    (2, 1, 4, [0, 3, 0], True),
    (2, 3, 4, [37, 0, 5, 64], False),
    (3, 2, 16, [100, 1], True),
    (8, 3, 16, [455], False),                 # 2 MB: three windows and a remainder of the last
    (8, 2, 16, [1900, 700], True),            # more windows than there are slots
    (1, 2, 4, [1 + i % 3 for i in range(1000)], False),
])
def test_import_export_round_trip(H, L, F, chunks, bf16):
    import torch
    from paper_2603_08453_amd import binding as lc
    blob = random_blob(lc, np.random.default_rng(len(chunks) + H), H, L, F, chunks, bf16)
    cfg = lc.lc_config_default(levels=L, fanout=F, max_chunks=max(chunks) + 2, max_tokens=5 * max(chunks) + 20,
                               center_dtype=lc.LC_CENTER_BF16 if bf16 else lc.LC_CENTER_F32)
    buf = torch.full((lc.lc_index_bytes(cfg, len(chunks), H),), 0xA5, dtype=torch.uint8, device="cuda")
    idx = lc.lc_index_import(cfg, blob, buf)
    assert lc.lc_index_export(idx) == blob
    if L > 1:                                 # the radii at import are the baseline of the drift figures
        drift = lc.lc_index_drift(idx, 1, torch.zeros(1 << 16, dtype=torch.uint8, device="cuda"))
        assert np.all(drift[..., 2] == 0) and np.array_equal(drift[..., 0], drift[..., 1])


@pytest.mark.parametrize("chunks", [[1, 255, 256], [4096, 4097], [9000, 0, 4351]])
def test_drift_counts_every_node(chunks):
    """Rounds of 16 nodes a thread with remainders: one node to a chunk, radii positive (float32 sums of n of them: n 2^-24 of the sum at most)."""
    import torch
    from paper_2603_08453_amd import binding as lc
    blob = random_blob(lc, np.random.default_rng(chunks[0]), 2, 2, 1, chunks, False)
    cfg = lc.lc_config_default(levels=2, fanout=1, max_chunks=max(chunks), max_tokens=5 * max(chunks) + 20)
    idx = lc.lc_index_import(cfg, blob, torch.zeros(lc.lc_index_bytes(cfg, len(chunks), 2), dtype=torch.uint8, device="cuda"))
    drift = lc.lc_index_drift(idx, 1, torch.zeros(1 << 16, dtype=torch.uint8, device="cuda"))
    for b, s in enumerate(lc.unpack_blob(blob)["seqs"]):
        for h, head in enumerate(s["heads"]):
            r = head[1]["radius"].astype(np.float64)
            r = r[np.isfinite(r)]
            assert drift[b, h, 3] == len(r) and drift[b, h, 2] == 0
            for total in drift[b, h, :2]:
                assert abs(total - r.sum()) <= max(len(r), 1) * 2.0 ** -24 * np.abs(r).sum()
