"""The decode step against the two separate calls, and both against the oracle on the stored index, around the sizes where
the step changes from one kernel to two."""
import numpy as np
import pytest

from oracle import lychee_oracle as orc
from tests import helpers

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G,centers", [(1, 0), (2, 1), (3, 0), (4, 0), (4, 1), (5, 0), (6, 1), (7, 0), (7, 1), (8, 0)])
@pytest.mark.parametrize("chunks", [[1], [63, 0], [64], [65, 2], [127], [128, 128], [129, 1]])
def test_few_chunks(chunks, G, centers):
    import torch
    from paper_2603_08453_amd import binding as lc
    from tests.gpu_common import attention_errors, levels_to_oracle_index
    H, B = 2, len(chunks)
    r = np.random.default_rng(sum(chunks) + G)
    bounds = [np.concatenate([[0], np.cumsum(r.integers(1, 30, size=m))]).astype(np.int32) for m in chunks]
    lens = [int(b[-1]) + 5 for b in bounds]                                  # (an open tail)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(G)
    K = torch.randn((B, H, max(lens), 128), generator=gen, device="cuda").to(torch.bfloat16)
    V = torch.randn((B, H, max(lens), 128), generator=gen, device="cuda").to(torch.bfloat16)
    q = torch.randn((B, H * G, 128), generator=gen, device="cuda").to(torch.bfloat16)
    cap = max(chunks)
    for sink, budget in ((0, 0), (0, 200), (40, 700), (0, 10 ** 6)):
        cfg = lc.lc_config_default(levels=2, fanout=8, kmeans_iters=2, max_chunks=cap, max_tokens=max(lens), center_dtype=centers,
                                   sink_tokens=sink)
        ib = torch.zeros(lc.lc_index_bytes(cfg, B, H), dtype=torch.uint8, device="cuda")
        ws = torch.zeros(lc.lc_workspace_bytes(cfg, B, H * G, H), dtype=torch.uint8, device="cuda")
        idx = lc.lc_build_index(cfg, K, lens, bounds, ib, ws)
        got = [torch.full((B, H, cap), -7, dtype=torch.int32, device="cuda") for _ in range(2)]
        n = [torch.full((B, H), -1, dtype=torch.int32, device="cuda") for _ in range(2)]
        out = [torch.full((B, H * G, 128), float("nan"), device="cuda") for _ in range(2)]
        lse = [torch.full((B, H * G), float("nan"), device="cuda") for _ in range(2)]
        lc.lc_retrieve(idx, q, budget, got[0], n[0], ws)
        lc.lc_sparse_decode(idx, q, K, V, got[0], n[0], out[0], ws, lse=lse[0])
        lc.lc_decode_step(idx, q, K, V, budget, out[1], ws, lse=lse[1], chunk_ids=got[1], counts=n[1])
        assert torch.equal(n[0], n[1])
        for b in range(B):
            for h in range(H):
                assert torch.equal(got[0][b, h, : n[0][b, h]], got[1][b, h, : n[1][b, h]])
        assert torch.allclose(out[0], out[1], rtol=1e-4, atol=2e-5) and torch.allclose(lse[0], lse[1], rtol=1e-5, atol=1e-5)
        # the oracle on the stored index: selection within the score band, attention over the selected chunks (the
        # acceptance bars of the other parity tests)
        seqs = lc.unpack_blob(lc.lc_index_export(idx))["seqs"]
        for b in range(B):
            for h in range(H):
                oi = levels_to_oracle_index(seqs[b]["heads"][h], bounds[b], lens[b], 8, orc.TOKEN_BALL)
                qh, ids = q[b, h * G:(h + 1) * G].double().cpu().numpy(), got[1][b, h, : n[1][b, h]].cpu().numpy()
                helpers.accept_ids(ids, orc.node_scores(oi, 0, qh), oi.lens(), budget, pinned=orc.pinned_chunks(oi, sink))
                ref, ref_lse = orc.sparse_decode(qh, K[b, h].double().cpu().numpy(), V[b, h].double().cpu().numpy(), oi.bounds, oi.T, ids)
                mx, rel = attention_errors(out[1][b, h * G:(h + 1) * G].cpu().numpy(), ref)
                assert mx <= 1e-2 and rel <= 2e-3
                assert np.abs(lse[1][b, h * G:(h + 1) * G].cpu().numpy() - ref_lse).max() <= 1e-3
