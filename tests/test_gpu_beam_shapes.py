"""Top-k per level against the oracle at the sizes where its kernel changes: lists around what one wavefront cuts and
what LDS holds, more nodes than one pass of the gather or the LDS copy of the parents takes, equal scores at the
cut, indexes of one level, pinned chunks."""
import numpy as np
import pytest

from oracle import lychee_oracle as orc

pytestmark = pytest.mark.gpu


def check(H, chunks, levels, F, beam, budget, sink=0, G=4, same=0, centers=0, seed=0):
    import torch
    from paper_2603_08453_amd import binding as lc
    from tests.gpu_common import levels_to_oracle_index
    r = np.random.default_rng(seed)
    bounds = [np.concatenate([[0], np.cumsum(r.integers(1, 4, size=m))]).astype(np.int32) for m in chunks]
    T = max(int(b[-1]) for b in bounds)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    K = torch.randn((len(chunks), H, T, 128), generator=g, device="cuda").to(torch.bfloat16)
    for b, bd in enumerate(bounds):
        K[b, :, : bd[min(same, len(bd) - 1)]] = K[b, :, :1].clone()
    q = torch.randn((len(chunks), H * G, 128), generator=g, device="cuda").to(torch.bfloat16)
    cfg = lc.lc_config_default(levels=levels, fanout=F, kmeans_iters=2, max_chunks=max(chunks), max_tokens=T, center_dtype=centers,
                               policy=lc.LC_POLICY_BEAM, beam=beam, sink_tokens=sink)
    ib = torch.zeros(lc.lc_index_bytes(cfg, len(chunks), H), dtype=torch.uint8, device="cuda")
    ws = torch.zeros(lc.lc_workspace_bytes(cfg, len(chunks), H * G, H), dtype=torch.uint8, device="cuda")
    idx = lc.lc_build_index(cfg, K, [int(b[-1]) for b in bounds], bounds, ib, ws)
    cap = max(chunks)
    ids = torch.full((len(chunks), H, cap), -7, dtype=torch.int32, device="cuda")
    counts = torch.full((len(chunks), H), -1, dtype=torch.int32, device="cuda")
    scores = torch.full((len(chunks), H, cap), float("nan"), dtype=torch.float32, device="cuda")
    lc.lc_retrieve(idx, q, budget, ids, counts, ws, scores=scores)
    seqs = lc.unpack_blob(lc.lc_index_export(idx))["seqs"]
    for b, s in enumerate(seqs):
        for h in range(H):
            oi = levels_to_oracle_index(s["heads"][h], s["bounds"], int(bounds[b][-1]), F, orc.TOKEN_BALL)
            qh = q[b, h * G:(h + 1) * G].double().cpu().numpy()
            ref = orc.retrieve_beam(oi, qh, budget, beam, sink)
            got = ids[b, h, : int(counts[b, h])].cpu().numpy()
            assert got.tolist() == ref.tolist(), (b, h, len(got), len(ref))
            sg, want = scores[b, h, : oi.M].cpu().numpy(), orc.node_scores(oi, 0, qh)
            seen = np.isfinite(sg)
            assert np.all(np.abs(sg[seen] - want[seen]) <= 2e-5 * np.maximum(1.0, np.abs(want[seen])))
            assert np.all(seen[np.setdiff1d(got, orc.pinned_chunks(oi, sink))])


@pytest.mark.parametrize("n", [1, 63, 64, 65, 255, 256, 257, 1023, 1024, 1025, 2100])
def test_nodes_of_the_top_level(n):
    check(2, [2 * n], 2, 2, [0, max(1, n // 7)], 60)


# Candidates of the top level beyond the first 256 come from a list that all wavefronts write and each reads from
# another: in LDS, and past 4096 of them in the workspace.  Every node is kept, so one lost entry shows in the ids.
@pytest.mark.parametrize("n", [300, 2000, 4096, 4097, 9000])
def test_list_of_the_top_level(n):
    check(1, [2 * n], 2, 2, [0, 0], 2 * n)
    check(2, [n], 1, 2, [0, 0], n, G=7, centers=1)


@pytest.mark.parametrize("n", [1, 3, 64, 257, 1024, 1025, 4096, 4097, 9000])
@pytest.mark.parametrize("levels", [1, 2])
def test_every_chunk_a_candidate(n, levels):
    check(1, [n], levels, 16, [0, 0], max(1, n // 3), sink=5)
    check(1, [n], levels, 16, [n // 5 + 1, 0], 10 ** 9, centers=1, G=7)


@pytest.mark.parametrize("chunks,levels,F,beam", [
    ([4095, 4096, 4097], 3, 16, [0, 30, 6]), ([12289], 3, 4, [0, 50, 20]), ([33000, 7], 4, 8, [0, 60, 20, 9]),
    ([40000], 3, 2, [0, 4000, 700]), ([900, 0, 1], 4, 4, [25, 9, 5, 2])])
def test_levels_beyond_one_pass(chunks, levels, F, beam):
    check(2, chunks, levels, F, beam, 200, sink=16)


@pytest.mark.parametrize("G", [1, 2, 3, 5, 6, 8])
def test_group_sizes(G):
    check(3, [1500, 333], 3, 16, [0, 12, 4], 90, G=G)
    check(1, [700], 3, 16, [0, 12, 4], 90, G=G, centers=1)


@pytest.mark.parametrize("chunks,same", [(300, 70), (900, 500), (3000, 2500), (6000, 5000)])
@pytest.mark.parametrize("limit,budget", [(0, 100), (40, 10 ** 9), (200, 10 ** 9)])
def test_equal_scores_at_the_cut(chunks, same, limit, budget):
    check(1, [chunks], 2, 8, [limit, 0], budget, same=same)
    check(1, [chunks], 3, 3, [limit, 25, 20], budget, same=same)


# Lists that the cutting wavefront holds in registers (25 to 256 and to 512 candidates), cut by the budget, by number and by both, with as
# many equal scores as its pairs take, more, and more than its bin takes.
@pytest.mark.parametrize("n", [24, 25, 64, 65, 255, 256, 257, 511, 512, 513])
@pytest.mark.parametrize("same", [0, 8, 9, 70])
def test_candidates_held_by_one_wavefront(n, same):
    for limit, budget in ((0, n // 2), (n // 3 + 1, 10 ** 9), (n // 4 + 1, n), (0, 0)):
        check(1, [n], 1, 2, [limit, 0], budget, same=same, seed=n)
    check(1, [2 * n], 2, 2, [0, n // 5 + 1], 60, same=2 * same, seed=n)
