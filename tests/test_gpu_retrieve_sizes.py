"""lc_retrieve where its selection changes shape: chunk counts around the rows of its selecting kernel and its largest, budgets that
end in the upper half of the scores' range, below it, nowhere, and inside large groups of equal scores."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def by_the_rule(scores, lens, starts, budget, sink):
    """Pinned chunks, and the longest prefix of the others (score descending, id ascending) that fits the budget."""
    pinned = starts < sink
    rest = np.flatnonzero(~pinned)
    order = rest[np.lexsort((rest, -scores[rest]))]
    fits = np.cumsum(lens[order]) <= max(budget, 0)
    return np.sort(np.concatenate([np.flatnonzero(pinned), order[: int(fits.sum())]]))


@pytest.mark.parametrize("geometry", [0, 1])                    # 1: scores of both signs
@pytest.mark.parametrize("distinct", [0, 37])                   # 37: the chunks repeat 37 contents, so scores are equal by the hundreds
@pytest.mark.parametrize("chunks", [65, 129, 1023, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193, 12287, 12288, 12289])
def test_selection_follows_the_scores(chunks, distinct, geometry):
    import torch
    from paper_2603_08453_amd import binding as lc
    B, H, G = 2, 2, 4
    r = np.random.default_rng(chunks + distinct)
    counts = [chunks, max(1, chunks // 3)]
    kinds = r.integers(0, 37, size=chunks)
    size = r.integers(1, 6, size=37)[kinds] if distinct else r.integers(1, 6, size=chunks)
    bounds = [np.concatenate([[0], np.cumsum(size[:m])]).astype(np.int32) for m in counts]
    lens = [int(b[-1]) + 2 for b in bounds]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(chunks)
    K = torch.randn((B, H, max(lens), 128), generator=gen, device="cuda").to(torch.bfloat16)
    if distinct:
        content = torch.randn((37, 5, 128), generator=gen, device="cuda").to(torch.bfloat16)
        kind = np.repeat(kinds, size)
        at = np.concatenate([np.arange(n) for n in size])
        K[:, :, : len(kind)] = content[torch.from_numpy(kind).cuda(), torch.from_numpy(at).cuda()]
    q = torch.randn((B, H * G, 128), generator=gen, device="cuda").to(torch.bfloat16)
    q[:, :G] *= 1.0 if chunks % 2 else 0.0                      # (no query: every score of head 0 is zero)
    total = int(bounds[0][-1])
    for sink, budget in ((0, 0), (3, 7), (0, total // 50 + 1), (total // 3, total // 9), (0, (9 * total) // 10), (0, total), (9, 10 ** 9)):
        cfg = lc.lc_config_default(levels=2, fanout=32, kmeans_iters=1, max_chunks=chunks, max_tokens=max(lens), sink_tokens=sink, prune=0,
                                   geometry=geometry)
        ib = torch.zeros(lc.lc_index_bytes(cfg, B, H), dtype=torch.uint8, device="cuda")
        ws = torch.zeros(lc.lc_workspace_bytes(cfg, B, H * G, H), dtype=torch.uint8, device="cuda")
        idx = lc.lc_build_index(cfg, K, lens, bounds, ib, ws)
        cap = max(1, min(chunks, budget + sink))
        ids = torch.full((B, H, cap), -7, dtype=torch.int32, device="cuda")
        n = torch.full((B, H), -1, dtype=torch.int32, device="cuda")
        scores = torch.full((B, H, chunks), float("nan"), device="cuda")
        lc.lc_retrieve(idx, q, budget, ids, n, ws, scores=scores)
        for b in range(B):
            m = counts[b]
            for h in range(H):
                want = by_the_rule(scores[b, h, :m].cpu().numpy(), np.diff(bounds[b]), bounds[b][:-1], budget, sink)
                assert int(n[b, h]) == len(want), (sink, budget, b, h)
                assert np.array_equal(ids[b, h, : len(want)].cpu().numpy(), want), (sink, budget, b, h)


@pytest.mark.parametrize("infinite", [False, True])
@pytest.mark.parametrize("geometry", [0, 1])
@pytest.mark.parametrize("chunks", [64, 65, 130, 241, 600, 1030, 2050, 4096])
def test_a_step_selects_the_same(chunks, geometry, infinite):
    import torch
    from paper_2603_08453_amd import binding as lc
    H, G = 2, 4
    size = np.random.default_rng(chunks).integers(1, 6, size=chunks)
    bounds = np.concatenate([[0], np.cumsum(size)]).astype(np.int32)
    T = int(bounds[-1]) + 2
    gen = torch.Generator(device="cuda")
    gen.manual_seed(chunks)
    K, V = (torch.randn((1, H, T, 128), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2))
    q = torch.randn((1, H * G, 128), generator=gen, device="cuda").to(torch.bfloat16)
    if infinite:
        K[0, 0, T // 2, 3], K[0, 1, T // 3, 5] = float("inf"), 3e38
    cfg = lc.lc_config_default(levels=2, fanout=32, kmeans_iters=1, max_chunks=chunks, max_tokens=T, prune=0, geometry=geometry)
    ib = torch.zeros(lc.lc_index_bytes(cfg, 1, H), dtype=torch.uint8, device="cuda")
    ws = torch.zeros(lc.lc_workspace_bytes(cfg, 1, H * G, H), dtype=torch.uint8, device="cuda")
    idx = lc.lc_build_index(cfg, K, [T], [bounds], ib, ws)
    for budget in (3, T // 40 + 1, T // 9, (9 * T) // 10, 10 ** 9):
        ids = [torch.full((1, H, chunks), -7, dtype=torch.int32, device="cuda") for _ in range(2)]
        n = [torch.full((1, H), -1, dtype=torch.int32, device="cuda") for _ in range(2)]
        out = torch.empty((1, H * G, 128), device="cuda")
        lc.lc_retrieve(idx, q, budget, ids[0], n[0], ws)
        lc.lc_decode_step(idx, q, K, V, budget, out, ws, chunk_ids=ids[1], counts=n[1])
        assert torch.equal(n[0], n[1]), budget
        for h in range(H):
            assert torch.equal(ids[0][0, h, : n[0][0, h]], ids[1][0, h, : n[1][0, h]]), (budget, h)


@pytest.mark.parametrize("others", [70, 1500, 9000])
@pytest.mark.parametrize("tied", [1, 15, 17, 64, 65, 255, 256, 257, 700])
def test_a_budget_that_ends_among_equal_scores(tied, others):
    """`tied` chunks of one score and different lengths between `others` of higher and lower ones: as many of them as the list of the
    cutoff bin holds, and one more and less.  (All tokens of a chunk are one row, so its score does not depend on its length.)"""
    import torch
    from paper_2603_08453_amd import binding as lc
    G, M = 4, tied + others
    r = np.random.default_rng(tied + others)
    size = r.integers(1, 6, size=M)
    bounds = np.concatenate([[0], np.cumsum(size)]).astype(np.int32)
    T = int(bounds[-1])
    level = r.permutation(np.concatenate([np.zeros(tied), r.normal(size=others)]))
    rows = np.zeros((M, 128), dtype=np.float32)
    rows[:, 0], rows[:, 1] = 8 + level, 0.25
    K = torch.from_numpy(np.repeat(rows, size, axis=0)).cuda().to(torch.bfloat16)[None, None].contiguous()
    q = torch.zeros((1, G, 128), device="cuda")
    q[0, :, 0] = torch.arange(G, 0, -1, device="cuda")
    q = q.to(torch.bfloat16)
    cfg = lc.lc_config_default(levels=2, fanout=32, kmeans_iters=1, max_chunks=M, max_tokens=T, prune=0)
    ib = torch.zeros(lc.lc_index_bytes(cfg, 1, 1), dtype=torch.uint8, device="cuda")
    ws = torch.zeros(lc.lc_workspace_bytes(cfg, 1, G, 1), dtype=torch.uint8, device="cuda")
    idx = lc.lc_build_index(cfg, K, [T], [bounds], ib, ws)
    higher, here = int(size[level > 0].sum()), int(size[level == 0].sum())
    for budget in (1, higher // 2, higher, higher + 1, higher + here // 3, higher + here - 1, higher + here, higher + here + 5, T // 3, T // 3 + 1, T - 1, T):
        ids = torch.full((1, 1, M), -7, dtype=torch.int32, device="cuda")
        n = torch.full((1, 1), -1, dtype=torch.int32, device="cuda")
        scores = torch.full((1, 1, M), float("nan"), device="cuda")
        lc.lc_retrieve(idx, q, budget, ids, n, ws, scores=scores)
        got = scores[0, 0].cpu().numpy()
        assert len(np.unique(got[level == 0])) == 1
        want = by_the_rule(got, size, bounds[:-1], budget, 0)
        assert int(n[0, 0]) == len(want), budget
        assert np.array_equal(ids[0, 0, : len(want)].cpu().numpy(), want), budget


@pytest.mark.parametrize("G", [7, 8])
@pytest.mark.parametrize("B,chunks", [(8, 1812), (8, 1813), (8, 2048), (8, 2049), (25, 256), (25, 257), (32, 512), (32, 513)])
def test_many_pairs_at_the_largest_group_sizes(B, chunks, G):
    """Both sides of the band in which one kernel scores and selects for many (sequence, head) pairs."""
    import torch
    from paper_2603_08453_amd import binding as lc
    H = 8
    r = np.random.default_rng(chunks + G)
    counts = [chunks if b % 3 != 1 else max(1, chunks // 2 - b) for b in range(B)]
    bounds = [np.concatenate([[0], np.cumsum(r.integers(1, 4, size=m))]).astype(np.int32) for m in counts]
    lens = [int(b[-1]) + 1 for b in bounds]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(chunks)
    K = torch.randn((B, H, max(lens), 128), generator=gen, device="cuda").to(torch.bfloat16)
    q = torch.randn((B, H * G, 128), generator=gen, device="cuda").to(torch.bfloat16)
    cfg = lc.lc_config_default(levels=2, fanout=32, kmeans_iters=1, max_chunks=chunks, max_tokens=max(lens), prune=0)
    ib = torch.zeros(lc.lc_index_bytes(cfg, B, H), dtype=torch.uint8, device="cuda")
    ws = torch.zeros(lc.lc_workspace_bytes(cfg, B, H * G, H), dtype=torch.uint8, device="cuda")
    idx = lc.lc_build_index(cfg, K, lens, bounds, ib, ws)
    for budget in (chunks // 8, chunks, 10 ** 9):
        ids = torch.full((B, H, chunks), -7, dtype=torch.int32, device="cuda")
        n = torch.full((B, H), -1, dtype=torch.int32, device="cuda")
        scores = torch.full((B, H, chunks), float("nan"), device="cuda")
        lc.lc_retrieve(idx, q, budget, ids, n, ws, scores=scores)
        ids, n, scores = ids.cpu().numpy(), n.cpu().numpy(), scores.cpu().numpy()
        for b in range(B):
            for h in range(H):
                want = by_the_rule(scores[b, h, : counts[b]], np.diff(bounds[b]), bounds[b][:-1], budget, 0)
                assert n[b, h] == len(want) and np.array_equal(ids[b, h, : len(want)], want), (budget, b, h)


@pytest.mark.parametrize("center_dtype", [0, 1])
@pytest.mark.parametrize("G", [1, 3, 7])
@pytest.mark.parametrize("B,H,chunks", [(1, 2, 65), (1, 2, 127), (8, 8, 300), (8, 8, 321), (16, 8, 1030)])
def test_scores_of_one_two_and_four_chunks_at_a_time(B, H, chunks, G, center_dtype):
    """The scoring kernel takes more chunks at a time the more there are in all: scores against 64 bits, and the level walk's (only
    some chunks wanted) the same bits where it scores at all, with the same chunks selected."""
    import torch
    from paper_2603_08453_amd import binding as lc
    r = np.random.default_rng(chunks + G)
    counts = [chunks if b % 3 != 1 else chunks // 2 + 1 for b in range(B)]
    bounds = [np.concatenate([[0], np.cumsum(r.integers(1, 4, size=m))]).astype(np.int32) for m in counts]
    lens = [int(b[-1]) + 1 for b in bounds]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(chunks)
    K = torch.randn((B, H, max(lens), 128), generator=gen, device="cuda").to(torch.bfloat16)
    q = torch.randn((B, H * G, 128), generator=gen, device="cuda").to(torch.bfloat16)
    budget, got = chunks // 4, {}
    for prune in (lc.LC_PRUNE_NEVER, lc.LC_PRUNE_ALWAYS):
        cfg = lc.lc_config_default(levels=2, fanout=32, kmeans_iters=1, max_chunks=chunks, max_tokens=max(lens), prune=prune,
                                   center_dtype=center_dtype, sink_tokens=5)
        ib = torch.zeros(lc.lc_index_bytes(cfg, B, H), dtype=torch.uint8, device="cuda")
        ws = torch.zeros(lc.lc_workspace_bytes(cfg, B, H * G, H), dtype=torch.uint8, device="cuda")
        idx = lc.lc_build_index(cfg, K, lens, bounds, ib, ws)
        ids = torch.full((B, H, chunks), -7, dtype=torch.int32, device="cuda")
        n = torch.full((B, H), -1, dtype=torch.int32, device="cuda")
        scores = torch.full((B, H, chunks), float("nan"), device="cuda")
        lc.lc_retrieve(idx, q, budget, ids, n, ws, scores=scores)
        got[prune] = scores.cpu().numpy(), ids.cpu().numpy(), n.cpu().numpy()
        if prune == lc.LC_PRUNE_NEVER:
            blob = lc.unpack_blob(lc.lc_index_export(idx))
    flat, walk = got[lc.LC_PRUNE_NEVER], got[lc.LC_PRUNE_ALWAYS]
    qd = q.double().cpu().numpy().reshape(B, H, G, 128)
    for b in range(B):
        m, pinned = counts[b], bounds[b][:-1] < 5
        for h in range(H):
            s = flat[0][b, h, :m]
            assert np.all(np.isneginf(s[pinned]))
            level = blob["seqs"][b]["heads"][h][0]
            mu, rad = level["center"].astype(np.float64), level["radius"].astype(np.float64)
            norm = np.linalg.norm(qd[b, h], axis=1)
            want = ((mu @ qd[b, h].T + rad[:, None] * norm) / np.sqrt(128)).max(axis=1)
            # 128 products and as many roundings of sums that are at most |q| (|mu| + r)
            bound = 132 * 2.0 ** -24 * norm.max() * (np.linalg.norm(mu, axis=1) + rad) / np.sqrt(128)
            assert np.all(np.abs(s - want)[~pinned] <= bound[~pinned]), (b, h)
            w = walk[0][b, h, :m]
            assert np.array_equal(w[~np.isneginf(w)], s[~np.isneginf(w)]), (b, h)
            k = flat[2][b, h]
            assert k == walk[2][b, h] and np.array_equal(flat[1][b, h, :k], walk[1][b, h, :k]), (b, h)
