"""Keys that are not a number or infinite.  The direction of a vector whose length is not a number is e_0, like the zero
vector's; an infinite component leaves a direction that compares with nothing, and such a point goes to cluster 0 of its
level whatever its neighbours are.  Every stored index stays inside its array, and no other chunk is affected beyond
what its cluster's mean is."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def setup(chunks, F, levels, iters, bad, H=2, centers=0, geometry=0, room=0, seed=0):
    """GPU index over one sequence of chunks of 1 to 3 tokens, some with a value of `bad` (chunk -> value) among their
    keys in head 0; head 1 has none."""
    import torch
    from paper_2603_08453_amd import binding as lc
    r = np.random.default_rng(seed)
    bounds = np.concatenate([[0], np.cumsum(r.integers(1, 4, size=chunks))]).astype(np.int32)
    T = int(bounds[-1])
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    K = torch.randn((1, H, T + room, 128), generator=g, device="cuda").to(torch.bfloat16)
    for j, value in bad.items():
        K[0, 0, bounds[j + 1] - 1, (37 * j) % 128] = value
    cfg = lc.lc_config_default(levels=levels, fanout=F, kmeans_iters=iters, max_chunks=chunks + room, max_tokens=T + room,
                               center_dtype=centers, geometry=geometry)
    ib = torch.zeros(lc.lc_index_bytes(cfg, 1, H), dtype=torch.uint8, device="cuda")
    ws = torch.full((lc.lc_workspace_bytes(cfg, 1, H, H),), 0xA5, dtype=torch.uint8, device="cuda")
    return lc, lc.lc_build_index(cfg, K, [T], [bounds], ib, ws), K, ws


def head(lc, idx, h=0):
    return lc.unpack_blob(lc.lc_index_export(idx))["seqs"][0]["heads"][h]


def directions(c):
    n2 = (c * c).sum(axis=1)
    e0 = np.eye(1, c.shape[1])
    return np.where((n2 > 0)[:, None], c * (1.0 / np.sqrt(np.where(n2 > 0, n2, 1.0)))[:, None], e0)


def check_labels(lab, x, cent):
    """Nearest centroid among those that compare; cluster 0 where none does."""
    s = x @ cent.T
    none = np.isnan(s).all(axis=1)
    assert np.all(lab[none] == 0)
    s = np.where(np.isnan(s), -np.inf, s)[~none]
    lab = lab[~none]
    assert np.all(s[np.arange(len(s)), lab] >= s.max(axis=1) - 3e-6)
    clear = np.partition(s, -2, axis=1)[:, -2] < s.max(axis=1) - 3e-6 if s.shape[1] > 1 else np.ones(len(s), bool)
    assert np.array_equal(lab[clear], s.argmax(axis=1)[clear])


def check_clustering(chunks, F, bad, centers=0):
    """The first two iterations of the chunk level's clustering."""
    heads = []
    with np.errstate(invalid="ignore"):
        for iters in (1, 2):
            lc, idx, _, _ = setup(chunks, F, 2, iters, bad, centers=centers)
            heads.append(head(lc, idx))
        x = directions(heads[0][0]["center"].astype(np.float64))
        k, lab = len(heads[0][1]["radius"]), heads[0][0]["parent"]
        assert np.isnan(x).any(axis=1).sum() == sum(np.isinf(v) for v in bad.values())
        cent = x[(np.arange(k) * chunks) // k].copy()
        check_labels(lab, x, cent)
        for c in range(k):
            s = x[lab == c].sum(axis=0)
            if s @ s > 0:                                    # (not where it is not a number: the centroid stays)
                cent[c] = s / np.sqrt(s @ s)
        check_labels(heads[1][0]["parent"], x, cent)


NAN, INF = float("nan"), float("inf")
# chunks that start a centroid and chunks that start none, neighbours, the first and the last
SOME = {0: INF, 5: NAN, 6: INF, 33: -INF, 64: -INF, 101: INF, 104: NAN, 199: INF}


@pytest.mark.parametrize("chunks,F,bad", [(200, 8, SOME), (200, 4, {7: INF}), (224, 112, SOME), (3, 2, {0: INF, 1: NAN, 2: INF}),
                                          (3, 1, {0: INF, 1: INF, 2: INF})])
def test_one_kernel_clustering(chunks, F, bad):
    check_clustering(chunks, F, bad)


# centroids in registers (up to 256 of them), then in tiles; every kernel of either kind by the number of points
@pytest.mark.parametrize("chunks,F", [(600, 16), (1100, 8), (1500, 6), (514, 2), (1300, 4), (2200, 4), (5001, 8), (10922, 2)])
def test_tiled_clustering(chunks, F):
    bad = {j: v for j, v in SOME.items() if j < chunks}
    bad.update({chunks // 2 + 3 * i: INF if i % 3 else NAN for i in range(40)})
    bad[chunks - 1] = -INF
    check_clustering(chunks, F, bad)
    check_clustering(chunks, F, {j: -INF for j in range(0, chunks, 2)}, centers=1)


def test_tiled_clustering_without_a_point_that_compares():
    check_clustering(1300, 4, {j: INF for j in range(1300)})


@pytest.mark.parametrize("value", [INF, -INF])
def test_neighbours_candidate_is_no_candidate(value):
    """The last chunk shares its lanes with one finite chunk alone, the one that starts the last centroid (the only
    centroid of the last step): the one similarity there that is a hit must not become the infinite chunk's candidate."""
    check_clustering(514, 2, {513: value})


def check_radii(levels):
    """Every node's radius covers the chunks below it of which the distance compares; none: no radius."""
    with np.errstate(invalid="ignore"):
        c0, r0 = levels[0]["center"].astype(np.float64), levels[0]["radius"].astype(np.float64)
        anc = np.arange(len(r0))
        for l in range(1, len(levels)):
            par = levels[l - 1]["parent"]
            k = len(levels[l]["radius"])
            assert np.all((par >= 0) & (par < k))
            anc = par[anc]
            assert np.array_equal(levels[l]["nchunk"], np.bincount(anc, minlength=k))
            assert np.array_equal(levels[l]["ntok"], np.bincount(anc, weights=levels[0]["ntok"], minlength=k).astype(np.int64))
            reach = np.full(k, -np.inf)
            np.fmax.at(reach, anc, np.linalg.norm(c0 - levels[l]["center"][anc].astype(np.float64), axis=1) + r0)
            got, some = levels[l]["radius"].astype(np.float64), ~np.isneginf(reach)
            assert np.all(np.isneginf(got[~some]))
            assert np.all(got[some] >= reach[some]) and np.all(got[some] <= reach[some] * (1.0 + 3e-5) + 1e-6)


@pytest.mark.parametrize("geometry", [0, 1])
@pytest.mark.parametrize("chunks,F,levels", [(200, 8, 3), (1300, 4, 4), (2275, 16, 4), (4500, 2, 2)])
def test_radii(chunks, F, levels, geometry):
    for value in (NAN, INF):
        lc, idx, _, _ = setup(chunks, F, levels, 3, {j: value for j in (0, 7, 8, 100, chunks - 1)}, geometry=geometry)
        for h in (0, 1):
            check_radii(head(lc, idx, h))


@pytest.mark.parametrize("value", [NAN, INF, -INF])
@pytest.mark.parametrize("chunks,levels", [(3, 2), (40, 3), (600, 3)])
def test_append(chunks, levels, value):
    """An appended chunk that compares with no level-1 node goes to the first one; later ones are grafted as ever."""
    import torch
    lc, idx, K, ws = setup(chunks, 8, levels, 2, {}, room=4)
    V = torch.zeros_like(K)
    before = [head(lc, idx, h) for h in (0, 1)]
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    for i in range(4):
        k = torch.randn((1, 2, 128), generator=g, device="cuda").to(torch.bfloat16)
        if i == 0:
            k[0, 0, 5] = value
        lc.lc_append(idx, K, V, k, k, [1], ws)
    with np.errstate(invalid="ignore"):
        for h in (0, 1):
            got = head(lc, idx, h)
            k1 = len(got[1]["radius"])
            new = got[0]["parent"][chunks:]
            assert np.all((new >= 0) & (new < k1)) and np.array_equal(got[0]["parent"][:chunks], before[h][0]["parent"])
            if h == 0 and np.isinf(value):
                assert new[0] == 0
            added = np.bincount(new, minlength=k1)
            assert np.array_equal(got[1]["nchunk"], before[h][1]["nchunk"] + added)
            calm = added == 0
            for name in ("center", "radius"):
                assert np.array_equal(got[1][name][calm], before[h][1][name][calm])
