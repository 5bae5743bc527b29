"""Index build against a plain float64 computation, at the sizes where its kernels change or have edges: number of
points and centroids around the tiles of each assignment kernel, clusters listed together, alone, by the whole
workgroup and beyond what a list holds, points with more equally near centroids than a candidate list holds."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def build(H, chunks, F, iters, levels=2, seed=0, same=0, centers=0, spread=1.0, **config):
    """GPU build over `chunks` (chunks per sequence) of 1 to 3 tokens; the first `same` chunks have identical keys."""
    import torch
    from paper_2603_08453_amd import binding as lc
    r = np.random.default_rng(seed)
    bounds = [np.concatenate([[0], np.cumsum(r.integers(1, 4, size=m))]).astype(np.int32) for m in chunks]
    T = max(int(b[-1]) for b in bounds)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    K = torch.randn((len(chunks), H, T, 128), generator=g, device="cuda")
    if spread != 1.0:                                        # clusters of very unequal sizes
        K[..., 0] += spread * torch.randn((len(chunks), H, T), generator=g, device="cuda").abs() ** 3
    K = K.to(torch.bfloat16)
    for b, bd in enumerate(bounds):
        if same:
            K[b, :, : bd[min(same, len(bd) - 1)]] = K[b, :, :1].clone()
    cfg = lc.lc_config_default(levels=levels, fanout=F, kmeans_iters=iters, max_chunks=max(chunks), max_tokens=T,
                               center_dtype=centers, **config)
    ib = torch.zeros(lc.lc_index_bytes(cfg, len(chunks), H), dtype=torch.uint8, device="cuda")
    ws = torch.full((lc.lc_workspace_bytes(cfg, len(chunks), H, H),), 0xA5, dtype=torch.uint8, device="cuda")
    idx = lc.lc_build_index(cfg, K, [int(b[-1]) for b in bounds], bounds, ib, ws)
    return lc.unpack_blob(lc.lc_index_export(idx))["seqs"]


def unit(x):
    return x / np.linalg.norm(x, axis=1, keepdims=True)


def check_labels(lab, x, cent):
    """Nearest centroid by inner product; a label may differ only where the two are equal to rounding."""
    s = x @ cent.T
    best = s.max(axis=1)
    got = s[np.arange(len(x)), lab]
    assert np.all(got >= best - 3e-6)
    clear = np.partition(s, -2, axis=1)[:, -2] < best - 3e-6 if cent.shape[0] > 1 else np.ones(len(x), bool)
    assert np.array_equal(lab[clear], s.argmax(axis=1)[clear])


def check_tree(head):
    """Centers, counts and radii of every level from the chunk level and the parents alone."""
    c0, r0 = head[0]["center"].astype(np.float64), head[0]["radius"].astype(np.float64)
    anc = np.arange(len(r0))
    for l in range(1, len(head)):
        anc = head[l - 1]["parent"][anc]
        k = len(head[l]["radius"])
        n = np.bincount(anc, minlength=k)
        assert np.array_equal(head[l]["nchunk"], n)
        assert np.array_equal(head[l]["ntok"], np.bincount(anc, weights=head[0]["ntok"], minlength=k).astype(np.int64))
        mean = np.zeros((k, 128))
        np.add.at(mean, anc, c0)
        full = n > 0
        mean[full] /= n[full, None]
        assert np.abs(head[l]["center"][full] - mean[full]).max() < 2e-5
        reach = np.full(k, -np.inf)
        np.maximum.at(reach, anc, np.linalg.norm(c0 - head[l]["center"][anc].astype(np.float64), axis=1) + r0)
        assert np.all(np.isneginf(head[l]["radius"][~full]))
        got = head[l]["radius"][full]
        assert np.all(got >= reach[full]) and np.all(got <= reach[full] * (1.0 + 3e-5) + 1e-6)


# points, centroids: one case for each assignment kernel and its remainders (heads and batch decide the wide ones)
SHAPES = [(8, [225], 15), (8, [640, 1], 15), (2, [700, 65], 16), (2, [1000], 11), (1, [1024], 8), (3, [1120], 7),
          (1, [1500], 8), (2, [1281], 5), (8, [4500, 300], 32), (8, [4160], 20), (1, [514], 2), (2, [777, 3], 2),
          (8, [2200, 2100], 4), (8, [5001, 4097], 8), (8, [10922], 2), (8, [4160], 33), (8, [4160], 22), (8, [5300], 20),
          (8, [5300, 700], 17), (4, [2050, 2048], 2),
          (8, [4160, 100], 17), (8, [4224], 16), (2, [2048], 4), (2, [2052], 4)]


@pytest.mark.parametrize("H,chunks,F", SHAPES)
def test_first_two_iterations(H, chunks, F):
    one, two = build(H, chunks, F, 1), build(H, chunks, F, 2)
    for s1, s2 in zip(one, two):
        for h in (0, H - 1):
            x = unit(s1["heads"][h][0]["center"].astype(np.float64))
            N, k = len(x), len(s1["heads"][h][1]["radius"])
            lab = s1["heads"][h][0]["parent"]
            cent = x[(np.arange(k) * N) // k]
            check_labels(lab, x, cent)
            total = np.zeros((k, 128))
            np.add.at(total, lab, x)
            some = np.bincount(lab, minlength=k) > 0
            cent = cent.copy()
            cent[some] = unit(total[some])
            check_labels(s2["heads"][h][0]["parent"], x, cent)
            check_tree(s2["heads"][h])


@pytest.mark.parametrize("centers", [0, 1])
@pytest.mark.parametrize("chunks,F", [([200, 1], 4), ([224], 14), ([16], 16), ([150, 30], 9)])
def test_small_levels_without_iterations(chunks, F, centers):
    """Every chunk in node 0, whose center is their mean; the other nodes keep their starting centroid."""
    for s, n in zip(build(2, chunks, F, 0, centers=centers), chunks):
        for lev in s["heads"]:
            x = lev[0]["center"].astype(np.float64)
            k = len(lev[1]["radius"])
            assert not lev[0]["parent"].any() and lev[1]["nchunk"].tolist() == [n] + [0] * (k - 1)
            assert lev[1]["ntok"][0] == lev[0]["ntok"].sum()
            want = np.concatenate([x.mean(axis=0)[None], unit(x)[(np.arange(1, k) * n) // k]])
            # a sum in float64 rounded once; a direction from a float32 norm of 128 squares
            assert np.abs(lev[1]["center"] - want).max() <= 2.0 ** -20 * np.abs(want).max()


@pytest.mark.parametrize("iters", [2, 4, 8])
@pytest.mark.parametrize("H,chunks,F,level,config", [
    (2, [143, 16, 9], 16, 0, {}), (2, [224, 65, 8], 14, 0, {}), (2, [224, 33, 7], 4, 0, {}), (1, [200], 12, 0, {}), (1, [225], 15, 0, {}), (2, [640, 256, 64], 10, 0, {}), (2, [1281, 1279], 9, 0, {}), (8, [2275], 16, 0, {}), (1, [4096], 17, 0, {}),
    (8, [2100, 1000], 17, 0, {}), (2, [10000, 300], 2, 1, {"levels": 3, "fanouts": [0, 2, 25]}),
    (1, [8320], 2, 1, {"levels": 3, "fanouts": [0, 2, 17]})])
def test_an_iteration_follows_from_the_one_before(H, chunks, F, level, config, iters):
    """Small clusterings in one kernel, up to 16 clusters and beyond; and clusters that are updated one by one from their members'
    bits, those without a change left alone: up to one window of 4096 points and beyond, blocks of 64 points with a
    remainder, batches of unequal sequences."""
    before, after = build(H, chunks, F, iters, **config), build(H, chunks, F, iters + 1, **config)
    checked = 0
    for s1, s2 in zip(before, after):
        for h in (0, H - 1):
            here1, here2 = s1["heads"][h], s2["heads"][h]
            if level and not np.array_equal(here1[0]["parent"], here2[0]["parent"]):
                continue                                    # (the level below is not at rest yet: other points)
            x = unit(here1[level]["center"].astype(np.float64))
            k = len(here1[level + 1]["radius"])
            lab = here1[level]["parent"]
            n = np.bincount(lab, minlength=k)
            if len(x) <= k or not n.all():
                continue
            total = np.zeros((k, 128))
            np.add.at(total, lab, x)
            check_labels(here2[level]["parent"], x, unit(total))
            check_tree(here2)
            checked += s1 is before[0]
    assert checked > 0                                      # (the first sequence, the one of the size that is asked for)


@pytest.mark.parametrize("H,chunks,F,levels,centers,spread", [
    (2, [2275], 16, 4, 0, 1.0), (2, [2275, 0, 17], 16, 4, 1, 1.0), (1, [4097], 3, 3, 0, 1.0), (1, [9000], 2, 4, 0, 1.0),
    (1, [6000], 16, 3, 1, 3.0), (1, [3000], 4, 2, 0, 6.0), (2, [300], 300, 2, 0, 1.0), (1, [5000], 1, 2, 0, 1.0)])
def test_nodes_of_every_level(H, chunks, F, levels, centers, spread):
    for s in build(H, chunks, F, 4, levels=levels, centers=centers, spread=spread):
        if len(s["bounds"]) > 1:
            for head in s["heads"]:
                check_tree(head)


@pytest.mark.parametrize("chunks,F,same", [(800, 8, 500), (1200, 2, 300), (3000, 3, 3000), (2400, 12, 40)])
def test_many_equally_near_centroids(chunks, F, same):
    """Identical chunks start identical centroids: all of them take the lowest one's number."""
    s = build(2, [chunks], F, 1, same=same)[0]
    for head in s["heads"]:
        x = unit(head[0]["center"].astype(np.float64))
        k = len(head[1]["radius"])
        check_labels(head[0]["parent"], x, x[(np.arange(k) * chunks) // k])
        assert np.all(head[0]["parent"][:same] == 0)
        check_tree(head)


@pytest.mark.parametrize("centers", [0, 1])
def test_chunk_lengths_around_a_pooling_batch(centers):
    """Means and radii of chunks just below, at and beyond what the pooling pass holds in registers and on chip."""
    import torch
    from paper_2603_08453_amd import binding as lc
    sizes = [1, 3, 4, 5, 29, 31, 32, 33, 36, 57, 59, 60, 61, 63, 64, 65, 92, 93, 96, 97, 130, 300]
    bounds = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    T = int(bounds[-1])
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    K = torch.randn((1, 2, T, 128), generator=g, device="cuda").to(torch.bfloat16)
    for lo, hi, n in zip(bounds[:-1], bounds[1:], range(len(sizes))):        # the farthest row: another one in every chunk
        K[0, :, lo + (7 * n + (hi - lo) - 1) % (hi - lo)] *= 3
    cfg = lc.lc_config_default(levels=2, fanout=4, kmeans_iters=1, max_chunks=len(sizes), max_tokens=T, center_dtype=centers)
    ib = torch.zeros(lc.lc_index_bytes(cfg, 1, 2), dtype=torch.uint8, device="cuda")
    ws = torch.zeros(lc.lc_workspace_bytes(cfg, 1, 2, 2), dtype=torch.uint8, device="cuda")
    heads = lc.unpack_blob(lc.lc_index_export(lc.lc_build_index(cfg, K, [T], [bounds], ib, ws)))["seqs"][0]["heads"]
    for h in range(2):
        keys = K[0, h].double().cpu().numpy()
        center, radius = heads[h][0]["center"].astype(np.float64), heads[h][0]["radius"]
        for j, (lo, hi) in enumerate(zip(bounds[:-1], bounds[1:])):
            mean = keys[lo:hi].mean(axis=0)
            assert np.abs(center[j] - mean).max() < (4e-3 * max(1.0, np.abs(mean).max()) if centers else 2e-6)
            reach = np.linalg.norm(keys[lo:hi] - center[j], axis=1).max()
            assert reach * (1 - 1e-6) - 1e-6 <= radius[j] <= reach * (1 + 3e-5) + 1e-5


def test_capacity_that_is_not_in_use_costs_a_build_nothing():
    """100 chunks in an index for 100 and in one for 131072: what a build clears does not grow with the capacity (as it did, three times the
    build's time)."""
    import torch
    from paper_2603_08453_amd import binding as lc
    H, chunks = 8, 100
    bounds = [np.arange(chunks + 1, dtype=np.int32) * 12]
    us = {}
    for most in (chunks, 131072):
        cfg = lc.lc_config_default(levels=2, fanout=16, kmeans_iters=1, max_chunks=most, max_tokens=max(most, 1200))
        K = torch.zeros((1, H, cfg.max_tokens, 128), dtype=torch.bfloat16, device="cuda")
        K[:, :, :1200] = torch.randn((1, H, 1200, 128), device="cuda").to(torch.bfloat16)
        ib = torch.zeros(lc.lc_index_bytes(cfg, 1, H), dtype=torch.uint8, device="cuda")
        ws = torch.zeros(lc.lc_workspace_bytes(cfg, 1, H, H), dtype=torch.uint8, device="cuda")
        took = []
        for _ in range(20):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            a.record()
            for _ in range(5):
                lc.lc_build_index(cfg, K, [1200], bounds, ib, ws)
            b.record()
            torch.cuda.synchronize()
            took.append(a.elapsed_time(b) * 200)
        us[most] = min(took)
    assert us[131072] < 1.6 * us[chunks], us


@pytest.mark.parametrize("chunks,F", [([224, 211], 14), ([209, 17, 34], 15), ([64, 65, 48], 8), ([128], 64)])
def test_up_to_16_clusters_of_a_small_level(chunks, F):
    """16 clusters and fewer, each listed by a wavefront: tiles of points and batches of 16 members with remainders."""
    for iters in (2, 3):
        test_an_iteration_follows_from_the_one_before(2, chunks, F, 0, {}, iters)


@pytest.mark.parametrize("chunks", [[224, 1, 0, 17], [2]])
@pytest.mark.parametrize("iters", [1, 10])
def test_one_cluster(chunks, iters):
    """Its centroid is the direction of the sum of all directions: a float32 sum of n unit vectors (n 2^-24 of their lengths together at
    most) over its length, which random keys leave at sqrt(n) at least."""
    for s, n in zip(build(2, chunks, 224, iters, geometry=1), chunks):
        for head in s["heads"] if n else []:
            x = unit(head[0]["center"].astype(np.float64))
            assert not head[0]["parent"].any() and head[1]["nchunk"].tolist() == [n]
            total = x.sum(axis=0)
            assert np.abs(head[1]["center"][0] - unit(total[None])[0]).max() <= (n + 8) * n * 2.0 ** -24 / np.linalg.norm(total)
