"""The attention kernel's P.V on the matrix cores: token counts around its steps (32 tokens of a wavefront), tiles and splits,
logits that rise and fall along the tokens (the softmax's reference moves late, or never), infinite, large and small values of V,
and tokens whose weight bfloat16 does not hold in three terms."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G", [1, 2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("tokens,splits", [(1, 0), (15, 1), (63, 1), (64, 1), (65, 1), (127, 1), (129, 2), (1025, 1), (2500, 2), (700, 0)])
def test_against_float64(tokens, splits, G):
    import torch
    from paper_2603_08453_amd import binding as lc
    H, T = 2, tokens
    gen = torch.Generator(device="cuda")
    gen.manual_seed(100 * T + G)
    draw = lambda *shape: torch.randn(shape, generator=gen, device="cuda")
    q = draw(1, H * G, 128)
    K, V = draw(1, H, T, 128), draw(1, H, T, 128)
    # head 0's keys lean towards the group's queries by an amount that rises along the tokens, head 1's falls
    lean = torch.linspace(0.0, 1.5, T, device="cuda")
    for h, w in enumerate((lean, lean.flip(0))):
        K[0, h] += w[:, None] * q[0, h * G:(h + 1) * G].sum(dim=0)
    q, K, V = q.to(torch.bfloat16), K.to(torch.bfloat16), V.to(torch.bfloat16)
    bounds = np.unique(np.concatenate([[0], np.arange(7, T, 13), [max(0, T - 3)]])).astype(np.int32)      # (an open tail)
    cfg = lc.lc_config_default(levels=2, fanout=8, kmeans_iters=1, max_chunks=max(1, len(bounds)), max_tokens=T, decode_splits=splits)
    ib = torch.zeros(lc.lc_index_bytes(cfg, 1, H), dtype=torch.uint8, device="cuda")
    ws = torch.zeros(lc.lc_workspace_bytes(cfg, 1, H * G, H), dtype=torch.uint8, device="cuda")
    idx = lc.lc_build_index(cfg, K, [T], [bounds], ib, ws)

    def step(V):
        out = torch.full((1, H * G, 128), float("nan"), device="cuda")
        lse = torch.full((1, H * G), float("nan"), device="cuda")
        lc.lc_decode_step(idx, q, K, V, 10 ** 6, out, ws, lse=lse)
        return out[0].double().cpu(), lse[0].double().cpu()

    out, lse = step(V)
    x = torch.stack([q[0, g].double().cpu() @ K[0, g // G].double().cpu().T for g in range(H * G)]) / 128 ** 0.5
    p = torch.softmax(x, dim=-1)
    v = V[0].double().cpu()
    ref = torch.stack([p[g] @ v[g // G] for g in range(H * G)])
    # a logit is a float32 sum of 128 products: off by at most 2^-24 * 8 of the sum of their sizes (the matrix instruction adds 32 at
    # a time), a probability by that relatively, and V's sum by that of the sum of |p v|, plus the roundings of the sums
    size = torch.stack([q[0, g].double().cpu().abs() @ K[0, g // G].double().cpu().abs().T for g in range(H * G)]) / 128 ** 0.5
    rel = 2.0 * (2.0 ** -21 * size.amax(dim=-1) + 2.0 ** -20)
    bound = rel[:, None] * torch.stack([p[g] @ v[g // G].abs() for g in range(H * G)])
    assert ((out - ref).abs() <= bound).all(), ((out - ref).abs() / bound).max()
    assert ((lse - torch.logsumexp(x, dim=-1)).abs() <= rel + 2.0 ** -22 * lse.abs()).all()

    # infinite values reach their column of the heads that weigh the token, and nothing else
    t = int(p[:, :].sum(dim=0).argmax())
    W = V.clone()
    W[0, :, t, 5], W[0, :, t, 77] = float("inf"), float("-inf")
    got, _ = step(W)
    heavy = p[:, t] > 1e-30
    assert heavy.any()
    assert (got[heavy, 5] == float("inf")).all() and (got[heavy, 77] == float("-inf")).all()
    rest = [c for c in range(128) if c not in (5, 77)]
    assert torch.equal(got[:, rest], out[:, rest])


def _attend(q, K, V, splits):
    """Output and log-sum-exp of a step that attends to every token of one sequence and of the two calls in its place, float64 on the CPU."""
    import torch
    from paper_2603_08453_amd import binding as lc
    H, T = K.shape[1], K.shape[2]
    bounds = np.unique(np.concatenate([[0], np.arange(7, T, 13), [max(0, T - 3)]])).astype(np.int32)      # (an open tail)
    cfg = lc.lc_config_default(levels=2, fanout=8, kmeans_iters=1, max_chunks=max(1, len(bounds)), max_tokens=T, decode_splits=splits)
    ib = torch.zeros(lc.lc_index_bytes(cfg, 1, H), dtype=torch.uint8, device="cuda")
    ws = torch.zeros(lc.lc_workspace_bytes(cfg, 1, q.shape[1], H), dtype=torch.uint8, device="cuda")
    idx = lc.lc_build_index(cfg, K, [T], [bounds], ib, ws)
    out = torch.full((1, q.shape[1], 128), float("nan"), device="cuda")
    lse = torch.full((1, q.shape[1]), float("nan"), device="cuda")
    lc.lc_decode_step(idx, q, K, V, 10 ** 6, out, ws, lse=lse)
    step = (out[0].double().cpu(), lse[0].double().cpu())
    ids = torch.full((1, H, len(bounds)), -7, dtype=torch.int32, device="cuda")
    n = torch.full((1, H), -1, dtype=torch.int32, device="cuda")
    lc.lc_retrieve(idx, q, 10 ** 6, ids, n, ws)
    lc.lc_sparse_decode(idx, q, K, V, ids, n, out.fill_(float("nan")), ws, lse=lse.fill_(float("nan")))
    return step, (out[0].double().cpu(), lse[0].double().cpu())


def _aimed(logits, G):
    """One-hot queries and keys of one KV head: `logits` (base 2) for head 0, 15/16 of it and so on for the next; the logits as they come out."""
    import torch
    q, K = torch.zeros((1, G, 128)), torch.zeros((1, 1, len(logits), 128))
    q[0, :, 0] = 1 - torch.arange(G) / 16
    K[0, 0, :, 0] = torch.as_tensor(logits, dtype=torch.float32) * float(np.log(2.0) * 128 ** 0.5)
    K = K.to(torch.bfloat16)
    x = q[0, :, :1].double() * K[0, 0, :, 0].double() / 128 ** 0.5
    return q.to(torch.bfloat16).cuda(), K.cuda(), x


@pytest.mark.parametrize("G", [1, 4, 7])
@pytest.mark.parametrize("tokens,splits", [(40, 1), (129, 1), (200, 1), (1025, 1), (2500, 2), (700, 0)])
def test_large_and_small_values(tokens, splits, G):
    """Every 64th token weighs some 2^7.5 times the others, late in its lane group's slice: the softmax's reference, set at the first tokens,
    does not move.  A column's largest value sits there alone, up to the largest of bfloat16: the result lies below it."""
    import torch
    T = tokens
    heavy = np.unique(np.concatenate([np.arange(63, T, 64), [T - 1]]))
    logits = np.zeros(T)
    logits[heavy] = 7.5
    q, K, x = _aimed(logits, G)
    p = torch.softmax(x, dim=-1)
    gen = torch.Generator()
    gen.manual_seed(T + G)
    noise = torch.randn((T, 128), generator=gen).clamp(-4, 4)
    noise[heavy] = 0.0
    for scale in (2.0 ** 127, -1.9921875 * 2.0 ** 127, 2.0 ** -110):
        V = noise * (2.0 ** -14 * scale)                            # (a column's other values together stay below the one)
        for c in range(128):
            V[heavy[c % len(heavy)], c] = scale
        V = V.to(torch.bfloat16).cuda()[None, None].contiguous()
        v = V[0, 0].double().cpu()
        # as above; and of values this small a sum is cut off at the last bit of float32's range, at most once per product and
        # term of its probability, divided by a sum of probabilities that are 2^-9 and more where they are largest
        rel = 2.0 * (2.0 ** -21 * x.abs().amax(dim=-1) + 2.0 ** -20)
        bound = rel[:, None] * (p @ v.abs()) + 3 * T * 2.0 ** -149 * 2.0 ** 9
        for out, lse in _attend(q, K, V, splits):
            assert torch.isfinite(out).all()
            assert ((out - p @ v).abs() <= bound).all(), ((out - p @ v).abs() / bound).max()
            assert ((lse - torch.logsumexp(x, dim=-1)).abs() <= rel + 2.0 ** -22 * lse.abs()).all()


@pytest.mark.parametrize("G", [1, 7, 8])
@pytest.mark.parametrize("below", [104, 112, 125, 145, 700])
@pytest.mark.parametrize("tokens,splits,light,heavy", [(3, 1, 2, 0), (40, 1, 0, 39), (200, 1, 13, 199), (200, 1, 199, 0), (1100, 1, 3, 1090), (2500, 2, 10, 2400), (4500, 64, 4400, 10), (700, 0, 650, 5)])
def test_values_of_light_tokens(tokens, splits, light, heavy, below, G):
    """One token weighs 2^-below of the heaviest.  An infinite value of it reaches its column whatever the weight, as it does in float64;
    a finite one is counted to float32's precision as far as the weight has a place in float32's range."""
    import torch
    T = tokens
    gen = torch.Generator()
    gen.manual_seed(T + below + G)
    logits = np.full(T, -3.0)
    logits[heavy], logits[light] = 0.0, -below
    q, K, x = _aimed(logits, G)
    p = torch.softmax(x, dim=-1)
    assert (p[:, light] > 0).all()
    V = torch.randn((T, 128), generator=gen)
    V[:, 9], V[:, 40] = 0.0, 0.0
    V[light, 9], V[light, 40] = 1.7 * 2.0 ** 127, -1.3 * 2.0 ** 100
    V = V.to(torch.bfloat16)
    W = V.clone()
    W[light, 5], W[light, 77] = float("inf"), float("-inf")
    rel = 2.0 * (2.0 ** -21 * x.abs().amax(dim=-1) + 2.0 ** -20)
    for values in (V, W):
        v = values.double()
        ref = p @ v
        # as above; the light token's probability is off by the last bit of float32's range at most (and at most one scaling on its
        # way loses as much again, twice), where the heaviest's is 1
        bound = rel[:, None] * (p @ v.abs()) + 3 * T * 2.0 ** -149 * 2.0 ** 9 + 4 * 2.0 ** -149 * v[light].abs()
        finite = torch.isfinite(v).all(dim=0)
        for out, lse in _attend(q, K, values[None, None].cuda(), splits):
            assert ((out - ref).abs() <= bound)[:, finite].all(), ((out - ref).abs() / bound)[:, finite].max()
            assert torch.equal(out[:, ~finite], ref[:, ~finite])       # infinities of the sign that float64 gives
            assert ((lse - torch.logsumexp(x, dim=-1)).abs() <= rel + 2.0 ** -22 * lse.abs()).all()


@pytest.mark.parametrize("top", [99, 100, 101, 102])
def test_infinite_values_where_three_terms_end(top):
    """Seven of eight tokens weigh 2^-top to 2^-(top + 1) of the eighth, in 200 K different ways: of so many, some have low bits that leave
    nothing for the second term where the bits run out.  All of them are infinite in one column, which is infinite then."""
    import torch
    T, G = 32768, 8
    gen = torch.Generator()
    gen.manual_seed(top)
    unit = float(np.log(2.0) * 128 ** 0.5)                          # of a logit to base 2
    q, K = torch.zeros((1, G, 128)), torch.zeros((1, 1, T, 128))
    q[0, :, :4] = 1.0
    q[0, :, 3] += torch.arange(G) / 16
    K[0, 0, :, 0] = torch.tensor(-(top + 0.5) * unit).to(torch.bfloat16)
    K[0, 0, :, 1] = -(top + 0.5) * unit - K[0, 0, 0, 0]
    K[0, 0, :, 2] = (torch.rand(T, generator=gen) - 0.5) * 0.9 * unit
    K[0, 0, :, 3] = (torch.rand(T, generator=gen) - 0.5) * 0.04 * unit
    K[0, 0, ::8] = 0.0
    K = K.to(torch.bfloat16)
    V = torch.randn((T, 128), generator=gen)
    V[:, 5] = float("inf")
    V[::8, 5] = 0.0
    q = q.to(torch.bfloat16)
    x = q[0, :, :4].double() @ K[0, 0, :, :4].double().T / unit
    light = x[:, torch.arange(T) % 8 != 0]
    assert (light < -top).all() and (light > -top - 1).all()
    for out, lse in _attend(q.cuda(), K.cuda(), V.to(torch.bfloat16)[None, None].cuda(), 4):
        assert (out[:, 5] == float("inf")).all()
        assert torch.isfinite(out[:, 6:]).all() and torch.isfinite(lse).all()
