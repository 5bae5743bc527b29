"""The calls that a program built on this library makes, at the sizes it makes them.

A case is one operation of the decode path's public entry points (paper_2603_08453_amd.binding):

  step       lc_decode_step, launched as it is: one layer's retrieval + attention for one token
  layers     the same for several layers, each with its own caches and index, replayed from one HIP
             graph (how a serving loop runs the layers of a model)
  separate   lc_retrieve, then lc_sparse_decode on its chunk list
  prefill    lc_build_index over a prompt's key cache, then the first decode step
  stream     a short generation: index build, then lc_append + lc_decode_step per token, chunks
             closing on the way
  recluster  lc_recluster, then lc_index_drift of every level above the chunks
  checkpoint lc_index_export, then lc_index_import of the blob into a second buffer and a decode step on it
  chunk      lc_chunk_tokens on a prompt's token texts (host)

Keys, values and queries follow the repository's synthetic workloads: keys are unit noise around a
per-chunk offset of standard deviation 0.5, queries lean towards three chunks, values are unit
noise, all bfloat16; chunk lengths are uniform in a range or log-normal (median 48).
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2603_08453_amd import binding as lc

D = lc.LC_HEAD_DIM
KMEANS_ITERS = 10


def _case(name, op, **kw):
    c = {"name": name, "op": op, "batch": 1, "q_heads": 32, "kv_heads": 8, "tokens": 32768, "ragged": False,
         "chunk_lo": 16, "chunk_hi": 128, "lognormal": False, "levels": 3, "fanout": 16, "tiers": False,
         "budget": 2048, "policy": "exact", "sink": 0, "centers": "f32", "geometry": "ball",
         "layers": 1, "new_tokens": 0}
    c.update(kw)
    return c


# the headline context: log-normal chunks (median 48), four levels, budget 4096
_LONG = dict(tokens=131072, chunk_lo=8, chunk_hi=256, lognormal=True, levels=4, budget=4096)
# the paper's tiers at that context: chunks of 8 to 16 tokens, two per fine cluster, 22 fine clusters per coarse unit
_TIERS = dict(tokens=131072, chunk_lo=8, chunk_hi=16, tiers=True, budget=1024)
# sixteen sequences of 16K to 64K tokens, group size 7
_RAGGED = dict(batch=16, q_heads=28, kv_heads=4, tokens=65536, ragged=True, chunk_lo=8, fanout=32)


def listed():
    return [
        # one layer, short context: the smallest call, where latency and launches are everything
        _case("step-4K", "step", tokens=4096, chunk_lo=8, chunk_hi=64, levels=2, budget=1024),
        # a small batch at an ordinary context, one layer at a time
        _case("step-32Kx4", "step", batch=4),
        # serving loop at the headline context: eight layers in one graph, every layer's rows cold in the caches
        _case("layers-128K", "layers", layers=8, **_LONG),
        # large ragged batch, chunk centers stored as bfloat16
        _case("step-ragged16", "step", centers="bf16", **_RAGGED),
        # the two separate calls (the caller wants the chunk list) over an index of small chunks
        _case("separate-128K-tiers", "separate", **_TIERS),
        # Algorithm 1's top-k per level over the same index, with the attention sink
        _case("beam-128K-tiers", "step", policy="beam", sink=16, **_TIERS),
        # prefill: index build and first decode step, headline context
        # (top-k per level, so that every level of the index decides what is attended)
        _case("prefill-128K", "prefill", policy="beam", **_LONG),
        # prefill of a large ragged batch
        _case("prefill-ragged16", "prefill", policy="beam", **_RAGGED),
        # a request of 64 generated tokens after a 32K prompt
        _case("stream-32K", "stream", chunk_hi=64, new_tokens=64),
        # drift control during a long generation: every level above the chunks rebuilt, index of small chunks
        _case("recluster-128K-tiers", "recluster", **_TIERS),
        # saving and restoring the index of a prompt (prefix cache)
        _case("checkpoint-32K", "checkpoint", policy="beam"),
        # cutting a prompt into chunks
        _case("chunk-32K", "chunk", chunk_lo=16, chunk_hi=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    op = rng.choice(["step", "step", "step", "layers", "separate", "separate", "prefill", "prefill",
                     "stream", "recluster", "checkpoint", "chunk"])
    if op == "chunk":
        lo = rng.randint(4, 32)
        return _unnamed(op, tokens=_log_int(rng, 1024, 32768), chunk_lo=lo, chunk_hi=lo + rng.randint(8, 96))
    kw = {}
    kw["tokens"] = _log_int(rng, 2048, 131072)
    kw["q_heads"], kw["kv_heads"] = rng.choice([(32, 8), (32, 8), (28, 4), (8, 2), (8, 8), (24, 8), (48, 8)])
    kw["chunk_lo"], kw["chunk_hi"], kw["lognormal"] = rng.choice(
        [(8, 64, False), (16, 128, False), (8, 16, False), (8, 128, False), (8, 256, True)])
    # chunks of the whole batch stay below what the largest listed index holds, and so do the tokens
    mean = _mean_chunk(kw)
    most_tokens = min(16 * 40960 * 4, int(8 * 131072 / 12 * mean)) // (kw["kv_heads"] * kw["tokens"])
    kw["batch"] = min(16, max(1, _log_int(rng, 1, max(1, min(16, most_tokens)))))
    kw["ragged"] = kw["batch"] > 1 and rng.random() < 0.5
    kw["tiers"] = kw["chunk_hi"] <= 16 and rng.random() < 0.5
    kw["levels"] = 3 if kw["tiers"] else rng.choice([2, 3, 4])
    kw["fanout"] = rng.choice([16, 32])
    kw["budget"] = min(_log_int(rng, 256, 4096), kw["tokens"] // 2)
    kw["centers"] = rng.choice(["f32", "f32", "bf16"])
    kw["geometry"] = rng.choice(["ball", "ball", "ball", "unit"])
    if op == "prefill" or (op in ("step", "separate") and rng.random() < 0.3):
        kw["policy"] = "beam"
        kw["sink"] = rng.choice([0, 16])
    if op == "layers":
        kw["layers"] = rng.randint(2, 8)
        kw["batch"] = max(1, kw["batch"] // kw["layers"])
        kw["ragged"] = kw["ragged"] and kw["batch"] > 1
    if op == "checkpoint":
        kw["tokens"] = min(kw["tokens"], 32768)
        kw["batch"], kw["ragged"] = 1, False
        kw["levels"], kw["policy"] = 3, "beam"
        kw["chunk_lo"], kw["chunk_hi"], kw["lognormal"], kw["tiers"] = 16, 128, False, False
    if op == "stream":
        kw["tokens"] = min(kw["tokens"], 49152)
        kw["batch"] = min(kw["batch"], 4)
        kw["budget"] = min(kw["budget"], 2048)
        kw["ragged"] = kw["ragged"] and kw["batch"] > 1
        kw["new_tokens"] = rng.randint(16, 64)
        most = max(work(x)["bytes"] for x in listed() if x["op"] == "stream")
        while kw["new_tokens"] > 4 and work(_unnamed(op, **kw))["bytes"] > most:
            kw["new_tokens"] -= 1
    return _unnamed(op, **kw)


def _unnamed(op, **kw):
    c = _case("", op, **kw)
    del c["name"]
    return c


# ------------------------------------------------------------------ sizes that follow from a case

def _mean_chunk(c):
    return 57.0 if c["lognormal"] else 0.5 * (c["chunk_lo"] + c["chunk_hi"])


def _seq_lens(c):
    """Tokens per sequence: all alike, or spread evenly from a quarter of `tokens` to `tokens`."""
    B, T = c["batch"], c["tokens"]
    if not c["ragged"]:
        return [T] * B
    return [max(64, T // 4 + (T - T // 4) * ((7 * b) % B + 1) // B - 3 * b) for b in range(B)]


def _fanouts(c):
    return {"fanouts": [0, 2, 22]} if c["tiers"] else {}


def _beam(c):
    return [0, 43, 8] if c["tiers"] else [0, 16] + [4] * (c["levels"] - 2)


def _level_sizes(c, chunks):
    n = [chunks]
    for l in range(1, c["levels"]):
        f = (2 if l == 1 else 22) if c["tiers"] else c["fanout"]
        n.append(max(1, -(-n[-1] // f)))
    return n


# ------------------------------------------------------------------ inputs

def _chunk_bounds(c, T, rng):
    """Ascending boundaries from 0 to T.  The number of chunks follows from T and the mean length; the drawn
    lengths are moved by ones, within their range, until they add up to T."""
    lo, hi = c["chunk_lo"], c["chunk_hi"]
    M = max(1, int(T / _mean_chunk(c)))
    if c["lognormal"]:
        lens = np.clip(np.rint(np.exp(rng.normal(math.log(48.0), 0.6, size=M))), lo, hi).astype(np.int64)
    else:
        lens = rng.integers(lo, hi + 1, size=M)
    while (off := int(T - lens.sum())) != 0:
        free = np.flatnonzero(lens < hi if off > 0 else lens > lo)
        if len(free) == 0:
            lens[-1] += off
            break
        lens[rng.permutation(free)[: abs(off)]] += 1 if off > 0 else -1
    return np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)


_VOCAB = ["the", " of", " to", " chunk", " a", " in", " cache", "ing", " key", "s", " is", " value", " that", " for",
          " layer", " x", " =", " 0", "(", "def", " return", ".", ".", ".", ",", ",", ":", ";", "\n", "\n\n", "}", "]",
          "。", "，", " ", "?", "```"]


class _Layer:
    """One attention layer of a request: caches, index, workspace, query and outputs."""

    def __init__(self, c, rng, gen):
        dev = torch.device("cuda:0")
        B, H, Hq = c["batch"], c["kv_heads"], c["q_heads"]
        new = c["new_tokens"]
        self.lens = _seq_lens(c)
        self.bounds = [_chunk_bounds(c, T, rng) for T in self.lens]
        most = max(len(b) - 1 for b in self.bounds)
        self.close = np.zeros((new, B), dtype=np.uint8)
        for b in range(B):                                   # chunks of 16 to 64 streamed tokens
            at = int(rng.integers(4, 64))
            while at < new:
                self.close[at, b] = 1
                at += int(rng.integers(16, 65))
        self.cfg = lc.lc_config_default(
            levels=c["levels"], fanout=c["fanout"], kmeans_iters=KMEANS_ITERS,
            geometry=lc.LC_GEOMETRY_PAPER_UNIT if c["geometry"] == "unit" else lc.LC_GEOMETRY_TOKEN_BALL,
            policy=lc.LC_POLICY_BEAM if c["policy"] == "beam" else lc.LC_POLICY_EXACT,
            beam=_beam(c) if c["policy"] == "beam" else [], sink_tokens=c["sink"],
            max_chunks=most + new + 8, max_tokens=max(self.lens) + new + 8,
            center_dtype=lc.LC_CENTER_BF16 if c["centers"] == "bf16" else lc.LC_CENTER_F32, **_fanouts(c))
        self.budget = c["budget"]
        rows = self.cfg.max_tokens
        self.K = torch.zeros((B, H, rows, D), dtype=torch.bfloat16, device=dev)
        self.V = torch.zeros_like(self.K)
        self.q = torch.empty((B, Hq, D), dtype=torch.bfloat16, device=dev)
        for b, (T, bd) in enumerate(zip(self.lens, self.bounds)):
            M = len(bd) - 1
            off = 0.5 * torch.randn((H, M, D), generator=gen, device=dev)
            of = torch.repeat_interleave(torch.arange(M, device=dev), torch.from_numpy(np.diff(bd)).to(dev))
            for h in range(H):
                self.K[b, h, :T] = torch.randn((T, D), generator=gen, device=dev).add_(off[h][of])
                self.V[b, h, :T] = torch.randn((T, D), generator=gen, device=dev)
            pick = torch.from_numpy(np.stack([rng.integers(0, M, size=3) for _ in range(H)])).to(dev)
            lean = torch.stack([off[h][pick[h]].sum(dim=0) for h in range(H)])
            self.q[b] = torch.randn((Hq, D), generator=gen, device=dev) + lean.repeat_interleave(Hq // H, dim=0)
        self.ib = torch.zeros(lc.lc_index_bytes(self.cfg, B, H), dtype=torch.uint8, device=dev)
        self.ws = torch.zeros(lc.lc_workspace_bytes(self.cfg, B, Hq, H), dtype=torch.uint8, device=dev)
        self.out = torch.zeros((B, Hq, D), dtype=torch.float32, device=dev)
        self.lse = torch.zeros((B, Hq), dtype=torch.float32, device=dev)

    def build(self):
        self.idx = lc.lc_build_index(self.cfg, self.K, self.lens, self.bounds, self.ib, self.ws)

    def step(self):
        lc.lc_decode_step(self.idx, self.q, self.K, self.V, self.budget, self.out, self.ws, lse=self.lse)


def prepare(case, seed):
    c = dict(case)
    rng = np.random.Generator(np.random.PCG64([int(seed), 11]))
    if c["op"] == "chunk":
        texts = [_VOCAB[i] for i in rng.integers(0, len(_VOCAB), size=c["tokens"])]
        return {"case": c, "texts": texts, "bounds": np.zeros(c["tokens"] + 1, dtype=np.int32)}
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(int(seed))
    s = {"case": c, "layers": [_Layer(c, rng, gen) for _ in range(c["layers"])]}
    y = s["layers"][0]
    dev = y.K.device
    B, H, Hq = c["batch"], c["kv_heads"], c["q_heads"]
    if c["op"] in ("step", "layers", "separate", "recluster", "checkpoint"):
        for z in s["layers"]:
            z.build()
    if c["op"] == "separate":
        cap = min(y.cfg.max_chunks, y.budget + c["sink"])
        s["ids"] = torch.zeros((B, H, cap), dtype=torch.int32, device=dev)
        s["counts"] = torch.zeros((B, H), dtype=torch.int32, device=dev)
    if c["op"] == "stream":
        n = c["new_tokens"]
        s["all_outs"] = torch.zeros((n, B, Hq, D), dtype=torch.float32, device=dev)
        s["outs"] = list(s["all_outs"])
        s["k_new"] = list(torch.randn((n, B, H, D), generator=gen, device=dev).to(torch.bfloat16))
        s["v_new"] = list(torch.randn((n, B, H, D), generator=gen, device=dev).to(torch.bfloat16))
        s["qs"] = list(torch.randn((n, B, Hq, D), generator=gen, device=dev).add_(0.5 * y.q.float()).to(torch.bfloat16))
        s["close"] = [[int(x) for x in row] for row in y.close]
    if c["op"] == "checkpoint":
        s["ib2"] = torch.zeros_like(y.ib)
    if c["op"] == "layers":
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            for z in s["layers"]:
                z.step()
            side.synchronize()
            s["graph"] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(s["graph"], stream=side):
                for z in s["layers"]:
                    z.step()
        torch.cuda.current_stream().wait_stream(side)
    return s


def run(s):
    c = s["case"]
    op = c["op"]
    if op == "chunk":
        bounds = lc.lc_chunk_tokens(s["texts"], c["chunk_lo"], c["chunk_hi"])
        s["bounds"][: len(bounds)] = bounds                  # (as many as there are, zeros behind them)
        return s["bounds"]
    y = s["layers"][0]
    if op == "step":
        y.step()
        return [y.out, y.lse]
    if op == "layers":
        s["graph"].replay()
        return [[z.out, z.lse] for z in s["layers"]]
    if op == "separate":
        lc.lc_retrieve(y.idx, y.q, y.budget, s["ids"], s["counts"], y.ws)
        lc.lc_sparse_decode(y.idx, y.q, y.K, y.V, s["ids"], s["counts"], y.out, y.ws, lse=y.lse)
        return [s["ids"], s["counts"], y.out, y.lse]
    if op == "prefill":
        y.build()
        y.step()
        return [y.out, y.lse]
    if op == "stream":
        y.build()
        for t in range(c["new_tokens"]):
            lc.lc_append(y.idx, y.K, y.V, s["k_new"][t], s["v_new"][t], s["close"][t], y.ws)
            lc.lc_decode_step(y.idx, s["qs"][t], y.K, y.V, y.budget, s["outs"][t], y.ws)
        return [s["all_outs"], y.K, y.V]
    if op == "recluster":
        lc.lc_recluster(y.idx, y.ws)
        return [lc.lc_index_drift(y.idx, l, y.ws) for l in range(1, c["levels"])]
    if op == "checkpoint":
        blob = lc.lc_index_export(y.idx)
        s["idx2"] = lc.lc_index_import(y.cfg, blob, s["ib2"])
        lc.lc_decode_step(s["idx2"], y.q, y.K, y.V, y.budget, y.out, y.ws, lse=y.lse)
        return [np.frombuffer(blob, dtype=np.float32), y.out, y.lse]
    raise ValueError(op)


# ------------------------------------------------------------------ what a pass cannot do without

def work(case):
    c = case
    op = c["op"]
    if op == "chunk":
        return {"bytes": 5.0 * c["tokens"], "flops": 4.0 * c["tokens"]}
    B, H, Hq = c["batch"], c["kv_heads"], c["q_heads"]
    lens = _seq_lens(c)
    chunks = [max(1, int(T / _mean_chunk(c))) for T in lens]
    center = D * (2 if c["centers"] == "bf16" else 4)
    attended = sum(min(T, c["budget"] + c["sink"]) for T in lens) * H
    # scoring: every chunk's center, radius and boundary (top-k per level: the top level, and the children of kept nodes)
    if c["policy"] == "beam":
        beam, nodes = _beam(c), 0
        for m in chunks:
            n = _level_sizes(c, m)
            nodes += n[-1] + sum(min(n[l - 1], beam[l] * max(1, n[l - 1] // n[l])) for l in range(1, c["levels"]))
        nodes *= H
    else:
        nodes = sum(chunks) * H
    step = {"bytes": nodes * (center + 8.0) + attended * 4.0 * D + B * Hq * D * 6.0,
            "flops": (nodes + 2.0 * attended) * (Hq // H) * 2.0 * D}
    # clustering: a fixed point takes at least two assignments
    levels = [_level_sizes(c, m) for m in chunks]
    pairs = H * sum(sum(n[l] * n[l + 1] for l in range(c["levels"] - 1)) for n in levels)
    upper = H * sum(sum(n[1:]) for n in levels)
    cluster = {"bytes": sum(chunks) * H * (center + 4.0) + upper * (4.0 * D + 20.0), "flops": 2.0 * 2.0 * D * pairs}
    build = {"bytes": sum(lens) * H * 2.0 * D + sum(chunks) * H * (center + 16.0) + upper * (4.0 * D + 20.0),
             "flops": cluster["flops"] + 5.0 * D * H * sum(lens)}
    if op in ("step", "separate"):
        return step
    if op == "layers":
        return {k: c["layers"] * v for k, v in step.items()}
    if op == "prefill":
        return {k: build[k] + step[k] for k in step}
    if op == "stream":
        return {k: build[k] + c["new_tokens"] * step[k] for k in step}
    if op == "recluster":
        return cluster
    if op == "checkpoint":                               # the index out to the host and back in
        nodes_out = sum(chunks) * H * (center + 16.0) + upper * (4.0 * D + 16.0)
        return {"bytes": 2.0 * nodes_out + step["bytes"], "flops": step["flops"]}
    raise ValueError(op)


def tolerance(case):
    if case["op"] == "chunk":
        return "exact"
    if case["op"] in ("recluster", "checkpoint"):
        # clusterings: an assignment can fall either way where two centroids are equally near to float32
        # rounding, and moves one point of a cluster then
        return {"rel": 2e-3, "max": 0.5, "differ": 0.005}
    # attention and scores: bfloat16 inputs, float32 sums; chunk ids are whole numbers
    if case["policy"] == "beam":
        return {"rel": 1e-3, "max": 0.05}               # (the clustering decides what is attended)
    return {"rel": 2e-5, "max": 1e-3}
