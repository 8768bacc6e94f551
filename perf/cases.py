"""The calls this library is timed on.

Every case is one call (or, for Greedy, one K-round run) through the Python
binding, at sizes of the library's own workloads (paper_2101_08763_amd/synth.py,
bench.py) or generic ones.  ``listed()`` names them, ``draw()`` makes more of
the same ranges, ``prepare()`` builds the inputs on the GPU from a seed,
``run()`` makes the call and ``exact()`` is the same value in 64 bits by plain
torch.
"""
from __future__ import annotations

import math

import torch

from paper_2101_08763_amd import api

DTYPES = {"fp32": torch.float32, "fp16": torch.float16, "bf16": torch.bfloat16}
BYTES = {"fp32": 4, "fp16": 2, "bf16": 2}


def _case(call, n, d, l, k, prec, clusters=50, empty=0.0, unit=False, pinned=True):
    return {"call": call, "n": n, "d": d, "l": l, "k": k, "prec": prec, "clusters": clusters,
            "empty": empty, "unit": unit, "pinned": pinned}


def listed():
    cases = {
        # The smallest call: an optimizer step on a toy problem, where launches
        # and host work are all there is.
        "tiny_fp32": _case("eval", 1000, 8, 16, 5, "fp32", clusters=0),
        # A serving loop that may not allocate: a few sets of different sizes
        # against a small 16-bit ground set, through the fixed scratch buffer.
        "serve_bf16": _case("noalloc", 10_000, 64, 48, 8, "bf16", empty=0.25),
        # One optimizer step on a mid-size clustered data set.
        "mix50k_fp32": _case("eval", 50_000, 32, 256, 10, "fp32", clusters=10),
        # The paper's default experiment (Section V-A: n = 50 000, d = 100,
        # l = 5 000, k = 10) in the two precisions it reports.
        "paper_fp32": _case("eval", 50_000, 100, 5000, 10, "fp32", clusters=0),
        "paper_fp16": _case("eval", 50_000, 100, 5000, 10, "fp16", clusters=0),
        # Low-dimensional points (positions on a plane).
        "plane_d2_fp32": _case("eval", 100_000, 2, 1024, 16, "fp32", clusters=0),
        # Nothing is a multiple of anything: odd n, d, l and k, sets of
        # different sizes.
        "ragged_d301_fp32": _case("eval", 30_011, 301, 333, 7, "fp32", empty=0.2),
        # One Greedy step over a candidate list, scored against a solution of
        # 19 points.
        "gain200k_fp32": _case("gain", 200_000, 100, 4096, 19, "fp32"),
        # The whole Greedy optimizer: 16 rounds over every point.
        "greedy_fp32": _case("greedy", 20_000, 100, 0, 16, "fp32"),
        # Text-embedding rows: long unit vectors in bf16.
        "embed_d1536_bf16": _case("eval", 20_000, 1536, 512, 16, "bf16", unit=True),
        # A ground set kept in host memory and streamed through the GPU.
        "streamed_fp16": _case("streamed", 400_000, 128, 256, 16, "fp16"),
        # The largest single-GPU workload: 10^6 points, the bench default.
        "large1m_fp16": _case("eval", 1_000_000, 256, 2048, 32, "fp16", clusters=100),
    }
    return [{"name": name, **c} for name, c in cases.items()]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choices(["eval", "noalloc", "gain", "greedy", "streamed"], [10, 2, 3, 2, 2])[0]
    if call == "greedy":
        n, d, K = _log(rng, 1000, 20_000), _log(rng, 2, 600), rng.randint(2, 16)
        while 2.0 * n * n * d * K > 1.3e12:  # no dearer than the largest listed case
            K, n = max(2, K * 3 // 4), n * 3 // 4
        return _case("greedy", n, d, 0, K, "fp32", clusters=rng.randint(8, 64))
    prec = "fp32" if call == "gain" else rng.choice(["fp32", "fp32", "fp16", "bf16"])
    n, d = _log(rng, 1000, 200_000), _log(rng, 2, 2048)
    l, k = _log(rng, 16, 5000), _log(rng, 1, 48)
    if call == "noalloc":
        n, l = _log(rng, 1000, 50_000), _log(rng, 16, 500)
    if call == "streamed":
        n = min(_log(rng, 20_000, 400_000), 50_000_000 // d)
    cap = (1.2e12 if d <= 512 else 6e11) if prec == "fp32" else 4e12
    per_set = 2.0 * n * d * (1 if call == "gain" else k)
    if call != "gain" and per_set * 16 > cap:  # keep at least a few sets
        k = max(1, int(cap / (16 * 2.0 * n * d)))
        per_set = 2.0 * n * d * k
    l = max(1, min(l, int(cap / per_set)))
    return _case(call, n, d, l, k, prec, clusters=rng.choice([0, 10, 50]),
                 empty=rng.choice([0.0, 0.0, 0.3]) if call != "gain" and k > 1 else 0.0,
                 unit=d >= 512 and rng.random() < 0.5, pinned=rng.random() < 0.7)


def _points(c, g):
    n, d = c["n"], c["d"]
    V = torch.randn(n, d, generator=g, device="cuda")
    if c["clusters"]:
        means = 5.0 * torch.randn(c["clusters"], d, generator=g, device="cuda")
        V += means[torch.randint(0, c["clusters"], (n,), generator=g, device="cuda")]
    if c["unit"]:
        V /= V.norm(dim=1, keepdim=True)
    return V.to(DTYPES[c["prec"]])


def _inputs(c, seed):
    """V, and the index tensors of the call, on the GPU."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    V = _points(c, g)
    n, l, k = c["n"], c["l"], c["k"]
    if c["call"] == "greedy":
        return V, ()
    if c["call"] == "gain":
        perm = torch.randperm(n, generator=g, device="cuda", dtype=torch.int64)[:k + l].to(torch.int32)
        return V, (perm[:k].contiguous(), perm[k:].contiguous())
    sets = torch.randint(0, n, (l, k), generator=g, device="cuda", dtype=torch.int32)
    if c["empty"]:
        blank = torch.rand(l, k, generator=g, device="cuda") < c["empty"]
        blank[:, 0] = False
        sets = torch.where(blank, torch.full_like(sets, -1), sets)
    return V, (sets,)


def prepare(case, seed):
    V, idx = _inputs(case, seed)
    s = {"call": case["call"], "V": V, "idx": idx, "K": case["k"]}
    if case["call"] == "noalloc":
        s["out"] = torch.empty(case["l"], dtype=torch.float32, device="cuda")
    if case["call"] == "streamed":
        host = torch.empty(V.shape, dtype=V.dtype, pin_memory=case["pinned"])
        host.copy_(V)
        s["V"], s["idx"] = host, (idx[0].cpu(),)
    return s


def run(s):
    call, V, idx = s["call"], s["V"], s["idx"]
    if call == "eval":
        return api.exemplar_eval(V, idx[0])
    if call == "noalloc":
        return api.exemplar_eval_noalloc(V, idx[0], s["out"])
    if call == "gain":
        return api.exemplar_gain(V, idx[0], idx[1])
    if call == "greedy":
        return api.exemplar_greedy(V, s["K"])
    return api.exemplar_eval_streamed(V, idx[0])


def work(case):
    n, d, l, k, es = case["n"], case["d"], case["l"], case["k"], BYTES[case["prec"]]
    if case["call"] == "greedy":  # every pair's product once
        return {"bytes": n * d * es + 8 * k, "flops": 2.0 * n * n * d}
    if case["call"] == "gain":  # S against every point once, then the candidates
        return {"bytes": n * d * es + 4 * k + 8 * l, "flops": 2.0 * n * (l + k) * d}
    return {"bytes": n * d * es + 4 * l * k + 4 * l, "flops": 2.0 * n * l * k * d}


def tolerance(case):
    # fp32 results from fp32 sums in every storage type (16-bit products are
    # exact in fp32).  Against 64 bits the results are 2e-8 .. 1.4e-7 off, and
    # 4.5e-7 for unit vectors of 1 536 coordinates, whose dot products nearly
    # cancel the norms; another order of the sums differs by as much again.
    return {"rel": 4e-6, "max": 4e-5, "differ": 0.0}


def _scores(V, sets, n):
    """f of every set in 64 bits: (2/n) sum_v max(0, max_s <v, s> - |s|^2 / 2)."""
    l, k = sets.shape
    out = torch.zeros(l, dtype=torch.float64, device="cuda")
    lb = max(1, min(l, 65_536 // k))
    for j in range(0, l, lb):
        part = sets[j:j + lb].reshape(-1)
        E = V[part.clamp(min=0).long()].double()
        bias = torch.where(part >= 0, -0.5 * (E * E).sum(1), torch.full_like(part, -math.inf, dtype=torch.float64))
        Et = E.t().contiguous()
        rows = max(1, 100_000_000 // Et.shape[1])
        for i in range(0, n, rows):
            H = V[i:i + rows].double() @ Et
            H += bias
            out[j:j + lb] += H.view(H.shape[0], -1, k).amax(2).clamp_(min=0).sum(0)
    return out * (2.0 / n)


def exact(case, seed):
    V, idx = _inputs(case, seed)
    n = case["n"]
    if case["call"] in ("eval", "noalloc", "streamed"):
        f = _scores(V, idx[0], n)
        return f.cpu() if case["call"] == "streamed" else f
    V = V.double()
    half = 0.5 * (V * V).sum(1)
    g = torch.zeros(n, dtype=torch.float64, device="cuda")

    def grow(g, c):
        return torch.maximum(g, V @ V[c] - half[c])

    def score(g, cands):
        out = torch.empty(cands.numel(), dtype=torch.float64, device="cuda")
        step = max(1, 200_000_000 // n)
        for j in range(0, cands.numel(), step):
            c = cands[j:j + step]
            H = V[c] @ V.t().contiguous() - half[c, None]
            out[j:j + step] = torch.maximum(H, g[None, :]).sum(1)
        return out * (2.0 / n)

    if case["call"] == "gain":
        for c in idx[0].tolist():
            g = grow(g, c)
        return score(g, idx[1].long())
    f_out = torch.empty(case["k"], dtype=torch.float64, device="cuda")
    every, free = torch.arange(n, device="cuda"), torch.ones(n, dtype=torch.bool, device="cuda")
    for i in range(case["k"]):
        f = score(g, every).masked_fill(~free, -math.inf)
        c = int(f.argmax())
        f_out[i], free[c] = f[c], False
        g = grow(g, c)
    return None, f_out
