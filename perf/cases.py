"""Work that users of this library have it do, as cases that can be timed.

A case is a dict of plain values.  ``prepare`` makes what a program holds
before the call (edge lists in device memory, or graph handles built from
them), ``run`` makes one pass through the public entry points and returns its
outputs in caller ids, ``work`` counts the bytes of the inputs and outputs, and
``exact`` gives the outputs from plain torch where that is quick.

Operations (``op``):

* ``degrees``  clique-degrees of a graph whose handle the program keeps
* ``build``    a handle built from raw pairs, and the vertex degrees (h = 2)
* ``core``     a handle built from raw pairs, and its (k, Psi)-core numbers
* ``app``      CoreApp on a kept handle
* ``peel``     PeelApp on a kept handle
* ``path``     the whole path on raw pairs: build, core numbers, CoreApp, CoreExact
* ``batch``    the core numbers of many small graphs in one call, handles kept

A handle remembers its core decomposition for each h, so ``core`` and ``path``
build a new one in every pass, as a program with a new graph does.

Graphs (``gen``): ``er`` a sparse uniform graph with a planted dense block (the
small graphs that are solved exactly), ``cl`` a Chung-Lu power-law graph with
planted blocks, ``rmat`` a recursive-matrix graph; ``mix`` the batch mixture.
They are the families of ``paper_1906_00341_amd.synth``, drawn on the GPU where
they are large.
"""
import math

import numpy as np
import torch

from paper_1906_00341_amd import dsd, synth


def listed():
    return [
        # one small graph, its handle kept: the shortest call, where latency and launches count
        {"name": "degrees_er2000_h3", "op": "degrees", "gen": "er", "n": 2000, "pairs": 10000, "h": 3},
        # the small graphs that are solved exactly: a new graph, every stage, the edge pattern
        {"name": "path_er2000_h2", "op": "path", "gen": "er", "n": 2000, "pairs": 10000, "h": 2},
        # a new mid-sized power-law graph of an odd size: triangle cores
        {"name": "core_cl30011_h3", "op": "core", "gen": "cl", "n": 30011, "pairs": 297109, "h": 3},
        # PeelApp on a power-law graph whose handle is kept
        {"name": "peel_cl100003_h3", "op": "peel", "gen": "cl", "n": 100003, "pairs": 1000030, "h": 3},
        # the large power-law graph: triangle density, every stage with the exact search
        {"name": "path_cl1000000_h3", "op": "path", "gen": "cl", "n": 1000000, "pairs": 10000000, "h": 3},
        # core numbers for the larger cliques on a skewed graph (many levels, most of them small)
        {"name": "core_rmat16_h5", "op": "core", "gen": "rmat", "n": 1 << 16, "pairs": 16 << 16, "h": 5},
        {"name": "core_rmat18_h4", "op": "core", "gen": "rmat", "n": 1 << 18, "pairs": 16 << 18, "h": 4},
        # the (k_max, Psi)-core alone of a large skewed graph
        {"name": "app_rmat20_h4", "op": "app", "gen": "rmat", "n": 1 << 20, "pairs": 16 << 20, "h": 4},
        # clique-degrees alone: larger cliques on a mid-sized graph, and the largest graph
        {"name": "degrees_rmat18_h5", "op": "degrees", "gen": "rmat", "n": 1 << 18, "pairs": 16 << 18, "h": 5},
        {"name": "degrees_rmat22_h4", "op": "degrees", "gen": "rmat", "n": 1 << 22, "pairs": 16 << 22, "h": 4},
        # loading the largest graph
        {"name": "build_rmat22", "op": "build", "gen": "rmat", "n": 1 << 22, "pairs": 16 << 22, "h": 2},
        # many small graphs at once (h = 2, 3, 4 mixed)
        {"name": "batch_mix1000", "op": "batch", "gen": "mix", "graphs": 1000},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["degrees", "build", "core", "core", "app", "peel", "path", "batch"])
    if op == "batch":
        return {"op": op, "gen": "mix", "graphs": _log_int(rng, 40, 1000)}
    if op == "path":
        if rng.random() < 0.5:
            n = _log_int(rng, 300, 4000)
            return {"op": op, "gen": "er", "n": n, "pairs": int(n * rng.uniform(3, 7)), "h": rng.choice([2, 3])}
        n = _log_int(rng, 100000, 900000)
        return {"op": op, "gen": "cl", "n": n, "pairs": int(n * rng.uniform(6, 10)), "h": 3}
    if op == "build":
        gen, h = rng.choice(["cl", "rmat"]), 2
        n = _log_int(rng, 2000, 1000000) if gen == "cl" else 1 << rng.randint(12, 22)
        return {"op": op, "gen": gen, "n": n, "pairs": int(n * rng.uniform(4, 15)), "h": h}
    if op == "peel":
        n = _log_int(rng, 2000, 100000)
        return {"op": op, "gen": "cl", "n": n, "pairs": int(n * rng.uniform(4, 10)), "h": rng.choice([2, 3])}
    gen = rng.choice(["er", "cl", "rmat"])
    if gen == "er":
        n = _log_int(rng, 300, 20000)
        return {"op": op, "gen": gen, "n": n, "pairs": int(n * rng.uniform(3, 10)), "h": rng.randint(2, 6)}
    if gen == "cl":
        n = _log_int(rng, 2000, 500000)
        return {"op": op, "gen": gen, "n": n, "pairs": int(n * rng.uniform(4, 10)), "h": rng.choice([2, 3, 4])}
    h = rng.choice([3, 4, 4, 5])
    top = {"degrees": {3: 22, 4: 21, 5: 18}, "app": {3: 20, 4: 20, 5: 16}, "core": {3: 18, 4: 17, 5: 15}}[op][h]
    n = 1 << rng.randint(11, top)
    return {"op": op, "gen": gen, "n": n, "pairs": int(n * rng.uniform(6, 16)), "h": h}


# ---------------------------------------------------------------- inputs

PLANTED, PLANT_SIZE, PLANT_P = 5, 200, 0.7     # a Chung-Lu graph's dense blocks
BETA = 2.1                                     # its exponent
RMAT_A, RMAT_B, RMAT_C = 0.57, 0.19, 0.19      # quadrant probabilities


def _pairs_rmat(n, pairs, seed, dev):
    g = torch.Generator(device=dev).manual_seed(seed)
    scale = n.bit_length() - 1
    perm = torch.randperm(n, generator=g, device=dev).to(torch.int32)
    src = torch.empty(pairs, dtype=torch.int32, device=dev)
    dst = torch.empty(pairs, dtype=torch.int32, device=dev)
    for lo in range(0, pairs, 1 << 24):
        k = min(1 << 24, pairs - lo)
        s = torch.zeros(k, dtype=torch.int32, device=dev)
        d = torch.zeros(k, dtype=torch.int32, device=dev)
        for _ in range(scale):
            r = torch.rand(k, generator=g, device=dev)
            s = s * 2 + (r >= RMAT_A + RMAT_B)
            d = d * 2 + (((r >= RMAT_A) & (r < RMAT_A + RMAT_B)) | (r >= RMAT_A + RMAT_B + RMAT_C))
        src[lo:lo + k] = perm[s.long()]
        dst[lo:lo + k] = perm[d.long()]
    return src, dst


def _pairs_cl(n, pairs, seed, dev, beta=BETA, planted=PLANTED):
    g = torch.Generator(device=dev).manual_seed(seed)
    w = torch.arange(1, n + 1, dtype=torch.float64, device=dev) ** (-1.0 / (beta - 1.0))
    w *= 2.0 * pairs / w.sum()
    for _ in range(8):                         # expected degrees of at most sqrt(their sum)
        w = torch.minimum(w, w.sum().sqrt())
        w *= 2.0 * pairs / w.sum()
    cdf = torch.cumsum(w, 0)
    cdf /= cdf[-1].clone()
    perm = torch.randperm(n, generator=g, device=dev).to(torch.int32)
    ends = []
    for _ in range(2):
        u = torch.rand(pairs, generator=g, device=dev, dtype=torch.float64)
        ends.append(perm[torch.searchsorted(cdf, u, right=True).clamp_(max=n - 1)])
    if not planted:
        return ends[0], ends[1]
    size = min(PLANT_SIZE, n // planted)
    blocks = torch.randperm(n, generator=g, device=dev)[:planted * size].to(torch.int32).reshape(planted, size)
    i, j = torch.triu_indices(size, size, 1, device=dev)
    src, dst = [ends[0]], [ends[1]]
    for b in blocks:
        keep = torch.rand(i.numel(), generator=g, device=dev) < PLANT_P
        src.append(b[i[keep]])
        dst.append(b[j[keep]])
    return torch.cat(src), torch.cat(dst)


def _edges(case, seed):
    dev = torch.device("cuda")
    if case["gen"] == "er":
        n, s, d = synth.er_planted(n=case["n"], m=case["pairs"], plant=60, p=0.4, seed=seed)
        return torch.from_numpy(s).to(dev), torch.from_numpy(d).to(dev)
    if case["gen"] == "cl":
        return _pairs_cl(case["n"], case["pairs"], seed, dev)
    return _pairs_rmat(case["n"], case["pairs"], seed, dev)


def _mix(case):
    """(n, pairs, exponent, h) of every graph of the batch mixture; the seed draws the edges only."""
    out = []
    for sp in synth.batch_specs(count=case["graphs"], seed=7):
        avg = min(sp["avg_deg"], sp["n"] - 1)
        out.append((sp["n"], int(round(sp["n"] * avg / 2)), sp["beta"], sp["h"]))
    return out


def prepare(case, seed):
    dev = torch.device("cuda")
    st = {"op": case["op"], "h": case.get("h")}
    if case["op"] == "batch":
        mix = _mix(case)
        sizes = [n for n, _, _, _ in mix]
        st["h"] = [h for _, _, _, h in mix]
        st["graphs"] = []
        for i, (n, pairs, beta, _) in enumerate(mix):
            src, dst = _pairs_cl(n, pairs, seed * 1000003 + i, dev, beta, planted=0)
            st["graphs"].append(dsd.build_csr(n, src, dst))
        st["core"] = torch.zeros(sum(sizes), dtype=torch.uint64, device=dev)
        st["outs"] = list(torch.split(st["core"], sizes))
        return st
    n = case["n"]
    src, dst = _edges(case, seed)
    st["n"] = n
    if case["op"] in ("build", "core", "path"):
        st["src"], st["dst"] = src, dst
    else:
        st["graph"] = dsd.build_csr(n, src, dst)
    if case["op"] in ("degrees", "build", "core", "path"):
        st["out64"] = torch.zeros(n, dtype=torch.uint64, device=dev)
    if case["op"] in ("app", "peel", "path"):
        st["out8"] = torch.zeros(n, dtype=torch.uint8, device=dev)
    if case["op"] == "path":
        st["exact8"] = torch.zeros(n, dtype=torch.uint8, device=dev)
    torch.cuda.synchronize()
    return st


# ---------------------------------------------------------------- one pass

def _i64(t):
    return t.view(torch.int64)


def run(state):
    op, h = state["op"], state["h"]
    if op == "degrees":
        deg, mu = dsd.clique_degrees(state["graph"], h, out=state["out64"])
        return {"deg": _i64(deg), "mu": mu}
    if op == "app":
        member, kmax, density = dsd.core_app(state["graph"], h, out=state["out8"])
        return {"member": member, "kmax": kmax, "density": [density.numerator, density.denominator]}
    if op == "peel":
        member, density, rounds, best = dsd.peel_app(state["graph"], h, out=state["out8"])
        return {"member": member, "density": [density.numerator, density.denominator], "rounds": rounds, "best": best}
    if op == "batch":
        res = dsd.batch_run(state["graphs"], state["h"], "core", outs=state["outs"])
        return {"core": _i64(state["core"]), "kmax": np.array([r["kmax"] for r in res], dtype=np.int64),
                "cliques": np.array([r["num_cliques"] for r in res], dtype=np.int64),
                "status": np.array([r["status"] for r in res], dtype=np.int64)}
    g = dsd.build_csr(state["n"], state["src"], state["dst"])
    try:
        if op == "build":
            deg, m = dsd.clique_degrees(g, 2, out=state["out64"])
            return {"deg": _i64(deg), "m": m}
        core, kmax = dsd.clique_core(g, h, out=state["out64"])
        if op == "core":
            return {"core": _i64(core), "kmax": kmax}
        member, kmax_app, density = dsd.core_app(g, h, out=state["out8"])
        dense, rho = dsd.core_exact(g, h, out=state["exact8"])
        return {"core": _i64(core), "kmax": [kmax, kmax_app], "member": member, "dense": dense,
                "density": [density.numerator, density.denominator, rho.numerator, rho.denominator]}
    finally:
        g.free()


def work(case):
    """Every pair (two 32-bit ids) read once and every per-vertex result written once."""
    if case["op"] == "batch":
        return {"bytes": float(sum(8 * pairs + 8 * n for n, pairs, _, _ in _mix(case))), "flops": 0.0}
    per_vertex = {"degrees": 8, "build": 8, "core": 8, "app": 1, "peel": 1, "path": 10}[case["op"]]
    return {"bytes": float(8 * case["pairs"] + per_vertex * case["n"]), "flops": 0.0}


# ---------------------------------------------------------------- plain results

def exact(case, seed):
    """Degrees from the distinct pairs, triangle-degrees from a dense product
    of 64-bit floats; the sequential decompositions have no quick plain form."""
    small = case["op"] == "degrees" and case["h"] in (2, 3) and case["n"] <= 4096
    if case["op"] != "build" and not small:
        return None
    n = case["n"]
    src, dst = (t.to(torch.int64) for t in _edges(case, seed))
    keep = src != dst
    lo, hi = torch.minimum(src, dst)[keep], torch.maximum(src, dst)[keep]
    key = torch.unique(lo * n + hi)
    a, b = key // n, key % n
    if case["h"] == 2:
        deg = torch.bincount(a, minlength=n) + torch.bincount(b, minlength=n)
        return {"deg": deg, "m" if case["op"] == "build" else "mu": int(key.numel())}
    adj = torch.zeros(n, n, dtype=torch.float64, device=src.device)
    adj[a, b] = 1.0
    adj[b, a] = 1.0
    deg = (((adj @ adj) * adj).sum(1) / 2).round().to(torch.int64)
    return {"deg": deg, "mu": int(deg.sum()) // 3}
