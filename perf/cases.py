"""Work that a user of this package has it do, as timed cases: graph builds of every size and
kind of vector, the call that allocates nothing, incremental construction, the merge, the
out-of-core build and the exact search, each through its public entry point.

Vectors are synthetic with the shapes the package's own configurations use: SIFT-shaped
(mixture, integers 0..255, as float32 or uint8), GIST-shaped (small non-negative, L1
normalised), DEEP-shaped (unit length, angular distance), directions of very different lengths
(cosine distance), histograms (chi-square distance) and uniform ones.
"""
from __future__ import annotations

import torch

import paper_2103_15386_amd as amd

DEV = "cuda:0"
ALGO_SEED = 42

METRIC = {"sift": amd.L2SQ_F32, "u8": amd.L2SQ_U8, "gist": amd.L2SQ_F32, "deep": amd.ANGULAR_F32,
          "lengths": amd.COSINE_F32, "hist": amd.CHI2_F32, "uniform": amd.L2SQ_F32}


def listed():
    return [
        # The smallest call: a 4096-point set built without allocating, where launches and
        # latency count (serving loops, captured graphs).  The package's small configuration.
        {"name": "static_uniform_4k_d16", "kind": "static", "data": "uniform", "n": 4096, "d": 16,
         "k": 10, "p": 8, "iters": 8},
        # A small collection of ragged size from vectors to graph in one call, context and
        # workspace made inside it; lists of 64.
        {"name": "fresh_sift_30k_d100_k64", "kind": "fresh", "data": "sift", "n": 30011, "d": 100,
         "k": 64, "p": 32, "iters": 5, "segmented": False},
        # The package's benchmark: a million SIFT-shaped vectors, k = p = 32, seven iterations
        # (Recall@10 0.95), the context kept by the program.
        {"name": "held_sift_1m_d128_k32", "kind": "held", "data": "sift", "n": 1_000_000, "d": 128,
         "k": 32, "p": 32, "iters": 7, "segmented": False},
        # Byte vectors with long lists (two entries per lane), as high-recall graphs have them.
        {"name": "held_u8_200k_d96_k96", "kind": "held", "data": "u8", "n": 200_000, "d": 96,
         "k": 96, "p": 32, "iters": 4, "segmented": False},
        # GIST-shaped global descriptors: very long float vectors.
        {"name": "held_gist_150k_d960_k32", "kind": "held", "data": "gist", "n": 150_000, "d": 960,
         "k": 32, "p": 32, "iters": 12, "segmented": False},
        # DEEP-shaped unit vectors, angular distance, more nodes than 2^20.
        {"name": "held_deep_1m5_d96_k32", "kind": "held", "data": "deep", "n": 1_500_000, "d": 96,
         "k": 32, "p": 32, "iters": 12, "segmented": False},
        # Raw embeddings of any length under the cosine distance; odd dimension, odd n.
        {"name": "fresh_cosine_100k_d75_k20", "kind": "fresh", "data": "lengths", "n": 99_991,
         "d": 75, "k": 20, "p": 12, "iters": 8, "segmented": False},
        # A large sample number (the paper varies p up to 42) on lists of 64.
        {"name": "held_sift_100k_p42_k64", "kind": "held", "data": "sift", "n": 100_000, "d": 128,
         "k": 64, "p": 42, "iters": 4, "segmented": False},
        # Histograms under the chi-square distance: the metric without an inner-product form.
        {"name": "held_chi2_100k_d96_k20", "kind": "held", "data": "hist", "n": 100_000, "d": 96,
         "k": 20, "p": 16, "iters": 6, "segmented": False},
        # Incremental construction: a batch of a tenth joins a resident collection.
        {"name": "append_deep_300k_30k_d96", "kind": "append", "data": "deep", "n": 300_000,
         "n2": 30_000, "d": 96, "k": 32, "p": 32, "iters": 6, "build_iters": 8},
        # Out of core: byte vectors in pinned host memory, four shards, every pair merged once
        # (two shards together are more than 2^20 nodes).
        {"name": "sharded_u8_4x600k_d128", "kind": "sharded", "data": "u8", "n": 2_400_000,
         "d": 128, "k": 32, "p": 32, "iters": 4, "build_iters": 8, "shards": 4},
        # Ground truth of the recall evaluation: 2000 nodes against a million, ten neighbours.
        {"name": "exact_deep_1m_d96_q2000", "kind": "exact", "data": "deep", "n": 1_000_000,
         "d": 96, "q": 2000, "k": 10},
    ]


def _log(rng, lo, hi):
    """A whole number from lo..hi, even over its logarithm."""
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


#: Dimensions by kind of vector: lowest, highest.
DIMS = {"sift": (8, 128), "u8": (8, 300), "gist": (64, 960), "deep": (16, 200),
        "lengths": (11, 300), "hist": (7, 200), "uniform": (4, 64)}


def draw(rng):
    kind = rng.choice(["static", "fresh", "held", "held", "fresh", "merge", "append", "sharded",
                       "exact"])
    data = rng.choice(["sift", "sift", "u8", "gist", "deep", "lengths", "hist", "uniform"])
    if kind == "sharded":
        data = rng.choice(["u8", "sift", "deep"])
    d = _log(rng, *DIMS[data])
    if kind == "exact":
        n = _log(rng, 3000, 1_000_000)
        return {"kind": kind, "data": data, "n": n, "q": _log(rng, 100, 2000),
                "d": min(d, 96), "k": rng.choice([1, 5, 10, 10, 32, 64])}
    k = rng.choice([5, 10, 16, 20, 24, 32, 32, 32, 33, 50, 64, 100, 128])
    p = min(k, rng.choice([5, 8, 12, 16, 24, 32, 32, 42, 64]))
    c = {"kind": kind, "data": data, "d": d, "k": k, "p": p, "iters": rng.randint(3, 8)}
    # the largest n of a kind: so many vector elements, and so many pairs, as its listed cases
    most = int(min(60e6 / d, 1.2e9 / (p * p) / max(1, d // 128)))
    if data == "hist" or p > 32:
        most = min(most, 60_000)
    if kind == "static":  # what fits the static scratch
        most = int(50e6 / (8 * k + 130 * p + d + 200))
    if kind == "sharded":
        c["shards"] = rng.choice([2, 3, 4, 5])
        c["build_iters"] = rng.randint(4, 8)
        c["iters"] = rng.randint(2, 4)
        c["k"], c["p"] = min(k, 32), min(p, 32)
        c["n"] = _log(rng, 20_000, max(20_000, min(most, 800_000)))
        return c
    c["n"] = _log(rng, 500, max(500, most))
    if kind in ("fresh", "held"):
        c["segmented"] = k in (64, 128) and rng.random() < 0.4
    if kind in ("merge", "append"):
        c["n2"] = _log(rng, max(200, c["n"] // 20), c["n"])
        c["build_iters"] = rng.randint(4, 8)
    return c


def _vectors(data, n, d, seed):
    g = torch.Generator(device=DEV).manual_seed(1000 + seed)

    def rand(*s):
        return torch.rand(s, generator=g, device=DEV)

    def randn(*s):
        return torch.randn(s, generator=g, device=DEV)

    if data == "uniform":
        return rand(n, d)
    comps = {"sift": 256, "u8": 64, "gist": 128, "deep": 1024, "lengths": 64, "hist": 64}[data]
    comps = max(2, min(comps, n // 50))
    comp = torch.randint(0, comps, (n,), generator=g, device=DEV)
    if data in ("sift", "u8"):
        x = (rand(comps, d) * 128.0)[comp].add_(randn(n, d), alpha=20.0).clamp_(0, 255).round_()
        return x.to(torch.uint8) if data == "u8" else x
    if data in ("gist", "hist"):
        x = randn(comps, d)[comp].add_(randn(n, d), alpha=0.3).abs_()
        return x.div_(x.sum(dim=1, keepdim=True))
    x = randn(comps, d)[comp].add_(randn(n, d), alpha=0.5)
    x.div_(x.norm(dim=1, keepdim=True))
    if data == "lengths":  # lengths from 0.05 to 40
        x.mul_(torch.exp(rand(n, 1) * 6.68 - 3.0))
    return x


def prepare(case, seed):
    c, kind, data = case, case["kind"], case["data"]
    n, d, k, metric = c["n"], c["d"], c["k"], METRIC[data]
    if kind in ("merge", "append"):
        # the collection's graph exists; so does the batch's where two graphs are merged
        x1, x2 = _vectors(data, n, d, 2 * seed), _vectors(data, c["n2"], d, 2 * seed + 1)
        p = min(c["p"], 32)
        ids1, dist1, ctx = amd.gnnd_build(x1, k, p, metric, ALGO_SEED, c["build_iters"])
        s = {"case": c, "x1": x1, "x2": x2, "g1": (ids1, dist1)}
        if kind == "merge":
            ids2, dist2, ctx2 = amd.gnnd_build(x2, k, p, metric, ALGO_SEED, c["build_iters"])
            s["g2"] = (ids2 + n, dist2)
            torch.cuda.synchronize()
            ctx2.close()
        torch.cuda.synchronize()
        ctx.close()
        return s
    x = _vectors(data, n, d, seed)
    s = {"case": c, "x": x}
    if kind == "sharded":
        s["x"] = torch.empty(x.shape, dtype=x.dtype, pin_memory=True)
        s["x"].copy_(x)
    elif kind == "held":
        s["ctx"] = _context(c, x)
    elif kind == "exact":
        g = torch.Generator(device=DEV).manual_seed(77 + seed)
        s["q"] = torch.randperm(n, generator=g, device=DEV)[:c["q"]].sort().values.int()
    return s


def _context(c, x):
    lists = amd.LISTS_SEGMENTED if c.get("segmented") else amd.LISTS_PLAIN
    return amd.Gnnd(x, c["k"], c["p"], METRIC[c["data"]], ALGO_SEED, list_mode=lists)


def run(state):
    c = state["case"]
    kind, k, metric = c["kind"], c["k"], METRIC[c["data"]]
    if kind == "static":
        return amd.gnnd_build_static(state["x"], k, c["p"], metric, ALGO_SEED, c["iters"])
    if kind == "held":
        state["ctx"].build(c["iters"], want_stats=False)
        return state["ctx"].graph()
    if kind == "fresh":
        ctx = _context(c, state["x"])
        ctx.build(c["iters"], want_stats=False)
        return ctx.graph()
    if kind == "merge":
        return amd.gnnd_merge(state["x1"], state["x2"], *state["g1"], *state["g2"], k, c["p"],
                              metric, ALGO_SEED, c["iters"])
    if kind == "append":
        return amd.gnnd_append(state["x1"], *state["g1"], state["x2"], k, c["p"], metric,
                               ALGO_SEED, c["build_iters"], c["iters"])
    if kind == "sharded":
        ids, dist, _ = amd.gnnd_build_sharded(state["x"], c["shards"], k, c["p"], metric,
                                              ALGO_SEED, c["build_iters"], c["iters"])
        return ids, dist
    return amd.exact_knn(state["x"], state["q"], k, metric)


def work(case):
    """Vectors read once, graphs read and written once; two operations per dimension of every
    distance.  A construction evaluates k distances per node for its first graph and about p^2
    per node and iteration (0.3 to 1.8 p^2 on the benchmark, less as lists settle); a merge
    about half of that.  That number depends on the data and is an estimate."""
    c, n, d, k = case, case["n"], case["d"], case["k"]
    elem = 1 if c["data"] == "u8" else 4
    if c["kind"] == "exact":
        return {"bytes": float(n * d * elem + c["q"] * (4 + 8 * k)),
                "flops": 2.0 * c["q"] * n * d}
    pp = c["p"] ** 2
    if c["kind"] in ("merge", "append"):
        m = n + c["n2"]
        evals = m * (k // 2 + c["iters"] * pp / 2)
        graphs = 8 * k * (n + m)
        if c["kind"] == "merge":
            graphs += 8 * k * c["n2"]
        else:
            evals += c["n2"] * (k + c["build_iters"] * pp)
        return {"bytes": float(m * d * elem + graphs), "flops": 2.0 * d * evals}
    if c["kind"] == "sharded":
        # every shard takes part in shards - 1 merges
        evals = n * (k + c["build_iters"] * pp
                     + (c["shards"] - 1) * (k // 2 + c["iters"] * pp / 2))
    else:
        evals = n * (k + c["iters"] * pp)
    return {"bytes": float(n * d * elem + 8 * k * n), "flops": 2.0 * d * evals}


def tolerance(case):
    """Distances are defined to the bit (float32, one fused multiply-add per dimension in
    dimension order; int32 for bytes) and every draw comes from a hash: two runs, and two
    correct implementations, give the same ids and the same distances."""
    return "exact"


def exact(case, seed):
    """Distances of the exact search in 64 bits (its ids may differ at ties).  Which neighbours
    a construction finds is decided step by step by comparisons of float32 distances, and its
    uint8 distances are whole numbers: no 64-bit value exists for those."""
    c = case
    if c["kind"] != "exact" or c["data"] == "u8":
        return None
    if c["data"] == "hist" and 1.0 * c["n"] * c["q"] * c["d"] > 2e10:
        return None
    s = prepare(case, seed)
    x, q, K = s["x"].double(), s["q"].long(), c["k"]
    a = x[q]
    na = (a * a).sum(1, keepdim=True)
    best = None
    step = max(1, int(2e8 / max(1, len(q) * (c["d"] if c["data"] == "hist" else 1))))
    for lo in range(0, c["n"], step):
        b = x[lo:lo + step]
        if c["data"] == "hist":
            u, v = a[:, None, :], b[None, :, :]
            t = u + v
            dist = torch.where(t > 0, (u - v) ** 2 / t, 0.0).sum(2)
        else:
            dot, nb = a @ b.T, (b * b).sum(1)[None, :]
            if METRIC[c["data"]] == amd.L2SQ_F32:
                dist = (na + nb - 2 * dot).clamp_(min=0)
            elif METRIC[c["data"]] == amd.ANGULAR_F32:
                dist = 1 - dot
            else:
                dist = 1 - dot / (na * nb).sqrt()
        own = (q >= lo) & (q < lo + len(b))
        dist[own.nonzero().flatten(), q[own] - lo] = float("inf")
        top = dist if best is None else torch.cat([best, dist], 1)
        best = top.topk(min(K, top.shape[1]), dim=1, largest=False).values
    return None, best.sort(1).values
