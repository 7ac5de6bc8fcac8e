"""Data that the 16-bit first pass of the float32 matrix-core join does not suit (distances small
against the rows' norms): nodes are then worked on in the float32 form, at once or after the first
pass has left too many pairs.  Every iteration against the oracle; dimensions that are and are not
multiples of 16 and of 4; builds and a merge."""
import numpy as np
import pytest
import torch

import oracle as og
import workloads as W

pytestmark = pytest.mark.gpu
SEED = W.ALGO_SEED


def _vectors(kind, n, d):
    rng = np.random.default_rng(881)
    x = rng.standard_normal((n, d), dtype=np.float32)
    if kind == "offset10":
        x += np.float32(10)
    elif kind == "offset30":
        x += np.float32(30)
    elif kind == "half":  # every other row far out: nodes of both forms
        x[::2] += np.float32(30)
    elif kind == "clusters":  # tight groups far from each other
        x += (np.float32(30) * rng.standard_normal((6, d), dtype=np.float32))[rng.integers(0, 6, n)]
    elif kind == "cone":  # directions close to each other
        x *= np.float32(0.02)
        x[:, 0] += np.float32(d ** 0.5)
        x /= np.sqrt((x * x).sum(axis=1, keepdims=True, dtype=np.float32))
    elif kind == "copies":  # equal distances en masse
        x = np.ascontiguousarray(np.repeat(x[:n // 40 + 1], 40, axis=0)[:n])
    return np.ascontiguousarray(x)


@pytest.mark.parametrize("kind,metric", [
    ("offset10", og.L2SQ_F32), ("offset30", og.L2SQ_F32), ("half", og.L2SQ_F32),
    ("clusters", og.L2SQ_F32), ("copies", og.L2SQ_F32), ("cone", og.ANGULAR_F32),
    ("cone", og.COSINE_F32), ("offset30", og.COSINE_F32)])
@pytest.mark.parametrize("d", [24, 49, 96])
def test_builds_match_oracle(kind, metric, d):
    import paper_2103_15386_amd as amd
    n, k, p = 900, 32, 32
    x = _vectors(kind, n, d)
    ctx = amd.Gnnd(torch.from_numpy(x).cuda(), k, p, metric, SEED)
    assert ctx.join_path() == amd.JOIN_GRAM
    ctx.init_random()
    g = og.init_random(x, k, metric, SEED)
    for it in range(1, 5):
        st = ctx.iterate()
        ref = og.iterate(x, metric, g, p, SEED, it)
        ids, dist, flags = ctx.graph(with_flags=True)
        assert (ids.cpu().numpy() == g.ids).all(), it
        assert (dist.cpu().numpy().astype(np.float64) == g.dist).all(), it
        assert (flags.cpu().numpy() == g.isnew).all(), it
        for key in ("inserts", "dist_evals", "sum_new", "sum_old", "proposals"):
            assert st[key] == ref[key], (it, key)
        assert st["dropped"] == 0
    ctx.close()


def test_a_merge_matches_oracle():
    import paper_2103_15386_amd as amd
    n, n1, d, k, p = 1300, 600, 49, 32, 32
    x = _vectors("offset30", n, d)
    graphs = []
    for lo, hi in ((0, n1), (n1, n)):
        ids, dist = og.bruteforce(x[lo:hi], og.L2SQ_F32, np.arange(hi - lo), k)
        graphs.append(og.Graph(ids + lo, dist, np.zeros_like(ids, dtype=np.uint8)))
    want, wstats = og.merge(x, n1, k, p, og.L2SQ_F32, SEED, graphs[0], graphs[1], 3)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (
        x[:n1], x[n1:], graphs[0].ids, graphs[0].dist.astype(np.float32), graphs[1].ids,
        graphs[1].dist.astype(np.float32))]
    ids, dist, stats = amd.gnnd_merge(*dev, k, p, og.L2SQ_F32, SEED, 3, want_stats=True)
    assert (ids.cpu().numpy() == want.ids).all()
    assert (dist.cpu().numpy().astype(np.float64) == want.dist).all()
    for a, b in zip(stats, wstats):
        for key in ("inserts", "dist_evals", "proposals"):
            assert a[key] == b[key], (key, a, b)
