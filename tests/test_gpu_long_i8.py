"""Sample lists of 65..128 objects on byte-valued data, left to the library (GNND_JOIN_AUTO): the
int8 matrix-core form of the long join against the oracle after every iteration.  Dimensions of
one to four steps of 32, lists that fill one to four blocks of 32, more samples than nodes."""
import numpy as np
import pytest
import torch

import oracle as og
import workloads as W

pytestmark = pytest.mark.gpu
SEED = W.ALGO_SEED


@pytest.mark.parametrize("n,d,k,p,metric,iters", [
    (1500, 128, 64, 42, og.L2SQ_F32, 4), (1200, 128, 128, 64, og.L2SQ_U8, 4),
    (900, 32, 40, 33, og.L2SQ_U8, 4), (800, 33, 48, 48, og.L2SQ_U8, 3),
    (700, 65, 70, 64, og.L2SQ_F32, 3), (90, 96, 50, 50, og.L2SQ_U8, 3),
    (600, 1, 64, 36, og.L2SQ_U8, 3),  # one dimension: equal distances everywhere
])
def test_long_lists_on_bytes_match_oracle(n, d, k, p, metric, iters):
    import paper_2103_15386_amd as amd
    x = (W.sift_like_u8 if metric == og.L2SQ_U8 else W.sift_like_f32)(n, d, seed=811, n_comp=4)
    ctx = amd.Gnnd(torch.from_numpy(x).cuda(), k, p, metric, SEED)
    assert ctx.join_path() == amd.JOIN_VALU
    ctx.init_random()
    g = og.init_random(x, k, metric, SEED)
    for it in range(1, iters + 1):
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


@pytest.mark.parametrize("k,p", [(64, 40), (128, 64)])
def test_merge_with_long_lists_on_bytes_matches_oracle(k, p):
    import paper_2103_15386_amd as amd
    n, n1 = 1400, 600
    x = W.sift_like_u8(n, 64, seed=812, n_comp=6)
    graphs = []
    for lo, hi in ((0, n1), (n1, n)):
        ids, dist = og.bruteforce(x[lo:hi], og.L2SQ_U8, np.arange(hi - lo), k)
        graphs.append(og.Graph(ids + lo, dist, np.zeros_like(ids, dtype=np.uint8)))
    want, wstats = og.merge(x, n1, k, p, og.L2SQ_U8, SEED, graphs[0], graphs[1], 3)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (
        x[:n1], x[n1:], graphs[0].ids, graphs[0].dist.astype(np.int32), graphs[1].ids,
        graphs[1].dist.astype(np.int32))]
    ids, dist, stats = amd.gnnd_merge(*dev, k, p, og.L2SQ_U8, SEED, 3, want_stats=True)
    assert (ids.cpu().numpy() == want.ids).all()
    assert (dist.cpu().numpy().astype(np.float64) == want.dist).all()
    for a, b in zip(stats, wstats):
        for key in ("inserts", "dist_evals", "proposals"):
            assert a[key] == b[key], (key, a, b)
