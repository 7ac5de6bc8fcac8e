"""Sample lists of 65..128 objects on byte-valued data, left to the library (GNND_JOIN_AUTO): the
int8 matrix-core form of the long join against the oracle after every iteration.  Dimensions of
one to four steps of 32, lists that fill one to four blocks of 32, more samples than nodes; enough
nodes that every persistent workgroup (at most nine of three, seven of four wavefronts per CU) works on
four and more, with and without nodes between them that have nothing to do."""
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


def _nodes(d, p, times):
    """`times` nodes and a few more per workgroup of the join (rows of d bytes)."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    waves = 7 if d <= 32 else 5 if d <= 96 else 4
    return cus * (4 * waves // (3 if p <= 48 else 4)) * times + 77


@pytest.mark.parametrize("d,k,p,metric", [
    (20, 40, 40, og.L2SQ_U8), (32, 64, 64, og.L2SQ_F32), (64, 48, 42, og.L2SQ_F32), (50, 64, 60, og.L2SQ_U8),
    (96, 50, 48, og.L2SQ_U8), (128, 64, 42, og.L2SQ_F32), (100, 64, 64, og.L2SQ_U8)])
def test_several_nodes_per_workgroup_match_oracle(d, k, p, metric):
    import paper_2103_15386_amd as amd
    n = _nodes(d, p, 4)
    x = (W.sift_like_u8 if metric == og.L2SQ_U8 else W.sift_like_f32)(n, d, seed=813, n_comp=8)
    ctx = amd.Gnnd(torch.from_numpy(x).cuda(), k, p, metric, SEED)
    assert ctx.join_path() == amd.JOIN_VALU
    ctx.init_random()
    _compare(ctx, x, metric, og.init_random(x, k, metric, SEED), p, 1, 3)


@pytest.mark.parametrize("d,k,p", [(16, 40, 40), (96, 64, 64), (128, 40, 40)])
@pytest.mark.parametrize("share", [0.02, 0.3])
def test_nodes_without_work_between_others_match_oracle(d, k, p, share):
    """A loaded graph in which `share` of the nodes have one NEW entry: the others, unless they stand in
    a NEW place, have OLD samples only, and a workgroup meets both kinds."""
    import paper_2103_15386_amd as amd
    n = _nodes(d, p, 4)
    rng = np.random.default_rng(5)
    x = W.sift_like_u8(n, d, seed=814, n_comp=8)
    g = og.init_random(x, k, og.L2SQ_U8, SEED)
    g.isnew[:] = 0
    rows = np.flatnonzero(rng.random(n) < share)
    g.isnew[rows, rng.integers(0, k, len(rows))] = 1
    ctx = amd.Gnnd(torch.from_numpy(x).cuda(), k, p, og.L2SQ_U8, SEED)
    ctx.set_graph(torch.from_numpy(g.ids).cuda(), torch.from_numpy(g.dist.astype(np.int32)).cuda(),
                  torch.from_numpy(g.isnew).cuda(), 3)
    _compare(ctx, x, og.L2SQ_U8, g, p, 4, 5)


def _compare(ctx, x, metric, g, p, first, last):
    for it in range(first, last + 1):
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


@pytest.mark.parametrize("d,k,p", [(16, 40, 40), (64, 64, 64), (128, 64, 40)])
def test_merge_of_several_nodes_per_workgroup_matches_oracle(d, k, p):
    import paper_2103_15386_amd as amd
    n = _nodes(d, p, 4)
    n1 = n // 3
    x = W.sift_like_u8(n, d, seed=815, n_comp=8)
    graphs = []
    for lo, hi in ((0, n1), (n1, n)):
        ids, dist = og.bruteforce(x[lo:hi], og.L2SQ_U8, np.arange(hi - lo), k)
        graphs.append(og.Graph(ids + lo, dist, np.zeros_like(ids, dtype=np.uint8)))
    want, wstats = og.merge(x, n1, k, p, og.L2SQ_U8, SEED, graphs[0], graphs[1], 2)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (
        x[:n1], x[n1:], graphs[0].ids, graphs[0].dist.astype(np.int32), graphs[1].ids,
        graphs[1].dist.astype(np.int32))]
    ids, dist, stats = amd.gnnd_merge(*dev, k, p, og.L2SQ_U8, SEED, 2, want_stats=True)
    assert (ids.cpu().numpy() == want.ids).all()
    assert (dist.cpu().numpy().astype(np.float64) == want.dist).all()
    for a, b in zip(stats, wstats):
        for key in ("inserts", "dist_evals", "proposals"):
            assert a[key] == b[key], (key, a, b)
