"""The float32 matrix-core join at the ends of float32's range, where the approximate distances of
its first pass say nothing about the canonical ones: products of two squared norms that overflow,
vanish or lose bits (cosine: the canonical distance divides by the root of that product), sums of
squared norms that overflow, squared norms in the denormal range.  Both forms of the first pass
(16-bit copies, float32 rows) against the oracle after every iteration."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle as og
import workloads as W

pytestmark = pytest.mark.gpu
SEED = W.ALGO_SEED


def _directions(n, d, lengths, seed=861):
    x = W.deep_like_f32(n, d, seed=seed, n_comp=5)
    rng = np.random.default_rng(seed + 1)
    picked = np.asarray(lengths, dtype=np.float64)[rng.integers(0, len(lengths), size=n)]
    with np.errstate(over="ignore", under="ignore"):
        return np.ascontiguousarray((x.astype(np.float64) * picked[:, None]).astype(np.float32))


def _check(x, metric, k, p, iters, short):
    """`short`: a workspace without room for the 16-bit copies."""
    import paper_2103_15386_amd as amd
    from paper_2103_15386_amd.binding import IterStats, make_params
    lib = amd.load_library()
    n, d = x.shape
    xd = torch.from_numpy(x).cuda()
    nbytes = amd.workspace_bytes(n, d, k, p, metric, join_path=amd.JOIN_GRAM) - (1 if short else 0)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    prm = make_params(n, d, k, p, metric, SEED, amd.JOIN_GRAM,
                      torch.cuda.current_stream().cuda_stream, ws)
    ctx = C.c_void_p()
    assert lib.gnnd_create(C.byref(ctx), C.byref(prm), xd.data_ptr()) == 0
    assert lib.gnnd_init_random(ctx) == 0
    g = og.init_random(x, k, metric, SEED)
    ids = torch.empty((n, k), dtype=torch.int32, device="cuda")
    dist = torch.empty((n, k), dtype=torch.float32, device="cuda")
    st = IterStats()
    for it in range(1, iters + 1):
        assert lib.gnnd_iterate(ctx, C.byref(st)) == 0
        ref = og.iterate(x, metric, g, p, SEED, it)
        assert lib.gnnd_get_graph(ctx, ids.data_ptr(), dist.data_ptr(), None) == 0
        torch.cuda.synchronize()
        assert (ids.cpu().numpy() == g.ids).all(), it
        assert (dist.cpu().numpy().astype(np.float64) == g.dist).all(), it
        got = st.as_dict()
        for key in ("inserts", "dist_evals", "proposals"):
            assert got[key] == ref[key], (it, key, got[key], ref[key])
    lib.gnnd_destroy(ctx)


@pytest.mark.parametrize("short", [False, True])
@pytest.mark.parametrize("d", [16, 24, 33, 96])
@pytest.mark.parametrize("lengths", [
    [1e-12], [1e-11], [1e-10], [1e-13, 1e-11], [1e-15], [1e10], [1e12], [1e19],
    [1.0, 1e-12], [1.0, 1e12], [1e-12, 1e12], [3e-10, 3e9, 1.0], [1e-16, 1e5, 1e14],
])
def test_cosine_of_very_short_and_very_long_rows_matches_oracle(lengths, d, short):
    if short and d < 24:
        pytest.skip("no 16-bit copies below 24 dimensions")
    _check(_directions(500, d, lengths), og.COSINE_F32, 16, 16, 3, short)


@pytest.mark.parametrize("short", [False, True])
@pytest.mark.parametrize("d", [16, 40])
@pytest.mark.parametrize("lengths", [[1.2e19], [1.5e19], [1.5e19, 1.0], [1e-14], [1e-16], [1e-18, 1e-14],
                                     [1e-20], [1e-16, 1.0]])
def test_squared_l2_of_very_short_and_very_long_rows_matches_oracle(lengths, d, short):
    if short and d < 24:
        pytest.skip("no 16-bit copies below 24 dimensions")
    _check(_directions(500, d, lengths), og.L2SQ_F32, 16, 16, 3, short)


@pytest.mark.parametrize("short", [False, True])
@pytest.mark.parametrize("d", [16, 40])
@pytest.mark.parametrize("lengths", [[1.0, 1e19], [1.0, 3e19], [1.0, 1e20], [1e-16], [1e-20, 1e-10], [1e-19, 1.0]])
def test_inner_products_of_very_short_and_very_long_rows_match_oracle(lengths, d, short):
    if short and d < 24:
        pytest.skip("no 16-bit copies below 24 dimensions")
    _check(_directions(500, d, lengths), og.ANGULAR_F32, 16, 16, 3, short)


@pytest.mark.parametrize("metric", [og.L2SQ_F32, og.ANGULAR_F32, og.COSINE_F32])
@pytest.mark.parametrize("d", [16, 40])
def test_rows_that_are_not_finite_equal_the_per_pair_join(metric, d):
    import paper_2103_15386_amd as amd
    x = _directions(400, d, [1.0, 3.0])
    x[5:9, 1] = np.inf
    x[20, 3] = -np.inf
    if metric == og.COSINE_F32:  # distance 1; the other metrics define none for such rows
        x[30:33, d - 1] = np.nan
    x[40:42] = 0.0
    xd = torch.from_numpy(x).cuda()
    graphs = []
    for path in (amd.JOIN_GRAM, amd.JOIN_VALU):
        ctx = amd.Gnnd(xd, 16, 16, metric, SEED, path)
        ctx.init_random()
        counts = [[s[f] for f in ("inserts", "dist_evals", "proposals")]
                  for s in (ctx.iterate() for _ in range(3))]
        ids, dist, flags = ctx.graph(with_flags=True)
        graphs.append((ids, dist.view(torch.int32), flags, counts))
        ctx.close()
    assert all(torch.equal(a, b) for a, b in zip(graphs[0][:3], graphs[1][:3]))
    assert graphs[0][3] == graphs[1][3]
