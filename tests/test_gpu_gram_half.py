"""The 16-bit first pass of the float32 matrix-core join: rows that have no 16-bit copy (norms
too small to divide by, infinite norms), zero rows, elements far below the row's largest, and
workspaces without room for the copies - everything against the oracle or the per-pair join."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle as og
import workloads as W

pytestmark = pytest.mark.gpu
SEED = W.ALGO_SEED


def _vectors(kind, n, d):
    x = W.scaled_directions_f32(n, d, seed=771, n_comp=5, zero_rows=2)
    if kind == "tiny_rows":  # squared norms about 2^-100, two rows with norms that underflow to 0
        x[5:9] *= 1e-15
        x[9:11] = 3e-24
    elif kind == "wide_range":  # single elements far below and far above the others
        x[:, 0] *= 1e4
        x[:, 1] *= 1e-9
    elif kind == "large":
        x *= 1e15
    return x


@pytest.mark.parametrize("metric", [og.L2SQ_F32, og.ANGULAR_F32, og.COSINE_F32])
@pytest.mark.parametrize("kind", ["tiny_rows", "wide_range", "large"])
@pytest.mark.parametrize("d", [24, 33, 96])
def test_rows_that_do_not_fit_16_bits_match_oracle(metric, kind, d):
    import paper_2103_15386_amd as amd
    x = _vectors(kind, 700, d)
    if kind == "large" and metric != og.L2SQ_F32:
        x *= 1e-10  # beyond, 1 - dot is -dot alone, and the cosine's product of norms overflows
    k, p = 20, 20
    ctx = amd.Gnnd(torch.from_numpy(x).cuda(), k, p, metric, SEED, amd.JOIN_GRAM)
    ctx.init_random()
    g = og.init_random(x, k, metric, SEED)
    for it in range(1, 4):
        st = ctx.iterate()
        ref = og.iterate(x, metric, g, p, SEED, it)
        ids, dist = ctx.graph()
        assert (ids.cpu().numpy() == g.ids).all(), it
        assert (dist.cpu().numpy().astype(np.float64) == g.dist).all(), it
        for key in ("inserts", "dist_evals", "proposals"):
            assert st[key] == ref[key], (it, key)
    ctx.close()


def test_infinite_norms_angular_equals_the_per_pair_join():
    import paper_2103_15386_amd as amd
    x = W.scaled_directions_f32(600, 40, seed=772, n_comp=4)
    x[3:6] *= 1e20  # the squared norm overflows, the inner products do not
    xd = torch.from_numpy(x).cuda()
    a = amd.Gnnd(xd, 16, 16, amd.ANGULAR_F32, SEED, amd.JOIN_GRAM)
    b = amd.Gnnd(xd, 16, 16, amd.ANGULAR_F32, SEED, amd.JOIN_VALU)
    for c in (a, b):
        c.build(4, want_stats=False)
    for s, t in zip(a.graph(with_flags=True), b.graph(with_flags=True)):
        assert torch.equal(s, t)
    a.close()
    b.close()


def test_a_workspace_without_room_for_the_copies_still_serves():
    import paper_2103_15386_amd as amd
    from paper_2103_15386_amd.binding import make_params
    lib = amd.load_library()
    x = torch.from_numpy(W.deep_like_f32(1500, 96, seed=773, n_comp=8)).cuda()
    k, p, metric = 16, 16, amd.ANGULAR_F32
    full = amd.workspace_bytes(1500, 96, k, p, metric)
    ref = amd.gnnd_build(x, k, p, metric, SEED, 4)
    copies = 1500 * 96 * 2
    for nbytes in (full - 1, full - (copies & ~255)):
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        prm = make_params(1500, 96, k, p, metric, SEED,
                              stream=torch.cuda.current_stream().cuda_stream, workspace=ws)
        ctx = C.c_void_p()
        assert lib.gnnd_create(C.byref(ctx), C.byref(prm), x.data_ptr()) == 0
        assert lib.gnnd_build(ctx, 4, 0.0, None) == 0
        ids, dist = torch.empty_like(ref[0]), torch.empty_like(ref[1])
        assert lib.gnnd_get_graph(ctx, ids.data_ptr(), dist.data_ptr(), None) == 0
        torch.cuda.synchronize()
        lib.gnnd_destroy(ctx)
        assert torch.equal(ids, ref[0]) and torch.equal(dist, ref[1])
    ref[2].close()
