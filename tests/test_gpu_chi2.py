"""The chi-square join sums every pair with the reciprocal instruction and the possible nearest
partners once more in the canonical arithmetic: ties en masse (more pairs than its list holds),
values outside the range of its error bound, single and several chunks of 64 dimensions."""
import numpy as np
import pytest
import torch

import oracle as og
import workloads as W

pytestmark = pytest.mark.gpu
SEED = W.ALGO_SEED


def _vectors(kind, n, d):
    x = W.gist_like_f32(n, d, seed=821, n_comp=4)
    if kind == "copies":  # every vector 20 times
        x = np.ascontiguousarray(np.repeat(x[:n // 20 + 1], 20, axis=0)[:n])
    elif kind == "small":  # squares of differences underflow
        x *= np.float32(1e-20)
    elif kind == "large":  # some squares of differences overflow
        x[::7] *= np.float32(1e21)
    elif kind == "zeros":
        x[x < np.median(x)] = 0.0
        x[:5] = 0.0
    elif kind == "negative":  # the distance skips dimensions with a + b <= 0
        x[3::11, 0] = -0.5
    elif kind == "signed":  # every node leaves the range: hardly one is tried in two passes
        x -= np.float32(x.mean())
    elif kind == "last_negative":  # seen in the last chunk of dimensions only
        x[:, d - 1] = -1.0
    return x


@pytest.mark.parametrize("kind", ["plain", "copies", "small", "large", "zeros", "negative",
                                  "signed", "last_negative"])
@pytest.mark.parametrize("d,k,p", [(64, 32, 32), (65, 20, 16), (130, 24, 20), (3, 10, 8)])
def test_chi2_join_matches_oracle(kind, d, k, p):
    import paper_2103_15386_amd as amd
    x = _vectors(kind, 800, d)
    ctx = amd.Gnnd(torch.from_numpy(x).cuda(), k, p, og.CHI2_F32, SEED)
    ctx.init_random()
    g = og.init_random(x, k, og.CHI2_F32, SEED)
    for it in range(1, 5):
        st = ctx.iterate()
        ref = og.iterate(x, og.CHI2_F32, g, p, SEED, it)
        ids, dist = ctx.graph()
        assert (ids.cpu().numpy() == g.ids).all(), it
        assert (dist.cpu().numpy().astype(np.float64) == g.dist).all(), it
        for key in ("inserts", "dist_evals", "sum_new", "sum_old", "proposals"):
            assert st[key] == ref[key], (it, key, st[key], ref[key])
    ctx.close()
