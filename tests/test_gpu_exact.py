"""Exhaustive search against the oracle's, element by element: every number of queries per
workgroup (1, 2, 4, 8, chosen by the number of queries), row counts around the tile of 128 rows (two
per lane; the last tile is moved back) and the round of 2048 rows (a wavefront's second tile),
dimensions around the chunk of 16 words (16 floats, 64 bytes) and of every alignment, the shortest
and longest result lists."""
import numpy as np
import pytest
import torch

import oracle as og
import workloads as W

pytestmark = pytest.mark.gpu

GEN = {
    og.L2SQ_F32: lambda n, d: W.uniform_f32(n, d, seed=401),
    og.ANGULAR_F32: lambda n, d: W.deep_like_f32(n, d, seed=402, n_comp=3),
    og.L2SQ_U8: lambda n, d: W.sift_like_u8(n, d, seed=403, n_comp=2),
    og.CHI2_F32: lambda n, d: W.gist_like_f32(n, d, seed=404, n_comp=3),
    og.COSINE_F32: lambda n, d: W.scaled_directions_f32(n, d, seed=405, n_comp=3, zero_rows=1),
}


@pytest.mark.parametrize("metric", list(GEN))
@pytest.mark.parametrize("n,d,nq,K", [
    (2, 1, 2, 1), (3, 4, 3, 64), (64, 33, 64, 64), (65, 32, 5, 10), (1023, 31, 40, 64),
    (1025, 36, 257, 10), (2100, 20, 300, 64), (1300, 66, 600, 7), (1090, 13, 1030, 10),
    (5000, 64, 1100, 33), (4097, 128, 1, 64),
    (127, 16, 30, 64), (128, 15, 20, 64), (128, 16, 128, 10), (129, 17, 129, 10), (129, 64, 5, 64),
    (2047, 64, 100, 10), (2048, 60, 300, 33), (2048, 16, 1030, 10), (2049, 65, 40, 64),
    (2049, 64, 600, 10), (2177, 68, 1100, 10),
])
def test_exact_knn_equals_brute_force(metric, n, d, nq, K):
    import paper_2103_15386_amd as amd
    x = GEN[metric](n, d)
    if n > 100:
        x[n // 2:n // 2 + 40] = x[:40]  # equal distances: the id decides
    q = W.sample_nodes(n, nq, seed=3) if nq <= n else np.arange(n, dtype=np.int32)
    ids, dist = amd.exact_knn(torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda(), K, metric)
    ids, dist = ids.cpu().numpy(), dist.cpu().numpy().astype(np.float64)
    k = min(K, n - 1)
    oi, od = og.bruteforce(x, metric, q, k)
    assert (ids[:, :k] == oi).all() and (dist[:, :k] == od).all()
    assert (ids[:, k:] == -1).all()  # ranks beyond the n - 1 other rows
