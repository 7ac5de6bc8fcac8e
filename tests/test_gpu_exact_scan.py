"""Exhaustive search with a workspace (matrix cores turn rows away) against the oracle and, on data
outside its bounds' range, against the form without one, bit for bit: row counts around the tile of 64,
dimensions around the 64-byte pieces of a copy, query counts around the group of 256 and the slice of
4096, rows and queries without a usable copy, lists that run over."""
import numpy as np
import pytest
import torch

import oracle as og
import workloads as W

pytestmark = pytest.mark.gpu

GEN = {
    og.L2SQ_F32: lambda n, d: W.uniform_f32(n, d, seed=411),
    og.ANGULAR_F32: lambda n, d: W.deep_like_f32(n, d, seed=412, n_comp=5),
    og.L2SQ_U8: lambda n, d: W.sift_like_u8(n, d, seed=413, n_comp=4),
    og.COSINE_F32: lambda n, d: W.scaled_directions_f32(n, d, seed=415, n_comp=5, zero_rows=1),
}


def _both(x, q, K, metric):
    """(ids, distances) of the form with and of the form without a workspace."""
    import paper_2103_15386_amd as amd
    lib = amd.load_library()
    (n, d), nq = x.shape, q.numel()
    need = int(lib.gnnd_exact_knn_workspace_bytes(n, d, metric, nq, K))
    assert need > 0
    with_ws = amd.exact_knn(x, q, K, metric)
    ids, dist = torch.empty_like(with_ws[0]), torch.empty_like(with_ws[1])
    assert lib.gnnd_exact_knn(x.data_ptr(), n, d, metric, q.data_ptr(), nq, K, ids.data_ptr(),
                              dist.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0
    return with_ws, (ids, dist)


@pytest.mark.parametrize("metric", list(GEN))
@pytest.mark.parametrize("n,d,nq,K", [
    (6016, 128, 600, 20), (6017, 97, 700, 1), (6079, 96, 769, 64), (6080, 65, 1023, 10),
    (6081, 64, 1025, 33), (7000, 63, 900, 10), (9000, 33, 1000, 10), (9001, 32, 1000, 20),
    (9000, 31, 1000, 64), (20000, 127, 257, 10), (20001, 76, 256, 64), (40000, 20, 300, 5),
    (20000, 4, 4100, 10), (16400, 128, 3, 32),
])
def test_scan_equals_brute_force(metric, n, d, nq, K):
    x = GEN[metric](n, d)
    x[n // 2:n // 2 + 40] = x[:40]  # equal distances: the id decides
    q = W.sample_nodes(n, nq, seed=3)
    (ids, dist), general = _both(torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda(), K, metric)
    assert torch.equal(ids, general[0]) and torch.equal(dist, general[1])
    some = np.r_[0:min(nq, 40), max(0, nq - 40):nq]
    oi, od = og.bruteforce(x, metric, q[some], K)
    assert (ids.cpu().numpy()[some] == oi).all()
    assert (dist.cpu().numpy().astype(np.float64)[some] == od).all()


def _hard(name, x):
    if name == "offset":
        x += 30
    elif name == "copies":  # more candidates than a list holds
        x[100:3000] = x[0]
    elif name == "lengths":
        x *= torch.exp(8 * torch.randn((len(x), 1), device=x.device,
                                       generator=torch.Generator(x.device).manual_seed(1)))
    elif name == "zeros":
        x[::3] = 0
    elif name == "ends":  # no usable copy: infinite, huge, tiny
        x[7], x[11], x[800], x[1200], x[1300] = float("inf"), 1e30, 1e25, 1e-25, 1e-38
    elif name == "nan":
        x[9, 3] = x[400, 2] = float("nan")
    return x


@pytest.mark.parametrize("metric", [og.L2SQ_F32, og.ANGULAR_F32, og.COSINE_F32])
@pytest.mark.parametrize("name", ["offset", "copies", "lengths", "zeros", "ends", "nan"])
def test_scan_on_data_its_bounds_do_not_suit(metric, name):
    x = _hard(name, torch.from_numpy(W.deep_like_f32(16000, 48, seed=416, n_comp=40)).cuda())
    q = torch.arange(0, 16000, 25, dtype=torch.int32, device="cuda")
    got, want = _both(x, q, 10, metric)
    assert torch.equal(got[0], want[0])
    assert torch.equal(got[1].view(torch.int32), want[1].view(torch.int32))


def _norm_in_parts(v, parts):
    """Squared norm in float32: every part (a list of dimensions) by itself, one fused multiply-add
    per dimension, then the parts' sums in pairs."""
    sums = np.zeros((len(v), len(parts)), np.float32)
    for i in range(len(parts[0])):
        x = v[:, [p[i] for p in parts]].astype(np.float64)
        sums = (x * x + sums).astype(np.float32)
    while sums.shape[1] > 1:
        sums = sums[:, 0::2] + sums[:, 1::2]
    return sums[:, 0]


def _at_the_end_of_the_range(rng):
    """64 dimensions of 11 significant bits (exact as float16) whose squared norm is just above 2^60
    or just not, as it is added up over the lanes of a wavefront or over groups of eight
    dimensions."""
    lanes = [[j] for j in range(64)]
    groups = [[c * 32 + g * 8 + e for c in range(2) for e in range(8)] for g in range(4)]
    while True:
        a = 2048 + rng.integers(-150, 150, 64)
        a = np.where(a > 2048, a & ~1, a)
        for j in np.nonzero(a < 2000)[0]:
            a[j] += np.clip(-((a * a).sum() - (1 << 28)) // (2 * a[j]), -40, 40)
        low = np.nonzero(a < 2046)[0]
        off = (a * a).sum() - (1 << 28)  # one up and one down moves it by twice their difference
        pairs = np.argwhere(2 * (a[low][:, None] - a[low][None, :]) + 2 + off == rng.integers(1, 32))
        if len(pairs) == 0 or pairs[0][0] == pairs[0][1]:
            continue
        a[low[pairs[0][0]]] += 1
        a[low[pairs[0][1]]] -= 1
        v = (a * 65536.0).astype(np.float32)[None]
        if _norm_in_parts(v, lanes)[0] > 2.0 ** 60 >= _norm_in_parts(v, groups)[0]:
            return v[0]


@pytest.mark.parametrize("seed", [1, 2, 3, 4])
def test_scan_query_at_the_end_of_the_range(seed):
    """A query whose squared norm is in the bounds' range or not as it is summed, all others a
    thousand times shorter: either it takes part and its length counts, or it does not.  Ten rows
    lie a little nearer to it than two hundred others, but their copies are rounded the other way,
    by all of their length."""
    rng = np.random.default_rng(seed)
    far = _at_the_end_of_the_range(rng)
    x = rng.standard_normal((16000, 64)).astype(np.float32)
    x *= 2.0 ** 19.5 / np.linalg.norm(x, axis=1, keepdims=True)
    ulp = np.where(far < 2.0 ** 27, 65536.0, 131072.0).astype(np.float32)
    x[400] = far
    x[1001:1200] = far - (0.45 + 0.01 * rng.random((199, 1), np.float32)) * ulp
    x[3001:3011] = far + (0.40 + 0.01 * rng.random((10, 1), np.float32)) * ulp
    q = torch.arange(0, 16000, 25, dtype=torch.int32, device="cuda")
    q[40:48] = q[60:68]  # (the rows around it are no queries: it is the only long one)
    got, want = _both(torch.from_numpy(x).cuda(), q, 10, og.L2SQ_F32)
    assert sorted(want[0][16].tolist()) == list(range(3001, 3011))
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


@pytest.mark.parametrize("metric,n,d,nq,K,by_class", [
    (og.L2SQ_F32, 20000, 20, 4096, 64, False), (og.L2SQ_U8, 20000, 96, 4096, 64, False),
    (og.ANGULAR_F32, 40000, 33, 5000, 64, False), (og.COSINE_F32, 17000, 8, 4097, 50, False),
    (og.L2SQ_F32, 60000, 48, 600, 10, True), (og.L2SQ_U8, 60000, 96, 600, 32, True),
])
def test_scan_leaves_no_query_over(metric, n, d, nq, K, by_class):
    """Many candidates per workgroup (thousands of queries, large K; rows in the order of their
    components, queries side by side): only a query's own list is a limit."""
    import paper_2103_15386_amd as amd
    lib = amd.load_library()
    x = W.uniform_f32(n, d, seed=421)
    if by_class:
        x = np.repeat(W.uniform_f32(n // 1000, d, seed=422), 1000, 0) + 0.2 * x
    if metric == og.L2SQ_U8:
        x = (x * 200).astype(np.uint8)
    x = torch.from_numpy(x).cuda()
    q = torch.arange(nq, dtype=torch.int32, device="cuda")
    _, want = _both(x, q, K, metric)
    ws = torch.empty(int(lib.gnnd_exact_knn_workspace_bytes(n, d, metric, nq, K)),
                     dtype=torch.uint8, device="cuda")
    ids, dist = torch.empty_like(want[0]), torch.empty_like(want[1])
    assert lib.gnnd_exact_knn_ws(x.data_ptr(), n, d, metric, q.data_ptr(), nq, K, ids.data_ptr(),
                                 dist.data_ptr(), ws.data_ptr(), ws.numel(),
                                 torch.cuda.current_stream().cuda_stream) == 0
    assert torch.equal(ids, want[0]) and torch.equal(dist, want[1])
    assert int((ws[:nq] != 0).sum()) == 0  # (the workspace begins with a byte per query)


def test_scan_takes_what_it_is_faster_for():
    """Sizes at which either form was clearly the faster one."""
    import paper_2103_15386_amd as amd
    need = amd.load_library().gnnd_exact_knn_workspace_bytes
    for n, d, metric, nq, K in [(14914, 4, og.L2SQ_F32, 1000, 1), (10325, 20, og.L2SQ_F32, 1000, 1),
                                (6711, 48, og.L2SQ_U8, 1000, 1), (26215, 48, og.L2SQ_U8, 16, 5),
                                (6000, 96, og.L2SQ_U8, 1000, 1), (13108, 128, og.L2SQ_U8, 16, 10),
                                (3000, 96, og.L2SQ_F32, 2000, 10)]:
        assert need(n, d, metric, nq, K) == 0
    for n, d, metric, nq, K in [(14914, 4, og.L2SQ_F32, 1000, 64), (10325, 20, og.L2SQ_F32, 1000, 64),
                                (6000, 96, og.L2SQ_U8, 1000, 64), (24577, 96, og.L2SQ_F32, 16, 1),
                                (10**6, 96, og.ANGULAR_F32, 16, 10), (10**6, 96, og.L2SQ_U8, 2000, 64)]:
        assert need(n, d, metric, nq, K) > 0


def test_scan_query_ids():
    x = torch.from_numpy(W.uniform_f32(16000, 48, seed=417)).cuda()
    q = torch.arange(0, 16000, 25, dtype=torch.int32, device="cuda")
    q[5], q[6], q[7], q[8] = -1, 16000, 15999, 15999
    got, want = _both(x, q, 64, og.L2SQ_F32)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    assert (got[0][5] == -1).all() and torch.equal(got[0][7], got[0][8])
    x[15998, 47] = float("nan")  # (its order among the others is the general form's to decide)
    got, want = _both(x, q, 64, og.L2SQ_F32)
    assert torch.equal(got[0], want[0]) and (got[0][5:7] == -1).all()
    assert torch.equal(got[1].view(torch.int32), want[1].view(torch.int32))


def test_scan_under_capture():
    x = torch.from_numpy(W.uniform_f32(16000, 48, seed=418)).cuda()
    q = torch.arange(0, 16000, 25, dtype=torch.int32, device="cuda")
    import paper_2103_15386_amd as amd
    want = amd.exact_knn(x, q, 10)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ids, dist = amd.exact_knn(x, q, 10)
    for _ in range(3):
        ids.fill_(-7)
        graph.replay()
        again = amd.exact_knn(x, q, 10)
        torch.cuda.synchronize()
        assert torch.equal(ids, want[0]) and torch.equal(dist, want[1])
        assert torch.equal(again[0], want[0])
