"""A context created and built inside a captured HIP graph (sample lists beyond 64, float32 vectors:
creating one reads nothing back there, byte-valued or not).  Every replay against the eager result."""
import ctypes as C

import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu
SEED = W.ALGO_SEED


@pytest.mark.parametrize("bytes_valued", [True, False])
def test_create_and_build_under_capture(bytes_valued):
    import paper_2103_15386_amd as amd
    from paper_2103_15386_amd.binding import make_params
    lib = amd.load_library()
    n, d, k, p, iters = 900, 64, 48, 40, 3
    x = (W.sift_like_f32 if bytes_valued else W.uniform_f32)(n, d, seed=891)
    xd = torch.from_numpy(x).cuda()
    want_ids, want_dist, ctx = amd.gnnd_build(xd, k, p, amd.L2SQ_F32, SEED, iters)
    ctx.close()
    ws = torch.empty(amd.workspace_bytes(n, d, k, p, amd.L2SQ_F32), dtype=torch.uint8, device="cuda")
    ids, dist = torch.empty_like(want_ids), torch.empty_like(want_dist)
    side = torch.cuda.Stream()
    handle = C.c_void_p()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        prm = make_params(n, d, k, p, amd.L2SQ_F32, SEED, stream=side.cuda_stream, workspace=ws)
        codes = [lib.gnnd_create(C.byref(handle), C.byref(prm), xd.data_ptr())]
        if codes[0] == 0:
            codes.append(lib.gnnd_build(handle, iters, 0.0, None))
            codes.append(lib.gnnd_get_graph(handle, ids.data_ptr(), dist.data_ptr(), None))
    assert codes == [0, 0, 0]
    for _ in range(3):
        ids.fill_(-7)
        dist.zero_()
        ws.fill_(0xAB)  # nothing may be left over from the replay before
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(ids, want_ids) and torch.equal(dist, want_dist)
        again, again_dist, ctx = amd.gnnd_build(xd, k, p, amd.L2SQ_F32, SEED, iters)
        ctx.close()
        assert torch.equal(again, want_ids) and torch.equal(again_dist, want_dist)
    lib.gnnd_destroy(handle)
