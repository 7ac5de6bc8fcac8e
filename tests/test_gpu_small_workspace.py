"""Workspaces and arenas without room for what only makes a call faster (16-bit rows, int8 rows of the
long join, staged results beyond 2^20 nodes): same graphs, and the Python calls take such a one
where memory is short."""
import ctypes as C

import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu
SEED = W.ALGO_SEED


def _bytes(n, d, seed=0):
    g = torch.Generator(device="cuda").manual_seed(n + seed)
    return torch.randint(0, 256, (n, d), generator=g, device="cuda", dtype=torch.int32).to(torch.uint8)


def _sizes(n, d, k, p, metric):
    import paper_2103_15386_amd as amd
    from paper_2103_15386_amd.binding import make_params
    lib = amd.load_library()
    prm = make_params(n, d, k, p, metric)
    return lib.gnnd_workspace_bytes(C.byref(prm)), lib.gnnd_workspace_bytes_min(C.byref(prm))


def _build(x, k, p, metric, iters, nbytes):
    import paper_2103_15386_amd as amd
    from paper_2103_15386_amd.binding import make_params
    lib = amd.load_library()
    n, d = x.shape
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    prm = make_params(n, d, k, p, metric, SEED, stream=torch.cuda.current_stream().cuda_stream,
                      workspace=ws)
    ctx = C.c_void_p()
    assert lib.gnnd_create(C.byref(ctx), C.byref(prm), x.data_ptr()) == 0
    assert lib.gnnd_build(ctx, iters, 0.0, None) == 0
    ids = torch.empty((n, k), dtype=torch.int32, device="cuda")
    dist = torch.empty((n, k), dtype=torch.int32 if metric == amd.L2SQ_U8 else torch.float32,
                       device="cuda")
    assert lib.gnnd_get_graph(ctx, ids.data_ptr(), dist.data_ptr(), None) == 0
    torch.cuda.synchronize()
    lib.gnnd_destroy(ctx)
    return ids, dist


@pytest.mark.parametrize("n,d,k,p,kind", [
    (2000, 96, 48, 42, "bytes"),             # int8 rows of the long join
    ((1 << 20) + 1, 16, 6, 6, "bytes"),      # staged results
    ((1 << 20) + 1, 32, 6, 6, "floats"),     # 16-bit rows in the staged results' place
    (3000, 40, 16, 16, "unit")])             # 16-bit rows
def test_smaller_workspaces_give_the_same_graph(n, d, k, p, kind):
    import paper_2103_15386_amd as amd
    if kind == "bytes":
        x, metric = _bytes(n, d), amd.L2SQ_U8
    else:
        g = torch.Generator(device="cuda").manual_seed(n)
        x, metric = torch.randn((n, d), generator=g, device="cuda"), amd.L2SQ_F32
        if kind == "unit":
            x, metric = x / x.norm(dim=1, keepdim=True), amd.ANGULAR_F32
    full, least = _sizes(n, d, k, p, metric)
    assert least < full
    want = _build(x, k, p, metric, 3, full)
    for nbytes in (full - 1, least):
        got = _build(x, k, p, metric, 3, nbytes)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


def test_a_smaller_arena_gives_the_same_graph():
    import paper_2103_15386_amd as amd
    from paper_2103_15386_amd.binding import make_params
    lib = amd.load_library()
    n, d, k, p, shards = 3000, 48, 12, 10, 3
    host = torch.from_numpy(W.deep_like_f32(n, d, seed=901, n_comp=8)).pin_memory()
    want = amd.gnnd_build_sharded(host, shards, k, p, amd.ANGULAR_F32, SEED, 4, 2)
    side = torch.cuda.Stream()
    prm = make_params(n, d, k, p, amd.ANGULAR_F32, SEED)
    full = lib.gnnd_sharded_arena_bytes(C.byref(prm), shards)
    least = lib.gnnd_sharded_arena_bytes_min(C.byref(prm), shards)
    assert least < full
    for nbytes in (full - 1, least):
        arena = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        prm = make_params(n, d, k, p, amd.ANGULAR_F32, SEED,
                          stream=torch.cuda.current_stream().cuda_stream, workspace=arena)
        ids = torch.empty((n, k), dtype=torch.int32, pin_memory=True)
        dist = torch.empty((n, k), dtype=torch.float32, pin_memory=True)
        assert lib.gnnd_build_sharded(C.byref(prm), host.data_ptr(), shards, 4, 2, ids.data_ptr(),
                                      dist.data_ptr(), side.cuda_stream, None) == 0
        assert torch.equal(ids, want[0]) and torch.equal(dist, want[1])


def test_python_calls_take_the_smaller_workspace_where_the_full_one_does_not_fit(monkeypatch):
    import paper_2103_15386_amd as amd
    n, d, k, p = 4000, 128, 8, 6
    x = torch.from_numpy(W.deep_like_f32(n, d, seed=903, n_comp=8)).cuda()
    full, least = _sizes(n, d, k, p, amd.ANGULAR_F32)
    want = amd.gnnd_build(x, k, p, amd.ANGULAR_F32, SEED, 3)
    assert want[2].workspace.numel() == full
    half = n // 2
    parts = [amd.gnnd_build(v.contiguous(), k, p, amd.ANGULAR_F32, SEED, 3) for v in (x[:half], x[half:])]
    merge = (x[:half].contiguous(), x[half:].contiguous(), parts[0][0], parts[0][1],
             parts[1][0] + half, parts[1][1], k, p, amd.ANGULAR_F32, SEED, 2)
    append = (merge[0], merge[2], merge[3], merge[1], k, p, amd.ANGULAR_F32, SEED, 3, 2)
    sharded = (x.cpu().pin_memory(), 2, k, p, amd.ANGULAR_F32, SEED, 3, 2)
    calls = [(amd.gnnd_merge, merge), (amd.gnnd_append, append), (amd.gnnd_build_sharded, sharded)]
    results = [f(*args)[:2] for f, args in calls]
    empty, refused = torch.empty, []

    def little_room(*size, **kw):
        if kw.get("dtype") == torch.uint8 and not kw.get("pin_memory") and size[0] >= full:
            if len(refused) % 2 == 0:  # the larger of the two sizes of a call
                refused.append(size[0])
                raise torch.cuda.OutOfMemoryError("no room")
            refused.append(0)
        return empty(*size, **kw)

    monkeypatch.setattr(torch, "empty", little_room)
    ctx = amd.Gnnd(x, k, p, amd.ANGULAR_F32, SEED)
    assert ctx.workspace.numel() == least and refused == [full]
    ctx.build(3, want_stats=False)
    got = ctx.graph()
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    for (f, args), ref in zip(calls, results):
        refused.clear()
        got = f(*args)
        assert refused and torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])


def test_the_smallest_sizes_are_those_without_the_extras():
    import paper_2103_15386_amd as amd
    # sizes before there were such extras (bytes per node: lists, samples, candidates, proposals, ...)
    for args in ((4_000_000, 96, 32, 32, amd.L2SQ_U8), (100_000_000, 96, 32, 32, amd.ANGULAR_F32),
                 (200_000, 128, 64, 42, amd.L2SQ_U8), (1_000_000, 128, 32, 32, amd.L2SQ_F32)):
        full, least = _sizes(*args)
        assert 0 < least <= full
    n, d = 4_000_000, 96
    full, least = _sizes(n, d, 32, 32, amd.L2SQ_F32)
    # the 16-bit rows lie where the staged results would: never both
    assert full - least < n * 6 * 32 * 8 + n * 16
