"""The reverse part of the sample lists where its kernels change their way of working: as many
candidates as there is room for and one more or less, up to 64, up to 128 and beyond; and the
proposal segments on both sides of the size from which the forward samples are added up."""
import numpy as np
import pytest
import torch

import oracle as og
import workloads as W

pytestmark = pytest.mark.gpu

SEED = W.ALGO_SEED


def _graph_with_degrees(n, k, p, rng):
    """Random lists (k = p: every entry is sampled) in which chosen nodes are entries of as many
    other lists, flagged NEW or OLD, as the comment above names."""
    isnew = (rng.random((n, k)) < rng.random((n, 1))).astype(np.uint8)
    free = [list(rng.permutation(k)) for _ in range(n)]
    ids = np.full((n, k), -1, np.int64)
    special = 0
    for kind in (1, 0):
        for want in range(13):
            v = special
            special += 1
            room = 2 * p - int((isnew[v] == kind).sum())
            deg = [0, 1, room - 1, room, room + 1, 63, 64, 65, 127, 128, 129, 193, 300][want]
            for s in rng.permutation(n):
                if deg <= 0:
                    break
                slots = [j for j in free[s] if isnew[s, j] == kind]
                if s == v or not slots or len(free[s]) <= k // 2:
                    continue
                ids[s, slots[0]] = v
                free[s].remove(slots[0])
                deg -= 1
    for s in range(n):
        fill = rng.choice(n - special, k + 1, replace=False) + special
        fill = [v for v in fill if v != s][:len(free[s])]
        ids[s, free[s]] = fill
    dist = np.broadcast_to(np.arange(1, k + 1, dtype=np.float64), (n, k)).copy()
    return ids.astype(np.int32), dist, isnew


@pytest.mark.parametrize("p", [5, 8, 31, 32, 33, 42, 64])
@pytest.mark.parametrize("seed", [1, 2])
def test_samples_match_the_oracle_at_chosen_reverse_degrees(p, seed):
    import paper_2103_15386_amd as amd
    n, k = 1100, p
    rng = np.random.default_rng(100 * p + seed)
    x = rng.random((n, 4), dtype=np.float32)
    g = og.init_random(x, k, og.L2SQ_F32, SEED)
    ids, dist, isnew = _graph_with_degrees(n, k, p, rng)
    g.ids[:], g.dist[:], g.isnew[:] = ids, dist, isnew
    ctx = amd.Gnnd(torch.from_numpy(x).cuda(), k, p, amd.L2SQ_F32, SEED)
    ctx.set_graph(torch.from_numpy(ids).cuda(), torch.from_numpy(dist.astype(np.float32)).cuda(),
                  torch.from_numpy(isnew).cuda(), 2)
    ctx.step_sample()
    got = [t.cpu().numpy() for t in ctx.samples()]
    snew, cnew, sold, cold = og.sample(g, p, SEED, 3)
    for a, b in zip(got, (snew, cnew, sold, cold)):
        assert (a == b).all()
    ctx.close()


@pytest.mark.parametrize("n", [(1 << 18) - 1, 1 << 18, (1 << 18) + 1, (1 << 18) + 4099])
@pytest.mark.parametrize("metric", [og.L2SQ_F32, og.L2SQ_U8])
def test_builds_match_the_oracle_around_the_segment_rule(n, metric):
    import paper_2103_15386_amd as amd
    x = W.uniform_f32(n, 4, seed=3)
    if metric == og.L2SQ_U8:
        x = (x * 255).astype(np.uint8)
    g, _ = og.build(x, 6, 5, metric, SEED, 2)
    ctx = amd.Gnnd(torch.from_numpy(x).cuda(), 6, 5, metric, SEED)
    st = ctx.build(2)
    ids, dist = ctx.graph()
    assert st["dropped"] == 0
    assert (ids.cpu().numpy() == g.ids).all() and (dist.cpu().numpy() == g.dist).all()
    ctx.close()


@pytest.mark.parametrize("k,p,every", [(65, 5, False), (40, 33, False), (6, 4, True)])
def test_builds_match_the_oracle_beyond_the_segment_rule(k, p, every):
    """The forms of sampling and reverse selection for long lists and for every evaluated pair where
    the forward samples are added up: a segment in a wrong place would mix two nodes' results."""
    import paper_2103_15386_amd as amd
    n = (1 << 18) + 33
    x = W.uniform_f32(n, 4, seed=6)
    ctx = amd.Gnnd(torch.from_numpy(x).cuda(), k, p, amd.L2SQ_F32, SEED, amd.JOIN_AUTO,
                   amd.UPDATE_ALL_PAIRS if every else amd.UPDATE_SELECTIVE)
    ctx.init_random()
    g = og.init_random(x, k, og.L2SQ_F32, SEED)
    for it in (1, 2):
        ctx.step_sample()
        got = [t.cpu().numpy() for t in ctx.samples()]
        snew, cnew, sold, cold = og.sample(g.copy(), p, SEED, it)
        for a, b in zip(got, (snew, cnew, sold, cold)):
            assert (a == b).all()
        ctx.step_join()
        st = ctx.step_update()
        want = og.iterate(x, og.L2SQ_F32, g, p, SEED, it, all_pairs=every)
        assert st["dropped"] == 0
        for key in ("inserts", "dist_evals", "sum_new", "sum_old", "proposals"):
            assert st[key] == want[key], key
    ids, dist = ctx.graph()
    assert (ids.cpu().numpy() == g.ids).all() and (dist.cpu().numpy() == g.dist).all()
    ctx.close()


@pytest.mark.parametrize("n,k,p", [(12288, 10, 10), (12289, 10, 10), (12287, 11, 10),
                                   (4096, 32, 32), (4097, 33, 32), (2048, 128, 64), (2049, 100, 64),
                                   (1000, 70, 64), (65, 64, 40), (7, 5, 3)])
def test_builds_match_the_oracle_where_small_collections_end(n, k, p):
    import paper_2103_15386_amd as amd
    x = W.uniform_f32(n, 8, seed=5)
    g, _ = og.build(x, k, p, og.L2SQ_F32, SEED, 3)
    ctx = amd.Gnnd(torch.from_numpy(x).cuda(), k, p, amd.L2SQ_F32, SEED)
    for _ in range(2):  # (the second build finds what the first one has left)
        st = ctx.build(3)
        ids, dist = ctx.graph()
        assert st["dropped"] == 0
        assert (ids.cpu().numpy() == g.ids).all() and (dist.cpu().numpy() == g.dist).all()
    ctx.close()


@pytest.mark.parametrize("n,d,k,p", [(1 << 14, 20, 12, 10), ((1 << 14) + 1, 96, 20, 20),
                                     (16000, 64, 33, 32), (16390, 128, 32, 32),
                                     (11264, 30, 33, 17), (11265, 100, 33, 17)])
def test_hand_out_of_small_byte_collections(n, d, k, p):
    """Results one by one up to 2^14 nodes (k > 32, p > 16: 11,264), staged beyond: the oracle's graph,
    and the counters of the staged form."""
    import paper_2103_15386_amd as amd
    x = torch.from_numpy(W.sift_like_u8(n, d, seed=9, n_comp=16)).cuda()
    seen = []
    for path in (amd.JOIN_AUTO, amd.JOIN_MFMA):
        ctx = amd.Gnnd(x, k, p, amd.L2SQ_U8, SEED, path)
        ctx.init_random()
        stats = [ctx.iterate() for _ in range(3)]
        seen.append(([{f: v for f, v in s.items() if not f.startswith("ms")} for s in stats],
                     *[t.cpu().numpy() for t in ctx.graph()]))
        ctx.close()
    g, _ = og.build(x.cpu().numpy(), k, p, og.L2SQ_U8, SEED, 3)
    assert seen[0][0] == seen[1][0]
    for _, ids, dist in seen:
        assert (ids == g.ids).all() and (dist == g.dist).all()


@pytest.mark.parametrize("n,k,targets,fit", [(13000, 8, 256, 12 * 1024),
                                             ((1 << 18) + 100, 24, 512, 36 * 1024)])
@pytest.mark.parametrize("more", [-1, 0, 1, 3000])
@pytest.mark.parametrize("kind", [0, 1])
def test_a_bucket_of_candidates_that_just_fits_or_does_not(n, k, targets, fit, more, kind):
    """The first `targets` nodes (one bucket of the counting sort) are entries of one kind of fit + more
    lists: the number a workgroup keeps in registers and LDS, and around it."""
    import paper_2103_15386_amd as amd
    rng = np.random.default_rng(7)
    x = rng.random((n, 4), dtype=np.float32)
    ids = (targets + (np.arange(n)[:, None] * 7 + 1 + np.arange(k) * 31) % (n - targets)).astype(np.int32)
    ids += ids == np.arange(n, dtype=np.int32)[:, None]
    ids[ids >= n] = targets
    isnew = rng.integers(0, 2, (n, k)).astype(np.uint8)
    at = targets * k + np.arange(fit + more)
    ids.reshape(-1)[at] = at % targets
    isnew.reshape(-1)[at] = kind
    dist = np.broadcast_to(np.arange(1, k + 1, dtype=np.float64), (n, k)).copy()
    g = og.init_random(x, k, og.L2SQ_F32, SEED)
    g.ids[:], g.dist[:], g.isnew[:] = ids, dist, isnew
    ctx = amd.Gnnd(torch.from_numpy(x).cuda(), k, k, amd.L2SQ_F32, SEED)
    ctx.set_graph(torch.from_numpy(ids).cuda(), torch.from_numpy(dist.astype(np.float32)).cuda(),
                  torch.from_numpy(isnew).cuda(), 2)
    ctx.step_sample()
    got = [t.cpu().numpy() for t in ctx.samples()]
    for a, b in zip(got, og.sample(g, k, SEED, 3)):
        assert (a == b).all()
    ctx.close()
