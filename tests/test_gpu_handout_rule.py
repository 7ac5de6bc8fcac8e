"""Whether the staged int8 join hands on every result it finds: one word behind the counters, which the
sampling stage writes for every context (only staged joins look at it).  The results are the same
either way, so the word itself is read here, from the workspace."""
import pytest
import torch

import workloads as W
from handout_word import handout_word, next_word

pytestmark = pytest.mark.gpu
def _vectors(n, d=16, seed=3):
    return torch.from_numpy(W.sift_like_u8(n, d, seed=seed, n_comp=16)).cuda()


def _random_graph(n, k):
    """Distinct ids that are no self loops, ascending made-up distances, every entry NEW."""
    ids = (torch.arange(n, device="cuda")[:, None] + 1 + 37 * torch.arange(k, device="cuda")) % n
    dist = torch.arange(1, k + 1, device="cuda").expand(n, k) * 1000
    return ids.int().contiguous(), dist.int().contiguous(), torch.ones((n, k), dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("n", [3000, 20_000])  # sampled by atomics, by the counting sort
def test_what_the_workspace_held_before_decides_nothing(n, monkeypatch):
    import paper_2103_15386_amd as amd
    from paper_2103_15386_amd import binding
    k, seen, real = 8, [], binding._workspace
    x = _vectors(n)
    # nothing; in the counters' layout: many results found before, none of them passed
    for left in ([0] * 8, [0, 0, 0, 0, -(1 << 40), 0, 0, 0]):
        def workspace(prm, dev):
            ws = real(prm, dev)
            ws.view(torch.int64).view(-1, 8)[:] = torch.tensor(left, device=dev)
            return ws
        monkeypatch.setattr(binding, "_workspace", workspace)
        ctx = amd.Gnnd(x, k, k, amd.L2SQ_U8, W.ALGO_SEED)
        ctx.set_graph(*_random_graph(n, k), 5)
        seen.append(handout_word(ctx.workspace, [ctx.iterate()]))
        ctx.close()
    assert seen[0] == seen[1]


def test_the_decision_follows_from_the_graph_and_the_iteration_before():
    """A fresh random graph: everything; then two thirds of the results of the iteration before; a loaded
    graph, whatever its iteration number and whatever the context worked on before: not everything."""
    import paper_2103_15386_amd as amd
    n, k = 20_000, 12
    ctx = amd.Gnnd(_vectors(n, 40), k, k, amd.L2SQ_U8, W.ALGO_SEED)
    stats, later = [], set()

    def iterate(expected):
        stats.append(ctx.iterate())
        assert handout_word(ctx.workspace, stats) == expected
        return next_word(stats[-1])

    ctx.init_random()
    word = iterate(1)
    for _ in range(6):
        later.add(word)
        word = iterate(word)
    assert later == {0, 1}
    for it in (0, 9):
        ctx.init_random()
        assert iterate(1) == 1
        ctx.set_graph(*_random_graph(n, k), it)
        word = iterate(0)
        iterate(word)
    ctx.close()


@pytest.mark.parametrize("iters", [1, 2, 4])
def test_a_merge_begins_with_everything(iters, monkeypatch):
    import paper_2103_15386_amd as amd
    from paper_2103_15386_amd import binding
    n1, n2, k, real, kept = 9000, 7000, 12, binding._workspace, []
    x = _vectors(n1 + n2, 40)
    a, b = x[:n1].contiguous(), x[n1:].contiguous()
    ids1, dist1, c1 = amd.gnnd_build(a, k, k, amd.L2SQ_U8, 42, 5)
    ids2, dist2, c2 = amd.gnnd_build(b, k, k, amd.L2SQ_U8, 43, 5)

    def workspace(prm, dev):
        kept.append(real(prm, dev))
        return kept[-1]
    monkeypatch.setattr(binding, "_workspace", workspace)
    *_, stats = amd.gnnd_merge(a, b, ids1, dist1, ids2 + n1, dist2, k, k, amd.L2SQ_U8, 42, iters,
                               want_stats=True)
    assert len(kept) == 1
    assert handout_word(kept[0], stats) == (1 if iters == 1 else next_word(stats[-2]))
    c1.close()
    c2.close()
