"""Whether the staged int8 join hands on every result it finds: one word behind the counters, which the
sampling stage writes for every context (only staged joins look at it).  The results are the same
either way, so the word itself is read here, from the workspace."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu
FIELDS = ("inserts", "dist_evals", "sum_new", "sum_old", "proposals", "dropped", "passed")


def _word(ws, stats):
    """The word, after the iterations of a context or merge whose statistics are `stats`: the counters
    are the 64 x 8 words whose column sums are theirs, it is the second word behind them."""
    w = ws.view(torch.int64)
    want = torch.tensor([sum(s[f] for s in stats) for f in FIELDS] + [0], device="cuda")
    at = (w.unfold(0, 512, 32).view(-1, 64, 8).sum(1) == want).all(1).nonzero().flatten().tolist()
    assert len(at) == 1
    return int(w[at[0] * 32 + 512 + 1])


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
        seen.append(_word(ctx.workspace, [ctx.iterate()]))
        ctx.close()
    assert seen[0] == seen[1]
