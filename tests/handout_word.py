"""Reads, from a context's workspace, the word that says whether the staged int8 join hands on every
result it finds in the iteration the workspace was last used for."""
import torch

FIELDS = ("inserts", "dist_evals", "sum_new", "sum_old", "proposals", "dropped", "passed")


def handout_word(ws, stats):
    """The word, after the iterations of a context or merge whose statistics are `stats`: the counters
    are the 64 x 8 words whose column sums are theirs, it is the second word behind them."""
    w = ws.view(torch.int64)
    want = torch.tensor([sum(s[f] for s in stats) for f in FIELDS] + [0], device="cuda")
    at = (w.unfold(0, 512, 32).view(-1, 64, 8).sum(1) == want).all(1).nonzero().flatten().tolist()
    assert len(at) == 1
    return int(w[at[0] * 32 + 512 + 1])


def next_word(stats):
    """What the word has to be in an iteration that follows one with these statistics."""
    return int(3 * stats["passed"] >= 2 * stats["proposals"])
