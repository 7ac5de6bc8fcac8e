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


def region_cursors(ws, handed):
    """How many results each of the 256 bucket regions has received in the last staged join, `handed`
    in all: those of the iteration's proposals that passed, or all of them."""
    w = ws.view(torch.int64)
    at = (w.unfold(0, 256, 32).sum(1) == handed).nonzero().flatten().tolist()
    assert at and at[-1] - at[0] < 8  # (fewer buckets: the last words are zero, and so may those before be)
    return w[at[-1] * 32:at[-1] * 32 + 256]
