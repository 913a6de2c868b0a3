"""What the backward lists of the rows with many lookups - the hint for the next forward, and the rows for the matrix cores -
against the lists that the counts give."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def listed(rows, D, B, counts, dtype="f32"):
    """counts[t]: lookups of every row of table t.  Spreads them over B bags per table at random, prepares the batch and returns
    the lists (hinted, dense) per table."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE
    g = torch.Generator().manual_seed(7)
    ids, lens = [], []
    for c in counts:
        i = torch.repeat_interleave(torch.arange(len(c)), c)
        ids.append(i[torch.randperm(i.numel(), generator=g)])
        lens.append(torch.bincount(torch.randint(0, B, (i.numel(),), generator=g), minlength=B))
    off = torch.zeros(len(rows) * B + 1, dtype=torch.int64)
    off[1:] = torch.cumsum(torch.cat(lens), 0)
    idx = torch.cat(ids).cuda()
    tbe = TBE(rows, D, dtype)
    ws = tbe.alloc_workspace(B, idx.numel())
    tbe.backward_prepare(idx, off.cuda(), B, ws)
    lists = tbe.debug_hot_rows(ws, B, idx.numel())
    tbe.close()
    return lists


def longest(c, at_least, most):
    """Rows of at least that many lookups, most lookups first, ties by id."""
    order = torch.argsort(c, descending=True, stable=True)
    return [int(r) for r in order if c[r] >= at_least][:most]


@pytest.mark.parametrize("total", [60_000, 300_000, 1_200_000, 2_500_000])   # rows are long from 65 / 129 / 257 / 513 lookups on
def test_the_hint_lists_rows_of_more_than_512_lookups(total):
    c0 = torch.tensor([513, 512, 900, 66, 511, 514, 900, 130, 300, 5000])
    c1 = torch.full((400,), (total - int(c0.sum())) // 400)
    hot, dense = listed([10, 400], [16, 16], 64, [c0, c1])
    assert hot == [longest(c0, 513, 256), longest(c1, 513, 256)]
    assert dense == [[], []]

