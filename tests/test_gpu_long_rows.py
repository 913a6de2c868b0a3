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


def uneven(n, low, spread, hot=()):
    """n rows of low .. low + spread - 1 lookups in no order; hot: (row, lookups) of the few above them."""
    c = low + torch.arange(n) * 7919 % spread
    for r, k in hot:
        c[r] = k
    return c


@pytest.mark.parametrize("n", [1, 127, 128, 129, 1023, 1024, 1025, 1500])
@pytest.mark.parametrize("low,spread", [(66, 1), (66, 23)])
def test_the_longest_rows_are_dense_whatever_their_number(n, low, spread):
    B, D = 1024, 1024                          # the smallest batch with dense rows; long from 65 lookups on
    c = torch.cat([uneven(n, low, spread, [(n // 2, 3000), (n - 1, 700)]), torch.tensor([64, 0, 1, 65, 64])])
    first = longest(c, 65, 128)
    if int(c[first].sum()) < 2 * B:
        first = []
    tiny = torch.tensor([3])
    hot, dense = listed([n + 5] + 7 * [1], 8 * [D], B, [c] + 7 * [tiny])      # 8 tables x 4 chunks x 4 column blocks
    assert hot == [longest(c, 513, 256)] + 7 * [[]]
    assert dense == [first] + 7 * [[]]
    hot, dense = listed([n + 5], [D], B, [c])  # a lone table: too few workgroups for the dense rows of so many long ones
    assert hot == [longest(c, 513, 256)]
    assert dense == [first if int((c > 64).sum()) <= 1024 else []]


def test_more_than_1024_rows_above_the_hint_border():
    # lengths that differ in the third byte, in the second, in the last, and not at all; 2.3 M lookups: long from 513 on
    c = uneven(2500, 700, 97, [(17, 70000), (900, 66000), (2400, 65999), (3, 40000), (4, 40000), (5, 39999)])
    d = torch.full((1100,), 600)
    tiny = torch.tensor([1])
    hot, dense = listed([2500, 1100] + 6 * [1], [64, 32] + 6 * [64], 8400, [c, d] + 6 * [tiny])
    assert hot == [longest(c, 513, 256), longest(d, 513, 256)] + 6 * [[]]
    assert dense == [longest(c, 513, 128)] + 7 * [[]]      # the second table's block is too small


def test_rows_beyond_the_ranked_ones_take_the_same_step():
    """1310 long rows, 128 of them dense, the rest in parts: the step of every row against 64-bit sums."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE
    T, R, D, B = 8, 1400, 1024, 1024
    c = uneven(R, 130, 9, [(5, 2500), (1398, 900)])          # 180 k lookups: long from 129 on
    c[1300:1390] = 3
    g = torch.Generator().manual_seed(2)
    idx = torch.repeat_interleave(torch.arange(R), c)
    idx = idx[torch.randperm(idx.numel(), generator=g)]
    bag = torch.sort(torch.randint(0, B, (idx.numel(),), generator=g)).values
    off = torch.full((T * B + 1,), idx.numel(), dtype=torch.int64)
    off[0] = 0
    off[1:B + 1] = torch.cumsum(torch.bincount(bag, minlength=B), 0)
    grad = torch.randn(B, T * D, generator=g)
    tbe = TBE([R] + (T - 1) * [1], T * [D], "f32")
    ws = tbe.alloc_workspace(B, idx.numel())
    w = torch.zeros(tbe.total_elems, device="cuda")
    tbe.backward_sgd(grad.cuda(), idx.cuda(), off.cuda(), B, w, ws, lr=1.0)
    assert [len(d) for d in tbe.debug_hot_rows(ws, B, idx.numel())[1]] == [128] + (T - 1) * [0]
    mine = grad[:, :D].double()[bag]
    want = torch.zeros(R, D, dtype=torch.float64).index_add_(0, idx, mine)
    size = torch.zeros(R, D, dtype=torch.float64).index_add_(0, idx, mine.abs())
    # an fp32 sum of n terms in any order: at most n * 2^-24 of the sum of their magnitudes; here within 4 sqrt(n)
    bound = 4.0 * c.double().sqrt()[:, None] * 2.0 ** -24 * size
    assert bool(((-w[:R * D].cpu().double().view(R, D) - want).abs() <= bound).all())
    assert float(w[R * D:].abs().sum()) == 0.0
    tbe.close()
