"""Long bags of the lane-group forward classes: the bound that follows a table's mean bag length, the error of the bags that lane
groups walk below it, and wavefronts that look at 4 to 128 bags."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("T,B,mean", [
    (5, 3500, 15),     # the class bounds hold (32 / 48 / 64), 4 bags per wavefront, tables that end inside one
    (5, 3501, 36),     # a bound of 72 for every class
    (1, 16390, 90),    # the highest bound (128)
    (6, 11000, 3),     # 16 bags per wavefront
    (5, 105000, 2),    # 128 bags per wavefront: two rounds of 64
])
def test_bags_on_both_sides_of_the_bound(dtype, T, B, mean):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE, binding
    v = 8 if dtype == "f16" else 4
    D = [v * w for w in (1, 8, 13, 32, 3, 16)][:T]        # 1 to 32 lanes per row
    R = 400
    g = torch.Generator().manual_seed(B)
    lens = torch.randint(0, 2 * mean + 1, (T * B,), generator=g)
    twice = 2 * int(lens.sum()) // (T * B)
    special = [0, 1] + [b + d for b in (32, 48, 64, 128, twice) for d in (-1, 0, 1)] + [300]
    for t in range(T):   # the first and last bags of every table, and some in between
        at = torch.cat([torch.arange(40), torch.arange(B - 40, B), torch.randperm(B - 80, generator=g)[:40] + 40]) + t * B
        lens[at] = torch.tensor(special * 8)[torch.randperm(120, generator=g)].clamp(min=0)
    off = torch.zeros(T * B + 1, dtype=torch.int64)
    off[1:] = torch.cumsum(lens, 0)
    idx = torch.randint(0, R, (int(off[-1]),), generator=g)
    tbe = TBE([R] * T, D, dtype)
    tbe.set_tunable("hot_rows_min_workgroups", -1)
    assert tbe.debug_forward_kernels(B, idx.numel()) == binding.FWD_LANE_GROUPS | binding.FWD_LONG_BAGS
    tabs = torch.empty(tbe.total_elems).uniform_(-0.01, 0.01, generator=g).to(tbe.torch_dtype).cuda()
    args = (idx.cuda(), off.cuda(), B, "sum")
    out = tbe.forward(tabs, *args)
    d0 = w0 = 0
    for t, d in enumerate(D):
        o = off[t * B:(t + 1) * B + 1]
        bag = torch.repeat_interleave(torch.arange(B), o[1:] - o[:-1])
        want = torch.zeros(B, d, dtype=torch.float64)
        want.index_add_(0, bag, tabs[w0:w0 + R * d].cpu().view(R, d).double()[idx[int(o[0]):int(o[-1])]])
        # a 32-bit sum of L values of at most 0.01: at most (L - 1) * 2^-24 * L * 0.01
        L = (o[1:] - o[:-1]).double()[:, None]
        assert ((out[:, d0:d0 + d].cpu().double() - want).abs() <= 2.0 ** -24 * 0.01 * L * L).all(), (t, d)
        d0 += d
        w0 += R * d
    # the kernel with hot rows, none listed yet, makes the same additions in the same order
    tbe.set_tunable("hot_rows_min_workgroups", 1)
    assert tbe.debug_forward_kernels(B, idx.numel()) == binding.FWD_HOT_ROWS | binding.FWD_LONG_BAGS
    assert torch.equal(tbe.forward(tabs, *args), out)
    assert not tbe.poll_index_error()
    tbe.close()


def _sum_by_wavefront(x, lanes):
    """fp32 sum over dim 1 as a whole wavefront makes it: 64 / lanes groups take the rows in turn and are folded pairwise."""
    G = 64 // lanes
    acc = torch.zeros(x.shape[0], G, x.shape[2])
    for k in range(x.shape[1]):
        acc[:, k % G] += x[:, k]
    while acc.shape[1] > 1:
        acc = acc[:, 0::2] + acc[:, 1::2]
    return acc[:, 0]


def _sum_by_lane_group(x, lanes):
    """... as a lane group makes it above the class bound: runs of 8 rows (16 of rows of 32 lanes, 4 of rows of at most 4) in fp32,
    their sums in 64 bits."""
    run = 16 if lanes == 32 else min(8, max(4, lanes))
    total = torch.zeros(x.shape[0], x.shape[2], dtype=torch.float64)
    for k0 in range(0, x.shape[1], run):
        acc = torch.zeros(x.shape[0], x.shape[2])
        for k in range(k0, min(k0 + run, x.shape[1])):
            acc += x[:, k]
        total += acc.double()
    return total.float()


@pytest.mark.parametrize("D,L", [(8, 100), (16, 40), (32, 40), (32, 100), (64, 62), (128, 100)])
def test_error_above_the_class_bounds(D, L):
    """A lane group that walks a bag above its class bound is no further from the sum in 64 bits than a whole wavefront is."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE, binding
    T, B, R = 6, 3000, 700
    g = torch.Generator().manual_seed(D + L)
    w = torch.randn(T, R, D, generator=g)
    idx = torch.randint(0, R, (T, B, L), generator=g)
    tbe = TBE([R] * T, [D] * T, "f32")
    assert tbe.debug_forward_kernels(B, idx.numel()) == binding.FWD_LANE_GROUPS | binding.FWD_LONG_BAGS
    out = tbe.forward(w.view(-1).cuda(), idx.view(-1).cuda(), torch.arange(T * B + 1, dtype=torch.int64).cuda() * L, B, "sum").cpu()
    lanes = 1 << ((D + 3) // 4 - 1).bit_length()
    err = err_wave = 0.0
    for t in range(T):
        x = w[t][idx[t]]
        want = x.double().sum(1)
        got = out[:, t * D:(t + 1) * D]
        assert torch.equal(got, _sum_by_lane_group(x, lanes))
        err += float(((got.double() - want) ** 2).sum())
        err_wave += float(((_sum_by_wavefront(x, lanes).double() - want) ** 2).sum())
    assert err <= err_wave
    tbe.close()


@pytest.mark.parametrize("D,long,short", [(32, 100, 5), (64, 70, 3), (128, 128, 1)])
def test_bound_follows_the_tables_own_mean(D, long, short):
    """One table of long bags among tables of short ones: its ordinary bags are summed by lane groups and not by whole wavefronts,
    and a bag of the same length among the short ones by a whole wavefront."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE, binding
    T, B, R = 9, 2100, 500
    g = torch.Generator().manual_seed(D)
    lens = torch.full((T, B), short)
    lens[4] = long
    lens[2, ::100] = long
    lens[4, ::70] = 2 * long + 1
    off = torch.zeros(T * B + 1, dtype=torch.int64)
    off[1:] = torch.cumsum(lens.view(-1), 0)
    w = torch.randn(T, R, D, generator=g)
    idx = torch.randint(0, R, (int(off[-1]),), generator=g)
    tbe = TBE([R] * T, [D] * T, "f32")
    assert tbe.debug_forward_kernels(B, idx.numel()) == binding.FWD_LANE_GROUPS | binding.FWD_LONG_BAGS
    lanes = D // 4
    for it in (torch.int64, torch.int32):
        out = tbe.forward_ex(w.view(-1).cuda(), idx.cuda().to(it), off.cuda().to(it), B, "sum").cpu()

        def check(t, bags, sums):
            at = off[t * B + bags]
            x = w[t][idx[at[:, None] + torch.arange(int(lens[t, bags[0]]))]]
            assert torch.equal(out[bags, t * D:(t + 1) * D], sums(x, lanes)), (it, t)

        every = torch.arange(B)
        check(4, every[every % 70 != 0], _sum_by_lane_group)
        check(4, every[::70], _sum_by_wavefront)
        check(2, every[::100], _sum_by_wavefront)
    tbe.close()


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("hot", [-1, 0])
def test_mean_pooling_on_both_sides_of_the_bound(dtype, hot):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE
    v = 8 if dtype == "f16" else 4
    D = [v * lanes for lanes in (2, 8, 13, 32)]
    B, R = 4100, 300   # (more bags than one wavefront each takes)
    g = torch.Generator().manual_seed(3)
    lens = torch.randint(0, 90, (4 * B,), generator=g)     # twice the mean is 89
    lens[::50] = torch.tensor([0, 31, 33, 47, 49, 63, 65, 88, 91, 127, 129, 260]).repeat(50)[:len(lens[::50])]
    off = torch.zeros(4 * B + 1, dtype=torch.int64)
    off[1:] = torch.cumsum(lens, 0)
    idx = torch.randint(0, R, (int(off[-1]),), generator=g)
    tbe = TBE([R] * 4, D, dtype)
    tbe.set_tunable("hot_rows_min_workgroups", hot)
    w = torch.empty(tbe.total_elems).uniform_(-1, 1, generator=g).to(tbe.torch_dtype)
    out = tbe.forward(w.cuda(), idx.cuda(), off.cuda(), B, "mean").cpu().double()
    d0 = w0 = 0
    for t, d in enumerate(D):
        o = off[t * B:(t + 1) * B + 1]
        L = (o[1:] - o[:-1]).double()[:, None]
        want = torch.zeros(B, d, dtype=torch.float64)
        want.index_add_(0, torch.repeat_interleave(torch.arange(B), o[1:] - o[:-1]), w[w0:w0 + R * d].view(R, d).double()[idx[int(o[0]):int(o[-1])]])
        want /= L.clamp(min=1.0)
        # a 32-bit sum of L values of at most 1 and one division: at most (L - 1 + 1) * 2^-24
        assert ((out[:, d0:d0 + d] - want).abs() <= 2.0 ** -24 * L).all(), (t, d)
        d0 += d
        w0 += R * d
    tbe.close()
