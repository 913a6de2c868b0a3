"""The pooled forward on both sides of the border between one wavefront per bag and lane groups: every class of row widths,
empty, ordinary and long bags, against 64-bit sums."""
import pytest
import torch

pytestmark = pytest.mark.gpu

WIDTHS = {"f32": [8, 20, 32, 36, 64, 100, 128, 136, 256], "f16": [8, 24, 64, 104, 128, 200, 256, 264, 512]}
BAGS = 16384


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("pooling", ["sum", "mean"])
@pytest.mark.parametrize("B", [1, 7, BAGS // 9, BAGS // 9 + 1, BAGS // 9 + 70])   # 9 tables: 16380 bags, then 16389
def test_forward_on_both_sides_of_the_small_batch_border(dtype, pooling, B):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE, binding
    D = WIDTHS[dtype]
    T, R, longest = len(D), 500, 200
    g = torch.Generator().manual_seed(B)
    lens = torch.randint(0, 24, (T * B,), generator=g)
    lens[torch.rand(T * B, generator=g) < 0.02] = longest
    off = torch.zeros(T * B + 1, dtype=torch.int64)
    off[1:] = torch.cumsum(lens, 0)
    idx = torch.randint(0, R, (int(off[-1]),), generator=g)
    tbe = TBE([R] * T, D, dtype)
    small = tbe.debug_forward_kernels(B, idx.numel()) == binding.FWD_WAVEFRONT_PER_BAG
    assert small == (T * B <= BAGS)          # 15 ids per bag on average: the border lies at the most bags it can
    tabs = torch.empty(tbe.total_elems).uniform_(-0.01, 0.01, generator=g).to(tbe.torch_dtype)
    out = tbe.forward(tabs.cuda(), idx.cuda(), off.cuda(), B, pooling).cpu().double()
    assert not tbe.poll_index_error()
    d0 = w0 = 0
    for t, d in enumerate(D):
        table = tabs[w0:w0 + R * d].view(R, d).double()
        o = off[t * B:(t + 1) * B + 1]
        want = torch.zeros(B, d, dtype=torch.float64)
        bag = torch.repeat_interleave(torch.arange(B), o[1:] - o[:-1])
        want.index_add_(0, bag, table[idx[int(o[0]):int(o[-1])]])
        if pooling == "mean":
            want /= (o[1:] - o[:-1]).clamp(min=1).double()[:, None]
        # a 32-bit sum of L values of at most 0.01: at most (L - 1) * 2^-24 * L * 0.01
        assert (out[:, d0:d0 + d] - want).abs().max() <= longest * 2.0 ** -24 * longest * 0.01, (t, d)
        d0 += d
        w0 += R * d
    tbe.close()


@pytest.mark.parametrize("D,dtype,L,border", [
    (8, "f32", 1, 9728), (8, "f32", 3, 14848), (32, "f32", 4, 16384),
    (16, "f16", 1, 6400), (64, "f16", 3, 8960), (32, "f16", 10, 16384),
    (64, "f32", 1, 13312), (256, "f16", 2, 14336), (128, "f32", 8, 16384),
])
def test_the_small_batch_border_follows_row_width_and_bag_length(D, dtype, L, border):
    """One wavefront per bag up to the border, lane groups (and the long bags they leave out) from the next bag on: the same
    sums on both sides."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE, binding
    R = 300
    tbe = TBE([R], [D], dtype)
    g = torch.Generator().manual_seed(D)
    table = torch.empty(R, D).uniform_(-0.01, 0.01, generator=g).to(tbe.torch_dtype)
    idx = torch.randint(0, R, ((border + 1) * L,), generator=g)
    want = table.double()[idx].view(border + 1, L, D).sum(1)
    for B in (border, border + 1):
        kernels = tbe.debug_forward_kernels(B, B * L)
        assert kernels == (binding.FWD_WAVEFRONT_PER_BAG if B == border else binding.FWD_LANE_GROUPS | binding.FWD_LONG_BAGS)
        off = torch.arange(0, B * L + 1, L)
        out = tbe.forward(table.view(-1).cuda(), idx[:B * L].cuda(), off.cuda(), B, "sum").cpu().double()
        assert (out - want[:B]).abs().max() <= L * 2.0 ** -24 * L * 0.01
    assert not tbe.poll_index_error()
    tbe.close()
