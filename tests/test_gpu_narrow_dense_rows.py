"""Dense rows of tables of up to 64 columns: both column groupings, up to 32 / 64 / 96 / 128 rows and one more, short last blocks and
chunks, counts in two bytes and in rounds.  Gradients are small integers and bag lengths under mean pooling powers of two, so that
every sum is exact in fp32 (below 2^24 units) and has to equal the 64-bit one."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,B,rows,repeat,pooling,io", [
    (32, 16640, 128, 0, "sum", torch.float32),                     # whole blocks
    (32, 16641, 33, 0, "mean", torch.float16),                     # a last block of one bag
    (28, 20000, 97, 300, "sum", torch.float32),
    (4, 131373, 32, 0, "mean", torch.float32),
    (36, 15000, 64, 300, "sum", torch.bfloat16),                   # the second group of columns has four
    (64, 8447, 65, 0, "mean", torch.bfloat16),
    (64, 8450, 129, 70000, "sum", torch.float16),
    (48, 12289, 20, 70000, "sum", torch.float32),
])
def test_exact_sums(D, B, rows, repeat, pooling, io):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE
    dev, other = "cuda", 12
    g = torch.Generator(device=dev).manual_seed(D + rows)
    lens = 2 ** torch.randint(1, 4, (2 * B,), generator=g, device=dev)
    lens[B + B // 2] += repeat                                     # the second table is the narrow one
    off = torch.zeros(2 * B + 1, dtype=torch.int64, device=dev)
    torch.cumsum(lens, 0, out=off[1:])
    first = int(off[B])
    n = int(off[-1])
    idx = torch.randint(0, 3, (n,), generator=g, device=dev)
    idx[first:] = torch.randint(0, rows, (n - first,), generator=g, device=dev) * 3
    if repeat:
        at = int(off[B + B // 2])
        idx[at:at + repeat] = 3
    grad = torch.randint(-3, 4, (B, other + D), generator=g, device=dev).to(io)
    tbe = TBE([3, 3 * rows], [other, D], "f32")
    ws = tbe.alloc_workspace(B, n)
    w = torch.zeros(tbe.total_elems, device=dev)
    tbe.backward_sgd(grad, idx, off, B, w, ws, pooling=pooling, lr=1.0)
    assert len(tbe.debug_hot_rows(ws, B, n)[1][1]) == min(rows, 128)
    bag = torch.repeat_interleave(torch.arange(2 * B, device=dev), lens)[first:] - B
    rows_grad = grad[:, other:].double()
    if pooling == "mean":
        rows_grad = rows_grad / lens[B:, None]
    want = torch.zeros(3 * rows, D, dtype=torch.float64, device=dev).index_add_(0, idx[first:], rows_grad[bag])
    assert torch.equal(-w[3 * other:].view(3 * rows, D).double(), want)
    tbe.close()


@pytest.mark.parametrize("D,B,io,pooling,value", [
    (32, 16641, torch.float32, "sum", float("inf")),               # the last block's only bag
    (48, 12289 + 37, torch.bfloat16, "mean", float("nan")),
    (64, 8447, torch.float16, "sum", float("-inf")),
    (64, 8450, torch.float32, "mean", float("inf")),
])
def test_a_non_finite_gradient_of_the_last_bag_stays_with_it(D, B, io, pooling, value):
    """The steps behind the batch's end read the last bag's gradient, with counts of zero; 0 * Inf is NaN.  The rows of that bag become
    non-finite, all others get the step they get without it (the sum of the same values in another order: both are within a few units
    of 2^-24 of the sum of up to 2000 lookups' sizes)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE
    R, hot = 400, 90
    g = torch.Generator().manual_seed(D + B)
    lens = torch.randint(2, 9, (B,), generator=g)
    off = torch.zeros(B + 1, dtype=torch.int64)
    off[1:] = torch.cumsum(lens, 0)
    idx = torch.randint(0, hot, (int(off[-1]),), generator=g) * 3
    weights = torch.empty(R * D).uniform_(-0.01, 0.01, generator=g)
    grad = torch.randn(B, D, generator=g).to(io)
    spoilt = grad.clone()
    spoilt[B - 1, D - 3] = value
    tbe = TBE([R], [D], "f32")
    ws = tbe.alloc_workspace(B, idx.numel())
    res = []
    for go in (grad, spoilt):
        w, st = weights.cuda(), torch.ones(R, device="cuda")
        tbe.backward_rowwise_adagrad_ex(go.cuda(), idx.cuda(), off.cuda(), B, w, st, ws, pooling=pooling, lr=0.05, eps=1e-8)
        assert len(tbe.debug_hot_rows(ws, B, idx.numel())[1][0]) == hot
        res.append((w.cpu().view(R, D).double(), st.cpu().double()))
    hit = torch.zeros(R, dtype=torch.bool)
    hit[idx[int(off[B - 1]):]] = True
    (w0, s0), (w1, s1) = res
    assert bool(torch.isfinite(w0).all()) and bool(torch.isfinite(s0).all())
    assert not bool(torch.isfinite(s1[hit]).any())
    torch.testing.assert_close(w1[~hit], w0[~hit], rtol=0.0, atol=0.05 * 1e-5)
    torch.testing.assert_close(s1[~hit], s0[~hit], rtol=1e-5, atol=0.0)
    tbe.close()


@pytest.mark.parametrize("D,B,io", [(48, 65536, torch.float32), (64, 131072, torch.float32), (36, 100_001, torch.float32), (64, 65536, torch.bfloat16)])
def test_the_error_of_a_narrow_dense_row(D, B, io):
    """Rows that every bag holds, N(0,1) gradients, against 64 bits: two accumulators take turns, so that a run is two sums of 256 bags
    and one addition; not more than one running sum of the 512, 5 * 2^-24 with the partial sums' own."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE
    g = torch.Generator(device="cuda").manual_seed(3)
    grad = torch.randn(B, D, generator=g, device="cuda").to(io)
    idx, off = torch.arange(3, device="cuda").repeat(B), torch.arange(0, 3 * B + 1, 3, device="cuda")
    tbe = TBE([3], [D], "f32")
    ws = tbe.alloc_workspace(B, idx.numel())
    w = torch.zeros(3 * D, device="cuda")
    tbe.backward_sgd(grad, idx, off, B, w, ws, lr=1.0)
    assert len(tbe.debug_hot_rows(ws, B, idx.numel())[1][0]) == 3
    want = grad.double().sum(0)
    assert float((w.view(3, D).double() + want).norm() / (3.0 ** 0.5 * want.norm())) < 5.0 * 2.0 ** -24
    tbe.close()


@pytest.mark.parametrize("D,B", [(32, 16641), (64, 8447)])
@pytest.mark.parametrize("scale", [1.0, 1e-20, 1e-28, 1e-33, 1e-36])
@pytest.mark.parametrize("pooling", ["sum", "mean"])
def test_tiny_gradients_of_narrow_rows(D, B, scale, pooling):
    """fp32 gradients whose last bits no bfloat16 can hold, so that a wrong second or third piece shows: B / 10 lookups per row and
    fp32 sums, within 2^-24 * sqrt(B / 10) of the row's norm."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE
    R, L = 60, 6
    g = torch.Generator().manual_seed(8)
    grad = torch.randn(B, D, generator=g) * scale
    idx = torch.randint(0, R, (B * L,), generator=g)
    tbe = TBE([R], [D], "f32")
    ws = tbe.alloc_workspace(B, B * L)
    w = torch.zeros(R * D, device="cuda")
    tbe.backward_sgd(grad.cuda(), idx.cuda(), torch.arange(0, B * L + 1, L).cuda(), B, w, ws, pooling=pooling, lr=1.0)
    assert len(tbe.debug_hot_rows(ws, B, B * L)[1][0]) == R
    want = torch.zeros(R, D, dtype=torch.float64).index_add_(0, idx, grad.double().repeat_interleave(L, 0)) / (L if pooling == "mean" else 1)
    err = (w.cpu().double().view(R, D) + want).norm(dim=1) / want.norm(dim=1)
    assert float(err.max()) < (B / 10) ** 0.5 * 2.0 ** -24
    tbe.close()


@pytest.mark.parametrize("D,B", [(32, 16641), (64, 8447)])
@pytest.mark.parametrize("scale", [1e-3, 2e-5, 3e-7])
def test_subnormal_binary16_gradients_of_narrow_rows(D, B, scale):
    """Multiples of 2^-24, whose sums an fp32 holds exactly while they stay below 1."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE
    R, L = 60, 6
    g = torch.Generator().manual_seed(9)
    grad = (torch.randn(B, D, generator=g) * scale).half()
    grad = torch.round(grad.double() * 2 ** 24).mul(2.0 ** -24).half()
    idx = torch.randint(0, R, (B * L,), generator=g)
    tbe = TBE([R], [D], "f32")
    ws = tbe.alloc_workspace(B, B * L)
    w = torch.zeros(R * D, device="cuda")
    tbe.backward_sgd(grad.cuda(), idx.cuda(), torch.arange(0, B * L + 1, L).cuda(), B, w, ws, lr=1.0)
    assert len(tbe.debug_hot_rows(ws, B, B * L)[1][0]) == R
    want = torch.zeros(R, D, dtype=torch.float64).index_add_(0, idx, grad.double().repeat_interleave(L, 0))
    assert float(want.abs().max()) < 1.0
    assert torch.equal(-w.cpu().double().view(R, D), want)
    tbe.close()
