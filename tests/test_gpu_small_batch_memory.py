"""Small batches of wide rows cut their long rows finer, which takes more memory for partial sums - but never a batch its place in the
fixed scratch array, and the size of a workspace still never shrinks when the batch or its lookups grow."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def small_steps(T):
    """Lookups on both sides of every border of the finer parts, and beyond them as far as they are felt."""
    borders = [4096 * T, 8192 * T, 12288, 28247, 32768, 40000, 62740, 65536, 131072]
    return sorted({1, 2000} | {n + e for n in borders if n <= 140_000 for e in (-1, 0, 1)})


@pytest.mark.parametrize("T,D,B,fit", [(30, 912, 1024, 28247), (32, 840, 1024, 62740), (31, 880, 1024, 40000), (2, 1024, 20, 16384), (30, 200, 3000, 65536)])
def test_batches_that_fit_the_scratch_array_with_coarse_parts_still_do(T, D, B, fit):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE, binding
    tbe = TBE([2000] * T, [D] * T, "f32")
    size = {n: tbe.workspace_bytes(B, n) for n in small_steps(T)}
    lookups = sorted(size)
    for small, large in zip(lookups, lookups[1:]):
        assert size[small] <= size[large], (small, large)
        assert tbe.workspace_bytes(B, large) <= tbe.workspace_bytes(B + 1, large)
    assert size[fit] <= binding.STATIC_SCRATCH_BYTES
    tbe.close()


def test_static_backward_at_the_end_of_the_scratch_array():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE
    T, R, D, B, N = 30, 2000, 912, 1024, 28247
    tbe = TBE([R] * T, [D] * T, "f32")
    g = torch.Generator().manual_seed(3)
    off = torch.zeros(T * B + 1, dtype=torch.int64)
    torch.cumsum(torch.bincount(torch.randint(0, T * B, (N,), generator=g), minlength=T * B), 0, out=off[1:])
    # a third of the lookups on three rows of each table: long rows at either size of the parts
    idx = torch.where(torch.rand(N, generator=g) < 0.33, torch.randint(0, 3, (N,), generator=g), torch.randint(0, R, (N,), generator=g))
    grad = torch.randn(B, T * D, generator=g).cuda()
    w0, s0 = torch.randn(T * R * D, generator=g).cuda(), torch.rand(T * R, generator=g).cuda()
    got = []
    for static in (True, False):
        w, s = w0.clone(), s0.clone()
        args = (grad, idx.cuda(), off.cuda(), B, w, s)
        if static:
            tbe.backward_rowwise_adagrad_static(*args, lr=0.1, eps=1e-8)
        else:
            tbe.backward_rowwise_adagrad(*args, tbe.alloc_workspace(B, N), lr=0.1, eps=1e-8)
        got.append((w, s))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    key = torch.searchsorted(off, torch.arange(N), right=True) - 1
    table, bag = key // B, key % B
    gsum = torch.zeros(T, R, D, dtype=torch.float64, device="cuda")
    gsum.index_put_((table.cuda(), idx.cuda()), grad.view(B, T, D).cuda()[bag.cuda(), table.cuda()].double(), accumulate=True)
    # sums of up to 110 terms of size 1 in fp32
    v = s0.double() + (gsum * gsum).sum(2).flatten()
    torch.testing.assert_close(got[0][1].double(), v, rtol=2e-5, atol=1e-6)
    tbe.close()
