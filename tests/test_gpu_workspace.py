"""A workspace made for a batch serves every smaller one: the size never shrinks when the batch or its lookups grow, on both
sides of every border at which the sort or the dense rows change their layout."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,D", [([4000] * 4, 1024), ([100_000] * 64, 128), ([50], 4), ([30_000] * 200, 8)])
def test_workspace_grows_with_the_batch(rows, D):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE
    tbe = TBE(rows, [D] * len(rows), "f32")
    batches = [1, 1023, 1024] + [256 * k + e for k in (4, 8, 16, 17, 32, 33, 41, 64, 65, 130) for e in (0, 1)]
    borders = [131072, 393216, 1572864, 1 << 21, 32 * 1024 * len(rows), 32 * 2048 * len(rows), 4 * 32 * 2048 * len(rows), 8192 * 4096]
    lookups = sorted({1} | {n + e for n in borders for e in (0, 1, 4097)})
    size = {(B, n): tbe.workspace_bytes(B, n) for B in batches for n in lookups}
    for n in lookups:
        for small, large in zip(batches, batches[1:]):
            assert size[small, n] <= size[large, n], (n, small, large)
    for B in batches:
        for small, large in zip(lookups, lookups[1:]):
            assert size[B, small] <= size[B, large], (B, small, large)
    tbe.close()


@pytest.mark.parametrize("D,B,per_bag", [([128] * 32, 16384, 1), ([32] * 31 + [1024], 4096, 1), ([1024] * 32, 16384, 1), ([256] * 64, 4096, 2)])
def test_dense_rows_of_a_batch_with_few_lookups_take_a_bounded_share_of_memory(D, B, per_bag):
    """Their partial sums depend on the tables' columns alone: bounded by 20 bytes per lookup and 16 MiB, or the fixed array's
    size, over what the batch needs for its streams and parts."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE, binding
    tbe = TBE([100_000] * len(D), D, "f32")
    n = len(D) * B * per_bag
    lean = 20.5 * n + 4 * (n // 192 + 4096 + 512 * len(D)) * max(D)
    bound = lean + 20 * n + (16 << 20)
    assert tbe.workspace_bytes(B, n) <= (min(bound, binding.STATIC_SCRATCH_BYTES) if lean <= binding.STATIC_SCRATCH_BYTES else bound)
    tbe.close()


def test_a_smaller_last_batch_uses_the_same_workspace():
    """33 blocks of bags in runs of two, then 32 blocks one by one: the second needs more partial sums, in the same memory."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE
    R, D, L = 300, 1024, 6
    tbe = TBE([R], [D], "f32")
    ws = tbe.alloc_workspace(33 * 256, 33 * 256 * L)
    B = 32 * 256
    g = torch.Generator().manual_seed(5)
    idx = torch.randint(0, 40, (B * L,), generator=g)
    grad = torch.randn(B, D, generator=g)
    w, st = torch.zeros(R * D, device="cuda"), torch.ones(R, device="cuda")
    tbe.backward_rowwise_adagrad(grad.cuda(), idx.cuda(), torch.arange(0, B * L + 1, L).cuda(), B, w, st, ws, lr=1.0, eps=0.0)
    ref = torch.zeros(R, D, dtype=torch.float64).index_add_(0, idx, grad.double().repeat_interleave(L, 0))
    v = 1.0 + (ref * ref).sum(1)
    # about 1200 fp32 additions of unit values per element: sums around 35, good to 1e-4 of the largest; then / sqrt(v) of 1100
    torch.testing.assert_close(st.cpu().double(), v, rtol=1e-5, atol=0.0)
    torch.testing.assert_close(w.cpu().double().view(R, D), -ref / v.sqrt()[:, None], rtol=0.0, atol=1e-5)
    tbe.close()


@pytest.mark.parametrize("T,B,L", [(2, 5399, 8), (12, 6478, 12), (6, 4756, 7), (1, 32768, 3)])
def test_a_small_batch_shares_its_bags_out_as_far_as_is_useful(T, B, L):
    """One chunk of partial sums per block of 256 bags, up to 32: with fewer workgroups the dense rows of a batch that does not
    fill the chip anyway take as many times longer."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE
    tbe = TBE([500_000] * T, [256] * T, "f32")
    chunks = 4 * 128 * 256 * T * min((B + 255) // 256, 32)
    assert tbe.workspace_bytes(B, T * B * L) >= chunks + 16 * T * B * L
    tbe.close()
