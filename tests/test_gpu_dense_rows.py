"""Rows reduced on the matrix cores (the hottest rows of a large gradient block) at the borders of that kernel: blocks of 256
bags and runs of them that do not divide the batch, column groups of 64 and 256, up to 32 / 64 / 128 rows and one more,
counts above 255 and above 65535 in one bag - against the oracle, with the harness's tolerances (fp32 sums of exact
products; the row's own sum error where it has thousands of lookups)."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,D,B,hot,repeat,dtype,pooling,io", [
    ([300, 40], [256, 24], 2305, 33, 0, "f32", "sum", "f32"),       # 9 blocks + 1 bag, 32 + 1 rows; the narrow table has no dense rows
    ([500], [64], 8300, 64, 0, "f16", "mean", "f32"),               # a wavefront per quarter of the bags
    ([400], [136], 8449, 65, 0, "f32", "sum", "bf16"),              # columns in the middle of a 64-column group
    ([400], [520], 1100, 31, 0, "f16", "sum", "f16"),               # three column blocks, binary16 pieces
    ([600], [32], 20001, 129, 0, "f32", "mean", "bf16"),            # several blocks per run, more hot rows than the kernel takes
    ([50], [128], 4200, 20, 300, "f32", "sum", "f32"),              # one bag holds an id 300 times: counts in two bytes
    # ... and 70000 times: counted in rounds (sum pooling: the harness bounds the forward sum of so long a bag for it only)
    ([50], [128], 4200, 20, 70000, "f32", "sum", "f16"),
])
def test_dense_rows_at_the_borders(rows, D, B, hot, repeat, dtype, pooling, io):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_harness as H
    from paper_2508_03854_amd import TBE
    rng = np.random.default_rng(B + hot)
    cfg = W.Config("dense", rows, D, dtype, B, pooling, ("fixed", 1), ("uniform",))
    cfg.c, cfg.lr, cfg.eps = 2.0, 0.05, 1e-8
    lens = rng.integers(2, 9, size=len(rows) * B)
    if repeat:
        lens[B // 2] += repeat
    off = torch.zeros(len(lens) + 1, dtype=torch.int64)
    off[1:] = torch.cumsum(torch.as_tensor(lens), 0)
    ids = []
    for t, R in enumerate(rows):
        n = int(lens[t * B:(t + 1) * B].sum())
        pick = rng.integers(0, min(hot, R), size=n) * 7 % R          # the hot rows, scattered; a tenth of the ids cold
        ids.append(np.where(rng.random(n) < 0.9, pick, rng.integers(0, R, size=n)))
    idx = torch.as_tensor(np.concatenate(ids))
    if repeat:
        idx[int(off[B // 2]):int(off[B // 2]) + repeat] = 7
    tabs = H.host_tables(cfg)
    flat = H.flat_from_tables(tabs)
    st = W.state_rows(cfg, torch.arange(cfg.total_rows)).numpy()
    state = torch.from_numpy(st.copy()).cuda()
    tbe = TBE(cfg.rows, cfg.D, dtype)
    ws = tbe.alloc_workspace(B, idx.numel())
    gout = torch.randn(B, cfg.sum_D, generator=torch.Generator().manual_seed(3))
    rep = H.check_step(cfg, tbe, flat, state, tabs, st, idx, off, gout, ws, index_dtype=torch.int32, io=io)
    assert rep["max_seg"] > 64
    tbe.close()


@pytest.mark.parametrize("D,dtype,pooling,io,value", [
    (128, "f32", "sum", torch.float32, float("inf")),
    (520, "f16", "mean", torch.bfloat16, float("nan")),            # three column blocks
    (136, "f32", "sum", torch.float16, float("-inf")),
])
def test_a_non_finite_gradient_stays_with_its_own_bag(D, dtype, pooling, io, value):
    """One element of one bag's gradient is not finite: the rows of that bag become so, all others get the step they get
    without it (the sum of the same values in another order: both are within a few units of 2^-24 of the lookups' sum, a
    binary16 weight may round to its neighbour)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE
    B, R, hot = 4500, 400, 60
    g = torch.Generator().manual_seed(D)
    lens = torch.randint(2, 9, (B,), generator=g)
    off = torch.zeros(B + 1, dtype=torch.int64)
    off[1:] = torch.cumsum(lens, 0)
    idx = torch.randint(0, hot, (int(off[-1]),), generator=g) * 7 % R
    bag = B // 3
    weights = torch.empty(R * D).uniform_(-0.01, 0.01, generator=g)
    grad = torch.randn(B, D, generator=g).to(io)
    spoilt = grad.clone()
    spoilt[bag, D - 3] = value
    tbe = TBE([R], [D], dtype)
    ws = tbe.alloc_workspace(B, idx.numel())
    res = []
    for go in (grad, spoilt):
        w, st = weights.to(tbe.torch_dtype).cuda(), torch.ones(R, device="cuda")
        tbe.backward_rowwise_adagrad_ex(go.cuda(), idx.cuda(), off.cuda(), B, w, st, ws, pooling=pooling, lr=0.05, eps=1e-8)
        res.append((w.cpu().view(R, D).double(), st.cpu().double()))
    hit = torch.zeros(R, dtype=torch.bool)
    hit[idx[int(off[bag]):int(off[bag + 1])]] = True
    assert 0 < int(hit.sum()) < hot
    (w0, s0), (w1, s1) = res
    assert bool(torch.isfinite(w0).all()) and bool(torch.isfinite(s0).all())
    assert not bool(torch.isfinite(s1[hit]).any())
    atol = 0.05 * 1e-5 + (2.0 ** -14 if dtype == "f16" else 0.0)
    torch.testing.assert_close(w1[~hit], w0[~hit], rtol=0.0, atol=atol)
    torch.testing.assert_close(s1[~hit], s0[~hit], rtol=1e-5, atol=0.0)
    tbe.close()


@pytest.mark.parametrize("D,B", [(256, 65536), (128, 65536), (32, 262144)])
def test_the_error_of_a_dense_row_is_that_of_short_sums(D, B):
    """Rows that every bag holds, N(0,1) gradients, relative error of the summed gradient against 64 bits.

    A running fp32 sum of magnitude v rounds with an error of about 0.42 * 2^-24 * v per addition (uniform over a unit in the
    last place that is 2^-23 to 2^-22 of v).  The matrix core rounds once for 8 bags, and a run has 512, at magnitudes of
    sqrt(8 i): 54 * 2^-24 per run.  The B / 512 runs of a row of norm sqrt(B) come to 54 / sqrt(512) = 2.4 * 2^-24 of it, the sums of
    run sums to 1 to 1.5 more, and the smaller pieces of an element round a second time: 4 in all (measured 3.98, 4.29, 4.26).
    One sum over the whole chunk of 2048 bags and more would be at 5.5 to 7."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE
    g = torch.Generator(device="cuda").manual_seed(3)
    grad = torch.randn(B, D, generator=g, device="cuda")
    idx, off = torch.arange(3, device="cuda").repeat(B), torch.arange(0, 3 * B + 1, 3, device="cuda")
    tbe = TBE([3], [D], "f32")
    ws = tbe.alloc_workspace(B, idx.numel())
    w = torch.zeros(3 * D, device="cuda")
    tbe.backward_sgd(grad, idx, off, B, w, ws, lr=1.0)
    assert len(tbe.debug_hot_rows(ws, B, idx.numel())[1][0]) == 3
    want = grad.double().sum(0)
    assert float((w.view(3, D).double() + want).norm() / (3.0 ** 0.5 * want.norm())) < 5.0 * 2.0 ** -24
    tbe.close()


@pytest.mark.parametrize("scale", [1.0, 1e-20, 1e-28, 1e-33, 1e-36])
@pytest.mark.parametrize("pooling", ["sum", "mean"])
def test_tiny_gradients_keep_their_precision(scale, pooling):
    """fp32 gradients whose last bits no bfloat16 can hold: the rows' sums stay as good as at N(0,1).  400 lookups per row and
    fp32 sums: within 2^-24 * sqrt(400) of the row's norm, where the pieces alone would leave 5e-5 and 7e-4 at 1e-36."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE
    B, R, D, L = 4200, 60, 128, 6
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
    assert float(err.max()) < 20.0 * 2.0 ** -24
    tbe.close()


@pytest.mark.parametrize("scale", [1e-3, 2e-5, 3e-7])
def test_subnormal_binary16_gradients_are_summed_exactly(scale):
    """binary16 has its subnormals below 6.1e-5, ordinary values in mixed-precision training: multiples of 2^-24 whose sums an
    fp32 holds exactly while they stay below 1."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE
    B, R, D, L = 4200, 60, 128, 6
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
    assert torch.equal(-w.cpu().double().view(R, D), want)
    tbe.close()
