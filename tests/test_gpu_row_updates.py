"""Row updates at the borders of their short-row rounds: rows of 1 to 9 lookups and around 64 next to each other, so that a
round's slots, the windows of 64 lookups and the whole-wavefront path all start and end between and inside them; one row per
wavefront and several, tables that end inside a pass, and 16 tables or more, whose rows the dies take in long spans - against the
oracle, with the harness's tolerances.  A wavefront takes a pass of as few rows as fill the chip, 1 to 8 in the small batches of
the first test; passes of 16 rows, in which rounds share a window, and wavefronts of several passes need the many rows of the
second."""
import ctypes

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

COUNTS = [1, 1, 2, 3, 4, 5, 1, 6, 7, 8, 9, 1, 1, 1, 30, 33, 1, 62, 2, 63, 64, 65, 1, 66, 12, 13]


@pytest.mark.parametrize("T,rows,widths,dtype,pooling,io", [
    (1, 3000, [256], "f16", "sum", "f32"),            # one row per wavefront, the variant of fewer wavefronts
    (1, 3000, [200], "f16", "mean", "f32"),           # ... lanes without a column
    (2, 1500, [136, 256], "f32", "mean", "bf16"),
    (3, 1111, [128, 20, 64], "f32", "sum", "f32"),
    (16, 203, [64, 8, 256], "f16", "sum", "bf16"),    # tables of too different widths for long spans
    (18, 180, [64, 40, 128], "f32", "sum", "f32"),    # long spans
    (23, 97, [32, 128, 4], "f32", "mean", "f16"),
    (40, 13, [16, 136], "f16", "mean", "f16"),        # fewer rows than a pass takes
])
def test_rows_of_few_lookups(T, rows, widths, dtype, pooling, io):
    rep = _step(T, rows, widths, dtype, pooling, io, COUNTS)
    assert rep["max_seg"] >= 64 or rows < 26


# as many rows of 1 to 3 lookups as leave COUNTS a sixth of the rows
FEW = [1, 1, 2, 1, 3] * 26 + COUNTS


def _rows_per_pass(U, max_d, wavefronts):
    """The rows of one pass of seg_update_kernel: 32 in batches of very many rows or narrow ones, else 16, halved while wavefronts
    would have less than two passes, down to the rows of the widest table that lie side by side in a wavefront."""
    if U // wavefronts >= (128 if max_d <= 8 else 2048):
        return 32
    least = 1 if max_d > 128 else 2 if max_d > 64 else 4 if max_d > 32 else 8
    rows = 16
    while rows > least and U // rows < 2 * wavefronts:
        rows //= 2
    return rows


@pytest.mark.parametrize("T,rows,widths,dtype,pooling,io,per_pass,spans", [
    (1, 245000, [256], "f16", "sum", "f32", 16, False),          # 7 wavefronts per SIMD: the weights ahead of the gradients
    (1, 245000, [200], "f16", "mean", "f32", 16, False),         # ... mean pooling, lanes without a column
    (2, 133000, [256, 136], "f16", "mean", "bf16", 16, False),   # 8 wavefronts per SIMD, one row per round
    (2, 133000, [128, 64], "f32", "mean", "f32", 16, False),     # 2 and 4 rows per round
    (3, 88000, [20, 8, 4], "f32", "sum", "f16", 16, False),      # 8, 32 and 64
    (3, 350500, [8, 4, 8], "f32", "sum", "f32", 32, False),      # passes of 32 rows, 32 and 64 side by side
    (17, 15700, [64, 64, 104], "f16", "sum", "bf16", 16, True),  # long spans that end inside tables
    (16, 8500, [136, 256], "f32", "mean", "f32", 8, True),       # ... of passes of 8 rows
])
def test_passes_of_many_rows(T, rows, widths, dtype, pooling, io, per_pass, spans):
    D = [widths[t % len(widths)] for t in range(T)]
    seven = dtype == "f16" and io == "f32" and 2 * sum(r for r, d in zip([rows] * T, D) if d > 128) > rows * T
    rep = _step(T, rows, widths, dtype, pooling, io, FEW)
    assert _rows_per_pass(rep["U"], max(D), 7168 if seven else 8192) == per_pass
    assert spans == (T >= 16 and max(D) * T <= 2 * sum(D) and 700 * sum(D) * (4 if io == "f32" else 2) <= T * (3 << 19))


@pytest.mark.parametrize("D,dtype,wavefronts", [
    (136, "f16", 7168),   # one row per round, the variant of fewer wavefronts: one pass at a time
    (12, "f32", 8192),    # 16 rows per round, two passes at a time
])
def test_passes_of_very_many_rows(D, dtype, wavefronts):
    """Passes of 32 rows, against the step in 64 bits: every row once, every seventh a second time."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE
    R, B, lr, eps, c = 2048 * wavefronts + 77, 1000, 0.01, 1e-8, 2.0
    assert _rows_per_pass(R, D, wavefronts) == 32
    g = torch.Generator(device="cuda").manual_seed(D)
    idx = torch.cat([torch.arange(R, device="cuda"), torch.arange(0, R, 7, device="cuda")])
    idx = idx[torch.randperm(idx.numel(), generator=g, device="cuda")]
    off = (torch.arange(B + 1, device="cuda", dtype=torch.int64) * idx.numel()) // B
    tbe = TBE([R], [D], dtype)
    tables = torch.empty(R * D, device="cuda").uniform_(-0.01, 0.01, generator=g).to(tbe.torch_dtype)
    state = torch.rand(R, generator=g, device="cuda") + 1.0
    grad = torch.randn(B, D, generator=g, device="cuda")
    w0, v0 = tables.view(R, D).clone(), state.clone()
    tbe.backward_rowwise_adagrad(grad, idx, off, B, tables, state, tbe.alloc_workspace(B, idx.numel()), pooling="sum", lr=lr, eps=eps,
                                 momentum_scale=c)
    assert not tbe.poll_index_error()
    order = torch.sort(idx, stable=True).indices
    bag = torch.searchsorted(off, order, right=True) - 1
    per_row = torch.ones(R, dtype=torch.int64, device="cuda")
    per_row[::7] = 2
    start = torch.cumsum(per_row, 0) - per_row
    g64, w1 = grad.double(), tables.view(R, D)
    for lo in range(0, R, 1 << 20):
        r = slice(lo, min(R, lo + (1 << 20)))
        two = per_row[r] == 2
        s = g64[bag[start[r]]]
        s[two] += g64[bag[start[r][two] + 1]]
        v = v0[r].double() + (s * s).sum(1)
        step = lr / (torch.sqrt(v / c) + eps)
        want = w0[r].double() - step[:, None] * s
        # moments: a sum of D squares in 32 bits; weights: 1e-5 of the row's step and the rounding to the table's type
        assert ((state[r].double() - v).abs() <= D * 2.0 ** -24 * v).all()
        bound = 1e-5 * step[:, None] * s.abs().amax(1, keepdim=True) + (2.0 ** -23 if dtype == "f32" else 2.0 ** -11) * want.abs() + 2.0 ** -25
        assert ((w1[r].double() - want).abs() <= bound).all()
    tbe.close()


def _step(T, rows, widths, dtype, pooling, io, counts):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_harness as H
    from paper_2508_03854_amd import TBE
    rng = np.random.default_rng(T * 1000 + rows)
    B = 700
    cfg = W.Config("rows", [rows + 5 * (t % 3) for t in range(T)], [widths[t % len(widths)] for t in range(T)], dtype, B, pooling,
                   ("fixed", 1), ("uniform",))
    cfg.c, cfg.lr, cfg.eps = 2.0, 0.01, 1e-8
    ids, lens = [], []
    for R in cfg.rows:
        of_table = np.repeat(np.arange(R), np.resize(np.roll(counts, int(rng.integers(len(counts)))), R))
        ids.append(rng.permutation(of_table))
        cuts = np.sort(rng.integers(0, len(of_table) + 1, size=B - 1))
        lens.append(np.diff(np.concatenate(([0], cuts, [len(of_table)]))))
    off = torch.zeros(T * B + 1, dtype=torch.int64)
    off[1:] = torch.cumsum(torch.as_tensor(np.concatenate(lens)), 0)
    idx = torch.as_tensor(np.concatenate(ids))
    tabs = H.host_tables(cfg)
    flat = H.flat_from_tables(tabs)
    st = W.state_rows(cfg, torch.arange(cfg.total_rows)).numpy()
    state = torch.from_numpy(st.copy()).cuda()
    tbe = TBE(cfg.rows, cfg.D, dtype)
    ws = tbe.alloc_workspace(B, idx.numel())
    gout = torch.randn(B, cfg.sum_D, generator=torch.Generator().manual_seed(T))
    rep = H.check_step(cfg, tbe, flat, state, tabs, st, idx, off, gout, ws, io=io)
    tbe.close()
    return rep


@pytest.mark.parametrize("T,B,rows,lookups,hot", [
    (16, 100, (50, 4000), 2500, 0),           # ascending sizes, no long row
    (26, 300, (20000, 30), 9000, 40),         # descending
    (16, 200, (150, 9000), 20000, 145),       # more long rows than lie in LDS at a time
    (20, 64, (3, 3), 10, 0),                  # fewer rows than a pass
    (4100, 7, (30, 20), 24, 0),               # more tables than the lists take one by one
])
def test_long_spans_of_equal_work(T, B, rows, lookups, hot):
    """The borders of the long spans, as the batch's lists hold them: a row weighs 16 lookups and its own, long rows only the 16."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE
    rng = np.random.default_rng(T * B)
    R = [round(rows[0] * (rows[1] / rows[0]) ** (t / (T - 1))) for t in range(T)]
    ids = []
    for r in R:
        h = min(hot, r)
        few = rng.integers(0, r, size=lookups - 130 * h)
        ids.append(rng.permutation(np.concatenate([np.repeat(rng.permutation(r)[:h], 130), few])))
    idx = torch.as_tensor(np.concatenate(ids)).cuda()
    off = torch.cat([torch.arange(B) * lookups // B + t * lookups for t in range(T)] + [torch.tensor([T * lookups])]).cuda()
    tbe = TBE(R, [64] * T, "f32")
    ws = tbe.alloc_workspace(B, idx.numel())
    tbe.backward_prepare(idx, off, B, ws)
    n = idx.numel()
    dev = tbe.debug_sorted_device(ws, B, n)
    ptrs = [ctypes.c_void_p() for _ in range(5)]
    assert tbe._lib.tbe_debug_sorted(tbe._h, ws.data_ptr(), B, n, *[ctypes.byref(p) for p in ptrs]) == 0
    at = ptrs[4].value - ws.data_ptr()   # the number of unique rows heads the counters: borders from word 16 on
    words = ws[at:at + 128].view(torch.int32).cpu().numpy().astype(np.int64)
    U = int(words[0])
    start = dev["seg_start"].cpu().numpy()
    length = np.diff(start)
    long_min = 64 if n <= 1 << 17 else 128 if n <= 3 << 17 else 256
    if hot:
        assert (length > long_min).sum() >= hot * T * 0.9
    weight = np.concatenate(([0], np.cumsum(16 + np.where(length > long_min, 0, length))))
    want = [int(np.searchsorted(weight, weight[-1] * q // 16)) for q in range(16)]
    assert words[16:32].tolist() == want
    tbe.close()
