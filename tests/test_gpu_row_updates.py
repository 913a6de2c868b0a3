"""Row updates at the borders of their short-row rounds: rows of 1 to 9 lookups and around 64 next to each other, so that a
round's slots, the windows of 64 lookups and the whole-wavefront path all start and end between and inside them; one row per
wavefront and several, tables that end inside a pass, and 16 tables or more, whose rows the dies take in long spans - against the
oracle, with the harness's tolerances."""
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
    (16, 203, [64, 8, 256], "f16", "sum", "bf16"),    # long spans
    (23, 97, [32, 128, 4], "f32", "mean", "f16"),
    (40, 13, [16, 136], "f16", "mean", "f16"),        # fewer rows than a pass takes
])
def test_rows_of_few_lookups(T, rows, widths, dtype, pooling, io):
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
        of_table = np.repeat(np.arange(R), np.resize(np.roll(COUNTS, int(rng.integers(len(COUNTS)))), R))
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
    assert rep["max_seg"] >= 64 or rows < 26
    tbe.close()
