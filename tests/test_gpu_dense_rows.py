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
