"""The one-launch sort of small batches where nearly all lookups are one table's: keys in LDS up to 31 per thread, in registers behind
them, up to the most that a batch of several tables may hold - against the library's stable sort, bit for bit."""
import pytest
import torch

import test_gpu_small_sort as base

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("idt", [torch.int64, torch.int32])
@pytest.mark.parametrize("rows,kind", [(90_000, "uniform"), (90_000, "near"), (5_000_000, "near"), (2000, "two"), (3, "uniform"), (77, "one"),
                                       (40_000, "invalid")])
@pytest.mark.parametrize("n", [12_289, 31_744, 31_745, 40_000, 64_513, 65_536])
def test_one_long_segment_among_short_ones(n, rows, kind, idt):
    short = [(0 if n > 65_000 else 7 * t, 500, "uniform") for t in range(7)]
    tables = short[:3] + [(n, rows, kind)] + short[3:] + [(65_536 - n if n > 65_000 else 1, 10, "uniform")]
    base.test_sorted_keys_bags_segments_and_long_rows(tables, 150, idt)


@pytest.mark.parametrize("a,b", [(32_000, 33_000), (16_384, 49_152), (1, 65_535)])
def test_two_long_segments(a, b):
    tables = [(a, 70_000, "near")] + [(0, 9, "one")] * 6 + [(b, 1_000_000, "near")]
    base.test_sorted_keys_bags_segments_and_long_rows(tables, 1000, torch.int64)
