"""Small batches of many tables, which are sorted in one launch while its workgroups need no more rounds of the chip than there would
be passes over digits: one range fewer and one more than that, at one, two and three passes."""
import pytest
import torch

import test_gpu_small_sort as base

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tables,B", [
    ([(2, 60, "uniform")] * 255, 2),                                            # 256 ranges
    ([(2, 60, "uniform")] * 252 + [(3, 60, "near")] * 3, 2),                    # 257
    ([(143, 200, "near")] * 199 + [(215, 200, "two")], 13),                     # 28672 ids: 256 again
    ([(143, 200, "near")] * 199 + [(216, 200, "two")], 13),
    ([(7, 1000, "uniform")] * 300, 4),
    ([(7, 2_000_000, "invalid")] * 300, 4),
    ([(15, 3000, "uniform")] * 500, 3),
    ([(15, 100_000, "uniform")] * 500, 3),                                      # three rounds
    ([(t % 97, 100_000 + t, "near") for t in range(512)], 3),                   # as many tables as go this way
    ([(96, 3000, "near")] * 255 + [(96, 3000, "two")], 13),                     # 24576 ids, two rounds and two passes
    ([(96, 3000, "near")] * 255 + [(97, 3000, "two")], 13),
    ([(31_000, 90_000, "near")] + [(40, 1000, "uniform")] * 255, 20),           # most ids in one of them
])
def test_many_tables(tables, B):
    base.test_sorted_keys_bags_segments_and_long_rows(tables, B, torch.int64)
