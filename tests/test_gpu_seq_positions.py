"""The non-pooled lookup with 64, 32, 16, 8 and 4 positions per wavefront, in batches on both sides of what a rule takes as small."""
import pytest
import torch

import test_gpu_seq_windows as windows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,D,dtype", [
    ([70001, 61070], [16, 16], "f32"),                  # 131071 positions and less: small where rows have more than 4 fragments
    ([70001, 61071, 3], [32, 32, 32], "f32"),
    ([30000, 35537], [128, 128], "f32"),
    ([30000, 35531, 1, 3], [128, 136, 120, 128], "f32"),
    ([20001, 12766], [256, 256], "f16"),
    ([20001, 12768, 7], [256, 264, 248], "f16"),
    ([9000, 1, 7390], [256, 512, 8], "f32"),            # 16391: on either side of 8 positions
    ([3000, 0, 5180, 13], [1024, 8, 1024, 1024], "f32"),
    ([33, 65, 2], [1024, 512, 1016], "f16"),
    ([15] * 40, [1024, 16] * 20, "f32"),                # windows across tables of two widths
])
@pytest.mark.parametrize("io", [torch.float32, torch.bfloat16])
def test_positions_per_wavefront(n, D, dtype, io):
    windows.test_rows_in_order_of_position(n, D, dtype, io)
