"""Row updates of the smallest batches of wide rows: with few lookups per table a row is cut into finer parts than the shortest row
that is cut at all."""
import pytest
import torch

from test_gpu_exact_updates import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 3])
@pytest.mark.parametrize("D", [132, 256, 260, 1024])
@pytest.mark.parametrize("each", [300, 512, 513])
def test_rows_on_both_sides_of_a_long_one(T, D, each):
    """Rows of one lookup fewer and more than 16, 32 and 64, with as many lookups per table as keep rows of 64 whole, and one more."""
    dev = "cuda"
    g = torch.Generator(device=dev).manual_seed(each + D)
    ids, lens = [], []
    for t in range(T):
        spans = ([17, 64, 65, 80], [16, 33, 63, 66, 96], [15, 32, 129])[t % 3]
        fixed = torch.cat([torch.full((s,), 7 * i + t, device=dev) for i, s in enumerate(spans)])
        more = torch.randint(200, 4000, (each - fixed.numel(),), generator=g, device=dev)
        ids.append(torch.cat([fixed, more])[torch.randperm(each, generator=g, device=dev)])
        lens.append(torch.bincount(torch.randint(0, 64, (each,), generator=g, device=dev), minlength=64))
    check(T, 4000, D, 64, torch.cat(lens), torch.cat(ids), seed=each)
