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


@pytest.mark.parametrize("D,N,spans", [
    (260, 12288, [[1023, 1024, 1025, 1026], [2048, 2000], [4090]]),            # 64 parts of 16 lookups, and of 64
    (1024, 12288, [[4096], [4000, 65], [17, 33, 65, 1100]]),
    (132, 24576, [[2047, 2048, 2049], [4095, 4033], [8000]]),                  # of 32 lookups
    (256, 8192, [[4096, 4000]]),
    (132, 65536, [[60000], [2100], []] + [[]] * 6),
])
def test_rows_of_many_fine_parts(D, N, spans):
    """Rows that have as many fine parts as a row may have, one more, and so many that coarse ones are more."""
    dev, T = "cuda", len(spans)
    g = torch.Generator(device=dev).manual_seed(N + D)
    ids, lens = [], []
    left = N - sum(map(sum, spans))
    for t in range(T):
        fixed = [torch.full((s,), 7 * i + t, device=dev) for i, s in enumerate(spans[t])]
        more = min(left, N // T // 3 + 5) if t < T - 1 else left
        left -= more
        all_ids = torch.cat(fixed + [torch.randint(200, 4000, (more,), generator=g, device=dev)])
        n = all_ids.numel()
        ids.append(all_ids[torch.randperm(n, generator=g, device=dev)])
        lens.append(torch.bincount(torch.randint(0, 64, (n,), generator=g, device=dev), minlength=64))
    check(T, 4000, D, 64, torch.cat(lens), torch.cat(ids), seed=N)
