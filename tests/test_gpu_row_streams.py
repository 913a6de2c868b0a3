"""Row updates past the caches: rows that fill whole 64-byte pieces, rows that do not, wide ones, and tables that begin inside a piece.
SGD of learning rate 1 on zero weights, small integers as gradients: every sum is exact."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,dtype,rows", [
    ([16], "f32", 4_600_000),
    ([20, 12], "f32", 2_300_000),
    ([12, 32], "f32", 1_700_003),              # the second table begins 16 bytes into a piece
    ([100, 104, 108], "f32", 240_001),
    ([24, 32], "f16", 2_600_001),
    ([128, 136], "f16", 530_001),
])
def test_rows_of_every_alignment(D, dtype, rows):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE
    dev, T = "cuda", len(D)
    size = 4 if dtype == "f32" else 2
    n = rows // 5 * 5                          # lookups per table, five to a bag, each of a row of its own but for one in a hundred
    B = n // 5
    assert rows * sum(D) * size * 0.98 > 256 << 20
    g = torch.Generator(device=dev).manual_seed(sum(D))
    ids = []
    for _ in D:
        i = torch.randperm(rows, generator=g, device=dev)[:n]
        i[::100] = i[1::100]
        ids.append(i)
    grad = torch.randint(-3, 4, (B, sum(D)), generator=g, device=dev).half()
    off = torch.arange(0, T * n + 1, 5, device=dev)
    tbe = TBE([rows] * T, D, dtype)
    ws = tbe.alloc_workspace(B, T * n)
    w = torch.zeros(tbe.total_elems, device=dev, dtype=tbe.torch_dtype)
    tbe.backward_sgd(grad, torch.cat(ids), off, B, w, ws, lr=1.0)
    at = col = 0
    for d, i in zip(D, ids):
        want = torch.zeros(rows, d, device=dev)
        want.index_add_(0, i, grad[:, col:col + d].float().repeat_interleave(5, 0))
        assert torch.equal(-w[at:at + rows * d].view(rows, d).float(), want)
        at, col = at + rows * d, col + d
    tbe.close()
