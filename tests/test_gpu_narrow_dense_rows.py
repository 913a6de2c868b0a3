"""Dense rows of tables of up to 64 columns: both column groupings, up to 32 / 64 / 96 / 128 rows and one more, short last blocks and
chunks, counts in two bytes and in rounds.  Gradients are small integers and bag lengths under mean pooling powers of two, so that
every sum is exact in fp32 (below 2^24 units) and has to equal the 64-bit one."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,B,rows,repeat,pooling,io", [
    (32, 16640, 128, 0, "sum", torch.float32),                     # whole blocks
    (32, 16641, 33, 0, "mean", torch.float16),                     # a last block of one bag
    (28, 20000, 97, 300, "sum", torch.float32),
    (4, 131373, 32, 0, "mean", torch.float32),
    (36, 15000, 64, 300, "sum", torch.bfloat16),                   # the second group of columns has four
    (64, 8447, 65, 0, "mean", torch.bfloat16),
    (64, 8450, 129, 70000, "sum", torch.float16),
    (48, 12289, 20, 70000, "sum", torch.float32),
])
def test_exact_sums(D, B, rows, repeat, pooling, io):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE
    dev, other = "cuda", 12
    g = torch.Generator(device=dev).manual_seed(D + rows)
    lens = 2 ** torch.randint(1, 4, (2 * B,), generator=g, device=dev)
    lens[B + B // 2] += repeat                                     # the second table is the narrow one
    off = torch.zeros(2 * B + 1, dtype=torch.int64, device=dev)
    torch.cumsum(lens, 0, out=off[1:])
    first = int(off[B])
    n = int(off[-1])
    idx = torch.randint(0, 3, (n,), generator=g, device=dev)
    idx[first:] = torch.randint(0, rows, (n - first,), generator=g, device=dev) * 3
    if repeat:
        at = int(off[B + B // 2])
        idx[at:at + repeat] = 3
    grad = torch.randint(-3, 4, (B, other + D), generator=g, device=dev).to(io)
    tbe = TBE([3, 3 * rows], [other, D], "f32")
    ws = tbe.alloc_workspace(B, n)
    w = torch.zeros(tbe.total_elems, device=dev)
    tbe.backward_sgd(grad, idx, off, B, w, ws, pooling=pooling, lr=1.0)
    assert len(tbe.debug_hot_rows(ws, B, n)[1][1]) == min(rows, 128)
    bag = torch.repeat_interleave(torch.arange(2 * B, device=dev), lens)[first:] - B
    rows_grad = grad[:, other:].double()
    if pooling == "mean":
        rows_grad = rows_grad / lens[B:, None]
    want = torch.zeros(3 * rows, D, dtype=torch.float64, device=dev).index_add_(0, idx[first:], rows_grad[bag])
    assert torch.equal(-w[3 * other:].view(3 * rows, D).double(), want)
    tbe.close()
