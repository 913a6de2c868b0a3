"""The non-pooled lookup's wavefronts of 64 positions: inside one table, across several of one width or of different ones, behind
the first 64 tables, ids outside their table - against a gather by the library, bit for bit (each value is converted once)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,D,dtype", [
    ([64, 64, 128], [32, 32, 32], "f32"),                         # borders between wavefronts
    ([63, 1, 65, 200], [12, 12, 12, 12], "f32"),                  # several tables of one width in a wavefront
    ([10, 0, 30, 24, 100, 3], [8, 512, 24, 1024, 40, 8], "f32"),  # ... of different widths, an empty one, the widest
    ([1], [4], "f32"),
    ([700, 900], [1016, 1024], "f16"),                            # rows of 127 and 128 fragments of 16 bytes, 254 and 256 of 8
    ([100, 29, 0, 500], [8, 104, 16, 264], "f16"),
    ([7] * 70 + [500, 5], [16] * 40 + [64] * 32, "f32"),          # tables behind the first round of 64
    ([0] * 200 + [130, 1] + [0] * 50, [8] * 252, "f16"),
])
@pytest.mark.parametrize("io", [torch.float32, torch.float16, torch.bfloat16])
def test_rows_in_order_of_position(n, D, dtype, io):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE
    g = torch.Generator().manual_seed(len(n) + sum(n))
    rows = [50 + 13 * t % 97 for t in range(len(n))]
    tbe = TBE(rows, D, dtype)
    flat = torch.randn(tbe.total_elems, generator=g).to(tbe.torch_dtype)
    ids = [torch.randint(0, r, (k,), generator=g) for r, k in zip(rows, n)]
    off = torch.zeros(len(n) + 1, dtype=torch.int64)
    off[1:] = torch.cumsum(torch.tensor(n), 0)
    want, at = [], 0
    for t, i in enumerate(ids):
        want.append(flat[at:at + rows[t] * D[t]].view(rows[t], D[t])[i].to(io).reshape(-1))
        at += rows[t] * D[t]
    want = torch.cat(want)
    out = torch.full((want.numel() + 64,), 7.0, dtype=io, device="cuda")
    for idt in (torch.int64, torch.int32):
        out.fill_(7.0)
        tbe.lookup_seq(flat.cuda(), torch.cat(ids).to(idt).cuda(), off.to(idt).cuda(), out[:want.numel()])
        assert not tbe.poll_index_error()
        assert torch.equal(out[:want.numel()].cpu(), want) and bool((out[want.numel():] == 7.0).all())
    # an id outside its table: its row reads as zeros, all others as before
    idx = torch.cat(ids)
    bad = idx.numel() // 2
    t = int(torch.searchsorted(off, torch.tensor(bad), right=True)) - 1
    idx[bad] = rows[t]
    first = sum(k * d for k, d in zip(n[:t], D[:t])) + (bad - int(off[t])) * D[t]
    want[first:first + D[t]] = 0
    tbe.lookup_seq(flat.cuda(), idx.cuda(), off.cuda(), out[:want.numel()])
    assert tbe.poll_index_error()
    assert torch.equal(out[:want.numel()].cpu(), want)
    tbe.close()
