"""Integer by-products of tbe_backward_prepare at the borders of the sort's dispatch: tile sizes, digit widths, the three
ways the run lengths find their place, table-by-table and linearised keys - against the library's stable sort, bit for bit."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,B,nnz,idt", [
    ([200], 1, 1, torch.int64),                                  # one lookup, one 8-bit pass
    ([200], 7, 1025, torch.int32),                               # one element behind a 1024 tile
    ([100_000], 500, 32_768, torch.int64),                       # 9-bit digits; last size whose run lengths count in the keys
    ([100_000], 500, 32_769, torch.int32),                       # one chunk more than small tiles are for
    ([3_000_000], 9000, 5000, torch.int64),                      # 11-bit digits, more bags than a tile has positions
    ([900_000, 5, 70_000], 3000, 150_000, torch.int64),          # 2048 tile, 10-bit digits
    ([4_000_000, 3_999_999], 333, 100_000, torch.int32),         # 2048 tile, 11-bit digits
    ([300, 1], 4001, 600_000, torch.int64),                      # 4096 tile, chunk histograms added up by the scatter
    ([70_000, 300, 2_000_000, 1, 9], 5003, (1 << 21) + 77, torch.int64),   # chunk histograms scanned by a kernel
    ([30_000 + 61_000 * t for t in range(64)], 1100, (1 << 21) + 5000, torch.int32),   # the same with few chunks per table
    ([1000, 50_000, 17], 20_011, 2048 * 2048 + 1, torch.int32),  # run-length counts scanned by a kernel
    ([7] * 5000, 3, 40_000, torch.int64),                        # too many tables to sort one by one
    ([40, 60], 100, 5000, torch.int64),                          # linearised keys of one 8-bit pass
])
def test_sorted_keys_bags_and_segments(rows, B, nnz, idt):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE
    T, dev = len(rows), "cuda"
    g = torch.Generator(device=dev).manual_seed(nnz + T)
    # bag lengths: every third bag empty, the rest share the lookups at random
    bag = torch.randint(0, T * B, (nnz,), generator=g, device=dev)
    bag = torch.where(bag % 3 == 1, (bag - 1).clamp(min=0), bag).sort().values
    off = torch.zeros(T * B + 1, dtype=torch.int64, device=dev)
    torch.cumsum(torch.bincount(bag, minlength=T * B), 0, out=off[1:])
    R = torch.tensor(rows, device=dev)[bag // B]
    u = torch.rand(nnz, generator=g, device=dev, dtype=torch.float64)
    ids = torch.minimum((u.pow(4) * R).to(torch.int64), R - 1)    # skewed: long runs of equal keys next to single ones
    base = torch.zeros(T, dtype=torch.int64, device=dev)
    base[1:] = torch.cumsum(torch.tensor(rows[:-1], device=dev), 0) if T > 1 else base[1:]
    want, order = torch.sort(base[bag // B] + ids, stable=True)
    head = torch.ones(nnz, dtype=torch.bool, device=dev)
    head[1:] = want[1:] != want[:-1]
    seg = head.nonzero().squeeze(1)
    tbe = TBE(rows, [4] * T, "f32")
    ws = tbe.alloc_workspace(B, nnz)
    ws.fill_(0xA5)
    for _ in range(2):                                            # the second call finds the first one's leavings
        tbe.backward_prepare(ids.to(idt), off.to(idt), B, ws)
    got = tbe.debug_sorted_device(ws, B, nnz)
    assert not tbe.poll_index_error()
    assert torch.equal(got["keys_sorted"], want) and torch.equal(got["vals_sorted"], bag[order])
    assert got["num_unique"] == seg.numel()
    assert torch.equal(got["unique_rows"], want[seg]) and torch.equal(got["seg_start"][:-1], seg)
    assert int(got["seg_start"][-1]) == nnz
    tbe.close()
