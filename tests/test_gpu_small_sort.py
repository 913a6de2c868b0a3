"""The one-launch sort of small batches where its ranges of 512 places can go wrong: range borders inside runs of one key, more
elements between two borders than a workgroup has threads, further digits, ids outside their table, sparse offsets - against the
library's stable sort, bit for bit."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def ids_of(kind, n, R, g):
    if kind == "uniform":
        return torch.randint(0, R, (n,), generator=g)
    if kind == "one":                                             # every range inside one run
        return torch.full((n,), R - 1)
    if kind == "two":                                             # the border between two runs inside a range
        return torch.where(torch.arange(n) % 3 == 0, 0, R - 1)
    if kind == "near":                                            # a heavy key with close neighbours: many share its upper digits
        u = torch.rand(n, generator=g)
        return torch.where(u < 0.6, R // 2, (R // 2 + torch.randint(-200, 200, (n,), generator=g)).clamp(0, R - 1))
    if kind == "invalid":                                         # a third of the ids outside their table
        i = torch.randint(0, R, (n,), generator=g)
        return torch.where(torch.arange(n) % 3 == 1, torch.where(i % 2 == 0, R + i, -1 - i), i)
    assert kind == "all invalid"
    return torch.full((n,), R)


@pytest.mark.parametrize("idt", [torch.int64, torch.int32])
@pytest.mark.parametrize("tables,B", [                            # (lookups, rows, kind) of every table
    ([(1, 1, "one")], 1),
    ([(511, 100_000, "uniform")], 7),
    ([(512, 100_000, "uniform")], 1),
    ([(513, 1000, "uniform")], 513),
    ([(12_288, 3, "uniform")], 300),                              # whole keys after one level, thousands of each
    ([(12_288, 100_000, "near")], 300),                           # a second level, then more than fits between the borders still
    ([(12_288, 40_000_000, "near")], 2049),                       # a third one; every second offset in LDS
    ([(12_000, 2_147_483_647, "uniform")], 9000),                 # the most rows a table can have; every eighth offset
    ([(12_288, 70_000, "one")], 40),
    ([(9000, 1_000_000, "two"), (3000, 5, "two")], 100),
    ([(0, 10, "uniform"), (600, 300, "all invalid"), (0, 7, "one"), (700, 300, "all invalid"), (5, 9, "uniform"), (1100, 300, "invalid")], 33),
    ([(8000, 50_000, "invalid")], 64),
    ([(63_000, 90_000, "near")] + [(8 * t, 1000, "uniform") for t in range(20)], 50),   # a segment too long for LDS
    ([(4000 + t, 1000 * 7 ** (t % 5), "near") for t in range(15)], 777),
    ([(t % 97, 100 + t, "uniform") for t in range(512)], 3),      # as many tables as go this way
])
def test_sorted_keys_bags_segments_and_long_rows(tables, B, idt):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE
    rows = [r for _, r, _ in tables]
    T, nnz = len(rows), sum(n for n, _, _ in tables)
    g = torch.Generator().manual_seed(nnz + T)
    ids = torch.cat([ids_of(k, n, r, g) for n, r, k in tables])
    if idt == torch.int32 and int(ids.abs().max()) >= 2 ** 31:
        pytest.skip("ids beyond the type")
    bag = torch.cat([(torch.randint(0, B, (n,), generator=g) // 3 * 3).sort().values + t * B for t, (n, _, _) in enumerate(tables)])
    off = torch.zeros(T * B + 1, dtype=torch.int64)
    torch.cumsum(torch.bincount(bag, minlength=T * B), 0, out=off[1:])
    base = torch.zeros(T + 1, dtype=torch.int64)
    base[1:] = torch.cumsum(torch.tensor(rows), 0)
    t = bag // B
    bad = (ids < 0) | (ids >= torch.tensor(rows)[t])
    # ids outside their table sort behind its rows; their key is the number of all rows
    _, order = torch.sort(torch.where(bad, base[t + 1] + t, base[t] + ids + t), stable=True)
    want = torch.where(bad, base[-1], base[t] + ids)[order]
    head = torch.ones(nnz, dtype=torch.bool)
    head[1:] = want[1:] != want[:-1]
    seg = head.nonzero().squeeze(1)
    tbe = TBE(rows, [4] * T, "f32")
    ws = tbe.alloc_workspace(B, nnz)
    ws.fill_(0xA5)
    for _ in range(2):
        tbe.backward_prepare(ids.to(idt).cuda(), off.to(idt).cuda(), B, ws)
    assert tbe.poll_index_error() == bool(bad.any())
    got = tbe.debug_sorted(ws, B, nnz)
    assert torch.equal(got["keys_sorted"].long(), want) and torch.equal(got["vals_sorted"].long(), bag[order])
    assert got["num_unique"] == seg.numel()
    assert torch.equal(got["unique_rows"].long(), want[seg])
    ends = torch.cat([seg, torch.tensor([nnz])])
    assert torch.equal(got["seg_start"].long(), ends)
    # the rows listed for the next forward come from the list of long rows (more than 64 lookups): those of more than 512
    hot, _ = tbe.debug_hot_rows(ws, B, nnz)
    n = ends[1:] - ends[:-1]
    for k in range(T):
        mine = (want[seg] >= base[k]) & (want[seg] < base[k + 1]) & (n > 512)
        assert sorted(hot[k]) == (want[seg][mine] - base[k]).tolist()
    tbe.close()
