"""The forward of narrow rows on both sides of the rule by which its output goes past the caches: parts of 64 bytes or more, of whole
64-byte pieces or not (odd widths, an output that begins inside a piece), outputs below and above the size from which wide parts do."""
import pytest
import torch

pytestmark = pytest.mark.gpu
EB = {torch.float32: 4, torch.float16: 2, torch.bfloat16: 2}


@pytest.mark.parametrize("weights", ["f32", "f16"])
@pytest.mark.parametrize("io", [torch.float32, torch.float16, torch.bfloat16])
@pytest.mark.parametrize("widths,megabytes", [((16, 16, 16), 1), ((32, 32, 32), 1), ((32, 64, 96), 47), ((32, 64, 96), 50), ((64, 64, 8), 50),
                                              ((24, 40, 104), 50), ((8, 8), 9), ((128, 256), 50)])
def test_pooled_output_beside_the_rule(widths, megabytes, io, weights):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE
    T, R = len(widths), 97
    B = megabytes * 1024 * 1024 // (sum(widths) * EB[io]) + 3
    tbe = TBE([R] * T, list(widths), weights)
    g = torch.Generator(device="cuda")
    g.manual_seed(B)
    # small whole numbers: every sum is exact in any order and in 16 bits
    table = torch.randint(-4, 5, (tbe.total_elems,), generator=g, device="cuda").to(tbe.torch_dtype)
    L = torch.randint(0, 4, (T * B,), generator=g, device="cuda")
    off = torch.zeros(T * B + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(L, 0, out=off[1:])
    idx = torch.randint(0, R, (int(off[-1]),), generator=g, device="cuda")
    want = torch.empty(B, sum(widths), dtype=io, device="cuda")
    col = first = 0
    for t, D in enumerate(widths):
        rows = table[first:first + R * D].view(R, D).float()
        a, b = int(off[t * B]), int(off[(t + 1) * B])
        bag = torch.repeat_interleave(torch.arange(B, device="cuda"), L[t * B:(t + 1) * B])
        want[:, col:col + D] = torch.zeros(B, D, device="cuda").index_add_(0, bag, rows[idx[a:b]]).to(io)
        col, first = col + D, first + R * D
    for shift in (0, 16 // EB[io]):
        room = torch.full((want.numel() + shift,), 77.0, dtype=io, device="cuda")
        out = room[shift:].view_as(want)
        tbe.forward_ex(table, idx, off, B, "sum", out=out)
        assert torch.equal(out, want), shift
    tbe.close()
