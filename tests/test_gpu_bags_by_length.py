"""The lane groups of large launches, which hand a workgroup's bags out by length: ragged ends, empty, ordinary, split and long bags,
every class of row widths and output type, on both sides of the line - against 64-bit sums."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lanes,dtype,pooling,io", [
    (4, "f32", "sum", torch.float32), (3, "f16", "mean", torch.float16), (8, "f32", "mean", torch.bfloat16), (7, "f16", "sum", torch.float32),
    (16, "f32", "sum", torch.float16), (13, "f16", "sum", torch.bfloat16), (32, "f32", "mean", torch.float32), (25, "f16", "mean", torch.float16),
])
def test_bags_of_large_launches(lanes, dtype, pooling, io):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE, binding
    T, R, dev = 3, 400, "cuda"
    D = lanes * (8 if dtype == "f16" else 4)
    per_wg = 256 // (4 if lanes <= 4 else 8 if lanes <= 8 else 16 if lanes <= 16 else 32)
    line = max(2048 // T * per_wg, 5600)                           # 2046 workgroups of whole bags, then 2049 (8 bags each: 2100 on, smaller batches go another way)
    tbe = TBE([R] * T, [D] * T, dtype)
    tbe.set_tunable("hot_rows_min_workgroups", -1)                 # plain lane groups at every size
    g = torch.Generator(device=dev).manual_seed(lanes)
    w = torch.empty(tbe.total_elems, device=dev).uniform_(-1, 1, generator=g).to(tbe.torch_dtype)
    for B in (line, line + 1, line + per_wg - 1):
        lens = torch.round(torch.exp(1.2 + torch.randn(T * B, generator=g, device=dev))).long().clamp_(0, 127)
        lens[::7] = 0
        lens[5::1009] = torch.tensor([31, 33, 47, 49, 63, 65, 127, 128, 129, 255, 300], device=dev).repeat(len(lens[5::1009]) // 11 + 1)[:len(lens[5::1009])]
        off = torch.zeros(T * B + 1, dtype=torch.int64, device=dev)
        torch.cumsum(lens, 0, out=off[1:])
        idx = torch.randint(0, R, (int(off[-1]),), generator=g, device=dev)
        assert tbe.debug_forward_kernels(B, idx.numel()) == binding.FWD_LANE_GROUPS | binding.FWD_LONG_BAGS
        out = tbe.forward_ex(w, idx.int(), off.int(), B, pooling, out=torch.full((B, T * D), 7.0, dtype=io, device=dev)).double()
        assert not tbe.poll_index_error()
        for t in range(T):
            o = off[t * B:(t + 1) * B + 1]
            L = (o[1:] - o[:-1]).double()[:, None]
            rows = w[t * R * D:(t + 1) * R * D].view(R, D).double()[idx[int(o[0]):int(o[-1])]]
            want = torch.zeros(B, D, dtype=torch.float64, device=dev)
            want.index_add_(0, torch.repeat_interleave(torch.arange(B, device=dev), o[1:] - o[:-1]), rows)
            if pooling == "mean":
                want /= L.clamp(min=1.0)
            # a 32-bit sum of L values of at most 1 (a mean: one L-th of that, and one division), rounded once to the output's type
            err = 2.0 ** -24 * (L * L if pooling == "sum" else L + 1.0) + want.abs() * {torch.float32: 0.0, torch.float16: 2.0 ** -11, torch.bfloat16: 2.0 ** -8}[io] + 2.0 ** -24
            assert ((out[:, t * D:(t + 1) * D] - want).abs() <= err).all(), (B, t)
    tbe.close()


@pytest.mark.parametrize("D,dtype", [(8, "f32"), (32, "f32"), (64, "f16"), (128, "f32")])
@pytest.mark.parametrize("length,odd", [(0, 0), (5, 0), (5, 1), (128, 0), (64, 3)])
def test_bags_of_one_length(D, dtype, length, odd):
    """Workgroups whose bags are all of one length keep their order; one bag of another length is enough to give them one."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE
    R, B, dev = 50, 70_001, "cuda"
    tbe = TBE([R], [D], dtype)
    tbe.set_tunable("hot_rows_min_workgroups", -1)
    g = torch.Generator(device=dev).manual_seed(D + length)
    w = torch.randint(-2, 3, (R * D,), generator=g, device=dev).to(tbe.torch_dtype)   # exact sums in any order
    lens = torch.full((B,), length, device=dev)
    lens[17::500] += odd
    off = torch.zeros(B + 1, dtype=torch.int64, device=dev)
    torch.cumsum(lens, 0, out=off[1:])
    idx = torch.randint(0, R, (int(off[-1]),), generator=g, device=dev)
    out = tbe.forward(w, idx, off, B, "sum", out=torch.full((B, D), 7.0, device=dev))
    counts = torch.zeros(B * R, device=dev)
    counts.index_add_(0, torch.repeat_interleave(torch.arange(B, device=dev), lens) * R + idx, torch.ones(idx.numel(), device=dev))
    assert torch.equal(out, counts.view(B, R) @ w.view(R, D).float())
    tbe.close()


@pytest.mark.parametrize("D,dtype,mean", [(16, "f32", 0.5), (32, "f32", 2), (64, "f16", 2), (64, "f32", 8), (128, "f16", 8), (128, "f32", 32), (256, "f16", 32)])
@pytest.mark.parametrize("fewer", [0, 1])
def test_bags_long_enough_on_average(D, dtype, mean, fewer):
    """Bags of very different lengths, with as many lookups as have them handed out by length, and one fewer."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE
    R, B, dev = 50, 32_768 if D > 32 else 132_000, "cuda"
    tbe = TBE([R], [D], dtype)
    tbe.set_tunable("hot_rows_min_workgroups", -1)
    g = torch.Generator(device=dev).manual_seed(D)
    w = torch.randint(-2, 3, (R * D,), generator=g, device=dev).to(tbe.torch_dtype)   # exact sums in any order
    n = int(B * mean) - fewer
    lens = torch.bincount((torch.rand(n, generator=g, device=dev) ** 1.5 * B).long().clamp_(max=B - 1), minlength=B)
    lens = lens[torch.randperm(B, generator=g, device=dev)]
    off = torch.zeros(B + 1, dtype=torch.int64, device=dev)
    torch.cumsum(lens, 0, out=off[1:])
    idx = torch.randint(0, R, (n,), generator=g, device=dev)
    out = tbe.forward(w, idx, off, B, "sum", out=torch.full((B, D), 7.0, device=dev))
    counts = torch.zeros(B * R, device=dev)
    counts.index_add_(0, torch.repeat_interleave(torch.arange(B, device=dev), lens) * R + idx, torch.ones(n, device=dev))
    assert torch.equal(out, counts.view(B, R) @ w.view(R, D).float())
    tbe.close()
