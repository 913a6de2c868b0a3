"""Row updates and their lists at the borders of three rules, with SGD of learning rate 1 on zero weights and small integers as
gradients: every sum is exact in fp32 (below 2^24) and has to equal the whole-number one."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def check(T, R, D, B, lens, idx, dtype="f32", io=torch.float32, seed=0):
    """One backward of T tables of R rows against integer sums; lens [T * B], idx local ids."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE
    dev = "cuda"
    off = torch.zeros(T * B + 1, dtype=torch.int64, device=dev)
    torch.cumsum(lens, 0, out=off[1:])
    g = torch.Generator(device=dev).manual_seed(seed)
    grad = torch.randint(-3, 4, (B, T * D), generator=g, device=dev)
    tbe = TBE([R] * T, [D] * T, dtype)
    ws = tbe.alloc_workspace(B, idx.numel())
    w = torch.zeros(tbe.total_elems, device=dev, dtype=tbe.torch_dtype)
    tbe.backward_sgd(grad.to(io), idx, off, B, w, ws, lr=1.0)
    for t in range(T):
        ids = idx[int(off[t * B]):int(off[(t + 1) * B])]
        bag = torch.repeat_interleave(torch.arange(B, device=dev), lens[t * B:(t + 1) * B])
        want = torch.zeros(R, D, dtype=torch.int32, device=dev)
        for c in range(0, ids.numel(), 1 << 22):
            want.index_add_(0, ids[c:c + (1 << 22)], grad[bag[c:c + (1 << 22)], t * D:(t + 1) * D].int())
        assert torch.equal(-w[t * R * D:(t + 1) * R * D].view(R, D).to(torch.int32), want), t
    tbe.close()


@pytest.mark.parametrize("B,dtype,D,io", [
    (40000, "f32", 128, torch.float32),        # 160 thousand rows and gradients in all 107 MB: within the caches
    (150000, "f32", 128, torch.float32),       # 384 MB: streamed
    (150000, "f16", 256, torch.bfloat16),      # two pieces of a row per lane
    (600000, "f32", 36, torch.float32),        # lanes without columns
    (1700000, "f16", 8, torch.float32),        # many rows per wavefront
    (9000, "f32", 1020, torch.float16),        # 147 MB of rows, a column of workgroups of its own
    (20000, "f32", 1020, torch.float16),
])
def test_rows_read_once(B, dtype, D, io):
    """Four lookups per bag, each of a row of its own but for one in a hundred, on both sides of what the last cache holds."""
    g = torch.Generator(device="cuda").manual_seed(B)
    idx = torch.randperm(4 * B, generator=g, device="cuda")
    idx[::100] = idx[1::100]
    check(1, 4 * B, D, B, torch.full((B,), 4, device="cuda"), idx, dtype, io)


@pytest.mark.parametrize("T", [1, 3])
@pytest.mark.parametrize("D,N", [(132, 8192), (132, 65536), (256, 8192), (260, 4096), (260, 8192), (1024, 4096), (1024, 32768)])
def test_parts_of_wide_rows(T, D, N):
    """Rows of one lookup fewer and more than the parts they are cut into, with as many lookups as a rule takes, and one more."""
    dev = "cuda"
    spans = [15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 66, 127, 128, 129, 300]
    for n in (N, N + 1):
        each = [n // T + (1 if t < n % T else 0) for t in range(T)]
        B, R = 512, 4000
        g = torch.Generator(device=dev).manual_seed(n)
        ids, lens = [], []
        for t in range(T):
            fixed = torch.cat([torch.full((s,), 7 * i + t, device=dev) for i, s in enumerate(spans)])
            more = torch.randint(200, R, (each[t] - fixed.numel(),), generator=g, device=dev)
            both = torch.cat([fixed, more])
            ids.append(both[torch.randperm(each[t], generator=g, device=dev)])
            lens.append(torch.bincount(torch.randint(0, B, (each[t],), generator=g, device=dev), minlength=B))
        check(T, R, D, B, torch.cat(lens), torch.cat(ids), seed=n)


@pytest.mark.parametrize("T,R,N", [
    (1, 300, (1 << 21) + 1), (4, 70000, 6_290_000), (4, 70000, 6_300_000), (2, 1000, 16_770_000), (2, 1000, 16_785_000),
    (200, 3000, 33_600_000), (300, 100, 34_000_000),              # the last: more chunks than the scan holds in registers
])
def test_scans_of_many_chunks(T, R, N):
    """Lookups on both sides of the numbers of chunks that the scan of their histograms holds in registers."""
    dev = "cuda"
    B = N // (8 * T)
    lens = torch.full((T * B,), 8, device=dev)
    lens[::1001] += 3
    lens[-1] += max(N - int(lens.sum()), 0)
    g = torch.Generator(device=dev).manual_seed(T)
    n = int(lens.sum())
    idx = (torch.rand(n, generator=g, device=dev) ** 3 * R).long().clamp_(max=R - 1)
    check(T, R, 4, B, lens, idx)
