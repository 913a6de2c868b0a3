"""The replica mean on either side of the size from which it reads past the caches, and around its workgroups' pieces - against
the sum in index order in fp32, one division, one rounding, bit for bit."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,count,dtype", [
    (2, 1, "f32"), (2, 7, "f16"), (3, 1023, "f32"), (3, 1025, "f32"), (2, 2049, "f16"), (16, 4097, "f16"),
    (2, (1 << 26) + 1027, "f32"),                                 # just above 512 MB together, a ragged end
    (4, (1 << 26) + 8 * 300 + 5, "f16"),
    (2, (1 << 26), "f32"),                                        # just not: one round of 16384 workgroups is not enough
    (5, 33_600_003, "f32"),
])
def test_mean_of_every_size(M, count, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_03854_amd import TBE
    dt = torch.float32 if dtype == "f32" else torch.float16
    g = torch.Generator(device="cuda").manual_seed(M + count)
    reps = [torch.empty(count + 16, dtype=dt, device="cuda").uniform_(-1, 1, generator=g) for _ in range(M)]
    want = reps[0].float().clone()            # (of fp32 replicas .float() is the replica itself)
    for r in reps[1:]:
        want += r.float()
    # the correctly rounded quotient (53 bits are more than twice 24 and two); in fp32 the library multiplies by a rounded 1 / M
    for part in want.split(1 << 24):
        part.copy_((part.double() / M).float())
    tails = [r[count:].clone() for r in reps]
    tbe = TBE([16], [8], dtype)
    tbe.replica_mean([r[:count] for r in reps])
    for r, tail in zip(reps, tails):
        assert torch.equal(r[:count], want[:count].to(dt)) and torch.equal(r[count:], tail)
    tbe.close()


@pytest.mark.parametrize("M,count,dtype", [
    (6, 1, "f32"), (6, 5, "f16"), (7, 1023, "f16"), (6, 1024 * 256 + 3, "f32"),
    (6, (1 << 26) // 6, "f32"), (6, (1 << 26) // 6 + 1, "f32"),               # 256 MB together, and just above
    (8, (1 << 24) + 9, "f16"), (9, (288 << 18) // 9, "f32"), (9, (288 << 18) // 9 + 2, "f32"), (16, (288 << 19) // 16 + 8, "f16"),
])
def test_mean_of_many_replicas(M, count, dtype):
    """More replicas than are always written past the caches, on either side of the sizes up to which they are not."""
    test_mean_of_every_size(M, count, dtype)
