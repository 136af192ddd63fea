"""FP32 rounding error of the packed kernel: no output carries the whole
summation in one accumulator.

The bound is the error of a plain FP32 emulation that adds chains of L
products one by one and then the chains, times 1.15 for the spread of a
finite sample (128 x 128 outputs or more: the error's own deviation is below
1%) and the different order within a chain."""
import pytest

from gpu_common import print_case

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
comet = pytest.importorskip("paper_2102_06827_amd")


def emulated_error(A, B, L):
    A, B = A[:128], B[:, :128]
    total = torch.zeros(A.shape[0], B.shape[1])
    for k0 in range(0, A.shape[1], L):
        part = torch.zeros_like(total)
        for k in range(k0, min(k0 + L, A.shape[1])):
            part += A[:, k:k + 1] * B[k:k + 1]
        total += part
    ref = A.double() @ B.double()
    return ((total.double() - ref).norm() / ref.norm()).item()


# L: the pieces that a summation of this size was cut into when workgroups
# shared every tile (1024 where only a part of the tiles was shared)
@pytest.mark.parametrize("spec", ["ij=ik*kj", "ij=ki*jk"])
@pytest.mark.parametrize("m,n,k,L", [(256, 256, 256, 128), (512, 512, 512, 128), (960, 960, 960, 128),
                                     (3072, 300, 1000, 128), (1200, 1200, 1200, 192),
                                     (1400, 1400, 1400, 320), (3072, 600, 1000, 320), (1601, 1603, 1599, 1024),
                                     (3072, 3072, 3072, 1024)])
def test_fp32_error(m, n, k, L, spec):
    print_case("fp32 error", spec, m, n, k)
    g = torch.Generator().manual_seed(96)
    A = torch.rand(m, k, generator=g) * 2 - 1
    B = torch.rand(k, n, generator=g) * 2 - 1
    Ad = (A if spec == "ij=ik*kj" else A.T.contiguous()).cuda()
    Bd = (B if spec == "ij=ik*kj" else B.T.contiguous()).cuda()
    got = comet.contract(spec, Ad, Bd)[:256].cpu().double()
    ref = A[:256].double() @ B.double()
    assert ((got - ref).norm() / ref.norm()).item() <= 1.15 * emulated_error(A, B, L)


@pytest.mark.parametrize("m,n,k", [(33, 65, 31), (64, 32, 257), (513, 511, 515), (1201, 1199, 1203), (1603, 1601, 261),
                                   (3071, 2303, 1061)])
def test_fp32_integers_exactly(m, n, k):
    """Sums below 2^24 bit for bit: no product lost or doubled between the
    sets and folds, at odd numbers of steps and in shared tiles."""
    print_case("fp32 integers", m, n, k)
    g = torch.Generator().manual_seed(97)
    A = torch.randint(-8, 9, (m, k), generator=g).float()
    B = torch.randint(-8, 9, (k, n), generator=g).float()
    C0 = torch.randint(-8, 9, (m, n), generator=g).float()
    C = C0.cuda()
    comet.contract("ij=ik*kj", A.cuda(), B.cuda(), C, alpha=2.0, beta=-1.0)
    assert torch.equal(C.cpu().double(), 2.0 * (A.double() @ B.double()) - C0.double())
