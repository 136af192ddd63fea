"""FP32 BF16x3 products of middle sizes, which were split in the gather kernel
and are now sliced into a workspace first: what the one answered the other
does not refuse or answer otherwise."""
import pytest

from gpu_common import print_case

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
comet = pytest.importorskip("paper_2102_06827_amd")


@pytest.mark.parametrize("n,fused", [(172600, False), (172829, True), (173000, True)])
def test_slices_at_the_scratch_limit(n, fused):
    """65 x n x 65: executions without allocation are taken on either side of
    the line and where an estimate of the slices lies below it but the slices
    with their exponents above."""
    print_case("scratch limit", n)
    g = torch.Generator().manual_seed(98)
    A = torch.randint(-3, 4, (65, 65), generator=g).float()
    B = torch.randint(-3, 4, (n, 65), generator=g).float()
    Ad, Bd = A.cuda(), B.cuda()
    plan = comet.Plan("ij=ik*jk", Ad, Bd, compute="split_bf16x3")
    assert plan.describe()["fused3"] is fused
    C = torch.full((65, n), float("nan"), device="cuda")
    plan.execute_noalloc(Ad, Bd, C)
    assert torch.equal(C.cpu(), A @ B.T)


@pytest.mark.parametrize("compute", ["split_bf16x3", "split_fp16x2"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("size", [(407, 409, 407), (130, 200, 100), (2049, 2047, 65)])
def test_not_finite_times_a_row_of_zeros(size, dtype, compute):
    """NaN and infinities of one operand reach every output of their column,
    also those of the other operand's rows of zeros; the other columns stay
    exact."""
    m, n, k = size
    print_case("zero rows", size, str(dtype), compute)
    g = torch.Generator().manual_seed(99)
    A = torch.randint(-3, 4, (m, k), generator=g).to(dtype)
    B = torch.randint(-3, 4, (k, n), generator=g).to(dtype)
    A[0], A[m // 2], A[m - 1] = 0, 0, 0
    B[3, 0], B[k - 1, n // 2], B[5, n - 1] = float("nan"), float("inf"), float("-inf")
    B[:, 7] = 0
    bad = torch.zeros(n, dtype=torch.bool)
    bad[[0, n // 2, n - 1]] = True
    got = comet.contract("ij=ik*kj", A.cuda(), B.cuda(), compute=compute).cpu()
    zero = [0, m // 2, m - 1]
    assert torch.isnan(got[zero][:, bad]).all()
    assert not torch.isfinite(got[:, bad]).any()
    assert torch.equal(got[:, ~bad], (A @ torch.where(torch.isfinite(B), B, torch.zeros_like(B)))[:, ~bad])
    # and the other way round
    got = comet.contract("ij=ki*kj", B.cuda(), A.T.contiguous().cuda(), compute=compute).cpu()
    assert torch.isnan(got[bad][:, zero]).all() and not torch.isfinite(got[bad]).any()
