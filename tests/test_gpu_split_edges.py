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
