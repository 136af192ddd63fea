"""The slice-pair product's tile on short summations into large outputs: many
rounds of workgroups, whose prologue and epilogue count as much as their
stages."""
import pytest

from gpu_common import print_case

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
comet = pytest.importorskip("paper_2102_06827_amd")


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("m,n,k", [(8192, 8192, 64), (8192, 8192, 130), (8192, 16384, 32), (4099, 4096, 200)])
def test_bf16x3_not_on_lone_workgroups(m, n, k, dtype, monkeypatch):
    """BF16x3: 128 x 128 tiles run one workgroup per CU, which on these sizes
    is 3% to 25% slower than 192 x 192 and 128 x 64 ones.  Integers bit for bit."""
    monkeypatch.setenv("COMET_FUSED3", "0")
    print_case("split short", m, n, k, str(dtype))
    g = torch.Generator().manual_seed(95)
    A = torch.randint(-8, 9, (m, k), generator=g).to(dtype).cuda()
    B = torch.randint(-8, 9, (k, n), generator=g).to(dtype).cuda()
    plan = comet.Plan("ij=ik*kj", A, B, compute="split_bf16x3")
    assert plan.describe()["split_block"] in ("192x192", "128x64", "96x96", "64x64")
    C = plan(A, B)
    # (a row block and a column block against the oracle's product on the CPU)
    assert torch.equal(C[:130].cpu().double(), A[:130].cpu().double() @ B.cpu().double())
    assert torch.equal(C[:, -70:].cpu().double(), A.cpu().double() @ B[:, -70:].cpu().double())
