"""The slice-pair product's block tiles for the classic splits: each tile the
size rule takes, at ragged edges, with C in whole 64-byte segments and not."""
import pytest

from gpu_common import print_case

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
comet = pytest.importorskip("paper_2102_06827_amd")

# sizes and the block tile that they get: tiles one row short and one over,
# C rows in whole 64-byte segments (n a multiple of 16) and not
CASES = [
    ((2, 3, 1), "64x64"),
    ((63, 65, 64), "64x64"),
    ((130, 80, 65), "64x64"),
    ((1435, 1437, 70), "96x96"),
    ((1441, 1424, 31), "96x96"),
    ((2045, 1930, 66), "128x128"),
    ((1921, 2048, 64), "128x128"),
    ((2838, 2091, 32), "128x64"),
    ((3001, 2999, 64), "192x192"),
    ((2881, 3072, 33), "192x192"),
]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("compute", ["split_bf16x3", "split_fp16x2"])
@pytest.mark.parametrize("size,block", CASES)
def test_split_block(size, block, compute, dtype, monkeypatch):
    """Values within the classic splits' bar (1e-5: 22 to 24 significand bits
    in FP32 accumulation), integers that every product and sum holds exactly
    bit for bit, beta's C read and the surroundings of C left alone."""
    monkeypatch.setenv("COMET_FUSED3", "0")   # FP32 BF16x3 through the slicer too
    m, n, k = size
    print_case("split block", size, compute, str(dtype))
    g = torch.Generator().manual_seed(91)
    A = (torch.rand(m, k, generator=g, dtype=torch.float64) - 0.5).to(dtype)
    B = (torch.rand(k, n, generator=g, dtype=torch.float64) - 0.5).to(dtype)
    Ai = torch.randint(-8, 9, (m, k), generator=g).to(dtype)
    Bi = torch.randint(-8, 9, (k, n), generator=g).to(dtype)
    # C as a plain matrix, and inside a larger one from a column that is not 64-byte aligned
    for pad in (0, 3):
        full = torch.randint(-8, 9, (m, n + 2 * pad), generator=g).to(dtype)
        dev = full.cuda()
        C = dev[:, pad:pad + n]
        plan = comet.Plan("ij=ik*kj", A.cuda(), B.cuda(), C, compute=compute)
        assert plan.describe()["split_block"] == block
        C0 = full[:, pad:pad + n].double()
        plan(A.cuda(), B.cuda(), C, alpha=2.0, beta=-0.5)
        ref = 2.0 * (A.double() @ B.double()) - 0.5 * C0
        assert (C.cpu().double() - ref).norm() <= 1e-5 * ref.norm()
        plan(Ai.cuda(), Bi.cuda(), C)
        want = full.clone()
        want[:, pad:pad + n] = (Ai.double() @ Bi.double()).to(dtype)
        assert torch.equal(dev.cpu(), want)
