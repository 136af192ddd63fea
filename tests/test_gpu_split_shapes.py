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


# FP32 BF16x3: operand orders and sizes on either side of the line between
# splitting in the gather kernel and slicing first
FUSED = [
    ("ij=ik*kj", dict(i=1024, j=1024, k=1024), True),
    ("ij=ik*kj", dict(i=1088, j=1088, k=1096), False),
    ("ij=ki*kj", dict(i=400, j=400, k=400), True),      # both contiguous along their rows
    ("ij=ki*kj", dict(i=408, j=408, k=408), False),
    ("ij=ik*kj", dict(i=405, j=405, k=405), True),      # element loads
    ("ij=ik*kj", dict(i=407, j=409, k=407), False),
    ("abij=acik*cbkj", dict(a=33, b=33, c=33, i=9, j=9, k=9), True),
    ("abij=ciak*bkjc", dict(a=32, b=32, c=32, i=16, j=16, k=16), False),   # contiguous along neither index
    ("ij=ik*jk", dict(i=63, j=3001, k=2001), True),     # few rows
    ("ij=ik*jk", dict(i=65, j=3001, k=2001), False),
    ("ij=ik*jk", dict(i=65, j=65, k=30001), False),     # slices of 128 MiB at most
    ("ij=ik*jk", dict(i=65, j=65, k=40001), True),
    ("bij=bik*bkj", dict(b=9, i=300, j=301, k=299), True),                 # batch entries
]


@pytest.mark.parametrize("spec,ext,fused", FUSED)
def test_fp32_bf16x3_rule(spec, ext, fused):
    """The path of each form, its values within the BF16x3 bar and integers
    bit for bit, through a plan (with and without allocation) and a call."""
    print_case("fp32 bf16x3 rule", spec, ext)
    out, rhs = spec.split("=")
    a, b = rhs.split("*")
    g = torch.Generator().manual_seed(92)
    eq = "%s,%s->%s" % (a, b, out)
    for ints in (False, True):
        make = (lambda t: torch.randint(-3, 4, [ext[x] for x in t], generator=g).float()) if ints else \
               (lambda t: torch.rand([ext[x] for x in t], generator=g) - 0.5)
        A, B = make(a), make(b)
        ref = torch.einsum(eq, A.double(), B.double())
        Ad, Bd = A.cuda(), B.cuda()
        plan = comet.Plan(spec, Ad, Bd, compute="split_bf16x3")
        assert plan.describe()["fused3"] is fused
        C1 = plan(Ad, Bd)
        C2 = torch.full_like(C1, float("nan"))
        plan.execute_noalloc(Ad, Bd, C2)
        C3 = comet.contract(spec, Ad, Bd, compute="split_bf16x3")
        for C in (C1, C2, C3):
            got = C.cpu().double()
            if ints:
                assert torch.equal(got, ref)
            else:
                assert (got - ref).norm() <= 1e-5 * ref.norm()


def test_plan_workspaces_of_two_streams():
    """Executions of one plan on two streams have a workspace each."""
    A = torch.rand(600, 600, device="cuda", dtype=torch.float64)
    plan = comet.Plan("ij=ik*kj", A, A, compute="split_bf16x3")
    s = torch.cuda.Stream()
    own = plan.workspace(A.device)
    with torch.cuda.stream(s):
        other = plan.workspace(A.device)
    assert own is plan.workspace(A.device) and other is not own
    assert plan.workspace(A.device, s) is other
