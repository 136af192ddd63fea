"""Contractions with batch labels: which kernel runs their entries, on either
side of each line of the rule, and a forced schedule that is taken."""
import pytest

from gpu_common import print_case

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
comet = pytest.importorskip("paper_2102_06827_amd")

# entries, m, n, k, dtype, whether the packed kernel runs them
CASES = [
    (40, 64, 64, 64, torch.float64, False),
    (40, 64, 64, 66, torch.float64, True),       # above 64 summation indices
    (3, 512, 512, 66, torch.float64, True),
    (3, 512, 520, 66, torch.float64, False),     # above 2^18 outputs: up to 96
    (3, 512, 520, 98, torch.float64, True),
    (40, 100, 100, 32, torch.float64, True),     # C in partial 64-byte segments
    (2, 1024, 1028, 32, torch.float64, False),   # ... of large entries
    (40, 64, 64, 96, torch.float32, False),
    (40, 64, 64, 100, torch.float32, True),
    (3, 1024, 1040, 96, torch.float32, False),
    (40, 104, 104, 32, torch.float32, True),     # partial segments
    (40, 32, 64, 64, torch.float32, True),       # half a tile
]


def operands(nb, m, n, k, dtype):
    g = torch.Generator().manual_seed(100)
    A = torch.randint(-4, 5, (nb, m, k), generator=g).to(dtype)
    B = torch.randint(-4, 5, (nb, k, n), generator=g).to(dtype)
    C0 = torch.randint(-4, 5, (nb, m, n), generator=g).to(dtype)
    return A, B, C0


def check(plan, A, B, C0):
    C = C0.cuda()
    plan(A.cuda(), B.cuda(), C, alpha=2.0, beta=-1.0)
    want = torch.stack([2.0 * (a.double() @ b.double()) for a, b in zip(A, B)]) - C0.double()
    assert torch.equal(C.cpu().double(), want)


@pytest.mark.parametrize("nb,m,n,k,dtype,packed", CASES)
def test_entry_kernel(nb, m, n, k, dtype, packed):
    print_case("batch entries", nb, m, n, k, str(dtype))
    A, B, C0 = operands(nb, m, n, k, dtype)
    plan = comet.Plan("xij=xik*xkj", A.cuda(), B.cuda(), C0.cuda())
    assert (plan.describe()["packed"] > 0) is packed
    check(plan, A, B, C0)


@pytest.mark.parametrize("spec,shape", [("xij=xik*xkj", (7, 64, 96, 64)), ("ij=ik*kj", (1, 96, 64, 12))])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_forced_schedule(spec, shape, dtype, monkeypatch):
    """COMET_PACKED=tile,whole,shares also where the rule would keep the
    vector-load tiles."""
    nb, m, n, k = shape
    A, B, C0 = operands(nb, m, n, k, dtype)
    if spec == "ij=ik*kj":
        A, B, C0 = A[0], B[0], C0[0]
    for tile in range(5):
        print_case("forced entries", spec, tile, str(dtype))
        monkeypatch.setenv("COMET_PACKED", "%d,1000,0" % tile)
        plan = comet.Plan(spec, A.cuda(), B.cuda(), C0.cuda())
        assert plan.describe()["packed"] == tile + 1
        if A.dim() == 3:
            check(plan, A, B, C0)
        else:
            C = C0.cuda()
            plan(A.cuda(), B.cuda(), C, alpha=2.0, beta=-1.0)
            assert torch.equal(C.cpu().double(), 2.0 * (A.double() @ B.double()) - C0.double())
