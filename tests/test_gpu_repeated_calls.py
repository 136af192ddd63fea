"""Calls that differ from an earlier one in a stride, a shape or the output
only: the remembered call arguments of one are not those of the other, and the
shared workspace grows between calls without losing one in flight."""
import pytest

from gpu_common import print_case

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
comet = pytest.importorskip("paper_2102_06827_amd")


def ints(*shape):
    g = torch.Generator().manual_seed(94)
    return torch.randint(-5, 6, shape, generator=g).double().cuda()


def forms(x):
    """x dense, transposed in memory, and with a gap between rows."""
    gap = torch.zeros(x.shape[0], x.shape[1] + 3, dtype=x.dtype, device=x.device)
    gap[:, 1:1 + x.shape[1]] = x
    return [x, x.T.contiguous().T, gap[:, 1:1 + x.shape[1]]]


@pytest.mark.parametrize("n", [1, 6, 40])
def test_forms_of_one_shape(n):
    print_case("repeated calls", n)
    x, y, z = ints(n, n), ints(n, n) + 1, ints(n, n) - 1
    for _ in range(2):
        for a in forms(x):
            for b in forms(y):
                assert torch.equal(comet.contract("ij=ik*kj", a, b), x @ y)
                out = forms(torch.full_like(x, float("nan")))[2]
                assert comet.contract("ij=ik*kj", a, b, out) is out and torch.equal(out, x @ y)
                assert torch.equal(comet.contract_chain("il=ij*jk*kl", [a, b, z]), x @ y @ z)
                chain = comet.contract_chain("il=ij*jk*kl", [a, b, z], C=torch.ones_like(x), beta=2.0)
                assert torch.equal(chain, x @ y @ z + 2.0)
            assert torch.equal(comet.permute("ji=ij", a), x.T)
            out = forms(torch.full_like(x, float("nan")))[2]
            assert torch.equal(comet.permute("ji=ij", a, out), x.T)
    with pytest.raises(ValueError):
        comet.contract("ij=ik*kj", x, y, ints(n + 1, n))
    with pytest.raises(ValueError):
        comet.permute("jik=ijk", x)
    with pytest.raises(TypeError):
        comet.contract("ij=ik*kj", x, y.float())
    assert comet.contract("ij=ik*kj", x[:0], y).shape == (0, n)
    assert torch.equal(comet.contract("ij=ik*kj", x[:, :0], y[:0]), torch.zeros_like(x))


def test_workspace_growth_between_streams():
    """A growing workspace on the default stream and on another."""
    s = torch.cuda.Stream()
    want, got = [], []
    for n in (150, 400, 1000, 150):
        a, b = ints(n, n), ints(n, n) + 1
        want += [a @ b, a @ b]
        torch.cuda.synchronize()
        got.append(comet.contract("ij=ik*kj", a, b, compute="split_int8"))
        with torch.cuda.stream(s):
            got.append(comet.contract("ij=ik*kj", a, b, compute="split_int8"))
        s.synchronize()
    torch.cuda.synchronize()
    for g, w in zip(got, want):
        assert torch.equal(g, w)
