"""The transpose kernel's three tile edges (16, 32, 64) at the sizes where the
choice turns and where tiles are ragged, dense and strided, with alpha and beta,
bit for bit against torch."""
import pytest

from gpu_common import print_case

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
comet = pytest.importorskip("paper_2102_06827_amd")


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("spec,shape", [
    ("ba=ab", (1, 2)), ("ba=ab", (16, 5000)), ("ba=ab", (17, 4999)), ("ba=ab", (33, 33)),
    ("ba=ab", (1024, 1024)), ("ba=ab", (1023, 1025)), ("ba=ab", (961, 1100)),      # 64 x 64 from 256 tiles on
    ("baji=abij", (31, 29, 15, 16)), ("baji=abij", (5, 3, 16, 17)), ("baji=abij", (20, 20, 40, 41)),
    ("baji=abij", (3, 1, 9, 2)), ("cba=abc", (37, 2, 70)), ("ijab=abij", (33, 31, 15, 13)),
])
def test_transpose_tiles(spec, shape, dtype):
    out, inp = spec.split("=")
    perm = [inp.index(ch) for ch in out]
    g = torch.Generator(device="cuda")
    g.manual_seed(9600)
    x = torch.randint(-50, 50, shape, device="cuda", generator=g).to(dtype)
    print_case("transpose tiles", spec, shape, dtype)
    want = x.permute(perm)
    assert torch.equal(comet.permute(spec, x), want)
    y = torch.randint(-50, 50, tuple(want.shape), device="cuda", generator=g).to(dtype)
    got = comet.permute(spec, x, y.clone(), alpha=2.0, beta=-1.0)
    assert torch.equal(got, 2.0 * want - y)
    # views: every second element of longer rows on both sides, one element off
    big = torch.full(tuple(shape[:-1]) + (2 * shape[-1] + 1,), float("nan"), dtype=dtype, device="cuda")
    xv = big[..., 1::2]
    xv.copy_(x)
    obig = torch.zeros(tuple(want.shape[:-1]) + (want.shape[-1] + 3,), dtype=dtype, device="cuda")
    ov = obig[..., 1:1 + want.shape[-1]]
    comet.permute(spec, xv, ov)
    assert torch.equal(ov, want) and float(obig[..., 0].abs().sum()) == 0.0 and float(obig[..., -2:].abs().sum()) == 0.0
