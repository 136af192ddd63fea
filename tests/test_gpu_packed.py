"""The packed gather kernel (single-element loads, any strides and extents):
every tile and operand order at the edges of its tiles and steps, split
summations whose shares lie inside, cover and cross tiles, batch labels,
streamed and plain output stores -- against the oracle, bit for bit on integer
inputs."""
import numpy as np
import pytest

from gpu_common import TOL, inputs, oracle, print_case, shape_of, to_np, torch_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
comet = pytest.importorskip("paper_2102_06827_amd")

DT = {"f64": torch.float64, "f32": torch.float32}
STEP = {"f64": 16, "f32": 32}
TILES = [(128, 128), (64, 64), (128, 64), (64, 32), (32, 64)]
# operands contiguous along the summation or along their free label
LAYOUTS = {"kk": "mn=mk*nk", "kn": "mn=mk*kn", "mn": "mn=km*kn", "mk": "mn=km*nk"}


def run(spec, ext, dtype, seed, beta=0.0, expect=None):
    A, B, C0 = inputs(spec, ext, seed, kind="integer", beta=True)
    Ad, Bd, Cd = (torch_dev(x, DT[dtype]) for x in (A, B, C0))
    if beta == 0.0:
        Cd.fill_(float("nan"))
    plan = comet.Plan(spec, Ad, Bd, Cd, path="gett")
    d = plan.describe()
    for key, value in (expect or {}).items():
        assert d[key] == value, d
    plan(Ad, Bd, Cd, alpha=2.0, beta=beta)
    torch.cuda.synchronize()
    assert np.array_equal(to_np(Cd), oracle.contract(spec, A, B, C0 if beta else None, alpha=2.0, beta=beta))


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("tile", range(5))
@pytest.mark.parametrize("layout", list(LAYOUTS))
def test_tile_and_step_edges(layout, tile, dtype, monkeypatch):
    bm, bn = TILES[tile]
    bk = STEP[dtype]
    monkeypatch.setenv("COMET_PACKED", "%d,1000000" % tile)
    # one element; one short of a tile and step; exactly two; one past
    for i, (m, n, k) in enumerate([(1, 2, 1), (bm - 1, bn - 1, bk - 1), (2 * bm, 2 * bn, 2 * bk),
                                   (bm + 1, 2 * bn + 1, 3 * bk + 1)]):
        print_case("packed", layout, tile, dtype, m, n, k)
        # (a single row is a matrix-vector product's)
        run(LAYOUTS[layout], dict(m=m, n=n, k=k), dtype, 9000 + i, beta=(0.0 if i % 2 else -1.0),
            expect={"packed": tile + 1, "packed_shares": 0} if m > 1 else None)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("tile,whole,shares", [
    (1, 0, 5),      # fewer shares than tiles: a share covers whole tiles and crosses into others
    (1, 2, 23),     # several shares a tile, some cross a boundary
    (0, 1, 7), (2, 0, 11), (3, 4, 37), (4, 0, 1),
    (1, 0, 10 ** 6),   # a share per step
])
def test_shared_summations(tile, whole, shares, dtype, monkeypatch):
    spec, ext = "abij=acik*bkcj", dict(a=9, b=7, c=11, i=17, j=19, k=13)   # 153 x 133, K = 143
    bm, bn = TILES[tile]
    T = -(-153 // bm) * -(-133 // bn)
    steps = -(-143 // STEP[dtype])
    want = min(shares, (T - whole) * steps)
    monkeypatch.setenv("COMET_PACKED", "%d,%d,%d" % (tile, whole, shares))
    print_case("packed shares", tile, whole, shares, dtype)
    for beta in (0.0, 0.5):
        run(spec, ext, dtype, 9100, beta=beta,
            expect={"packed": tile + 1, "packed_whole": whole, "packed_shares": want})
    A, B, _ = inputs(spec, ext, 9101)
    Ad, Bd = torch_dev(A, DT[dtype]), torch_dev(B, DT[dtype])
    got = to_np(comet.Plan(spec, Ad, Bd, path="gett")(Ad, Bd))
    cast = np.float64 if dtype == "f64" else np.float32
    assert oracle.relerr(got, oracle.contract(spec, A.astype(cast), B.astype(cast))) <= TOL[dtype]


@pytest.mark.parametrize("spec,ext", [
    ("bij=bik*bkj", dict(b=5, i=67, j=33, k=35)),
    ("ibj=kbi*jbk", dict(b=3, i=65, j=129, k=17)),
    ("bij=ki*bkj", dict(b=1, i=70, j=40, k=100)),
    ("xiyj=xkyi*ykxj", dict(x=3, y=2, i=31, j=64, k=33)),   # two batch labels
])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("tile", [0, 1, 4])
def test_batch_labels(tile, dtype, spec, ext, monkeypatch):
    monkeypatch.setenv("COMET_PACKED", str(tile) + ",1000000")
    print_case("packed batch", spec, tile, dtype)
    run(spec, ext, dtype, 9200, beta=1.0, expect={"packed": tile + 1})


def test_operands_anywhere_in_memory():
    """Strided, broadcast and unaligned operands and outputs; the output in
    whole 64-byte segments, but from a base that is not."""
    spec, ext = "abij=acik*bkcj", dict(a=6, b=5, c=7, i=16, j=16, k=9)
    for dtype in ("f64", "f32"):
        A, B, C0 = inputs(spec, ext, 9300, kind="integer", beta=True)
        ref = oracle.contract(spec, A, B, C0, alpha=1.0, beta=1.0)
        for shift in (0, 1, 3):
            print_case("packed unaligned", dtype, shift)
            views = []
            for x in (A, B, C0):
                buf = torch.full((x.size + 8,), float("nan"), dtype=DT[dtype], device="cuda")
                v = buf[shift:shift + x.size].view(x.shape)
                v.copy_(torch_dev(x, DT[dtype]))
                views.append(v)
            plan = comet.Plan(spec, *views)
            assert plan.describe()["packed"] > 0
            plan(views[0], views[1], views[2], beta=1.0)
            torch.cuda.synchronize()
            assert np.array_equal(to_np(views[2]), ref)
    # every second element of a longer tensor, and one operand broadcast
    big = torch_dev(inputs("ij=ik*kj", dict(i=40, j=30, k=50), 9301, kind="integer")[0], torch.float64)
    A = big[:, ::2]
    B = torch_dev(np.arange(25.0) - 12, torch.float64)[:, None].expand(25, 30)
    plan = comet.Plan("ij=ik*kj", A, B)
    assert plan.describe()["packed"] > 0
    assert np.array_equal(to_np(plan(A, B)), oracle.contract("ij=ik*kj", to_np(A), to_np(B.contiguous())))


@pytest.mark.parametrize("where", ["row", "summation"])
def test_non_finite_values_stay_in_their_row(where, monkeypatch):
    """Rows past the edge repeat the last one and steps past the end are
    zeros: an infinity in the last row or summation index reaches the outputs
    it belongs to and no other."""
    monkeypatch.setenv("COMET_PACKED", "1,1000000")
    A, B, _ = inputs("ij=ik*kj", dict(i=65, j=63, k=17), 9400, kind="integer")
    B = np.abs(B) + 1.0
    if where == "row":
        A[64, 3] = np.inf
    else:
        A[7, 16] = np.nan
    plan = comet.Plan("ij=ik*kj", torch_dev(A, torch.float64), torch_dev(B, torch.float64))
    got = to_np(plan(torch_dev(A, torch.float64), torch_dev(B, torch.float64)))
    bad = np.zeros(got.shape, bool)
    bad[64 if where == "row" else 7] = True
    assert not np.isfinite(got[bad]).any() and np.isfinite(got[~bad]).all()


def test_schedule_keeps_within_the_static_workspace():
    """Plans that fitted comet_plan_execute_noalloc's buffer still do: the
    partial tiles stay within it, also behind TTGT's copies."""
    for n, path in ((3025, "gett"), (3072, "gett"), (2500, "ttgt")):
        A = torch.zeros((n, n), dtype=torch.float32, device="cuda")
        plan = comet.Plan("ij=ik*kj", A, A.clone(), path=path)
        assert plan.workspace_bytes <= 128 << 20, plan.describe()


def test_switched_off(monkeypatch):
    monkeypatch.setenv("COMET_PACKED", "0")
    A = torch.zeros((75, 75), dtype=torch.float64, device="cuda")
    assert comet.Plan("ij=ik*kj", A, A.clone()).describe()["packed"] == 0


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("cls", [None, "0", "1", "2", "3"])
def test_batch_of_odd_problems(cls, dtype, monkeypatch):
    """The batch on the packed tile product: odd extents in every tile class,
    batch labels, a dense copy of an operand (all of them in one launch),
    an empty summation and alpha = 0 beside them, run twice."""
    if cls is not None:
        monkeypatch.setenv("COMET_BATCH_CLASS", cls)
    rng = np.random.default_rng(9500)
    host = []
    for t, spec in enumerate(["abij=acik*bkcj", "abij=ciak*bkjc", "ajbi=kcia*cjkb", "bij=bik*bkj", "abij=ciak*bkjc",
                              "abij=ijcd*cdab", "ij=ik*kj", "ij=ik*kj"]):
        ext = {ch: int(rng.integers(3, 21)) for ch in set(spec) - set("=*")}
        if t == 6:
            ext["k"] = 0
        A, B, C0 = inputs(spec, ext, 9500 + 10 * t, kind="integer", beta=True)
        host.append((spec, A, B, C0, 0.0 if t == 7 else 2.0, 0.0 if t == 1 else -1.0))
    dev = [dict(spec=s, A=torch_dev(A, DT[dtype]), B=torch_dev(B, DT[dtype]), C=torch_dev(C0, DT[dtype]), alpha=al,
                beta=be) for s, A, B, C0, al, be in host]
    print_case("packed batch", dtype, cls)
    bt = comet.Batch(dev, dtype=DT[dtype])
    d = bt.describe()
    assert d["copies"] >= 2
    if cls in ("0", "1", "2"):
        assert d["classes"][int(cls)] > 0
    want = [C0 for _, _, _, C0, _, _ in host]
    for _ in range(2):
        bt()
        torch.cuda.synchronize()
        want = [oracle.contract(s, A, B, C, alpha=al, beta=be) for (s, A, B, _, al, be), C in zip(host, want)]
        for (s, *_), x, ref in zip(host, dev, want):
            assert np.array_equal(to_np(x["C"]), ref), s


@pytest.mark.parametrize("m,n,k,dtype,kernel", [
    (3072, 2304, 12, "f32", "gather"),      # half a step of summation, C in whole segments
    (3072, 2305, 12, "f32", "packed"),      # ... and not
    (3072, 2304, 17, "f32", "packed"),
    (4096, 4096, 16, "f32", "packed"),      # 2^24 outputs
    (3072, 2304, 12, "f64", "packed"),
    (5888, 5632, 16, "f64", "packed"),      # 2024 tiles of 128 x 128: less than 8 rounds of a workgroup per CU
    (5800, 5888, 16, "f64", "shortk"),      # 2116
    (8192, 8400, 32, "f32", "shortk"),      # 4224
    (8000, 8192, 32, "f32", "packed"),      # 4032 tiles, two workgroups a CU
])
def test_short_summations(m, n, k, dtype, kernel):
    """Which kernel takes a short summation, and its integers bit for bit."""
    print_case("short summations", m, n, k, dtype)
    g = torch.Generator().manual_seed(93)
    A = torch.randint(-3, 4, (m, k), generator=g).to(DT[dtype])
    B = torch.randint(-3, 4, (n, k), generator=g).to(DT[dtype])
    C = torch.full((m, n), float("nan"), dtype=DT[dtype], device="cuda")
    plan = comet.Plan("mn=mk*nk", A.cuda(), B.cuda(), C)
    d = plan.describe()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    if cus == 256:
        assert ("shortk" if d["shortk"] else "packed" if d["packed"] else "gather") == kernel, d
    plan(A.cuda(), B.cuda(), C)
    assert torch.equal(C.cpu(), A @ B.T)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("spec,ext", [
    ("abij=ciak*bkjc", dict(a=60, b=61, c=59, i=16, j=17, k=16)),
    ("abij=icak*kbjc", dict(a=60, b=30, c=33, i=18, j=21, k=20)),      # B the larger copy
    ("ijab=bkjc*ciak", dict(a=33, b=60, c=35, i=21, j=18, k=19)),      # C transposed, A copied
    ("jbia=ciak*bkjc", dict(a=45, b=25, c=31, i=16, j=33, k=29)),
])
def test_one_copied_operand(spec, ext, dtype):
    """Unit strides on different summation labels: one operand is copied, the
    other and C are used in place, strided ones too; integers bit for bit, with
    beta, and through the call without a plan."""
    print_case("one copied operand", spec, dtype)
    A, B, C0 = inputs(spec, ext, 9701, kind="integer", beta=True)
    Ad, Bd, Cd = (torch_dev(x, DT[dtype]) for x in (A, B, C0))
    want = oracle.contract(spec, A, B, C0, alpha=2.0, beta=-1.0)
    for strided in (False, True):
        if strided:   # every other plane of a larger tensor
            Ad, Bd, Cd = (torch.stack([x, torch.full_like(x, float("nan"))], 1)[:, 0] for x in (Ad, Bd, Cd))
        plan = comet.Plan(spec, Ad, Bd, Cd)
        d = plan.describe()
        assert d["path"] == "ttgt" and [d["ttgt"][x] for x in ("copyA", "copyB", "copyC")].count(True) == 1, d["ttgt"]
        out = Cd if strided else Cd.clone()
        plan(Ad, Bd, out, alpha=2.0, beta=-1.0)
        assert np.array_equal(to_np(out), want)
        assert np.array_equal(to_np(comet.contract(spec, Ad, Bd)), oracle.contract(spec, A, B))
