"""The autotuner times what a plan without tuning would do among its
candidates, records it and finds it again: tuning never leaves a plan with a
slower lowering than it had without."""
import json

import pytest

from gpu_common import oracle, print_case, shape_of, synth, to_np, torch_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
comet = pytest.importorskip("paper_2102_06827_amd")

SPEC = "abij=ciak*bkjc"   # unit strides on different summation labels: one operand is copied


@pytest.fixture
def cache(tmp_path):
    yield tmp_path / "tune.json"
    comet.autotune(None, 0)


def operands(v, o):
    ext = dict(a=v, b=v, c=v, i=o, j=o, k=o)
    A = torch_dev(synth.integers(21, shape_of("ciak", ext)), torch.float64)
    B = torch_dev(synth.integers(22, shape_of("bkjc", ext)), torch.float64)
    return A, B


def lowering(plan):
    d = plan.describe()
    return d["path"], d.get("ttgt")


def test_one_copied_operand_is_a_candidate(cache):
    """957^3: 52 us with one operand copied, 64 with three permutes, 111 by
    element loads."""
    A, B = operands(33, 29)
    print_case("autotune one copy")
    untuned = comet.Plan(SPEC, A, B)
    assert untuned.describe()["path"] == "ttgt"
    comet.autotune(str(cache), 2)
    plan = comet.Plan(SPEC, A, B)
    (key, entry), = json.loads(cache.read_text())["entries"].items()
    assert entry["path"] == 2 and entry["packed"] == 1
    assert lowering(plan) == lowering(untuned) and plan.workspace_bytes == untuned.workspace_bytes
    # from the cache, without timing
    comet.autotune(str(cache), 1)
    mtime = cache.stat().st_mtime_ns
    again = comet.Plan(SPEC, A, B)
    assert cache.stat().st_mtime_ns == mtime and lowering(again) == lowering(untuned)
    assert torch.equal(again(A, B), untuned(A, B))


def test_recorded_for_a_problem_that_has_none(cache):
    """An entry of the class that says so, and a problem whose untuned plan
    reads both operands in place: its own schedule."""
    spec, ext = "abij=acik*bkcj", dict(a=13, b=11, c=12, i=5, j=6, k=7)
    A, B = synth.integers(23, shape_of("acik", ext)), synth.integers(24, shape_of("bkcj", ext))
    Ad, Bd = torch_dev(A, torch.float64), torch_dev(B, torch.float64)
    print_case("autotune other class member")
    comet.autotune(str(cache), 2)
    comet.Plan(spec, Ad, Bd)
    data = json.loads(cache.read_text())
    (key, entry), = data["entries"].items()
    cache.write_text(cache.read_text().replace('"path": %d' % entry["path"], '"path": 2')
                     .replace('"packed": %d' % entry["packed"], '"packed": 1'))
    comet.autotune(None, 0)
    untuned = comet.Plan(spec, Ad, Bd)
    comet.autotune(str(cache), 1)
    plan = comet.Plan(spec, Ad, Bd)
    assert lowering(plan) == lowering(untuned)
    assert (to_np(plan(Ad, Bd)) == oracle.contract(spec, A, B)).all()
