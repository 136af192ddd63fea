"""Workspaces that outlive a call: those a plan keeps for its streams, and the
library's own growing while kernels that use them are in flight."""
import pytest

from gpu_common import print_case

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
comet = pytest.importorskip("paper_2102_06827_amd")


def ints(m, n, seed):
    g = torch.Generator().manual_seed(seed)
    return torch.randint(-5, 6, (m, n), generator=g).double().cuda()


@pytest.mark.parametrize("other", [False, True])
def test_library_workspace_grows_in_flight(other):
    """Calls that grow the shared workspace are enqueued behind one another, on
    the default stream and on another, without a synchronisation between
    them; the results are compared at the end."""
    print_case("workspace grows in flight", other)
    s = torch.cuda.Stream()
    # larger products first in time: each keeps its buffer busy while the next asks for more
    sizes = [(1600, 1600, 200), (1600, 1600, 900), (300, 300, 300), (2200, 2200, 1500), (150, 150, 150), (2600, 2600, 2000)]
    work = [(ints(m, k, 2 * i), ints(k, n, 2 * i + 1)) for i, (m, n, k) in enumerate(sizes)]
    want = [a @ b for a, b in work]
    for mode in ("split_int8", "split_bf16x3"):   # (two plans' slices in the same buffer)
        torch.cuda.synchronize()
        got = []
        for _ in range(2):
            for a, b in work:
                got.append(comet.contract("ij=ik*kj", a, b, compute=mode))
                if other:
                    with torch.cuda.stream(s):
                        got.append(comet.contract("ij=ik*kj", a, b, compute=mode))
        torch.cuda.synchronize()
        per = 2 if other else 1
        for i, c in enumerate(got):
            assert torch.equal(c, want[(i // per) % len(want)])


def test_plan_keeps_a_bounded_number():
    """A plan called from many streams keeps KEEP_WORKSPACES workspaces, with
    the same results."""
    print_case("plan workspaces")
    A, B = ints(400, 300, 50), ints(300, 500, 51)
    want = A @ B
    plan = comet.Plan("ij=ik*kj", A, B, compute="split_bf16x3")
    assert plan.workspace_bytes > 0
    streams = [torch.cuda.Stream() for _ in range(3 * plan.KEEP_WORKSPACES)]
    torch.cuda.synchronize()
    got = []
    for _ in range(2):
        for s in streams:
            with torch.cuda.stream(s):
                got.append(plan(A, B))
            assert len(plan._ws) <= plan.KEEP_WORKSPACES
        got.append(plan(A, B, stream=streams[0]))
        torch.cuda.synchronize()   # (its output was allocated on the default stream)
    for c in got:
        assert torch.equal(c, want)


def test_captured_workspace_stays():
    """The workspace a graph was captured with is not given up to other
    streams: replays between their calls give the same results."""
    print_case("captured workspace")
    A, B = ints(400, 300, 52), ints(300, 500, 53)
    want = A @ B
    plan = comet.Plan("ij=ik*kj", A, B, compute="split_bf16x3")
    C = torch.zeros_like(want)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        plan(A, B, C)   # warm-up on the stream to be captured: its workspace is there already
        own = plan.workspace(A.device)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        plan(A, B, C)
    others = [torch.cuda.Stream() for _ in range(2 * plan.KEEP_WORKSPACES)]
    for o in others:
        with torch.cuda.stream(o):
            plan(A, B)
        torch.cuda.synchronize()
        # memory that a workspace given up would have come from
        junk = torch.full((plan.workspace_bytes // 8,), -1.0, dtype=torch.float64, device="cuda")
        C.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(C, want)
        del junk
    assert plan.workspace(A.device, s) is own
    assert len(plan._ws) <= plan.KEEP_WORKSPACES + 1
