"""Batches on a stream that is being captured (needs a GPU): those that go as kernel
arguments are recorded and replay; one that needs its tables is refused and leaves
the capture intact."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2605_15547_amd import crmath  # noqa: E402
from test_gpu_batch_routes import EDGES, _batch, _need_gpu, _same  # noqa: E402

CALLS = [crmath.eval_batch, crmath.eval_batch_noalloc]


def _graph(body):
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, capture_error_mode="thread_local"):
        body()
    return g


@pytest.mark.parametrize("call", CALLS, ids=lambda c: c.__name__)
@pytest.mark.parametrize("num", [1, 96, 97, 300])
def test_captured_batch_replays(num, call):
    """Every replay, with eager work and a synchronisation in between, gives the eager
    result on the buffers' contents of that time."""
    _need_gpu()
    ptrs, out, want, x = _batch(num, EDGES, 900 + num)
    call(ptrs)
    assert _same(out, want)
    keep, other = x.clone(), torch.rand_like(x) * 0.9 + 0.05
    g = _graph(lambda: call(ptrs))
    assert _same(out, want)
    for k in range(4):
        x.copy_(other if k % 2 else keep)
        out.fill_(-3.0)
        if k % 2:
            call(ptrs)
            again = out.clone()
            out.fill_(-3.0)
        torch.cuda.synchronize()
        g.replay()
        assert _same(out, again if k % 2 else want), k


@pytest.mark.parametrize("call", CALLS, ids=lambda c: c.__name__)
def test_a_batch_that_needs_tables_is_refused_under_capture(call):
    _need_gpu()
    ptrs, out, want, _x = _batch(385, (5, 64), 990, impls=(1,))
    y = torch.zeros(8, device="cuda")

    def body():
        y.add_(1.0)
        with pytest.raises(crmath.CrError) as e:
            call(ptrs)
        assert e.value.status == -6
        y.add_(1.0)

    g = _graph(body)  # the capture ends without an error
    torch.cuda.synchronize()
    assert bool((out == -3.0).all())
    g.replay()
    assert bool((y == 2.0).all())
    call(ptrs)  # and the call works again
    assert _same(out, want)


def test_destroying_a_captured_plan_leaves_no_error():
    """A plan launched eagerly and then into a capture: its destruction (after the
    graph's) waits for the eager launch and nothing else, and the next calls work."""
    _need_gpu()
    ptrs, out, want, x = _batch(40, EDGES, 991)
    plan = crmath.BatchPlan(ptrs)
    before = crmath.lib().cr_last_hip_error()
    plan.launch()
    g = _graph(plan.launch)
    out.fill_(-3.0)
    g.replay()
    assert _same(out, want)
    plan.launch()
    del g
    plan.destroy()
    y = crmath.evaluate("expf", x)
    again = crmath.BatchPlan(ptrs)
    out.fill_(-3.0)
    again.launch()
    assert _same(out, want)
    again.destroy()
    assert torch.equal(y, crmath.evaluate("expf", x))
    assert crmath.lib().cr_last_hip_error() == before


def test_captured_large_plan_replays():
    """More than 2^26 elements: eagerly a graph of per-function kernels, in a capture
    the kernels themselves."""
    _need_gpu()
    ptrs, out, want, _x = _batch(70, (1 << 20, (1 << 20) - 3), 992)
    assert sum(p[3] for p in ptrs) > 1 << 26
    plan = crmath.BatchPlan(ptrs)
    plan.launch()
    assert _same(out, want)
    g = _graph(plan.launch)
    for _ in range(3):
        out.fill_(-3.0)
        torch.cuda.synchronize()
        g.replay()
        assert _same(out, want)
        out.fill_(-3.0)
        plan.launch()
        assert _same(out, want)
    del g
    plan.destroy()
