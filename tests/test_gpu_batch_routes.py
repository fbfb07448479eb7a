"""Every route of a batch -- requests as kernel arguments, tables in device memory,
per-function kernels of a large plan -- against one cr_eval call per request (which
the parity tests compare with the oracle), bit for bit (needs a GPU).

Requests lie packed end to end, so a store outside its own range shows in a
neighbour; counts stand at the edges of the kernel-argument launches (96 requests of
an implementation each, four launches), lengths at the edges of steps and tiles."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2605_15547_amd import crmath  # noqa: E402

F32 = crmath.FUNCS32
EDGES = (1, 2, 3, 4, 5, 1019, 1020, 1021, 1023, 1024, 1025, 1027, 2047, 2048, 2049, 4095, 4096,
         4097, 4099, 8193)


def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _batch(num, lengths, seed, impls=(1, 2)):
    """requests, output arena and the expected arena"""
    r = np.random.default_rng(seed)
    reqs, ni, no = [], 0, 0
    for k in range(num):
        f, n = F32[int(r.integers(len(F32)))], int(lengths[k % len(lengths)])
        reqs.append((f, ni, no, n, impls[int(r.integers(len(impls)))]))
        ni += n
        no += 2 * n if f == "sincosf" else n
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.rand(ni + 4, generator=g, device="cuda") * 0.9 + 0.05
    out = torch.full((no + 4,), -3.0, device="cuda")
    want = torch.full((no + 4,), -3.0, device="cuda")
    for f, i, o, n, impl in reqs:
        crmath.eval_ptr(f, x.data_ptr() + 4 * i, want.data_ptr() + 4 * o, n, impl, 0,
                        crmath._stream_ptr(None))
    ptrs = [(f, x.data_ptr() + 4 * i, out.data_ptr() + 4 * o, n, impl) for f, i, o, n, impl in reqs]
    return ptrs, out, want, x


def _same(out, want):
    torch.cuda.synchronize()
    return torch.equal(out.view(torch.int32), want.view(torch.int32))


@pytest.mark.parametrize("num", [1, 2, 63, 64, 65, 95, 96, 97, 192, 193, 384, 385, 769])
def test_request_counts(num):
    _need_gpu()
    ptrs, out, want, _x = _batch(num, EDGES, 600 + num)
    for call in (crmath.eval_batch, crmath.eval_batch_noalloc):
        out.fill_(-3.0)
        call(ptrs)
        assert _same(out, want), call.__name__
    plan = crmath.BatchPlan(ptrs)
    for _ in range(2):
        out.fill_(-3.0)
        plan.launch()
        assert _same(out, want), "plan"
    plan.destroy()


@pytest.mark.parametrize("impl", [1, 2])
def test_one_implementation_at_the_launch_edge(impl):
    """384 requests of one implementation: four launches of 96."""
    _need_gpu()
    for num in (383, 384, 385):
        ptrs, out, want, _x = _batch(num, (5, 1025, 64), 70 + num, impls=(impl,))
        crmath.eval_batch(ptrs)
        assert _same(out, want), num


@pytest.mark.parametrize("total_log2", [20, 21, 22, 23])
def test_tile_sizes(total_log2):
    """Totals around the steps from tiles of 1024 to 2048 to 4096 elements."""
    _need_gpu()
    for d in (-4099, 0, 4099):
        n = (1 << total_log2) + d
        ptrs, out, want, _x = _batch(37, (n // 37, n // 37 + 1), total_log2)
        crmath.eval_batch(ptrs)
        assert _same(out, want), n
        plan = crmath.BatchPlan(ptrs)
        out.fill_(-3.0)
        plan.launch()
        assert _same(out, want), n
        plan.destroy()


def test_large_plan_runs_per_function_kernels():
    """More than 2^26 elements, every function in both implementations."""
    _need_gpu()
    ptrs, out, want, _x = _batch(90, (1 << 20, 70001, 1 << 20, (1 << 20) - 3), 81)
    assert sum(p[3] for p in ptrs) > 1 << 26
    plan = crmath.BatchPlan(ptrs)
    for _ in range(3):
        out.fill_(-3.0)
        plan.launch()
        assert _same(out, want)
    plan.destroy()


def test_forced_accurate_path():
    _need_gpu()
    ptrs, out, want, _x = _batch(60, EDGES, 82)
    plan = crmath.BatchPlan(ptrs, flags=crmath.FLAG_FORCE_FALLBACK)
    plan.launch()
    assert _same(out, want)
    plan.destroy()


def test_captured_plan_replays():
    """A plan launched on a stream being captured: every replay, with eager work and
    synchronisation in between, gives the eager result."""
    _need_gpu()
    ptrs, out, want, _x = _batch(50, EDGES, 83)
    plan = crmath.BatchPlan(ptrs)
    plan.launch()
    assert _same(out, want)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, capture_error_mode="thread_local"):
        plan.launch()
    for _ in range(4):
        out.fill_(-3.0)
        torch.cuda.synchronize()
        g.replay()
        assert _same(out, want)
    del g
    plan.destroy()
