"""Partial last tiles of every kernel that takes more than one 128-bit vector a
thread (needs a GPU): the last tile holds one vector, one less and one more than a
vector per thread, and all but one.

Results against the oracle, bit for bit; a guard longer than a tile on either side
of the output keeps its value, so a store of the last tile that goes past the end
of the array by any part of a tile shows."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2605_15547_amd import crmath, inputs  # noqa: E402

BLOCK = 256
GUARD = 8192 + 32  # elements: more than the largest tile (16 to a thread)


def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.fixture(autouse=True)
def _default_configuration():
    crmath.tune_reset()
    yield
    crmath.tune_reset()


def check(oracle, func, impl, per_thread, flags=0, mode=None):
    """Lengths around the edges of the last tile for tiles of per_thread elements a
    thread, at an aligned and a shifted output."""
    f64 = func in crmath.FUNCS64
    vn = 2 if f64 else 4
    u = per_thread // vn
    vectors = sorted({r for k in range(1, u + 1) for r in (k * BLOCK - 1, k * BLOCK, k * BLOCK + 1)} | {1})
    lengths = [vn * (2 * BLOCK * u + r) + t for r in vectors if r <= BLOCK * u for t in (0, vn - 1)]
    lengths += [vn * r for r in vectors if r <= BLOCK * u]  # the only tile
    nmax = max(lengths)
    x = inputs.workload_f64(func, nmax, seed=77) if f64 else inputs.workload_f32(func, nmax, seed=78)
    ref = oracle.evaluate(func, x) if mode is None else oracle.evaluate(func, x, mode=mode)
    ref = ref.reshape(-1, nmax)
    xt = torch.from_numpy(x).cuda()
    es, it = x.dtype.itemsize, torch.int64 if f64 else torch.int32
    rt = torch.from_numpy(np.ascontiguousarray(ref)).cuda()
    for n in lengths:
        want = rt[:, :n].reshape(-1).view(it)
        for off in (0, 1):
            a = GUARD + off
            out = torch.full((a + want.numel() + GUARD,), 7.25, dtype=xt.dtype, device="cuda")
            crmath.eval_ptr(func, xt.data_ptr(), out.data_ptr() + es * a, n, impl, flags,
                            crmath._stream_ptr(None))
            assert torch.equal(out[a:a + want.numel()].view(it), want), (n, off)
            assert bool((out[:a] == 7.25).all()) and bool((out[a + want.numel():] == 7.25).all()), (n, off)


@pytest.mark.parametrize("impl", [crmath.IMPL_F64_INTERNAL, crmath.IMPL_SPLIT_F32])
def test_sincosf(oracle, impl):
    _need_gpu()
    check(oracle, "sincosf", impl, 8)


@pytest.mark.parametrize("variant,per_thread", [(0, 8), (1, 2), (2, 4), (3, 8)])
@pytest.mark.parametrize("func", crmath.FUNCS64)
def test_binary64_variants(oracle, func, variant, per_thread):
    _need_gpu()
    crmath.tune_set(func, crmath.IMPL_F64_INTERNAL, variant, 16)
    check(oracle, func, crmath.IMPL_F64_INTERNAL, per_thread)


@pytest.mark.parametrize("mode", ("rz", "ru", "rd"))
@pytest.mark.parametrize("func", ("expf", "logf", "tanf", "sincosf"))
def test_directed_modes(oracle, func, mode):
    _need_gpu()
    check(oracle, func, crmath.IMPL_F64_INTERNAL, 8, crmath.ROUND_FLAGS[mode], mode)


VARIANTS = list(enumerate(crmath.tune_variants()))


@pytest.mark.parametrize("func,impl", [("log1pf", crmath.IMPL_F64_INTERNAL),
                                       ("sinf", crmath.IMPL_F64_INTERNAL),
                                       ("expf", crmath.IMPL_SPLIT_F32)])
@pytest.mark.parametrize("variant,per_thread", [(v, s[0]) for v, s in VARIANTS])
def test_binary32_variants(oracle, func, impl, variant, per_thread):
    _need_gpu()
    crmath.tune_set(func, impl, variant, 16)
    check(oracle, func, impl, per_thread)


@pytest.mark.parametrize("impl", [crmath.IMPL_F64_INTERNAL, crmath.IMPL_SPLIT_F32])
@pytest.mark.parametrize("variant,per_thread", [(v, s[0]) for v, s in VARIANTS])
def test_the_variant_that_is_set_runs(variant, per_thread, impl):
    """Of a forced call each workgroup that has a tile queues 512 elements, 8 waves of
    them, at its end, so the counted waves tell the tile's size; the array is shorter
    than the length up to which the default is the smallest tile."""
    _need_gpu()
    n, tile = 300_000, 256 * per_thread
    x = torch.rand(n, device="cuda")
    out = torch.empty_like(x)

    def waves():
        crmath.stats_reset()
        crmath.eval_ptr("expf", x.data_ptr(), out.data_ptr(), n, impl,
                        crmath.FLAG_FORCE_FALLBACK, crmath._stream_ptr(None))
        return crmath.stats_read()["fallback_waves"]

    crmath.tune_set("expf", impl, variant, 16)
    assert waves() == 8 * -(-n // tile)
    crmath.tune_reset()
    assert waves() == 8 * -(-n // 1024)
