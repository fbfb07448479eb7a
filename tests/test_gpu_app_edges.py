"""The application kernels at the edges of their forms (needs a GPU): the DFT around
four-term strides, one and several slices, one wave's and more slices in the final sum;
sinh and cosh from one exponential over their whole range; complex elements whose
ingredients fail their tests."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import apps as A  # noqa: E402
from paper_2605_15547_amd import crmath, inputs  # noqa: E402


def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("n,m", [(0, 2), (1, 1), (255, 1), (256, 3), (257, 1), (1023, 2), (1024, 1),
                                 (1025, 2), (16383, 1), (16384, 2), (16385, 2), (16385, 1),
                                 (133121, 1), (140001, 1)])
def test_dft_sizes(n, m):
    _need_gpu()
    x, w = inputs.dft_workload(max(n, 4), m, seed=7100 + n)
    x = x[:n]
    w[0] = 0.0 if m > 1 else w[0]  # a zero frequency among several
    X = crmath.dft(torch.from_numpy(np.ascontiguousarray(x)).cuda(), torch.from_numpy(w).cuda()).cpu().numpy()
    if n == 0:
        assert np.all(X == 0.0)
        return
    ref, mag = A.dft(x, w)
    err = np.abs(X - ref) - (np.spacing(np.abs(ref)) + n * 2.0 ** -100 * mag)
    assert not np.any(err > 0), (n, m, err.max())


def test_dft_forced_accurate_path_gives_the_same_sums():
    _need_gpu()
    x, w = inputs.dft_workload(20001, 3, seed=7200)
    xt, wt = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    a = crmath.dft(xt, wt)
    b = crmath.dft(xt, wt, flags=crmath.FLAG_FORCE_FALLBACK)
    assert torch.equal(a.view(torch.int64), b.view(torch.int64))


@pytest.mark.parametrize("func", crmath.COMPLEX)
def test_complex_over_wide_arguments(func):
    """Both parts over [-88, 88], hard and tiny arguments among them, and every element
    through the accurate paths too."""
    _need_gpu()
    st = inputs.Stream(7300)
    parts = [inputs.uniform_f32(st, 40001, -88.0, 88.0), inputs.uniform_f32(st, 8000, -1.5, 1.5),
             inputs.uniform_f32(st, 4000, -1.0, 1.0) * np.float32(2.0 ** -20)]
    for f in ("expf", "sinf", "cosf", "sinhf", "coshf"):
        h = inputs.hard_set(f)
        parts.append(h[np.abs(h) < 88.0][:2000])
    z = np.concatenate(parts).astype(np.float32)
    z = np.ascontiguousarray(np.concatenate([z, np.roll(z, 12345)])[:2 * (z.size - 1) + 2])
    if func == "clogf":
        z = z[np.abs(z) > 2.0 ** -40]
        z = z[:z.size // 2 * 2]
    zt = torch.from_numpy(z).cuda()
    want = A.evaluate_complex(func, z).view(np.uint32)
    for flags in (0, crmath.FLAG_FORCE_FALLBACK):
        got = crmath.evaluate(func, zt, flags=flags).cpu().numpy().view(np.uint32)
        bad = np.nonzero(got != want)[0]
        assert bad.size == 0, (func, flags, bad.size, z[bad[0] // 2 * 2:bad[0] // 2 * 2 + 2])
