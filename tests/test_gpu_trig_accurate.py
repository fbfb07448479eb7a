"""The double-double path of the trigonometric functions next to a zero of the
cosine, where all 128 fraction bits of its reduction count (needs a GPU): the one
argument whose directed-mode results depend on them, and neighbours."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2605_15547_amd import crmath, inputs  # noqa: E402


@pytest.mark.parametrize("mode", ["rn", "rz", "ru", "rd"])
@pytest.mark.parametrize("func", ["sinf", "cosf", "sincosf", "tanf"])
def test_next_to_a_zero_of_the_cosine(oracle, func, mode):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    b = np.arange(0x6946e3bb - 8, 0x6946e3bb + 9, dtype=np.uint32)
    x = inputs.f32_bits(np.concatenate([b, b | np.uint32(0x80000000)]))
    xt = torch.from_numpy(np.ascontiguousarray(x)).cuda()
    want = np.asarray(oracle.evaluate(func, x, mode=mode)).view(np.uint32).ravel()
    for flags in (0, crmath.FLAG_FORCE_FALLBACK):
        got = crmath.evaluate(func, xt, impl=crmath.IMPL_F64_INTERNAL,
                              flags=crmath.ROUND_FLAGS[mode] | flags).cpu().numpy()
        assert np.array_equal(got.view(np.uint32).ravel(), want), (func, mode, flags)
