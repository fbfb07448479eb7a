"""The directed modes' fast paths against their accurate paths on every binary32
encoding (needs a GPU): the mode's default call and the same call with the
accurate path forced on every element give the same bits."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2605_15547_amd import crmath  # noqa: E402

CHUNK = 1 << 28


@pytest.mark.parametrize("mode", ("rz", "ru", "rd"))
@pytest.mark.parametrize("func", crmath.FUNCS32)
def test_fast_path_is_the_accurate_path(func, mode):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    fl = crmath.ROUND_FLAGS[mode]
    n, nout = CHUNK, (2 * CHUNK if func == "sincosf" else CHUNK)
    fast = torch.empty(nout, dtype=torch.float32, device="cuda")
    slow = torch.empty(nout, dtype=torch.float32, device="cuda")
    crmath.stats_reset()
    for c in range((1 << 32) // CHUNK):
        x = torch.arange(c * n, (c + 1) * n, dtype=torch.int64, device="cuda").to(torch.int32)
        for flags, out in ((fl, fast), (fl | crmath.FLAG_FORCE_FALLBACK, slow)):
            crmath.eval_ptr(func, x.data_ptr(), out.data_ptr(), n, crmath.IMPL_F64_INTERNAL, flags,
                            crmath._stream_ptr(None))
        a, b = fast.view(torch.int32), slow.view(torch.int32)
        if not torch.equal(a, b):
            k = int(torch.nonzero(a != b)[0])
            raise AssertionError("%s %s: input 0x%08x: fast 0x%08x, accurate 0x%08x"
                                 % (func, mode, (c * n + k % n) & 0xffffffff,
                                    int(a[k]) & 0xffffffff, int(b[k]) & 0xffffffff))
    st = crmath.stats_read()
    assert st["escapes"] == 0
    assert st["fallback_lanes"] >= 1 << 32  # the forced pass took every element there
