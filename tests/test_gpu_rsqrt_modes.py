"""rsqrtf in the directed rounding modes on every positive binary32 number (needs a
GPU), against an exact decision in integers: toward -infinity and zero, y is the
largest binary32 number with y^2 x <= 1; toward +infinity, the smallest with
y^2 x >= 1.

The decision is made on [1, 4); every other binade repeats it, since the function of
4 x is half that of x, exactly."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2605_15547_amd import crmath  # noqa: E402

N = 1 << 24  # the binary32 numbers of [1, 4)
ONE = 0x3F800000


def _rsqrt(bits, mode):
    x = bits.to(torch.int32)
    out = torch.empty(x.numel(), dtype=torch.float32, device="cuda")
    crmath.eval_ptr("rsqrtf", x.data_ptr(), out.data_ptr(), x.numel(), crmath.IMPL_F64_INTERNAL,
                    crmath.ROUND_FLAGS[mode], crmath._stream_ptr(None))
    return out.view(torch.int32).to(torch.int64)


def _sign(my, mx, e):
    """The sign of (my 2^-24)^2 mx 2^-e - 1, exactly: my^2 mx against 2^(48 + e) in two parts."""
    sq = my * my
    low = (sq & 0xFFFFFF) * mx
    hi = (sq >> 24) * mx + (low >> 24)
    d = torch.sign(hi - (1 << (24 + e)))
    return torch.where((d == 0) & ((low & 0xFFFFFF) > 0), torch.ones_like(d), d)


@pytest.mark.parametrize("mode", ("rz", "ru", "rd"))
def test_every_positive_number(mode):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    bits = torch.arange(N, dtype=torch.int64, device="cuda") + ONE
    y = _rsqrt(bits, mode)
    # x^-1/2 lies in (1/2, 1]: 1/2 itself where a result just above it is rounded down
    assert bool(((y >= ONE - (1 << 23)) & (y <= ONE)).all())
    my = torch.where(y == ONE, torch.full_like(y, 1 << 24), (y & 0x7FFFFF) | 0x800000)
    mx = (bits & 0x7FFFFF) | 0x800000
    for half, e in ((slice(0, N // 2), 23), (slice(N // 2, N), 22)):
        m, x = my[half], mx[half]
        if mode == "ru":
            assert bool((_sign(m, x, e) >= 0).all())
            assert bool((_sign(m - 1, x, e) < 0).all())
        else:
            up = m + torch.where(m == 1 << 24, 2, 1)  # the next binary32 number
            assert bool((_sign(m, x, e) <= 0).all())
            assert bool((_sign(up, x, e) > 0).all())
    # the other binades: 4^k times the same numbers
    for k in range(-63, 64):
        lo = ONE + (k << 24)
        b = torch.arange(N, dtype=torch.int64, device="cuda") + lo
        keep = (b >= 1 << 23) & (b < 0x7F800000)  # the normal numbers
        assert torch.equal(_rsqrt(b[keep], mode), y[keep] - (k << 23)), k
    # the subnormal ones: j 2^-149 = 2 j 4^-75
    j = torch.arange(1, 1 << 23, dtype=torch.int64, device="cuda")
    normal = (2 * j).to(torch.float32).view(torch.int32)  # exact
    assert torch.equal(_rsqrt(j, mode), _rsqrt(normal, mode) + (75 << 23))
