"""Every length and alignment through the map kernels' one launch: tails of 1-3
elements after the last 128-bit vector, tile edges, and input and output at
different offsets from a 16-byte boundary (needs a GPU).

Results against the oracle, bit for bit; the elements next to the output range
keep their values."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import apps as A  # noqa: E402
from paper_2605_15547_amd import crmath, inputs  # noqa: E402

LENGTHS = (1, 2, 3, 4, 5, 7, 511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049, 4099)
CASES = [("expf", 0), ("log1pf", 0), ("sincosf", 0), ("tanf", 2), ("sincosf", 2), ("exp", 0),
         ("log", 3), ("cexpf", 0), ("clogf", 0)]
GUARD = 8


@pytest.mark.parametrize("func,impl", CASES)
def test_every_length_and_alignment(oracle, func, impl):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    f64, cplx = func in crmath.FUNCS64, func in crmath.COMPLEX
    per_in = 2 if cplx else 1
    nmax = max(LENGTHS)
    if cplx:
        x = inputs.complex_workload(nmax, seed=91)
        ref = A.evaluate_complex(func, x)
    else:
        x = inputs.workload_f64(func, nmax, seed=92) if f64 else inputs.workload_f32(func, nmax, seed=93)
        ref = oracle.evaluate(func, x)
    es = x.dtype.itemsize
    ib = np.uint64 if f64 else np.uint32
    sp = crmath._stream_ptr(None)
    offsets = (0, 1) if f64 else (0, 1, 2, 3)
    for n in LENGTHS:
        if func == "sincosf":
            want = np.concatenate([ref.reshape(2, -1)[0, :n], ref.reshape(2, -1)[1, :n]])
        else:
            want = ref[:per_in * n]
        for io in offsets:
            for oo in offsets:
                src = np.zeros(io + per_in * n, x.dtype)
                src[io:] = x[:per_in * n]
                xt = torch.from_numpy(src).cuda()
                ot = torch.full((oo + want.size + 2 * GUARD,), 7.25, dtype=xt.dtype, device="cuda")
                crmath.eval_ptr(func, xt.data_ptr() + es * io, ot.data_ptr() + es * (GUARD + oo), n,
                                impl, 0, sp)
                got = ot.cpu().numpy()
                a, b = GUARD + oo, GUARD + oo + want.size
                assert np.array_equal(got[a:b].view(ib), np.ascontiguousarray(want).view(ib)), (n, io, oo)
                assert np.all(got[:a] == 7.25) and np.all(got[b:] == 7.25), (n, io, oo)


def test_one_map_at_every_offset_of_a_slice(oracle):
    """In place on a slice, and past the grid's first pass over the tiles."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = (1 << 22) + (1 << 20) + 3
    x = inputs.uniform_f32(inputs.Stream(94), n, -20.0, 20.0)
    whole = torch.from_numpy(x).cuda()
    want = crmath.evaluate("expf", whole).cpu().numpy()
    for k in (1, 2, 3):
        y = whole.clone()
        crmath.evaluate("expf", y[k:], out=y[k:])
        got = y.cpu().numpy()
        assert np.array_equal(got[k:].view(np.uint32), want[k:].view(np.uint32)), k
        assert np.array_equal(got[:k].view(np.uint32), x[:k].view(np.uint32)), k
    part = slice(n - 5000, n)
    assert np.array_equal(want[part].view(np.uint32), oracle.evaluate("expf", x[part]).view(np.uint32))
