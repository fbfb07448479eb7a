"""The calls by which the library's speed is measured: what a program that uses
it asks for, through the Python binding's public entry points.

Four kinds of case:
  map    one evaluate() call: a function over one array, with the implementation
         and the rounding mode that the caller may choose, on a whole allocation
         or on a slice that starts `shift` elements into one
  dft    one dft() call (spectral interpolation by a brute-force transform)
  plan   one launch of a BatchPlan of requests of mixed functions and lengths
  batch  one eval_batch() call on such requests, tables and all

Inputs are drawn on the GPU from the seed.  wide = False: the values that a
program meets day by day (network activations, angles of some turns,
magnitudes near one); wide = True: the function's whole domain, with one
element in a hundred a raw bit pattern (infinities, NaN, subnormals, arguments
outside the domain).
"""
import math

import numpy as np
import torch

from paper_2605_15547_amd import crmath

FUNCS32 = list(crmath.FUNCS32)
FUNCS64 = list(crmath.FUNCS64)
COMPLEX = list(crmath.COMPLEX)
MODES = {"rn": 0, "rz": crmath.FLAG_ROUND_TOWARD_ZERO, "ru": crmath.FLAG_ROUND_UP,
         "rd": crmath.FLAG_ROUND_DOWN}
IMPLS = {"auto": crmath.IMPL_AUTO, "split": crmath.IMPL_SPLIT_F32, "log128": crmath.IMPL_LOG128}

# (low, high) of the ordinary arguments, drawn uniformly
ORDINARY = {"expf": (-20, 20), "exp2f": (-30, 30), "exp10f": (-10, 10), "expm1f": (-4, 4),
            "logf": (1e-3, 100), "log2f": (1e-3, 100), "log10f": (1e-3, 100), "log1pf": (-0.9, 20),
            "rsqrtf": (1e-3, 1000), "sinf": (-100, 100), "cosf": (-100, 100),
            "sincosf": (-100, 100), "tanf": (-10, 10), "asinf": (-1, 1), "acosf": (-1, 1),
            "atanf": (-30, 30), "sinhf": (-10, 10), "coshf": (-10, 10), "tanhf": (-5, 5),
            "exp": (-20, 20), "log": (1e-3, 100), "exp2": (-20, 20)}
# the whole domain of the functions whose results leave the format beyond it;
# the others take any magnitude, drawn with a uniform exponent
DOMAIN = {"expf": (-103.9, 88.7), "exp2f": (-150, 128), "exp10f": (-45.15, 38.53),
          "expm1f": (-103.9, 88.7), "asinf": (-1, 1), "acosf": (-1, 1), "sinhf": (-89.4, 89.4),
          "coshf": (-89.4, 89.4), "tanhf": (-10, 10), "exp": (-745, 709.7), "exp2": (-1074, 1024)}
POSITIVE = ("logf", "log2f", "log10f", "rsqrtf", "log")


def _map(name, func, n, wide=False, shift=0, impl="auto", mode="rn"):
    return {"name": name, "kind": "map", "func": func, "n": n, "wide": wide, "shift": shift,
            "impl": impl, "mode": mode}


def listed():
    return [
        # the softmax or gate of one token: one short row, where latency is all
        _map("expf_1k", "expf", 1000),
        # a mid-sized array of no round length (a record count)
        _map("log1pf_100k_odd", "log1pf", 100003),
        # a slice x[1:] of a signal, written to a new array
        _map("sinf_1m_slice", "sinf", (1 << 20) - 1, shift=1),
        # the elementwise pass of the benchmark's size: 2^26 over the domain
        _map("expf_64m", "expf", 1 << 26, wide=True),
        # tangents of arguments of every magnitude (large-argument reduction)
        _map("tanf_16m_wide", "tanf", 1 << 24, wide=True),
        # phases to unit vectors (rotary tables, mixers), of no round length
        _map("sincosf_10m_odd", "sincosf", 10000001),
        # binary64: log-likelihoods
        _map("log64_16m", "log", 1 << 24),
        # the complex workload of the benchmark, a quarter of its length
        _map("csinf_4m", "csinf", 1 << 22),
        # an upper bound in interval arithmetic
        _map("logf_up_4m", "logf", 1 << 22, mode="ru"),
        # spectral interpolation: 2^18 samples at 64 frequencies
        {"name": "dft_256k_64", "kind": "dft", "n": 1 << 18, "m": 64},
        # a ragged batch of mixed requests, each in buffers of its own, replayed
        {"name": "plan_512", "kind": "plan", "num": 512, "max_log2": 18, "packed": False,
         "impl": "auto"},
        # what a server collects in one tick: short requests packed in one arena
        {"name": "batch_48_packed", "kind": "batch", "num": 48, "max_log2": 13, "packed": True,
         "impl": "auto"},
    ]


def _log_int(rng, lo, hi):
    """An integer spread evenly over the logarithm of [lo, hi]; even ones made odd half the time."""
    n = int(math.exp(rng.uniform(math.log(lo), math.log(hi))))
    return max(lo, min(hi, n | rng.randrange(2)))


def draw(rng):
    kind = rng.choices(["map", "dft", "plan", "batch"], [8, 1, 1, 1])[0]
    if kind == "dft":
        return {"kind": "dft", "n": _log_int(rng, 1 << 10, 1 << 18), "m": _log_int(rng, 1, 64)}
    if kind == "plan":
        return {"kind": "plan", "num": _log_int(rng, 4, 512), "max_log2": rng.randint(8, 18),
                "packed": rng.random() < 0.5, "impl": rng.choice(["auto", "auto", "split"])}
    if kind == "batch":
        return {"kind": "batch", "num": _log_int(rng, 1, 256), "max_log2": rng.randint(6, 16),
                "packed": rng.random() < 0.7, "impl": rng.choice(["auto", "auto", "split"])}
    func = rng.choice(FUNCS32 * 2 + FUNCS64 * 2 + COMPLEX)
    impl = mode = None
    if func in FUNCS32:
        impl = rng.choice(["auto", "auto", "auto", "split"])
        mode = rng.choice(["rn", "rn", "rz", "ru", "rd"]) if impl == "auto" else "rn"
    elif func == "log":
        impl = rng.choice(["auto", "auto", "log128"])
    c = _map("", func, _log_int(rng, 256, 1 << 24), wide=rng.random() < 0.5 and func not in COMPLEX,
             shift=rng.choice([0, 0, 0, 1, 2, 3]), impl=impl or "auto", mode=mode or "rn")
    del c["name"]
    return c


# ---------------------------------------------------------------------- inputs
def _uniform(g, n, lo, hi, dtype):
    return (torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * (hi - lo) + lo).to(dtype)


def _values(g, func, n, wide):
    """n arguments of func."""
    f64 = func in FUNCS64
    dtype = torch.float64 if f64 else torch.float32
    if func in COMPLEX:  # both parts in [-40, 40], as in the benchmark
        return _uniform(g, 2 * n, -40.0, 40.0, dtype)
    if not wide:
        return _uniform(g, n, *ORDINARY[func], dtype)
    itype, bits, mant = (torch.int64, 64, 52) if f64 else (torch.int32, 32, 23)
    raw = torch.randint(-(1 << (bits - 1)), (1 << (bits - 1)) - 1, (n,), generator=g, device="cuda",
                        dtype=torch.int64).to(itype)
    if func in DOMAIN:
        x = _uniform(g, n, *DOMAIN[func], dtype)
    else:  # any sign (if the domain has both) and any normal exponent
        e = torch.randint(1, (1 << (bits - 1 - mant)) - 1, (n,), generator=g, device="cuda",
                          dtype=torch.int64).to(itype)
        keep = (1 << mant) - 1
        if func not in POSITIVE:
            keep -= 1 << (bits - 1)  # the sign bit too
        x = ((raw & keep) | (e << mant)).view(dtype)
        if func == "log1pf":
            x = torch.where(x < -1, x.abs(), x)
    some = torch.rand(n, generator=g, device="cuda") < 0.01
    return torch.where(some, raw.view(dtype), x)


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(1000003 * int(seed) + 17)


def _dft_inputs(case, seed):
    g = _generator(seed)
    n, m = case["n"], case["m"]
    x = _uniform(g, n, -1.0, 1.0, torch.float32)
    f = torch.rand(m, generator=g, device="cuda", dtype=torch.float64) * (n / 2.0)
    return x, (2.0 * math.pi * f / n).to(torch.float32)


def _batch_layout(case):
    """[(func, length, first input element, first output element)] and the sizes
    of the two arenas: requests packed end to end, or each at a 256-byte boundary.
    The functions and lengths belong to the case; the seed draws the values."""
    r = np.random.default_rng([case["num"], case["max_log2"]])
    step = 1 if case["packed"] else 64
    out, i, o = [], 0, 0
    for _ in range(case["num"]):
        func = FUNCS32[int(r.integers(len(FUNCS32)))]
        n = int(2.0 ** (case["max_log2"] * r.random()))
        nout = 2 * n if func == "sincosf" else n
        out.append((func, n, i, o))
        i += -(-n // step) * step
        o += -(-nout // step) * step
    return out, i, o


def _batch_inputs(case, seed):
    layout, ni, no = _batch_layout(case)
    pool = {f: _values(_generator(1000 * int(seed) + k), f, 1 << case["max_log2"], False)
            for k, f in enumerate(FUNCS32)}
    x = torch.zeros(ni, dtype=torch.float32, device="cuda")
    for k, (func, n, i, _) in enumerate(layout):
        x[i:i + n] = torch.roll(pool[func], k)[:n]
    return layout, x, no


def _map_input(case, seed):
    """The array, `shift` elements into an allocation of its own."""
    v = _values(_generator(seed), case["func"], case["n"], case["wide"])
    if not case["shift"]:
        return v
    whole = torch.empty(v.numel() + case["shift"], dtype=v.dtype, device="cuda")
    whole[case["shift"]:] = v
    return whole[case["shift"]:]


# ------------------------------------------------------------------- the calls
def prepare(case, seed):
    if case["kind"] == "map":
        return {"kind": "map", "func": case["func"], "x": _map_input(case, seed),
                "impl": IMPLS[case["impl"]], "flags": MODES[case["mode"]]}
    if case["kind"] == "dft":
        x, w = _dft_inputs(case, seed)
        return {"kind": "dft", "x": x, "w": w}
    layout, x, no = _batch_inputs(case, seed)
    out = torch.zeros(no, dtype=torch.float32, device="cuda")
    impl = IMPLS[case["impl"]]
    reqs = [(f, x.data_ptr() + 4 * i, out.data_ptr() + 4 * o, n, impl) for f, n, i, o in layout]
    state = {"kind": case["kind"], "x": x, "out": out, "reqs": reqs}
    if case["kind"] == "plan":
        state["plan"] = crmath.BatchPlan(reqs)
    return state


def run(state):
    if state["kind"] == "map":
        return crmath.evaluate(state["func"], state["x"], impl=state["impl"], flags=state["flags"])
    if state["kind"] == "dft":
        return crmath.dft(state["x"], state["w"])
    if state["kind"] == "plan":
        state["plan"].launch()
    else:
        crmath.eval_batch(state["reqs"])
    return state["out"]


def work(case):
    """Bytes: each input read once and each output written once.  flops: the
    binary64 operations of a polynomial of the needed degree and the reduction
    around it, about 30 for each function value."""
    if case["kind"] == "map":
        n, func = case["n"], case["func"]
        per = 16 if func in FUNCS64 + COMPLEX else 12 if func == "sincosf" else 8
        return {"bytes": per * n, "flops": (90 if func in COMPLEX else 30) * n}
    if case["kind"] == "dft":
        n, m = case["n"], case["m"]
        return {"bytes": 4 * n + 20 * m, "flops": 64 * n * m}
    # the mean length of 2^(L u), u uniform, and one output more for sincosf
    mean = (2.0 ** case["max_log2"] - 1) / (case["max_log2"] * math.log(2.0))
    n = case["num"] * mean
    return {"bytes": int(n * (8 + 4 / 19)), "flops": int(30 * n)}


# ------------------------------------------------------------ in 64 bits, plain
def _plain(func, x):
    if func in COMPLEX:
        z = torch.view_as_complex(x.double().view(-1, 2))
        if func == "csinf":  # as products, so that each part keeps its own accuracy
            r = torch.stack([z.real.sin() * z.imag.cosh(), z.real.cos() * z.imag.sinh()], -1)
        else:
            r = torch.view_as_real(z.exp() if func == "cexpf" else z.log())
        return r.reshape(-1)
    x = x.double()
    if func == "sincosf":
        return torch.stack([x.sin(), x.cos()])
    if func == "exp10f":
        return torch.pow(torch.full_like(x, 10.0), x)
    if func == "rsqrtf":
        return 1.0 / x.sqrt()
    return getattr(torch, func[:-1] if func in FUNCS32 else func)(x)


def _overflowed(v, mode):
    """v with what lies beyond binary32 as IEEE 754 has it (Sec. 7.4): an
    infinity, or the largest finite number where the mode rounds toward zero."""
    big = float(np.finfo(np.float32).max)
    limit = big * (1.0 + 2.0 ** -25) if mode == "rn" else big
    top = big if mode in ("rz", "rd") else math.inf
    low = -big if mode in ("rz", "ru") else -math.inf
    inf = v.abs() == math.inf  # of an infinite argument, or beyond binary64 as well
    v = torch.where((v > limit) & ~inf, torch.full_like(v, top), v)
    return torch.where((v < -limit) & ~inf, torch.full_like(v, low), v)


def exact(case, seed):
    if case["kind"] == "map":
        x, func = _map_input(case, seed), case["func"]
        v = _plain(func, x)
        if func in FUNCS64:
            return v
        # beyond binary64 too, the argument being finite: an overflow like the others
        arg = x if v.shape == x.shape else x.expand_as(v)
        v = torch.where((v.abs() == math.inf) & arg.isfinite() & (arg.abs() > 1), v.sign() * 1e300, v)
        return _overflowed(v, case["mode"])
    if case["kind"] == "dft":
        x, w = _dft_inputs(case, seed)
        i = torch.arange(case["n"], device="cuda", dtype=torch.float32)
        rows = []
        for k in range(case["m"]):
            t = (w[k] * i).double()  # the angle is rounded to binary32, as documented
            rows.append(torch.stack([(t.cos() * x).sum(), -(t.sin() * x).sum()]))
        return torch.stack(rows)
    layout, x, no = _batch_inputs(case, seed)
    out = torch.zeros(no, dtype=torch.float64, device="cuda")
    for func, n, i, o in layout:
        v = _plain(func, x[i:i + n]).reshape(-1)
        out[o:o + v.numel()] = v
    return out
