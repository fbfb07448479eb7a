// cr_f32_trig.h -- correctly rounded sinf, cosf, sincosf, tanf (device).
//
// Paper, Sec. II-A: the trigonometric kernels branch only for large-argument
// reduction.  Here every lane runs the same reduction, branch-free, whatever the
// size of its argument: N = x 32/pi, k = nearest(N), f = N - k in [-1/2, 1/2],
// r = f pi/32, |r| <= pi/64, and q = k mod 64.
//
// Fast path: binary64, with the idea of Payne and Hanek (SIGNUM Newsletter 18(1),
// 1983) that the leading bits of 32/pi only add multiples of 64 to N: they are
// dropped from a constant chosen by the argument's exponent (16 rows for groups of
// 8 exponents), whose first two 29-bit parts give exact products with the 24-bit
// argument (trig_fast_core).
//
// Accurate path: Payne-Hanek in 32-bit integer arithmetic.
//   x = M 2^E (M a 24-bit integer).  N = x 32/pi = M 2^(E+4) sum_i g_i 2^-i
//   with g_i the bits of 2/pi.  Bits with i <= E - 2 only add multiples of 64
//   to N, so a 160-bit window W of 2/pi starting at bit E - 1 suffices:
//   N = M W 2^-154 (mod 64), truncation error < 2^24 2^-154 = 2^-130.
//   The window is read from an 11-word table (two zero words, then 288 bits
//   of 2/pi) with funnel shifts; the binary point of P = M W is always bit
//   154.  The zero words let the window start before the binary point, so the
//   reduction is also right for small arguments (down to 2^-37).
//
//   With theta = q pi/32 = quad pi/2 + j pi/32 (j = q mod 16), a 16-entry table
//   gives sin and cos of j pi/32 (double-double); quadrant symmetries give
//   sin/cos theta, and
//       sin x = sin theta cos r + cos theta sin r,
//       cos x = cos theta cos r - sin theta sin r,   tan x = sin x / cos x.
//   Near the zeros of sin/cos (j = 0) the table terms are exactly 0 and +-1,
//   so the result is +-sin r or +-cos r without cancellation.
#pragma once
#include "cr_consts.h"
#include "cr_round.h"

namespace cr {

enum { TRIGK_SIN = 0, TRIGK_COS = 1, TRIGK_TAN = 2, TRIGK_SINCOS = 3 };

struct TrigTab {
  double4 sc[16];
  double4 red[16];
  unsigned w[11];
};

__device__ __forceinline__ void trig_tab_load(TrigTab& t, int tid) {
  if (tid < 16) {
    t.sc[tid] = SINCOS_T[tid];
    t.red[tid] = TRIG_RED[tid];
  }
  if (tid < 11) t.w[tid] = TWO_OVER_PI_W[tid];
}

struct Reduced {
  int q;                  // k mod 64
  long long fhi;          // f = (fhi + flo 2^-64) 2^-64, signed
  unsigned long long flo;
};

// The 32-bit words of the window W that starts at bit sp of the zero-prefixed
// bit string of 2/pi: word k is bits [sp + 32k, sp + 32k + 32), the funnel
// shift of w[b + k] and w[b + k + 1] right by c, with b = ceil(sp / 32) - 1 and
// c = -sp mod 32 (c = 0 when sp is a multiple of 32: word k is then
// w[b + k + 1] itself), so that the shift count stays in [0, 31].
struct Window {
  int b;
  unsigned c;
};
__device__ __forceinline__ Window window_of(int sp) {
  return {((sp + 31) >> 5) - 1, (unsigned)(-sp) & 31u};
}
// ((hi:lo) >> c) mod 2^32 for c in [0, 31]: one funnel shift
__device__ __forceinline__ uint32_t funnel(uint32_t hi, uint32_t lo, unsigned c) {
  return __builtin_amdgcn_alignbit(hi, lo, c);
}
__device__ __forceinline__ uint32_t window_word(uint32_t hi, uint32_t lo, unsigned c) {
  return funnel(hi, lo, c);
}

// Payne-Hanek reduction of |x| (ax = its encoding), 2^-37 <= |x| finite;
// other encodings are clamped to in-range table indices (their result is
// discarded by the caller).
__device__ __forceinline__ Reduced payne_hanek(uint32_t ax, const unsigned* w) {
  int E = (int)(ax >> 23) - 150;
  E = E < -60 ? -60 : (E > 105 ? 105 : E);
  uint32_t M = (ax & 0x007fffffu) | 0x00800000u;
  const Window win = window_of(E - 2 + 64);  // window start: [2, 167]
  const unsigned* t = w + win.b;             // words b .. b + 5 <= 10
  uint32_t W0 = window_word(t[0], t[1], win.c);
  uint32_t W1 = window_word(t[1], t[2], win.c);
  uint32_t W2 = window_word(t[2], t[3], win.c);
  uint32_t W3 = window_word(t[3], t[4], win.c);
  uint32_t W4 = window_word(t[4], t[5], win.c);
  // P = M W, least significant word first (each step is one 32x32+64 multiply-add)
  uint64_t a = (uint64_t)M * W4;
  uint32_t p0 = (uint32_t)a;
  a = (uint64_t)M * W3 + (a >> 32);
  uint32_t p1 = (uint32_t)a;
  a = (uint64_t)M * W2 + (a >> 32);
  uint32_t p2 = (uint32_t)a;
  a = (uint64_t)M * W1 + (a >> 32);
  uint32_t p3 = (uint32_t)a;
  a = (uint64_t)M * W0 + (a >> 32);
  uint32_t p4 = (uint32_t)a;
  // integer bits 154..159 = p4[31:26]; fraction bits 153..26, by 32-bit words
  // the funnel shifts of (p4:p3), (p3:p2), (p2:p1), (p1:p0) right by 26
  Reduced R;
  R.q = (int)((((p4 >> 25) + 1) >> 1) & 63);  // round to nearest: + fraction bit 153
  R.fhi = (long long)(((uint64_t)funnel(p4, p3, 26) << 32) | funnel(p3, p2, 26));  // f - 1 when f >= 1/2
  R.flo = ((uint64_t)funnel(p2, p1, 26) << 32) | funnel(p1, p0, 26);
  return R;
}

// sin/cos of theta = q pi/32 as double-doubles, from the table and the quadrant
struct SinCosTheta {
  double sh, sl, ch, cl;
};

__device__ __forceinline__ SinCosTheta theta_of(int q, const TrigTab& tb) {
  // quad 0: (S, C); 1: (C, -S); 2: (-S, -C); 3: (-C, S).  The swap of odd
  // quadrants picks which half of the 32-byte table row is read for each
  // pair (an address offset instead of selects on four doubles), and the
  // signs are flipped on the sign bits.
  const int quad = q >> 4;
  const int swap = quad & 1;
  const double2* row = reinterpret_cast<const double2*>(&tb.sc[q & 15]);
  const double2 S = row[swap], C = row[swap ^ 1];
  const long long ms = (long long)(quad >= 2) << 63;
  const long long mc = (long long)(quad == 1 || quad == 2) << 63;
  SinCosTheta r;
  r.sh = __longlong_as_double(__double_as_longlong(S.x) ^ ms);
  r.sl = __longlong_as_double(__double_as_longlong(S.y) ^ ms);
  r.ch = __longlong_as_double(__double_as_longlong(C.x) ^ mc);
  r.cl = __longlong_as_double(__double_as_longlong(C.y) ^ mc);
  return r;
}

// Branch-free: res is always written (meaningful only when true is returned).
__device__ __forceinline__ bool trig_special(float xf, float& res, int kind) {
  const bool nan = xf != xf;
  const bool inf = (f32_bits(xf) & 0x7fffffffu) == 0x7f800000u;
  const bool zero = xf == 0.0f;
  float v = zero ? (kind == TRIGK_COS ? 1.0f : xf) : bits_f32(0x7fc00000u);  // sin, tan keep -0
  res = nan_or(xf, v);
  return nan | inf | zero;
}

// The fast path's special cases: NaN (returned quieted: canonicalize keeps its sign
// and payload) and infinities (the default NaN).  Zeros and tiny arguments
// need no case of their own: the reduction keeps a relative error down to the smallest
// subnormal, so for |x| < 2^-12, where sin x and tan x lie within 2^-25.5 |x| of x and
// cos x within 2^-25 of 1, the value is less than half a spacing away from x (or 1), on
// which it rounds; where its low bits come within the test's reach of the midpoint
// (cos x near |x| = 2^-12) the accurate path decides.
__device__ __forceinline__ bool trig_special_fast(float xf, float& res) {
  const float q = __builtin_canonicalizef(xf);
  res = fabsf(xf) == INFINITY ? bits_f32(0x7fc00000u) : q;
  return __builtin_amdgcn_class(xf, 0x207);
}

// v with its sign flipped where the mask m has bit 31 set (one operation on
// the high word)
__device__ __forceinline__ double flip(double v, uint32_t m) {
  return __hiloint2double(__double2hiint(v) ^ (int)(m & 0x80000000u), __double2loint(v));
}

// Fast path: binary64 sin and cos of |x| up to the quadrant's signs: sin |x| is s
// with its sign flipped by the mask ss (bit 31), cos |x| is c flipped by sc.
struct TrigFast {
  double s, c;
  uint32_t ss, sc;  // sign masks
};

// Bound by VALU issue.  The reduction takes 8 binary64 operations and two LDS reads
// for every argument; it replaced an integer Payne-Hanek reduction on 96 bits of 2/pi
// (three 64-bit multiply-adds, five funnel shifts, two conversions) with a branch to a
// three-part Cody-Waite form for waves whose arguments all lay below 2^23 (14
// operations), each with an absolute error that sent results below 2^-12 to the
// accurate path.  Measured at 2^24 elements, arguments of every magnitude: sinf 47.6 ->
// 37.5 us, cosf 48.4 -> 38.7, tanf 56.1 -> 44.3, sincosf 58.8 -> 50.2; in (0.05, 0.95):
// sinf 34.2 -> 31.2, tanf 42.0 -> 34.9, sincosf 42.0 -> 38.8.
__device__ __forceinline__ TrigFast trig_fast_core(float xf, const TrigTab& tb) {
  const uint32_t ax = f32_bits(xf) & 0x7fffffffu;
  const double a = (double)bits_f32(ax);
  // Row g of the table serves |x| in [2^(8g+1), 2^(8g+9)), row 0 all smaller
  // arguments too (the exponent field is at most 255: g <= 15).  With c1 + c2 + c3 =
  // 32/pi less the bits that only add multiples of 64 to N:
  //  * a c1 < 2^37 is an exact product (24 + 29 bits), a multiple of 2^-23, and a c2 <
  //    2^8 is exact too; their sum is rounded by at most 2^-17, and adding 1.5 2^52
  //    rounds it to the integer k, whose low bits are the low word of t;
  //  * a c1 - k is exact (below 2^8 + 1 in magnitude, a multiple of 2^-23);
  //  * f = (a c1 - k) + a c2 + a c3, |f| <= 1/2 + 2^-17, carries two roundings
  //    relative to the sums themselves and the rounding of c3 times a: f is within
  //    2^-52 |f| + 2^-74 of N - k (mod 64).
  const double4& w = tb.red[max(ax >> 26, 16u) - 16u];
  const double p2 = a * w.y;
  const double t = fma(a, w.x, p2) + 0x1.8p52;
  const double f = fma(a, w.z, fma(a, w.x, -(t - 0x1.8p52)) + p2);
  const uint32_t q = (uint32_t)__double2loint(t);  // bits 0..5 are used
  // r = f pi/32; the polynomials are in f
  const double f2 = f * f;
  const double sr = f * fma(fma(fma(SIN_F[3], f2, SIN_F[2]), f2, SIN_F[1]), f2, SIN_F[0]);  // sin r
  const double cm1 = f2 * fma(fma(COS_F[2], f2, COS_F[1]), f2, COS_F[0]);  // cos r - 1
  // theta = q pi/32 = quad pi/2 + j pi/32, with T1, T2 = sin, cos of j pi/32
  // (the high parts of table row j) swapped in odd quadrants: an offset of
  // the two reads, from bit 4 of q.  Then
  //   sin x = +-(T1 + T1 (cos r - 1) + T2 sr'),
  //   cos x = +-(T2 + T2 (cos r - 1) - T1 sr'),
  // with sr' = sin r negated in odd quadrants and the outer signs given by
  // bit 5 of q (sin) and bit 4 xor bit 5 (cos).
  const double* row = reinterpret_cast<const double*>(&tb.sc[q & 15]);
  const uint32_t sw = (q >> 3) & 2;
  const double T1 = row[sw], T2 = row[sw ^ 2];
  const double srq = flip(sr, q << 27);
  TrigFast o;
  o.s = T1 + fma(T1, cm1, T2 * srq);
  o.c = T2 + fma(T2, cm1, -(T1 * srq));
  o.ss = q << 26;
  o.sc = (q ^ (q << 1)) << 26;
  // Errors: sin r within 2^-50.8 |r| + 2^-77 (the reduction, pi/32 to 2^-54, the
  // polynomial's last addition and the product; its approximation and its other
  // coefficients far below), cos r - 1 within 2^-56 (the bound tests re-derive both
  // approximation errors); the table entries within 2^-54 each; three roundings of
  // terms below 0.05 and the final one of y.  With |sin x|, |cos x| >= 0.049 unless
  // j = 0 this is below 2^-52 absolute, i.e. 2^-47.6 |y|.  For j = 0 the table terms are
  // exactly 0 and 1 and y is +-sin r or +-cos r; no binary32 x lies closer than
  // 2^-30 to a multiple of pi/2, other than below pi/64 itself, so sin r is within
  // 2^-46 |y| there, and cos r within 2^-52 |y|.  Bound used: 2^-45 |y|.
  return o;
}

// bit 31 set when x is negative
__device__ __forceinline__ uint32_t sign_mask(float xf) { return f32_bits(xf); }

// The rounding test of the sin and cos fast paths, read off the bits of yh: the bound
// above is below 256 ulps of yh, which are at least 2^-53 |yh| (just below a power of
// two; 2^-52 |yh| at one), so a binary32 midpoint can lie within the error only when
// the 29 low bits of yh come within 256 of the midpoint pattern 2^28 (cr_round.h,
// round_f32_bits); 512 leaves a factor of 2.  All results are normal numbers but those
// of tiny arguments, which lie next to a binary32 number (trig_special_fast).
// tan x is the quotient within 2^-52 (div_fast) of two such values: at j = 0 one within
// 2^-46 and one within 2^-52 of theirs, elsewhere both within 2^-47.6.  2^-45.9 |yh| in
// either case, again below 256 ulps: the same test.
constexpr unsigned TRIG_TEST_E = 512;
__device__ __forceinline__ float round_trig_fast(double yh, bool& ok) {
  return round_f32_bits<TRIG_TEST_E>(yh, ok);
}

// ------------------------------------------------------------ accurate path
__device__ __forceinline__ dd dd_div(dd a, dd b) {
  double q1 = a.hi / b.hi;
  dd p = dd_mul_d(b, q1);
  dd r = dd_add(a, dd_neg(p));
  double q2 = r.hi / b.hi;
  return fast_two_sum(q1, q2);
}

// Round h + l to binary32 given an absolute error bound e (accurate path).
__device__ __forceinline__ float round_f32_dd_abs(double h, double l, double e, bool& ok) {
  dd lo = fast_two_sum(h, l - e);
  dd hi = fast_two_sum(h, l + e);
  float a = (float)ro53(lo.hi, lo.lo);
  float b = (float)ro53(hi.hi, hi.lo);
  ok = a == b;
  return b;
}

struct TrigAcc {
  dd s, c;
  double eabs;  // absolute error bound on each of s, c
};

// sin x and cos x in double-double: 128-bit reduction, Taylor series of
// sin r and cos r (|r| <= pi/64; terms of index >= 4 in binary64).
__device__ __forceinline__ TrigAcc trig_acc_core(float xf, const TrigTab& tb) {
  uint32_t ax = f32_bits(xf) & 0x7fffffffu;
  double axd = (double)bits_f32(ax);
  bool small = axd < PI64;
  Reduced R = payne_hanek(ax, tb.w);
  double d1 = (double)(R.fhi >> 11) * 0x1p-53;
  double d2 = (double)(((uint64_t)(R.fhi & 0x7ff) << 42) | (R.flo >> 22)) * 0x1p-106;
  double d3 = (double)(R.flo & 0x3fffff) * 0x1p-128;
  dd f = dd_add_d(fast_two_sum(d1, d2), d3);
  dd r = dd_mul(f, dd{PI32_HI, PI32_MID});
  r = dd_add_d(r, f.hi * PI32_LO);
  int q = R.q;
  if (small) {
    r = {axd, 0.0};
    q = 0;
  }
  dd r2 = dd_mul(r, r);
  double ph = SIN_TAYLOR[TRIG_TAYLOR_N].x;
#pragma unroll
  for (int k = TRIG_TAYLOR_N - 1; k >= 4; k--) ph = fma(ph, r2.hi, SIN_TAYLOR[k].x);
  dd ps = {ph, 0.0};
#pragma unroll
  for (int k = 3; k >= 0; k--) {
    double2 c = SIN_TAYLOR[k];
    ps = dd_add(dd_mul(ps, r2), dd{c.x, c.y});
  }
  dd sr = dd_mul(ps, r);
  ph = COS_TAYLOR[TRIG_TAYLOR_N].x;
#pragma unroll
  for (int k = TRIG_TAYLOR_N - 1; k >= 4; k--) ph = fma(ph, r2.hi, COS_TAYLOR[k].x);
  dd pc = {ph, 0.0};
#pragma unroll
  for (int k = 3; k >= 0; k--) {
    double2 c = COS_TAYLOR[k];
    pc = dd_add(dd_mul(pc, r2), dd{c.x, c.y});
  }
  SinCosTheta th = theta_of(q, tb);
  dd S = {th.sh, th.sl}, C = {th.ch, th.cl};
  TrigAcc o;
  o.s = dd_add(dd_mul(S, pc), dd_mul(C, sr));
  o.c = dd_add(dd_mul(C, pc), dd_neg(dd_mul(S, sr)));
  // reduction: |f| error < 2^-129 (window 2^-130, conversion 2^-130), so r is
  // within 2^-102 |r| + 2^-132; double-double arithmetic adds < 2^-98 |result|
  o.eabs = small ? 0.0 : 0x1p-128;
  return o;
}

template <int KIND>
__device__ __noinline__ AccResult trig_accurate(float xf, const TrigTab& tb) {
  float sp;
  if (trig_special(xf, sp, KIND)) return {sp, 1};
  TrigAcc A = trig_acc_core(xf, tb);
  bool neg = xf < 0.0f;
  dd y;
  double e;
  if (KIND == TRIGK_COS) {
    y = A.c;
    e = fma(fabs(y.hi), 0x1p-95, A.eabs);
  } else if (KIND == TRIGK_SIN) {
    y = neg ? dd_neg(A.s) : A.s;
    e = fma(fabs(y.hi), 0x1p-95, A.eabs);
  } else {
    y = dd_div(A.s, A.c);
    if (neg) y = dd_neg(y);
    // relative errors of s and c add; the absolute parts scale with 1/|c|
    double ic = 1.0 / fabs(A.c.hi);
    e = fma(fabs(y.hi), 0x1p-93, A.eabs * ic * (1.0 + fabs(y.hi)) * 2.0);
  }
  bool ok;
  float r = round_f32_dd_abs(y.hi, y.lo, e, ok);
  return {r, ok ? 1 : 0};
}

// sincos accurate path: both results (sin in r, cos in r2)
struct AccResult2 {
  float s, c;
  int ok;
};

__device__ __noinline__ AccResult2 sincos_accurate(float xf, const TrigTab& tb) {
  float ss, cs;
  if (trig_special(xf, ss, TRIGK_SIN)) {
    trig_special(xf, cs, TRIGK_COS);
    return {ss, cs, 1};
  }
  TrigAcc A = trig_acc_core(xf, tb);
  dd s = xf < 0.0f ? dd_neg(A.s) : A.s;
  bool ok1, ok2;
  float rs = round_f32_dd_abs(s.hi, s.lo, fma(fabs(s.hi), 0x1p-95, A.eabs), ok1);
  float rc = round_f32_dd_abs(A.c.hi, A.c.lo, fma(fabs(A.c.hi), 0x1p-95, A.eabs), ok2);
  return {rs, rc, (ok1 && ok2) ? 1 : 0};
}

template <int KIND>
__device__ __forceinline__ float trig_fast(float xf, const TrigTab& tb, bool& ok) {
  TrigFast F = trig_fast_core(xf, tb);
  const uint32_t xs = sign_mask(xf);
  float res;
  if (KIND == TRIGK_COS) {
    res = round_trig_fast(flip(F.c, F.sc), ok);
  } else if (KIND == TRIGK_SIN) {
    res = round_trig_fast(flip(F.s, F.ss ^ xs), ok);
  } else {
    res = round_trig_fast(flip(div_fast(F.s, F.c), F.ss ^ F.sc ^ xs), ok);
  }
  float sp;
  if (trig_special_fast(xf, sp)) {
    res = sp;
    ok = true;
  }
  return res;
}

// sincos fast path: returns sin in the result, cos in *c
__device__ __forceinline__ float sincos_fast(float xf, const TrigTab& tb, float& c, bool& ok) {
  TrigFast F = trig_fast_core(xf, tb);
  bool ok1, ok2;
  float s = round_trig_fast(flip(F.s, F.ss ^ sign_mask(xf)), ok1);
  c = round_trig_fast(flip(F.c, F.sc), ok2);
  ok = ok1 && ok2;
  float sp;
  if (trig_special_fast(xf, sp)) {
    s = c = sp;
    ok = true;
  }
  return s;
}

}  // namespace cr
