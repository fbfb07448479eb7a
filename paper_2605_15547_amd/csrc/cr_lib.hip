// cr_lib.hip -- kernels and the C ABI of libcr (gfx950).
//
// One elementwise map kernel per function (a template over the function's
// evaluator).  Each workgroup stages the function's <= 16-entry tables in LDS
// once, then each thread loads U float4 vectors (128-bit, coalesced: lane i of
// a wave touches bytes [16 i, 16 i + 16) of a contiguous 1 KiB span), evaluates
// the 4U elements and stores U float4 vectors.  One launch takes any length and
// any pointers aligned to their element.
#include <hip/hip_runtime.h>

#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <vector>
#include <mutex>
#include <new>

#include "../../include/cr.h"
#include "cr_f32_exp.h"
#include "cr_f32_log.h"
#include "cr_f32_rsqrt.h"
#include "cr_f32_trig.h"
#include "cr_f32_atan.h"
#include "cr_f32_hyp.h"
#include "cr_f64.h"
#include "cr_f32_dir.h"
#include "cr_split_exp.h"
#include "cr_split_log.h"
#include "cr_split_trig.h"
#include "cr_split_rsqrt.h"
#include "cr_split_atan.h"
#include "cr_split_hyp.h"
#include "cr_split_acc.h"

using namespace cr;

namespace {

// Counters are spread over NSLOT cache lines (slot = block index mod NSLOT)
// so that concurrent workgroups do not serialise on one address; the host
// sums them when they are read.
constexpr int NSLOT = 64;
struct alignas(128) CounterSlot {
  unsigned long long fallback_lanes, fallback_waves;
  unsigned long long pad[14];
};
struct DevStats {
  CounterSlot slot[NSLOT];
  unsigned long long escapes;
  unsigned long long escape_index[16];
};

// Launch-shape knobs (compile-time; the grid size is a run-time knob).
#ifndef CR_TILE_U
#define CR_TILE_U 2
#endif
#ifndef CR_PREFETCH
#define CR_PREFETCH 1
#endif
#ifndef CR_BLOCKS_PER_CU
#define CR_BLOCKS_PER_CU 16
#endif
constexpr int BLOCK = 256;
constexpr int TILE_U = CR_TILE_U;           // float4 vectors per thread per tile (sincosf)
constexpr int TILE = 4096;                  // elements of a batch tile, at most
constexpr int QCAP = 512;                   // deferred elements held in LDS
constexpr int QCHECK = 8;                   // tiles between two looks at the queue
constexpr int QFLUSH = QCAP / 2;            // flush when the queue is fuller than this

// Streaming accesses: each input is read once and each output written once, so
// the 128-bit loads and stores carry the nontemporal hint (measured on MI355X: a
// plain 2^26-float copy moves 5.1-5.5 TB/s without it and 5.8-6.6 TB/s with it,
// depending on the grid).
//
// Tiles of the map kernels.  T is float or double, VN elements make a 128-bit
// vector, and a tile is U vectors per thread (vector u of thread t is vector
// t + u BLOCK of the tile); nv = n / VN whole vectors.  The BLOCK vectors u of a tile
// are accessed through a buffer descriptor of their own, whose base is the first of
// them and whose size ends at nv, built by scalar instructions from the tile's
// number: the hardware drops stores past the end and returns 0 for loads there, so
// the ragged last tile takes the same instructions as any other and no lane computes
// a 64-bit address or a bounds check (expf 4% faster than with per-lane addresses at
// 2^24 elements, binary64 log 4%, sincosf 3%).  One descriptor for the tile and u in
// the access's scalar offset would save a few scalar instructions, but the builtins
// exclude the scalar offset from the range check: it is always 0 here, and the vector
// offset alone, 16 bytes times the thread, is what the hardware checks.
// gfx950 takes 128-bit accesses at any 4-byte address, so a slice of an array, a
// cosine block behind an odd number of sines and an aligned buffer all run the
// same kernel.  The n % VN elements after the last vector are evaluated one to a
// thread by the workgroup that takes the last tile.
#ifndef CR_NT
#define CR_NT 1
#endif
typedef unsigned v4u_t __attribute__((ext_vector_type(4)));
template <class T>
struct Vec;
template <>
struct Vec<float> {
  using type = float4;
  static constexpr int N = 4;
};
template <>
struct Vec<double> {
  using type = double2;
  static constexpr int N = 2;
};

// Vectors u, one a thread, of the tile of BLOCK U vectors that starts at vector t0 of
// the nv vectors at p (counts of vectors fit in 32 bits: LAUNCH_ELEMS elements a
// launch).
template <class T, int U>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(const T* p, int t0, int nv, int u) {
  // the same in every lane: scalar registers (and past the end: an empty tile)
  t0 = min(__builtin_amdgcn_readfirstlane(t0), nv);
  const int left = 16 * min(nv - t0, BLOCK * U);
  char* base = (char*)const_cast<T*>(p) + 16 * (size_t)(unsigned)t0;
  // 0x00020000: raw buffer, 32-bit data format, bounds checked by the byte
  return __builtin_amdgcn_make_buffer_rsrc(
      base + 16 * BLOCK * u, 0, u == 0 ? left : max(left - 16 * BLOCK * u, 0), 0x00020000);
}
template <class T, int U>
__device__ __forceinline__ void tile_load(typename Vec<T>::type (&v)[U], const T* in, int t0,
                                          int nv) {
#pragma unroll
  for (int u = 0; u < U; u++) {
    const v4u_t x = __builtin_amdgcn_raw_buffer_load_b128(tile_rsrc<T, U>(in, t0, nv, u),
                                                          16 * threadIdx.x, 0, CR_NT ? 2 : 0);
    __builtin_memcpy(&v[u], &x, 16);
  }
}
template <class T, int U>
__device__ __forceinline__ void tile_store(const typename Vec<T>::type (&v)[U], T* out, int t0,
                                           int nv) {
#pragma unroll
  for (int u = 0; u < U; u++) {
    v4u_t x;
    __builtin_memcpy(&x, &v[u], 16);
    __builtin_amdgcn_raw_buffer_store_b128(x, tile_rsrc<T, U>(out, t0, nv, u), 16 * threadIdx.x, 0,
                                           CR_NT ? 2 : 0);
  }
}
// Bit VN u + c is set where vector u of the tile lies below nv.
template <class T, int U>
__device__ __forceinline__ unsigned tile_live(int t0, int nv) {
  constexpr int VN = Vec<T>::N;
  unsigned m = 0;
#pragma unroll
  for (int u = 0; u < U; u++)
    m |= (int)threadIdx.x + u * BLOCK < nv - t0 ? ((1u << VN) - 1u) << (VN * u) : 0u;
  return m;
}
// The tail's elements go to the workgroup that takes the tile containing vector nv
// (a ragged tile, or the one after the last full tile): the workgroup's last tile
// or, t0 being where it left the loop, the next.
__device__ __forceinline__ bool takes_tail(int t0, int step, int nv, int tv) {
  const int d = nv - t0, e = d + step;
  return (d >= 0 && d < tv) || (e >= 0 && e < tv);
}

// ------------------------------------------------------------ evaluators
// Op::fast(x, tab, ok): binary64 fast path and rounding test (inlined).
// Op::accurate(x, tab): double-double path from x alone (out of line).
// Op::fast_dir<RM>, Op::dir<RM>: the same two in a directed rounding mode.
template <int K>
struct OpExp {
  using Tab = ExpTab;
  static constexpr int qcheck = QCHECK;
  static __device__ __forceinline__ void load(Tab& t, int tid) { exp_tab_load(t, tid); }
  static __device__ __forceinline__ float fast(float x, const Tab& t, bool& ok) {
    return exp_fast<K>(x, t, ok);
  }
  static __device__ __forceinline__ AccResult accurate(float x, const Tab& t) {
    return exp_accurate<K>(x, t);
  }
  template <int RM>
  static __device__ __forceinline__ float fast_dir(float x, const Tab& t, bool& ok) {
    return exp_fast_dir<K, RM>(x, t, ok);
  }
  template <int RM>
  static __device__ __forceinline__ AccResult dir(float x, const Tab& t) {
    return exp_dir<K, RM>(x, t);
  }
};

// sincos: two outputs per element (planar)
struct SinCosF64 {
  using Tab = TrigTab;
  static constexpr int qcheck = QCHECK;
  static __device__ __forceinline__ void load(Tab& t, int tid) { trig_tab_load(t, tid); }
  static __device__ __forceinline__ float fast(float x, const Tab& t, float& c, bool& ok) {
    return sincos_fast(x, t, c, ok);
  }
  static __device__ __forceinline__ AccResult2 accurate(float x, const Tab& t) {
    return sincos_accurate(x, t);
  }
  template <int RM>
  static __device__ __forceinline__ float fast_dir(float x, const Tab& t, float& c, bool& ok) {
    return sincos_fast_dir<RM>(x, t, c, ok);
  }
  template <int RM>
  static __device__ __forceinline__ AccResult2 dir(float x, const Tab& t) {
    return sincos_dir<RM>(x, t);
  }
};
struct SinCosSplit {
  using Tab = STrigTab;
  static constexpr int qcheck = 1;
  static __device__ __forceinline__ void load(Tab& t, int tid) { strig_tab_load(t, tid); }
  static __device__ __forceinline__ float fast(float x, const Tab& t, float& c, bool& ok) {
    return ssincos_fast(x, t, c, ok);
  }
  static __device__ __forceinline__ AccResult2 accurate(float x, const Tab& t) {
    return ssincos_acc(x, t.w);
  }
};

struct OpSRsqrt {
  using Tab = NoTab;
  static constexpr int qcheck = QCHECK;
  static __device__ __forceinline__ void load(Tab&, int) {}
  static __device__ __forceinline__ float fast(float x, const Tab&, bool& ok) {
    return srsqrt_fast(x, ok);
  }
  static __device__ __forceinline__ AccResult accurate(float x, const Tab&) {
    bool ok;
    return {srsqrt_fast(x, ok), 1};
  }
};

template <int KIND>
struct OpSAtan {
  using Tab = SAtanTab;
  static constexpr int qcheck = 1;  // more lanes fail: look at the queue every tile
  static __device__ __forceinline__ void load(Tab& t, int tid) { satan_tab_load(t, tid); }
  static __device__ __forceinline__ float fast(float x, const Tab& t, bool& ok) {
    return satan_fast<KIND>(x, t, ok);
  }
  static __device__ __forceinline__ AccResult accurate(float x, const Tab& t) {
    return satan_acc<KIND>(x);
  }
};

template <int KIND>
struct OpSHyp {
  using Tab = SHypTab;
  static constexpr int qcheck = 1;  // more lanes fail: look at the queue every tile
  static __device__ __forceinline__ void load(Tab& t, int tid) { shyp_tab_load(t, tid); }
  static __device__ __forceinline__ float fast(float x, const Tab& t, bool& ok) {
    return shyp_fast<KIND>(x, t, ok);
  }
  static __device__ __forceinline__ AccResult accurate(float x, const Tab& t) {
    return shyp_acc<KIND>(x);
  }
};

template <int KIND>
struct OpSTrig {
  using Tab = STrigTab;
  static constexpr int qcheck = 1;  // more lanes fail: look at the queue every tile
  static __device__ __forceinline__ void load(Tab& t, int tid) { strig_tab_load(t, tid); }
  static __device__ __forceinline__ float fast(float x, const Tab& t, bool& ok) {
    return strig_fast<KIND>(x, t, ok);
  }
  static __device__ __forceinline__ AccResult accurate(float x, const Tab& t) {
    return strig_acc<KIND>(x, t.w);
  }
};

// binary32-only (float-float) fast paths; failing lanes take the triple-float
// step (cr_split_acc.h): no binary64 operation on the whole path
template <int K>
struct OpSExp {
  using Tab = SExpTab;
  static constexpr int qcheck = 1;  // more lanes fail: look at the queue every tile
  static __device__ __forceinline__ void load(Tab& t, int tid) { sexp_tab_load<K>(t, tid); }
  static __device__ __forceinline__ float fast(float x, const Tab& t, bool& ok) {
    return sexp_fast<K>(x, t, ok);
  }
  static __device__ __forceinline__ AccResult accurate(float x, const Tab& t) {
    return sexp_acc<K>(x);
  }
};

template <int K>
struct OpSLog {
  using Tab = SLogTab;
  static constexpr int qcheck = 1;  // more lanes fail: look at the queue every tile
  static __device__ __forceinline__ void load(Tab& t, int tid) { slog_tab_load<K>(t, tid); }
  static __device__ __forceinline__ float fast(float x, const Tab& t, bool& ok) {
    return slog_fast<K>(x, t, ok);
  }
  static __device__ __forceinline__ AccResult accurate(float x, const Tab& t) {
    return slog_acc<K>(x);
  }
};

template <int K>
struct OpLog {
  using Tab = LogTab;
  static constexpr int qcheck = QCHECK;
  static __device__ __forceinline__ void load(Tab& t, int tid) { log_tab_load<K>(t, tid); }
  static __device__ __forceinline__ float fast(float x, const Tab& t, bool& ok) {
    return log_fast<K>(x, t, ok);
  }
  static __device__ __forceinline__ AccResult accurate(float x, const Tab& t) {
    return log_accurate<K>(x, t);
  }
  template <int RM>
  static __device__ __forceinline__ float fast_dir(float x, const Tab& t, bool& ok) {
    return log_fast_dir<K, RM>(x, t, ok);
  }
  template <int RM>
  static __device__ __forceinline__ AccResult dir(float x, const Tab& t) {
    return log_dir<K, RM>(x, t);
  }
};

// rsqrtf decides its rounding exactly in the fast path: nothing is deferred.
struct OpRsqrt {
  using Tab = NoTab;
  static constexpr int qcheck = QCHECK;
  static __device__ __forceinline__ void load(Tab&, int) {}
  static __device__ __forceinline__ float fast(float x, const Tab&, bool& ok) {
    return rsqrt_fast(x, ok);
  }
  static __device__ __noinline__ AccResult accurate(float x, const Tab&) {
    bool ok;
    return {rsqrt_fast(x, ok), 1};
  }
  template <int RM>
  static __device__ __forceinline__ float fast_dir(float x, const Tab&, bool& ok) {
    ok = true;
    return rsqrt_fast_dir<RM>(x);
  }
  template <int RM>
  static __device__ __forceinline__ AccResult dir(float x, const Tab&) {
    return rsqrt_dir<RM>(x);
  }
};

template <int KIND>
struct OpTrig {
  using Tab = TrigTab;
  static constexpr int qcheck = QCHECK;
  static __device__ __forceinline__ void load(Tab& t, int tid) { trig_tab_load(t, tid); }
  static __device__ __forceinline__ float fast(float x, const Tab& t, bool& ok) {
    return trig_fast<KIND>(x, t, ok);
  }
  static __device__ __forceinline__ AccResult accurate(float x, const Tab& t) {
    return trig_accurate<KIND>(x, t);
  }
  template <int RM>
  static __device__ __forceinline__ float fast_dir(float x, const Tab& t, bool& ok) {
    return trig_fast_dir<KIND, RM>(x, t, ok);
  }
  template <int RM>
  static __device__ __forceinline__ AccResult dir(float x, const Tab& t) {
    return trig_dir<KIND, RM>(x, t);
  }
};

template <int KIND>
struct OpAtan {
  using Tab = AtanTab;
  static constexpr int qcheck = QCHECK;
  static __device__ __forceinline__ void load(Tab& t, int tid) { atan_tab_load(t, tid); }
  static __device__ __forceinline__ float fast(float x, const Tab& t, bool& ok) {
    return atan_fast<KIND>(x, t, ok);
  }
  static __device__ __forceinline__ AccResult accurate(float x, const Tab& t) {
    return atan_accurate<KIND>(x, t);
  }
  template <int RM>
  static __device__ __forceinline__ float fast_dir(float x, const Tab& t, bool& ok) {
    return atan_fast_dir<KIND, RM>(x, t, ok);
  }
  template <int RM>
  static __device__ __forceinline__ AccResult dir(float x, const Tab& t) {
    return atan_dir<KIND, RM>(x, t);
  }
};

template <int KIND>
struct OpHyp {
  using Tab = ExpTab;
  static constexpr int qcheck = QCHECK;
  static __device__ __forceinline__ void load(Tab& t, int tid) { exp_tab_load(t, tid); }
  static __device__ __forceinline__ float fast(float x, const Tab& t, bool& ok) {
    return hyp_fast<KIND>(x, t, ok);
  }
  static __device__ __forceinline__ AccResult accurate(float x, const Tab& t) {
    return hyp_accurate<KIND>(x, t);
  }
  template <int RM>
  static __device__ __forceinline__ float fast_dir(float x, const Tab& t, bool& ok) {
    return hyp_fast_dir<KIND, RM>(x, t, ok);
  }
  template <int RM>
  static __device__ __forceinline__ AccResult dir(float x, const Tab& t) {
    return hyp_dir<KIND, RM>(x, t);
  }
};

// Block-level bookkeeping of the accurate path, kept in LDS.
struct Deferred {
  unsigned n;                 // entries in the queue
  unsigned lanes, waves;      // counters of this workgroup
  unsigned idx[QCAP];         // element index (relative to the launch)
  float x[QCAP];              // the input value (the output may alias it)
};

__device__ __forceinline__ void note_escape(DevStats* st, long long idx) {
  unsigned long long slot = atomicAdd(&st->escapes, 1ull);
  if (slot < 16) st->escape_index[slot] = (unsigned long long)idx;
}

// Runs body(k) on every queued entry k, 256 at a time (whole waves).
// FINAL = false: then empties the queue; all threads of the workgroup take
// part.  FINAL = true: the workgroup's last flush, after its final barrier; no
// barrier follows, so waves with no entry retire at once and free their slots
// for the next workgroup while the others run the accurate path, and the
// workgroup's counters go to the device statistics.
template <bool FINAL, class Q, class Body>
__device__ __forceinline__ void run_queue(Q& q, DevStats* st, Body body) {
  // q.n counts every enqueue attempt; entries past QCAP were never stored
  // (those elements took the accurate path in place), so only QCAP are valid
  const unsigned n = q.n < QCAP ? q.n : QCAP;
  for (unsigned k = threadIdx.x; k < n; k += BLOCK) body(k);
  if (FINAL) {
    if (threadIdx.x == 0) {
      const unsigned lanes = q.lanes + n, waves = q.waves + (n + 63) / 64;
      if (lanes) {
        CounterSlot& c = st->slot[blockIdx.x % NSLOT];
        atomicAdd(&c.fallback_lanes, (unsigned long long)lanes);
        atomicAdd(&c.fallback_waves, (unsigned long long)waves);
      }
    }
  } else {
    if (threadIdx.x == 0) {
      q.lanes += n;
      q.waves += (n + 63) / 64;
    }
    __syncthreads();
    if (threadIdx.x == 0) q.n = 0;
    __syncthreads();
  }
}

template <class Op, bool FINAL = false>
__device__ __forceinline__ void flush_queue(Deferred& q, const typename Op::Tab& tab, float* out,
                                            DevStats* st, long long elem_base) {
  run_queue<FINAL>(q, st, [&](unsigned k) {
    AccResult a = Op::accurate(q.x[k], tab);
    out[q.idx[k]] = a.r;
    if (!a.ok) note_escape(st, elem_base + q.idx[k]);
  });
}

// ---------------------------------------------------------------- kernels
// Persistent elementwise map.  Each workgroup walks tiles of 1024 U elements
// (tile t, t + gridDim.x, ...).  Per tile every thread loads U float4 (lane i of
// a wave touches bytes [16 i, 16 i + 16) of a contiguous 1 KiB span), runs the
// fast path on its 4U elements and stores.
// Elements whose fast result is not certified are queued in LDS (index and
// input value) and re-evaluated by the accurate path a whole workgroup at a
// time -- when the queue passes QFLUSH and at the end -- so a rare failing
// lane does not make a 64-lane wave run the slow path for it alone.
// The call's whole range is one launch at any length and alignment, bound by
// the VALU work per element (large arrays) or by the launch (small ones).
// Measured against a scalar kernel for heads, tails and pointers of different
// alignment beside a 16-byte aligned body: expf of 2^22 - 1 elements 10.4 -> 8.1
// us (one launch instead of two), of 2^26 elements from a slice x[1:] 159 -> 97
// us (scalar accesses before), sincosf of a slice of 2^24 73 -> 49 us.
// Launch-shape variants (chosen per function by the autotuner, cr_autotune):
//   U   float4 vectors per thread per tile (4U elements per thread),
//   PF  1: the next tile's vectors are loaded while this one is evaluated,
//   TP  table placement: 0 = staged in LDS per workgroup, 1 = read from a
//       device-global copy through the vector caches (no staging).
template <class Op>
__device__ typename Op::Tab g_tab;

template <class Op>
__global__ void k_tab_init() {
  Op::load(g_tab<Op>, threadIdx.x);
}

template <class Op, int U, int PF, int TP>
__global__ void __launch_bounds__(BLOCK)
    k_map_f32(const float* in, float* out, long long n, DevStats* st, unsigned flags,
              long long elem_base) {
  __shared__ typename Op::Tab lds_tab;
  __shared__ Deferred q;
  constexpr int TV = BLOCK * U;  // vectors per tile
  const typename Op::Tab& tab = TP ? g_tab<Op> : lds_tab;
  if (!TP) Op::load(lds_tab, threadIdx.x);
  if (threadIdx.x == 0) {
    q.n = 0;
    q.lanes = q.waves = 0;
  }
  __syncthreads();
  const bool force = flags & CR_FLAG_FORCE_FALLBACK;
  const int n4 = (int)(n >> 2), step = (int)gridDim.x * TV;
  int t0 = (int)blockIdx.x * TV;
  // queue element i (of this launch) with input x, or run its accurate path in
  // place when the queue is full (only with pathological inputs or force)
  auto enqueue = [&](unsigned i, float x, float& res) {
    unsigned pos = atomicAdd(&q.n, 1u);
    if (pos < QCAP) {
      q.idx[pos] = i;
      q.x[pos] = x;
    } else {
      AccResult a = Op::accurate(x, tab);
      res = a.r;
      atomicAdd(&q.lanes, 1u);
      if (!a.ok) note_escape(st, elem_base + i);
    }
  };
  // software pipelining: the next tile's vectors are loaded while this tile is
  // evaluated
  float4 nxt[U];
  if (PF) tile_load<float, U>(nxt, in, t0, n4);
  int iter = 0;
  for (; t0 < n4; t0 += step, iter++) {
    float4 v[U];
    if (PF) {
#pragma unroll
      for (int u = 0; u < U; u++) v[u] = nxt[u];
      tile_load<float, U>(nxt, in, t0 + step, n4);
    } else {
      tile_load<float, U>(v, in, t0, n4);
    }
    // Evaluate every element of the tile first -- straight-line code with no
    // branch between elements, so the scheduler can interleave their
    // dependency chains -- then queue the elements that failed the test.
    float xin[4 * U];
    unsigned fail = 0;
#pragma unroll
    for (int u = 0; u < U; u++) {
      float* e = reinterpret_cast<float*>(&v[u]);
#pragma unroll
      for (int c = 0; c < 4; c++) {
        bool ok;
        xin[4 * u + c] = e[c];
        e[c] = Op::fast(e[c], tab, ok);
        fail |= (unsigned)(!ok || force) << (4 * u + c);
      }
    }
    if (t0 + TV > n4) fail &= tile_live<float, U>(t0, n4);
    if (fail) {
      const unsigned i0 = 4 * ((unsigned)t0 + threadIdx.x);
#pragma unroll
      for (int u = 0; u < U; u++) {
        float* e = reinterpret_cast<float*>(&v[u]);
#pragma unroll
        for (int c = 0; c < 4; c++)
          if (fail & (1u << (4 * u + c))) enqueue(i0 + 4 * u * BLOCK + c, xin[4 * u + c], e[c]);
      }
    }
    tile_store<float, U>(v, out, t0, n4);
    if (iter % Op::qcheck == Op::qcheck - 1) {
      // every thread must see the same fill level: read it between two
      // barriers (no thread can queue more elements before all have read it)
      __syncthreads();
      const unsigned nq = __builtin_amdgcn_readfirstlane(q.n);
      __syncthreads();
      if (nq > QFLUSH) flush_queue<Op>(q, tab, out, st, elem_base);
    }
  }
  if ((n & 3) > threadIdx.x && takes_tail(t0, step, n4, TV)) {
    const long long i = 4 * n4 + threadIdx.x;
    bool ok;
    const float x = in[i];
    float r = Op::fast(x, tab, ok);
    if (!ok || force) enqueue((unsigned)i, x, r);
    out[i] = r;
  }
  __syncthreads();
  flush_queue<Op, true>(q, tab, out, st, elem_base);
}

// sincosf: the map kernel with two planar outputs (sin block, cos block).
template <class SC, bool FINAL = false>
__device__ __forceinline__ void flush_queue_sincos(Deferred& q, const typename SC::Tab& tab,
                                                   float* os, float* oc, DevStats* st,
                                                   long long elem_base) {
  run_queue<FINAL>(q, st, [&](unsigned k) {
    AccResult2 a = SC::accurate(q.x[k], tab);
    os[q.idx[k]] = a.s;
    oc[q.idx[k]] = a.c;
    if (!a.ok) note_escape(st, elem_base + q.idx[k]);
  });
}

template <class SC>
__global__ void __launch_bounds__(BLOCK)
    k_map_sincos(const float* in, float* outs, float* outc, long long n, DevStats* st,
                 unsigned flags, long long elem_base) {
  __shared__ typename SC::Tab tab;
  __shared__ Deferred q;
  constexpr int TV = BLOCK * TILE_U;  // vectors per tile
  SC::load(tab, threadIdx.x);
  if (threadIdx.x == 0) {
    q.n = 0;
    q.lanes = q.waves = 0;
  }
  __syncthreads();
  const bool force = flags & CR_FLAG_FORCE_FALLBACK;
  const int n4 = (int)(n >> 2), step = (int)gridDim.x * TV;
  // element i of this launch: fast path, queue or accurate path in place
  auto one = [&](unsigned i, float x, float& s, float& c) {
    bool ok;
    s = SC::fast(x, tab, c, ok);
    if (!ok || force) {
      unsigned pos = atomicAdd(&q.n, 1u);
      if (pos < QCAP) {
        q.idx[pos] = i;
        q.x[pos] = x;
      } else {
        AccResult2 a = SC::accurate(x, tab);
        s = a.s;
        c = a.c;
        atomicAdd(&q.lanes, 1u);
        if (!a.ok) note_escape(st, elem_base + i);
      }
    }
  };
  int t0 = (int)blockIdx.x * TV;
  int iter = 0;
  for (; t0 < n4; t0 += step, iter++) {
    float4 v[TILE_U], c4[TILE_U];
    tile_load<float, TILE_U>(v, in, t0, n4);
    const unsigned i0 = 4 * ((unsigned)t0 + threadIdx.x);
#pragma unroll
    for (int u = 0; u < TILE_U; u++) {
      if (t0 + (int)threadIdx.x + u * BLOCK < n4) {
        float* e = reinterpret_cast<float*>(&v[u]);
        float* ec = reinterpret_cast<float*>(&c4[u]);
#pragma unroll
        for (int c = 0; c < 4; c++) one(i0 + 4 * u * BLOCK + c, e[c], e[c], ec[c]);
      }
    }
    tile_store<float, TILE_U>(v, outs, t0, n4);
    tile_store<float, TILE_U>(c4, outc, t0, n4);
    if (iter % SC::qcheck == SC::qcheck - 1) {
      __syncthreads();
      const unsigned nq = __builtin_amdgcn_readfirstlane(q.n);
      __syncthreads();
      if (nq > QFLUSH) flush_queue_sincos<SC>(q, tab, outs, outc, st, elem_base);
    }
  }
  if ((n & 3) > threadIdx.x && takes_tail(t0, step, n4, TV)) {
    const long long i = 4 * n4 + threadIdx.x;
    float s, c;
    one((unsigned)i, in[i], s, c);
    outs[i] = s;
    outc[i] = c;
  }
  __syncthreads();
  flush_queue_sincos<SC, true>(q, tab, outs, outc, st, elem_base);
}

// ------------------------------------------------------------ binary64 map
struct OpExp64 {
  using Tab = Exp64Tab;
  static constexpr int qcheck = QCHECK;
  static __device__ __forceinline__ void load(Tab& t, int tid) { exp64_tab_load(t, tid); }
  static __device__ __forceinline__ double fast(double x, const Tab& t, bool& ok) {
    return exp64_fast(x, t, ok);
  }
  static __device__ __forceinline__ AccResultD accurate(double x, const Tab& t) {
    return exp64_accurate(x, t);
  }
};
struct OpLog64 {
  using Tab = Log64Tab;
  static constexpr int qcheck = QCHECK;
  static __device__ __forceinline__ void load(Tab& t, int tid) { log64_tab_load(t, tid); }
  static __device__ __forceinline__ double fast(double x, const Tab& t, bool& ok) {
    return log64_fast(x, t, ok);
  }
  static __device__ __forceinline__ AccResultD accurate(double x, const Tab& t) {
    return log64_accurate(x, t);
  }
};

// binary64 log with the paper's 128-entry scaled-integer table (main path);
// lanes that fail its test take the 16-entry accurate path
struct OpLog128 {
  using Tab = Log128Tab;
  static constexpr int qcheck = QCHECK;
  static __device__ __forceinline__ void load(Tab& t, int tid) { log128_tab_load(t, tid); }
  static __device__ __forceinline__ double fast(double x, const Tab& t, bool& ok) {
    return log128_fast(x, t, ok);
  }
  static __device__ __forceinline__ AccResultD accurate(double x, const Tab& t) {
    return log64_accurate(x, t.acc);
  }
};
struct OpExp2_64 {
  using Tab = Exp2_64Tab;
  static constexpr int qcheck = QCHECK;
  static __device__ __forceinline__ void load(Tab& t, int tid) { exp2_64_tab_load(t, tid); }
  static __device__ __forceinline__ double fast(double x, const Tab& t, bool& ok) {
    return exp2_64_fast(x, t, ok);
  }
  static __device__ __forceinline__ AccResultD accurate(double x, const Tab& t) {
    return exp2_64_accurate(x, t);
  }
};

struct Deferred64 {
  unsigned n, lanes, waves;
  unsigned idx[QCAP];
  double x[QCAP];
};

template <class Op, bool FINAL = false>
__device__ __forceinline__ void flush_queue64(Deferred64& q, const typename Op::Tab& tab,
                                              double* out, DevStats* st, long long elem_base) {
  run_queue<FINAL>(q, st, [&](unsigned k) {
    AccResultD a = Op::accurate(q.x[k], tab);
    out[q.idx[k]] = a.r;
    if (!a.ok) note_escape(st, elem_base + q.idx[k]);
  });
}

// The binary64 form of k_map_f32: tiles of BLOCK U double2 vectors (U per
// thread).  Launch-shape variants (chosen per function by the autotuner):
//   SL 0: each element is evaluated and, if its test fails, queued before the
//         next one (a branch between elements),
//   SL 1: as in k_map_f32, every element of the tile is evaluated in
//         straight-line code first (the scheduler interleaves their
//         dependency chains) and the failing ones are queued afterwards.
template <class Op, int U, int SL>
__global__ void __launch_bounds__(BLOCK)
    k_map_f64(const double* in, double* out, long long n, DevStats* st, unsigned flags,
              long long elem_base) {
  __shared__ typename Op::Tab tab;
  __shared__ Deferred64 q;
  constexpr int TV = BLOCK * U;  // vectors per tile
  Op::load(tab, threadIdx.x);
  if (threadIdx.x == 0) {
    q.n = 0;
    q.lanes = q.waves = 0;
  }
  __syncthreads();
  const bool force = flags & CR_FLAG_FORCE_FALLBACK;
  // queue element j (of this launch) with input x, or run its accurate path in
  // place when the queue is full
  auto enqueue = [&](unsigned j, double x, double& res) {
    unsigned pos = atomicAdd(&q.n, 1u);
    if (pos < QCAP) {
      q.idx[pos] = j;
      q.x[pos] = x;
    } else {
      AccResultD a = Op::accurate(x, tab);
      res = a.r;
      atomicAdd(&q.lanes, 1u);
      if (!a.ok) note_escape(st, elem_base + j);
    }
  };
  const int n2 = (int)(n >> 1), step = (int)gridDim.x * TV;
  int t0 = (int)blockIdx.x * TV;
  int iter = 0;
  for (; t0 < n2; t0 += step, iter++) {
    const unsigned j0 = 2 * ((unsigned)t0 + threadIdx.x);
    double2 v[U];
    tile_load<double, U>(v, in, t0, n2);
    if (SL) {
      // slots past the end hold 0: evaluated, never stored or queued
      double xin[2 * U];
      unsigned fail = 0;
#pragma unroll
      for (int u = 0; u < U; u++) {
        double* e = reinterpret_cast<double*>(&v[u]);
#pragma unroll
        for (int c = 0; c < 2; c++) {
          bool ok;
          xin[2 * u + c] = e[c];
          e[c] = Op::fast(e[c], tab, ok);
          fail |= (unsigned)(!ok || force) << (2 * u + c);
        }
      }
      if (t0 + TV > n2) fail &= tile_live<double, U>(t0, n2);
      if (fail) {
#pragma unroll
        for (int u = 0; u < U; u++) {
          double* e = reinterpret_cast<double*>(&v[u]);
#pragma unroll
          for (int c = 0; c < 2; c++)
            if ((fail >> (2 * u + c)) & 1u)
              enqueue(j0 + 2 * u * BLOCK + c, xin[2 * u + c], e[c]);
        }
      }
    } else {
#pragma unroll
      for (int u = 0; u < U; u++) {
        if (t0 + (int)threadIdx.x + u * BLOCK < n2) {
          double* e = reinterpret_cast<double*>(&v[u]);
#pragma unroll
          for (int c = 0; c < 2; c++) {
            bool ok;
            double x = e[c];
            e[c] = Op::fast(x, tab, ok);
            if (!ok || force) enqueue(j0 + 2 * u * BLOCK + c, x, e[c]);
          }
        }
      }
    }
    tile_store<double, U>(v, out, t0, n2);
    if (iter % Op::qcheck == Op::qcheck - 1) {
      __syncthreads();
      const unsigned nq = __builtin_amdgcn_readfirstlane(q.n);
      __syncthreads();
      if (nq > QFLUSH) flush_queue64<Op>(q, tab, out, st, elem_base);
    }
  }
  if ((n & 1) > threadIdx.x && takes_tail(t0, step, n2, TV)) {
    const long long i = 2 * n2;
    bool ok;
    const double x = in[i];
    double r = Op::fast(x, tab, ok);
    if (!ok || force) enqueue((unsigned)i, x, r);
    out[i] = r;
  }
  __syncthreads();
  flush_queue64<Op, true>(q, tab, out, st, elem_base);
}

// ------------------------------------------------- directed rounding modes
// The map kernels over a function's directed-mode paths (cr_f32_dir.h; the
// paper's GPU runs leave these modes out, Sec. III-C).  Measured against every
// element through the double-double evaluation, toward +infinity, 2^24 elements of
// the benchmark's inputs (5% of them hard to round in the exp/log family): expf
// 155 -> 36 us, logf 169 -> 38, sinf 235 -> 52, sincosf 265 -> 64, tanf 284 -> 60,
// acosf 231 -> 57, tanhf 191 -> 42, rsqrtf 45 -> 32.
template <class Op, int RM>
struct OpDir {
  using Tab = typename Op::Tab;
  static constexpr int qcheck = QCHECK;
  static __device__ __forceinline__ void load(Tab& t, int tid) { Op::load(t, tid); }
  static __device__ __forceinline__ float fast(float x, const Tab& t, bool& ok) {
    return Op::template fast_dir<RM>(x, t, ok);
  }
  static __device__ __forceinline__ AccResult accurate(float x, const Tab& t) {
    return Op::template dir<RM>(x, t);
  }
};
template <class SC, int RM>
struct SinCosDir {
  using Tab = typename SC::Tab;
  static constexpr int qcheck = QCHECK;
  static __device__ __forceinline__ void load(Tab& t, int tid) { SC::load(t, tid); }
  static __device__ __forceinline__ float fast(float x, const Tab& t, float& c, bool& ok) {
    return SC::template fast_dir<RM>(x, t, c, ok);
  }
  static __device__ __forceinline__ AccResult2 accurate(float x, const Tab& t) {
    return SC::template dir<RM>(x, t);
  }
};

// ------------------------------------------------- application workloads
// The paper's two synthetic applications built on the correctly rounded
// binary32 functions (Sec. III-A): complex expf, logf and sinf accurate to
// 2 ulps, and spectral interpolation by a brute-force DFT that spends its time
// in sincosf.  Each correctly rounded ingredient is evaluated by its fast path; an
// element with an ingredient whose rounding test fails (rare on these workloads: no
// hard-to-round inputs are planted) is evaluated again with the accurate paths in
// place, out of line.  The steps between the ingredients are single IEEE operations
// in the stated formats.
//   CF::fast(x, y, tab, ok)            every ingredient by its fast path, branch-free
//   CF::eval(x, y, tab, force, count)  each with its accurate path where needed

// One binary32 function, correctly rounded: fast path, accurate path if needed.
struct LaneCount {
  unsigned fails;
  unsigned escapes;
};
template <class Op>
__device__ __forceinline__ float cr1(float x, const typename Op::Tab& t, bool force, LaneCount& lc) {
  bool ok;
  float r = Op::fast(x, t, ok);
  if (!ok || force) {
    AccResult a = Op::accurate(x, t);
    r = a.r;
    lc.fails++;
    lc.escapes += a.ok ? 0u : 1u;
  }
  return r;
}
__device__ __forceinline__ float cr_sincos(float x, const TrigTab& t, float& c, bool force,
                                           LaneCount& lc) {
  bool ok;
  float s = sincos_fast(x, t, c, ok);
  if (!ok || force) {
    AccResult2 a = sincos_accurate(x, t);
    s = a.s;
    c = a.c;
    lc.fails++;
    lc.escapes += a.ok ? 0u : 1u;
  }
  return s;
}

// exp(x + iy) = e^x cos y + i e^x sin y: re = RN32(expf(x) cosf(y)),
// im = RN32(expf(x) sinf(y)).  Each part is the correctly rounded product of
// two correctly rounded factors: within 2 ulps.
struct CExpF {
  struct Tab {
    ExpTab e;
    TrigTab t;
  };
  static __device__ __forceinline__ void load(Tab& T, int tid) {
    exp_tab_load(T.e, tid);
    trig_tab_load(T.t, tid);
  }
  static __device__ __forceinline__ float2 fast(float x, float y, const Tab& T, bool& ok) {
    bool oke, okt;
    float C;
    const float E = exp_fast<EXPK_E>(x, T.e, oke);
    const float S = sincos_fast(y, T.t, C, okt);
    ok = oke && okt;
    return make_float2(E * C, E * S);
  }
  static __device__ __forceinline__ float2 eval(float x, float y, const Tab& T, bool force,
                                                LaneCount& lc) {
    const float E = cr1<OpExp<EXPK_E>>(x, T.e, force, lc);
    float C;
    const float S = cr_sincos(y, T.t, C, force, lc);
    return make_float2(E * C, E * S);
  }
};

// sin(x + iy) = sin x cosh y + i cos x sinh y, each product of correctly
// rounded factors rounded once: within 2 ulps.
struct CSinF {
  struct Tab {
    ExpTab e;
    TrigTab t;
  };
  static __device__ __forceinline__ void load(Tab& T, int tid) {
    exp_tab_load(T.e, tid);
    trig_tab_load(T.t, tid);
  }
  static __device__ __forceinline__ float2 fast(float x, float y, const Tab& T, bool& ok) {
    bool okt, okh;
    float C, Sh, Ch;
    const float S = sincos_fast(x, T.t, C, okt);
    sinh_cosh_fast(y, T.e, Sh, Ch, okh);
    ok = okt && okh;
    return make_float2(S * Ch, C * Sh);
  }
  static __device__ __forceinline__ float2 eval(float x, float y, const Tab& T, bool force,
                                                LaneCount& lc) {
    float C;
    const float S = cr_sincos(x, T.t, C, force, lc);
    const float Ch = cr1<OpHyp<HYPK_COSH>>(y, T.e, force, lc);
    const float Sh = cr1<OpHyp<HYPK_SINH>>(y, T.e, force, lc);
    return make_float2(S * Ch, C * Sh);
  }
};

// log(x + iy) = log|z| + i atan2(y, x), valid for finite z with
// 2^-63 <= |z| < 2^63.  With a = max(|x|, |y|), b = min(|x|, |y|):
//  * imaginary part: A = atanf(RN32(b / a)) correctly rounded, then in
//    binary64 v = A, v = RN64(pi/2) - v if |y| > |x|, v = RN64(pi) - v if
//    x < 0; the result is RN32(v) with the sign of y (below 1.5 ulps: the
//    quotient's rounding moves atan by at most 2^-24 t/(1 + t^2));
//  * real part: s = RN64(a^2 + b^2) (the squares are exact in binary64).
//    For 0.5 <= s < 2, d = RN64((a^2 - 1) + b^2) (a^2 - 1 exact), d = dh + dl
//    with dh = RN32(d) and dl exact, and log|z| = (log1pf(dh) + dl/(1 + dh))/2;
//    otherwise s = sh + sl, sh = RN32(s), and log|z| = (logf(sh) + sl/sh)/2,
//    the correction term's second-order error being below 2^-46 relative:
//    below 1.5 ulps.
struct CLogF {
  struct Tab {
    AtanTab a;
    LogTab l;
  };
  static __device__ __forceinline__ void load(Tab& T, int tid) {
    atan_tab_load(T.a, tid);
    log_tab_load<LOGK_E>(T.l, tid);  // logf and log1pf share the natural-log table
  }
  // the steps around the two ingredients, shared by both forms: atan1(q) and
  // log1(v, one_plus) evaluate them
  template <class A, class L>
  static __device__ __forceinline__ float2 compose(float x, float y, const A& atan1,
                                                   const L& log1) {
    const float ax = fabsf(x), ay = fabsf(y);
    const float a = fmaxf(ax, ay), b = fminf(ax, ay);
    double v = (double)atan1(b / a);
    if (ay > ax) v = 0x1.921fb54442d18p+0 - v;  // RN64(pi/2) - v
    if (x < 0.0f) v = 0x1.921fb54442d18p+1 - v;  // RN64(pi) - v
    const float im = copysignf((float)v, y);
    const double a2 = (double)a * (double)a, b2 = (double)b * (double)b;
    const double s = a2 + b2;
    const bool near1 = s >= 0.5 && s < 2.0;
    const double d = near1 ? (a2 - 1.0) + b2 : s;
    const float dh = (float)d;
    const double dl = d - (double)dh;
    const float l = log1(dh, near1);
    const double re = 0.5 * ((double)l + dl / (near1 ? 1.0 + (double)dh : (double)dh));
    return make_float2((float)re, im);
  }
  static __device__ __forceinline__ float2 fast(float x, float y, const Tab& T, bool& ok) {
    bool oka, okl;
    const float2 r = compose(
        x, y, [&](float q) { return atan_fast<ATANK_ATAN>(q, T.a, oka); },
        [&](float v, bool near1) {
          return near1 ? log_fast<LOGK_1P>(v, T.l, okl) : log_fast<LOGK_E>(v, T.l, okl);
        });
    ok = oka && okl;
    return r;
  }
  static __device__ __forceinline__ float2 eval(float x, float y, const Tab& T, bool force,
                                                LaneCount& lc) {
    return compose(
        x, y, [&](float q) { return cr1<OpAtan<ATANK_ATAN>>(q, T.a, force, lc); },
        [&](float v, bool near1) {
          return near1 ? cr1<OpLog<LOGK_1P>>(v, T.l, force, lc)
                       : cr1<OpLog<LOGK_E>>(v, T.l, force, lc);
        });
  }
};

// An element whose fast path failed: its value and the number of ingredients that
// failed, bit 31 set if the accurate path could not certify one of them.
struct ComplexSlow {
  float re, im;
  unsigned fails;
};
template <class CF>
__device__ __noinline__ ComplexSlow complex_slow(float x, float y, const typename CF::Tab& tab,
                                                 bool force) {
  LaneCount lc = {0u, 0u};
  const float2 r = CF::eval(x, y, tab, force, lc);
  return {r.x, r.y, lc.fails | (lc.escapes ? 0x80000000u : 0u)};
}

// Complex map: interleaved (re, im) binary32 pairs, two complex numbers per
// 128-bit load and store, at any 4-byte alignment; the last one of an odd
// number is loaded and stored by itself.  Persistent grid, tables staged in LDS.
// Bound by VALU issue.  Both elements of a thread are evaluated in straight-line code,
// the next two loaded meanwhile; before, each ingredient was followed by a branch to
// its accurate path, and csinf evaluated the exponential twice.  Measured at 2^22
// complex numbers: csinf 22.4 -> 18.4 us (21.2 with the present sine and cosine), cexpf
// 19.6 -> 17.6, clogf 26.3 -> 24.1.
template <class CF>
__global__ void __launch_bounds__(BLOCK)
    k_complex(const float* in, float* out, long long n, DevStats* st, unsigned flags,
              long long elem_base) {
  __shared__ typename CF::Tab tab;
  __shared__ unsigned fails;
  CF::load(tab, threadIdx.x);
  if (threadIdx.x == 0) fails = 0;
  __syncthreads();
  const bool force = flags & CR_FLAG_FORCE_FALLBACK;
  const int n2 = (int)(n >> 1), step = (int)gridDim.x * BLOCK;  // pairs
  unsigned mine = 0;
  auto slow = [&](float x, float y, long long i) {
    const ComplexSlow r = complex_slow<CF>(x, y, tab, force);
    mine += r.fails & 0x7fffffffu;
    if (r.fails >> 31) note_escape(st, elem_base + i);
    return make_float2(r.re, r.im);
  };
  int t0 = (int)blockIdx.x * BLOCK;
  float4 nxt[1];
  tile_load<float, 1>(nxt, in, t0, n2);
  for (; t0 < n2; t0 += step) {
    const float4 v = nxt[0];
    tile_load<float, 1>(nxt, in, t0 + step, n2);
    bool ok0, ok1;
    float2 r0 = CF::fast(v.x, v.y, tab, ok0);
    float2 r1 = CF::fast(v.z, v.w, tab, ok1);
    if (!(ok0 && ok1) || force) {
      const int i = t0 + (int)threadIdx.x;
      if (i < n2) {
        if (!ok0 || force) r0 = slow(v.x, v.y, 2LL * i);
        if (!ok1 || force) r1 = slow(v.z, v.w, 2LL * i + 1);
      }
    }
    const float4 r[1] = {make_float4(r0.x, r0.y, r1.x, r1.y)};
    tile_store<float, 1>(r, out, t0, n2);
  }
  if ((n & 1) && threadIdx.x == 0 && takes_tail(t0, step, n2, BLOCK)) {
    const long long i = n - 1;
    const float x = in[2 * i], y = in[2 * i + 1];
    bool ok;
    float2 r = CF::fast(x, y, tab, ok);
    if (!ok || force) r = slow(x, y, i);
    out[2 * i] = r.x;
    out[2 * i + 1] = r.y;
  }
  if (mine) atomicAdd(&fails, mine);
  __syncthreads();
  if (threadIdx.x == 0 && fails) {
    CounterSlot& c = st->slot[blockIdx.x % NSLOT];
    atomicAdd(&c.fallback_lanes, (unsigned long long)fails);
    atomicAdd(&c.fallback_waves, 1ull);
  }
}

// Brute-force DFT of real samples at per-output angles (spectral
// interpolation): X_k = sum_n x[n] (cos t - i sin t), t = RN32(w_k n), with
// sincosf correctly rounded.  Each product x[n] cos t is exact in binary64;
// the sums are carried as double-doubles (TwoSum per term), so X_k is within
// about N 2^-104 sum |x c| of the exact sum of the exact products before its
// final rounding.  Block (s, k) covers samples [s L, (s + 1) L) of output k
// and writes its partial sums (re.hi, re.lo, im.hi, im.lo); a second kernel
// adds the S partials of each k in a fixed order, so results do not depend
// on timing.
__device__ __forceinline__ void dd_acc(double& hi, double& lo, double p) {
  const dd t = two_sum(hi, p);
  hi = t.hi;
  lo += t.lo;
}
__device__ __forceinline__ void dd_acc2(double& hi, double& lo, double h2, double l2) {
  const dd t = two_sum(hi, h2);
  const dd u = fast_two_sum(t.hi, t.lo + (lo + l2));
  hi = u.hi;
  lo = u.lo;
}

// One term: the correctly rounded sine and cosine of th and their exact products.
struct DftSum {
  double rh, rl, ih, il;
};
__device__ __forceinline__ void dft_add(DftSum& a, float xv, float s, float c) {
  const double xd = (double)xv;
  dd_acc(a.rh, a.rl, xd * (double)c);
  dd_acc(a.ih, a.il, xd * (double)s);
}
__device__ __forceinline__ void dft_add2(DftSum& a, const DftSum& b) {
  dd_acc2(a.rh, a.rl, b.rh, b.rl);
  dd_acc2(a.ih, a.il, b.ih, b.il);
}
// xor butterfly over the wave, in a fixed order
__device__ __forceinline__ void dft_wave_sum(DftSum& a) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1)
    dft_add2(a, {__shfl_xor(a.rh, off), __shfl_xor(a.rl, off), __shfl_xor(a.ih, off),
                 __shfl_xor(a.il, off)});
}

// Bound by VALU issue: 77 instructions a term, half of them binary64, against 4
// bytes of samples that the outputs share.  A thread takes DFT_U terms at a time, a
// block's stride apart, evaluated in straight-line code with one branch for the lanes
// whose rounding test failed; a term at a time with its own branch it took 120
// instructions.  Measured, with the present sine and cosine: 2^20 samples at 256
// frequencies 886 -> 550 us (302 -> 488 G terms/s), 2^18 at 64 80 -> 46 us, 2000 at
// 41 23 -> 5.3 us (no workspace).
constexpr int DFT_U = 4;
template <bool ONE>  // ONE: a single slice, whose sums are the result
__global__ void __launch_bounds__(BLOCK)
    k_dft(const float* x, int n, const float* w, int slice, double4* part, double2* X, int S,
          DevStats* st, unsigned flags, long long k0) {
  __shared__ TrigTab tab;
  __shared__ DftSum red[BLOCK / 64];
  __shared__ unsigned fails;
  trig_tab_load(tab, threadIdx.x);
  if (threadIdx.x == 0) fails = 0;
  __syncthreads();
  const bool force = flags & CR_FLAG_FORCE_FALLBACK;
  const int k = blockIdx.y;
  const float wk = w[k];
  const int n0 = (int)blockIdx.x * slice;
  const int n1 = min(n0 + slice, n);
  DftSum sum = {0.0, 0.0, 0.0, 0.0};
  LaneCount lc = {0u, 0u};
  int i = n0 + (int)threadIdx.x;
  // RN32(w_k n) with n < 2^24 exact
  for (; i + (DFT_U - 1) * BLOCK < n1; i += DFT_U * BLOCK) {
    float xv[DFT_U], s[DFT_U], c[DFT_U];
    bool ok = true;
#pragma unroll
    for (int u = 0; u < DFT_U; u++) xv[u] = x[i + u * BLOCK];
#pragma unroll
    for (int u = 0; u < DFT_U; u++) {
      bool o;
      s[u] = sincos_fast(wk * (float)(i + u * BLOCK), tab, c[u], o);
      ok = ok && o;
    }
    if (!ok || force) {
#pragma unroll
      for (int u = 0; u < DFT_U; u++)
        s[u] = cr_sincos(wk * (float)(i + u * BLOCK), tab, c[u], force, lc);
    }
#pragma unroll
    for (int u = 0; u < DFT_U; u++) dft_add(sum, xv[u], s[u], c[u]);
  }
  for (; i < n1; i += BLOCK) {
    float c;
    const float s = cr_sincos(wk * (float)i, tab, c, force, lc);
    dft_add(sum, x[i], s, c);
  }
  if (lc.escapes) note_escape(st, k0 + k);
  dft_wave_sum(sum);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sum;
  if (lc.fails) atomicAdd(&fails, lc.fails);
  __syncthreads();
  if (threadIdx.x == 0) {
    DftSum acc = red[0];
    for (int q = 1; q < BLOCK / 64; q++) dft_add2(acc, red[q]);
    if (ONE)
      X[k] = make_double2(acc.rh + acc.rl, -(acc.ih + acc.il));
    else
      part[(long long)k * S + blockIdx.x] = make_double4(acc.rh, acc.rl, acc.ih, acc.il);
    if (fails) {
      CounterSlot& cs = st->slot[(blockIdx.y * gridDim.x + blockIdx.x) % NSLOT];
      atomicAdd(&cs.fallback_lanes, (unsigned long long)fails);
      atomicAdd(&cs.fallback_waves, 1ull);
    }
  }
}

// The slices' sums of each output, one wave to an output: lane q adds slices q,
// q + 64, ... in order, then the wave's butterfly (a thread to an output, adding its S
// slices one after the other, took 7.5 us for 32 slices of 64 outputs; now 4.0).
__global__ void __launch_bounds__(BLOCK)
    k_dft_finish(const double4* part, int S, long long m, double2* X) {
  const long long k = (long long)blockIdx.x * (BLOCK / 64) + (threadIdx.x >> 6);
  if (k >= m) return;
  DftSum acc = {0.0, 0.0, 0.0, 0.0};
  for (int q = threadIdx.x & 63; q < S; q += 64) {
    const double4 p = part[k * S + q];
    dft_add2(acc, {p.x, p.y, p.z, p.w});
  }
  dft_wave_sum(acc);
  if ((threadIdx.x & 63) == 0) X[k] = make_double2(acc.rh + acc.rl, -(acc.ih + acc.il));
}

// ------------------------------------------------------------ ragged batch
// One persistent kernel evaluates a whole batch: the requests sorted by
// (implementation, function) and cut into tiles of 1024, 2048 or 4096 elements,
// tile t of the batch being tile t - tile0 of its request.  Workgroup b takes the
// tiles [b per, (b + 1) per): the function changes rarely along them, and where it
// does the workgroup runs the accurate path on its queue and stages the next tables.
// Bound by the latency of a workgroup's look-ups and first loads (small batches) and
// by VALU issue (large ones).  Before, every batch ran one kernel per function
// present, 19 of them for most, from a graph (125-140 us a launch whatever the work)
// or one after the other (cr_eval_batch, 100 us and more).  Measured: a plan of 48
// requests (40259 elements) 131 -> 7.9 us, of 512 requests (12.4e6) 125 -> 38 us,
// cr_eval_batch of 48 requests 115 -> 6.4 us, of 512 requests 184 -> 59 us.
struct BReq {
  const float* in;
  float* out;
  unsigned n;
  unsigned tile0;  // the request's first tile
  int key;         // func, + BSPLIT for the binary32-only implementation
  int orig;        // index of the request in the caller's array
};
constexpr int BSPLIT = 32;

// Up to BARG requests go to the kernel as its arguments, with nothing to allocate
// or copy (first tiles apart, for the search); larger batches and plans keep a
// request table and the request of every tile in device memory.
constexpr int BARG = 96;
// The tables do not change while a kernel reads them: the constant address space
// makes the accesses that are the same in every lane scalar loads.
typedef const __attribute__((address_space(4))) BReq* BReqTab;
typedef const __attribute__((address_space(4))) unsigned* BTileTab;
struct BArgs {
  unsigned tile0[128];  // 0xffffffff beyond the last request
  BReq req[BARG];
};

// Static device memory of the library.  Each device the library runs on holds
// its own copy, zero-initialised when the code object loads, until the
// process ends.  Host code never passes these names to a kernel or a copy
// (in host code they are host-side stand-ins): get_state() resolves their
// per-device addresses with hipGetSymbolAddress.
//   g_dev_stats  the statistics counters and escape list of every entry point
//   scratch      the request and tile tables of cr_eval_batch_noalloc:
//                CR_NOALLOC_MAX_REQUESTS BReq, then the request of each of up to
//                CR_NOALLOC_MAX_TILES tiles
__device__ __align__(256) DevStats g_dev_stats;
constexpr size_t NOALLOC_REQ_BYTES =
    ((size_t)CR_NOALLOC_MAX_REQUESTS * sizeof(BReq) + 255) / 256 * 256;
constexpr size_t SCRATCH_BYTES =
    NOALLOC_REQ_BYTES + (size_t)CR_NOALLOC_MAX_TILES * sizeof(unsigned);
static __device__ __align__(256) unsigned char scratch[SCRATCH_BYTES];

struct BDeferred {
  unsigned n, lanes, waves;
  unsigned req[QCAP];
  unsigned idx[QCAP];
  float x[QCAP];
};

// Escapes of a batch are recorded as (request << 32) | element index within
// the request.
__device__ __forceinline__ long long batch_escape_id(unsigned req, unsigned idx) {
  return (long long)(((unsigned long long)req << 32) | idx);
}

// A function's evaluator for the batch: one output (Op) or two (SC, sincosf).
template <class Op>
struct BOne {
  using Tab = typename Op::Tab;
  static constexpr bool TWO = false;
  static constexpr int qcheck = Op::qcheck;
  static __device__ __forceinline__ void load(Tab& t, int tid) { Op::load(t, tid); }
  static __device__ __forceinline__ float fast(float x, const Tab& t, float&, bool& ok) {
    return Op::fast(x, t, ok);
  }
  static __device__ __forceinline__ AccResult2 accurate(float x, const Tab& t) {
    const AccResult a = Op::accurate(x, t);
    return {a.r, 0.0f, a.ok};
  }
};
template <class SC>
struct BTwo : SC {
  static constexpr bool TWO = true;
};

constexpr size_t cmax(size_t a, size_t b) { return a > b ? a : b; }
struct BShared {
  BDeferred q;
  __align__(16) unsigned char tab[cmax(
      cmax(cmax(sizeof(ExpTab), sizeof(LogTab)), cmax(sizeof(TrigTab), sizeof(AtanTab))),
      cmax(cmax(cmax(sizeof(SExpTab), sizeof(SLogTab)), cmax(sizeof(STrigTab), sizeof(SAtanTab))),
           sizeof(SHypTab)))];
};

// Element idx of request R failed its test: queued, or its accurate path in place
// when the queue is full (pathological inputs, or force).
template <class E>
__device__ __forceinline__ void batch_enqueue(BDeferred& q, const typename E::Tab& tab, int ri,
                                              int orig, unsigned idx, float x, float& s, float& c,
                                              DevStats* st) {
  unsigned pos = atomicAdd(&q.n, 1u);
  if (pos < QCAP) {
    q.req[pos] = ri;
    q.idx[pos] = idx;
    q.x[pos] = x;
  } else {
    const AccResult2 a = E::accurate(x, tab);
    s = a.s;
    c = a.c;
    atomicAdd(&q.lanes, 1u);
    if (!a.ok) note_escape(st, batch_escape_id(orig, idx));
  }
}

// cnt elements from element `start` of request ri, 1024 at a time: four a thread
// in straight-line code, the next four loaded meanwhile.  The cnt % 4 elements
// after the last whole vector are the lane's that would take the next vector.
template <class E>
__device__ __forceinline__ void batch_tile(BReq R, int ri, unsigned start, unsigned cnt,
                                           const typename E::Tab& tab, BDeferred& q, bool force,
                                           DevStats* st) {
  const float* in = R.in + start;
  float* out = R.out + start;
  float* outc = E::TWO ? out + R.n : out;
  const int n4 = (int)(cnt >> 2), rem = (int)(cnt & 3u), orig = R.orig;
  const int steps = (int)((cnt + 4 * BLOCK - 1) / (4 * BLOCK));
  float4 nxt[1];
  tile_load<float, 1>(nxt, in, 0, n4);
#pragma unroll 1
  for (int k = 0; k < steps; k++) {
    const int t0 = k * BLOCK, i = t0 + (int)threadIdx.x;
    float4 v[1] = {nxt[0]}, vc[1];
    tile_load<float, 1>(nxt, in, t0 + BLOCK, n4);
    float* e = reinterpret_cast<float*>(&v[0]);
    float* ec = reinterpret_cast<float*>(&vc[0]);
    unsigned live = 0xfu;
    if (t0 + BLOCK > n4) {  // the tile's last step
      live = i < n4 ? 0xfu : i == n4 ? (1u << rem) - 1u : 0u;
      if (i == n4) {
#pragma unroll
        for (int c = 0; c < 3; c++)
          if (c < rem) e[c] = in[4 * i + c];
      }
    }
    float x[4];
    unsigned fail = 0;
#pragma unroll
    for (int c = 0; c < 4; c++) {
      bool ok;
      x[c] = e[c];
      e[c] = E::fast(x[c], tab, ec[c], ok);
      fail |= (unsigned)(!ok || force) << c;
    }
    fail &= live;
    if (fail) {
#pragma unroll
      for (int c = 0; c < 4; c++)
        if (fail & (1u << c))
          batch_enqueue<E>(q, tab, ri, orig, start + 4 * i + c, x[c], e[c], ec[c], st);
    }
    tile_store<float, 1>(v, out, t0, n4);
    if (E::TWO) tile_store<float, 1>(vc, outc, t0, n4);
    if (i == n4) {
#pragma unroll
      for (int c = 0; c < 3; c++) {
        if (c < rem) out[4 * i + c] = e[c];
        if (E::TWO && c < rem) outc[4 * i + c] = ec[c];
      }
    }
  }
}

// The accurate path on the queued elements, 256 at a time.
template <class E>
__device__ __forceinline__ void batch_flush(BDeferred& q, const typename E::Tab& tab,
                                            BReqTab reqs, DevStats* st) {
  const unsigned n = q.n < QCAP ? q.n : QCAP;  // see run_queue
  for (unsigned k = threadIdx.x; k < n; k += BLOCK) {
    const AccResult2 a = E::accurate(q.x[k], tab);
    const unsigned ri = q.req[k], idx = q.idx[k];
    float* out = reqs[ri].out;
    out[idx] = a.s;
    if (E::TWO) out[(size_t)reqs[ri].n + idx] = a.c;
    if (!a.ok) note_escape(st, batch_escape_id(reqs[ri].orig, idx));
  }
  if (threadIdx.x == 0) {
    q.lanes += n;
    q.waves += (n + 63) / 64;
  }
}

// The workgroup's tiles t, t + step, ... < t1 that share the function of request ri;
// t and ri move past them.  find(t): the request of tile t.
template <class E, class Find>
__device__ __forceinline__ void batch_segment(BReqTab reqs, int& t, int step, int t1, int& ri,
                                              int tile, const Find& find, BShared& sh, bool force,
                                              DevStats* st) {
  typename E::Tab& tab = *reinterpret_cast<typename E::Tab*>(sh.tab);
  BDeferred& q = sh.q;
  E::load(tab, threadIdx.x);
  if (threadIdx.x == 0) q.n = 0;
  __syncthreads();
  // the next tile's request is looked up while this tile is evaluated
  BReq R = {reqs[ri].in, reqs[ri].out, reqs[ri].n, reqs[ri].tile0, reqs[ri].key, reqs[ri].orig};
  const int key = R.key;
  int iter = 0, next;
  do {
    const unsigned start = (unsigned)(t - (int)R.tile0) * (unsigned)tile;
    next = t + step < t1 ? find(t + step) : ri;
    const BReq N = {reqs[next].in,    reqs[next].out, reqs[next].n,
                    reqs[next].tile0, reqs[next].key, reqs[next].orig};
    batch_tile<E>(R, ri, start, min(R.n - start, (unsigned)tile), tab, q, force, st);
    R = N;
    if (++iter % E::qcheck == 0) {
      __syncthreads();
      const unsigned nq = __builtin_amdgcn_readfirstlane(q.n);
      __syncthreads();
      if (nq > QFLUSH) {
        batch_flush<E>(q, tab, reqs, st);
        __syncthreads();
        if (threadIdx.x == 0) q.n = 0;
        __syncthreads();
      }
    }
    t += step;
    ri = next;
  } while (t < t1 && R.key == key);
  __syncthreads();
  batch_flush<E>(q, tab, reqs, st);
  if (t < t1) __syncthreads();  // the tables and the queue are free for the next function
}

// The workgroup's counters to the device statistics.
__device__ __forceinline__ void batch_count(const BDeferred& q, DevStats* st) {
  if (threadIdx.x == 0 && q.lanes) {
    CounterSlot& c = st->slot[blockIdx.x % NSLOT];
    atomicAdd(&c.fallback_lanes, (unsigned long long)q.lanes);
    atomicAdd(&c.fallback_waves, (unsigned long long)q.waves);
  }
}

template <bool SPLIT, class Find>
__device__ __forceinline__ void batch_run(BReqTab reqs, int t, int t1, int tile,
                                          const Find& find, DevStats* st, unsigned flags) {
  __shared__ BShared sh;
  if (threadIdx.x == 0) sh.q.lanes = sh.q.waves = 0;
  const bool force = flags & CR_FLAG_FORCE_FALLBACK;
  int ri = find(t);
#define CR_SEG(id, ...)                                                                 \
  case id:                                                                              \
    batch_segment<__VA_ARGS__>(reqs, t, 1, t1, ri, tile, find, sh, force, st);          \
    break
  while (t < t1) {
    if (!SPLIT) {
      switch (__builtin_amdgcn_readfirstlane(reqs[ri].key)) {
        CR_SEG(CR_EXPF, BOne<OpExp<EXPK_E>>);
        CR_SEG(CR_EXP2F, BOne<OpExp<EXPK_2>>);
        CR_SEG(CR_EXP10F, BOne<OpExp<EXPK_10>>);
        CR_SEG(CR_EXPM1F, BOne<OpExp<EXPK_EM1>>);
        CR_SEG(CR_LOGF, BOne<OpLog<LOGK_E>>);
        CR_SEG(CR_LOG2F, BOne<OpLog<LOGK_2>>);
        CR_SEG(CR_LOG10F, BOne<OpLog<LOGK_10>>);
        CR_SEG(CR_LOG1PF, BOne<OpLog<LOGK_1P>>);
        CR_SEG(CR_RSQRTF, BOne<OpRsqrt>);
        CR_SEG(CR_SINF, BOne<OpTrig<TRIGK_SIN>>);
        CR_SEG(CR_COSF, BOne<OpTrig<TRIGK_COS>>);
        CR_SEG(CR_SINCOSF, BTwo<SinCosF64>);
        CR_SEG(CR_TANF, BOne<OpTrig<TRIGK_TAN>>);
        CR_SEG(CR_ASINF, BOne<OpAtan<ATANK_ASIN>>);
        CR_SEG(CR_ACOSF, BOne<OpAtan<ATANK_ACOS>>);
        CR_SEG(CR_ATANF, BOne<OpAtan<ATANK_ATAN>>);
        CR_SEG(CR_SINHF, BOne<OpHyp<HYPK_SINH>>);
        CR_SEG(CR_COSHF, BOne<OpHyp<HYPK_COSH>>);
        CR_SEG(CR_TANHF, BOne<OpHyp<HYPK_TANH>>);
        default: return;  // not reached: the host builds the keys
      }
    } else {
      switch (__builtin_amdgcn_readfirstlane(reqs[ri].key) - BSPLIT) {
        CR_SEG(CR_EXPF, BOne<OpSExp<EXPK_E>>);
        CR_SEG(CR_EXP2F, BOne<OpSExp<EXPK_2>>);
        CR_SEG(CR_EXP10F, BOne<OpSExp<EXPK_10>>);
        CR_SEG(CR_EXPM1F, BOne<OpSExp<EXPK_EM1>>);
        CR_SEG(CR_LOGF, BOne<OpSLog<LOGK_E>>);
        CR_SEG(CR_LOG2F, BOne<OpSLog<LOGK_2>>);
        CR_SEG(CR_LOG10F, BOne<OpSLog<LOGK_10>>);
        CR_SEG(CR_LOG1PF, BOne<OpSLog<LOGK_1P>>);
        CR_SEG(CR_RSQRTF, BOne<OpSRsqrt>);
        CR_SEG(CR_SINF, BOne<OpSTrig<TRIGK_SIN>>);
        CR_SEG(CR_COSF, BOne<OpSTrig<TRIGK_COS>>);
        CR_SEG(CR_SINCOSF, BTwo<SinCosSplit>);
        CR_SEG(CR_TANF, BOne<OpSTrig<TRIGK_TAN>>);
        CR_SEG(CR_ASINF, BOne<OpSAtan<ATANK_ASIN>>);
        CR_SEG(CR_ACOSF, BOne<OpSAtan<ATANK_ACOS>>);
        CR_SEG(CR_ATANF, BOne<OpSAtan<ATANK_ATAN>>);
        CR_SEG(CR_SINHF, BOne<OpSHyp<HYPK_SINH>>);
        CR_SEG(CR_COSHF, BOne<OpSHyp<HYPK_COSH>>);
        CR_SEG(CR_TANHF, BOne<OpSHyp<HYPK_TANH>>);
        default: return;
      }
    }
  }
#undef CR_SEG
  batch_count(sh.q, st);
}

// One function's tiles [t0, t1) of a large plan, strided over the grid.
template <class E>
__global__ void __launch_bounds__(BLOCK)
    k_tiles(BReqTab reqs, BTileTab tile_req, int t0, int t1, int tile, DevStats* st,
            unsigned flags) {
  __shared__ BShared sh;
  if (threadIdx.x == 0) sh.q.lanes = sh.q.waves = 0;
  const auto find = [&](int k) { return (int)__builtin_amdgcn_readfirstlane(tile_req[k]); };
  int t = t0 + (int)blockIdx.x, ri = find(t);
  batch_segment<E>(reqs, t, (int)gridDim.x, t1, ri, tile, find, sh,
                   flags & CR_FLAG_FORCE_FALLBACK, st);
  batch_count(sh.q, st);
}

// Tiles [t0, t1) of the batch, `per` to a workgroup, tables in device memory.
template <bool SPLIT>
__global__ void __launch_bounds__(BLOCK)
    k_batch(BReqTab reqs, BTileTab tile_req, int t0, int t1, int per, int tile,
            DevStats* st, unsigned flags) {
  const int t = t0 + (int)blockIdx.x * per;
  batch_run<SPLIT>(reqs, t, min(t + per, t1), tile,
                   [&](int k) { return (int)__builtin_amdgcn_readfirstlane(tile_req[k]); }, st,
                   flags);
}
// The same with the requests as kernel arguments (the first argument lies at the
// start of the kernel argument segment, read in place).  Tile k belongs to the
// last request whose first tile is not beyond k: a count over the wave's lanes.
template <bool SPLIT>
__global__ void __launch_bounds__(BLOCK)
    k_batch_args(const BArgs args, int t1, int per, int tile, DevStats* st, unsigned flags) {
  typedef const __attribute__((address_space(4))) BArgs* ArgTab;
  const ArgTab a = (ArgTab)__builtin_amdgcn_kernarg_segment_ptr();
  const int lane = threadIdx.x & 63;
  const unsigned lo = a->tile0[lane], hi = a->tile0[lane + 64];
  const int t = (int)blockIdx.x * per;
  batch_run<SPLIT>(a->req, t, min(t + per, t1), tile,
                   [&](int k) {
                     return __popcll(__ballot(lo <= (unsigned)k)) +
                            __popcll(__ballot(hi <= (unsigned)k)) - 1;
                   },
                   st, flags);
}

__global__ void k_zero_stats(DevStats* st) {
  unsigned long long* p = reinterpret_cast<unsigned long long*>(st);
  for (int i = threadIdx.x; i < (int)(sizeof(DevStats) / 8); i += blockDim.x) p[i] = 0;
}

// ------------------------------------------------------------- host side
constexpr int MAX_DEV = 64;
std::mutex g_mu;
std::atomic<unsigned long long> g_elems[MAX_DEV];
thread_local int t_last_hip = 0;

int hip_fail(hipError_t e) {
  t_last_hip = (int)e;
  return CR_E_HIP;
}

// Per-device addresses of the library's static device memory (g_dev_stats,
// scratch), resolved once per device with that device current.
struct DevState {
  DevStats* stats;
  unsigned char* scratch;
};
DevState g_state[MAX_DEV];
std::atomic<bool> g_state_ok[MAX_DEV];

int get_state(DevState** out, int* device = nullptr) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e);
  if (dev < 0 || dev >= MAX_DEV) return CR_E_HIP;
  if (device) *device = dev;
  if (g_state_ok[dev].load(std::memory_order_acquire)) {  // every call but the first
    *out = &g_state[dev];
    return CR_OK;
  }
  std::lock_guard<std::mutex> lk(g_mu);
  if (!g_state_ok[dev].load(std::memory_order_relaxed)) {
    void* ps = nullptr;
    void* pb = nullptr;
    e = hipGetSymbolAddress(&ps, HIP_SYMBOL(g_dev_stats));
    if (e != hipSuccess) return hip_fail(e);
    e = hipGetSymbolAddress(&pb, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_fail(e);
    if (!ps || !pb) return CR_E_HIP;
    g_state[dev].stats = static_cast<DevStats*>(ps);
    g_state[dev].scratch = static_cast<unsigned char*>(pb);
    g_state_ok[dev].store(true, std::memory_order_release);
  }
  *out = &g_state[dev];
  return CR_OK;
}

int get_stats(DevStats** out) {
  DevState* ds = nullptr;
  int rc = get_state(&ds);
  if (rc) return rc;
  *out = ds->stats;
  return CR_OK;
}

std::atomic<int> g_cus{0};  // compute units of the current device (cached on first use)

int num_cus() {
  int n = g_cus.load(std::memory_order_relaxed);
  if (!n) {
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess)
      (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    g_cus = n = cus > 0 ? cus : 256;
  }
  return n;
}

// default workgroups per compute unit of the persistent grids
int default_bpc() {
  static int per = 0;
  if (!per) {
    int v = CR_BLOCKS_PER_CU;
    if (const char* e = getenv("CR_BLOCKS_PER_CU")) v = atoi(e);
    per = v < 1 ? 1 : (v > 64 ? 64 : v);
  }
  return per;
}

// The table copy read by the global-placement variants, filled once per device
// (synchronously, on first use).
template <class Op>
int ensure_gtab() {
  static std::atomic<unsigned long long> done{0};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e);
  const unsigned long long bit = 1ull << (dev & 63);
  if (done.load() & bit) return CR_OK;
  std::lock_guard<std::mutex> lk(g_mu);
  if (done.load() & bit) return CR_OK;
  hipLaunchKernelGGL(k_tab_init<Op>, dim3(1), dim3(BLOCK), 0, 0);
  e = hipDeviceSynchronize();
  if (e != hipSuccess) return hip_fail(e);
  done |= bit;
  return CR_OK;
}

constexpr size_t LAUNCH_ELEMS = (size_t)1 << 31;

template <class Op, int U, int PF, int TP>
int launch_map_f32(const float* in, float* out, size_t n, hipStream_t s, unsigned flags,
                   DevStats* st, int grid) {
  if (TP) {
    int rc = ensure_gtab<Op>();
    if (rc) return rc;
  }
  // the kernel counts elements in 32 bits (its deferred queue): at most
  // LAUNCH_ELEMS a launch
  for (size_t done = 0; done < n;) {
    const size_t cnt = n - done < LAUNCH_ELEMS ? n - done : LAUNCH_ELEMS;
    const size_t tiles = (cnt + BLOCK * 4 * U - 1) / (BLOCK * 4 * U);
    const size_t g = tiles < (size_t)grid ? tiles : (size_t)grid;
    hipLaunchKernelGGL((k_map_f32<Op, U, PF, TP>), dim3((unsigned)g), dim3(BLOCK), 0, s, in + done,
                       out + done, (long long)cnt, st, flags, (long long)done);
    done += cnt;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e);
  return CR_OK;
}

// The launch variants the autotuner chooses from: {U, PF, TP} of k_map_f32.
constexpr int NVARIANT = 7;
constexpr int VARIANTS[NVARIANT][3] = {{2, 1, 0}, {1, 1, 0}, {4, 1, 0}, {2, 0, 0},
                                       {4, 0, 0}, {1, 0, 0}, {2, 1, 1}};

// The variant of a function whose configuration is not set (DEFAULT_VARIANT).  Arrays
// that give the compute units at most four workgroups of the smallest tile (1024
// elements) each take that tile, and no prefetch: each workgroup has one tile, and
// its length is the call's.  Graph launches back to back, variant 0 (2048 elements,
// prefetch) against it, at 10^3, 3 10^5 and 2^20 elements of the benchmark's inputs:
// expf 2.44 -> 2.14 us, 3.82 -> 3.52, 4.77 -> 4.46; tanf 3.08 -> 2.51, 5.36 -> 4.64,
// 6.67 -> 5.76; binary32-only expf 5.23 -> 4.35, 6.09 -> 5.41, 7.35 -> 6.72, tanf
// 5.22 -> 3.55, 8.57 -> 7.06, 10.75 -> 9.60; no function slower at any of the three.
// Beyond, at 3 10^6, expf 6.2 -> 7.4, sinf 10.1 -> 10.2.  A configuration that was set
// is launched as it is.
constexpr int DEFAULT_VARIANT = -1;
int default_variant(size_t n, int grid) {
  return n <= (size_t)num_cus() * 4096 && n <= (size_t)grid * 1024 ? 5 : 0;
}
template <class Op>
int launch_variant(const float* in, float* out, size_t n, hipStream_t s, unsigned flags,
                   DevStats* st, int variant, int grid) {
  switch (variant == DEFAULT_VARIANT ? default_variant(n, grid) : variant) {
    case 0: return launch_map_f32<Op, 2, 1, 0>(in, out, n, s, flags, st, grid);
    case 1: return launch_map_f32<Op, 1, 1, 0>(in, out, n, s, flags, st, grid);
    case 2: return launch_map_f32<Op, 4, 1, 0>(in, out, n, s, flags, st, grid);
    case 3: return launch_map_f32<Op, 2, 0, 0>(in, out, n, s, flags, st, grid);
    case 4: return launch_map_f32<Op, 4, 0, 0>(in, out, n, s, flags, st, grid);
    case 5: return launch_map_f32<Op, 1, 0, 0>(in, out, n, s, flags, st, grid);
    case 6: return launch_map_f32<Op, 2, 1, 1>(in, out, n, s, flags, st, grid);
  }
  return CR_E_TUNE;
}

template <class SC>
int launch_sincos(const float* in, float* out, size_t n, hipStream_t s, unsigned flags,
                  DevStats* st, int grid) {
  float* outc = out + n;
  for (size_t done = 0; done < n;) {
    const size_t cnt = n - done < LAUNCH_ELEMS ? n - done : LAUNCH_ELEMS;
    const size_t tiles = (cnt + BLOCK * 4 * TILE_U - 1) / (BLOCK * 4 * TILE_U);
    const size_t g = tiles < (size_t)grid ? tiles : (size_t)grid;
    hipLaunchKernelGGL(k_map_sincos<SC>, dim3((unsigned)g), dim3(BLOCK), 0, s, in + done,
                       out + done, outc + done, (long long)cnt, st, flags, (long long)done);
    done += cnt;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e);
  return CR_OK;
}

template <class Op, int U, int SL>
int launch_map_f64(const double* in, double* out, size_t n, hipStream_t s, unsigned flags,
                   DevStats* st, int grid) {
  for (size_t done = 0; done < n;) {
    const size_t cnt = n - done < LAUNCH_ELEMS ? n - done : LAUNCH_ELEMS;
    const size_t tiles = (cnt + BLOCK * 2 * U - 1) / (BLOCK * 2 * U);
    const size_t g = tiles < (size_t)grid ? tiles : (size_t)grid;
    hipLaunchKernelGGL((k_map_f64<Op, U, SL>), dim3((unsigned)g), dim3(BLOCK), 0, s, in + done,
                       out + done, (long long)cnt, st, flags, (long long)done);
    done += cnt;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e);
  return CR_OK;
}

// The binary64 launch variants: {U, SL} of k_map_f64 (variant 0: four vectors
// per thread, an element at a time).
constexpr int NVARIANT64 = 4;
template <class Op>
int launch_variant64(const double* in, double* out, size_t n, hipStream_t s, unsigned flags,
                     DevStats* st, int variant, int grid) {
  switch (variant == DEFAULT_VARIANT ? 0 : variant) {
    case 0: return launch_map_f64<Op, 4, 0>(in, out, n, s, flags, st, grid);
    case 1: return launch_map_f64<Op, 1, 1>(in, out, n, s, flags, st, grid);
    case 2: return launch_map_f64<Op, 2, 1>(in, out, n, s, flags, st, grid);
    case 3: return launch_map_f64<Op, 4, 1>(in, out, n, s, flags, st, grid);
  }
  return CR_E_TUNE;
}

// Complex binary32 map (n complex numbers, interleaved), two a thread.
template <class CF>
int launch_complex(const float* in, float* out, size_t n, hipStream_t s, unsigned flags,
                   DevStats* st, int grid) {
  for (size_t done = 0; done < n;) {
    const size_t cnt = n - done < LAUNCH_ELEMS ? n - done : LAUNCH_ELEMS;
    size_t g = (cnt + 2 * BLOCK - 1) / (2 * BLOCK);
    if (g > (size_t)grid) g = grid;
    hipLaunchKernelGGL(k_complex<CF>, dim3((unsigned)g), dim3(BLOCK), 0, s, in + 2 * done,
                       out + 2 * done, (long long)cnt, st, flags, (long long)done);
    done += cnt;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e);
  return CR_OK;
}

bool func_complex(int f) { return f == CR_CEXPF || f == CR_CLOGF || f == CR_CSINF; }
bool impl_valid(int impl) {
  return impl == CR_IMPL_AUTO || impl == CR_IMPL_F64_INTERNAL || impl == CR_IMPL_SPLIT_F32 ||
         impl == CR_IMPL_LOG128;
}
bool func_f64(int f) { return f == CR_EXP || f == CR_LOG || f == CR_EXP2; }
bool func_valid(int f) { return (f >= 0 && f < CR_NUM_F32) || func_f64(f) || func_complex(f); }
bool func_built(int f) {
  return (f >= CR_EXPF && f <= CR_TANHF) || func_f64(f) || func_complex(f);
}
// bytes of one input element (complex: two binary32) and of the output per element
size_t elem_bytes(int f) { return func_f64(f) || func_complex(f) ? 8 : 4; }
// functions with a binary32-only (split) implementation
bool split_built(int f) { return f >= CR_EXPF && f <= CR_TANHF; }

int dispatch_f32_split(int f, const float* in, float* out, size_t n, hipStream_t s,
                       unsigned flags, DevStats* st, int v, int g) {
  switch (f) {
    case CR_EXPF: return launch_variant<OpSExp<EXPK_E>>(in, out, n, s, flags, st, v, g);
    case CR_EXP2F: return launch_variant<OpSExp<EXPK_2>>(in, out, n, s, flags, st, v, g);
    case CR_EXP10F: return launch_variant<OpSExp<EXPK_10>>(in, out, n, s, flags, st, v, g);
    case CR_EXPM1F: return launch_variant<OpSExp<EXPK_EM1>>(in, out, n, s, flags, st, v, g);
    case CR_LOGF: return launch_variant<OpSLog<LOGK_E>>(in, out, n, s, flags, st, v, g);
    case CR_LOG2F: return launch_variant<OpSLog<LOGK_2>>(in, out, n, s, flags, st, v, g);
    case CR_LOG10F: return launch_variant<OpSLog<LOGK_10>>(in, out, n, s, flags, st, v, g);
    case CR_LOG1PF: return launch_variant<OpSLog<LOGK_1P>>(in, out, n, s, flags, st, v, g);
    case CR_RSQRTF: return launch_variant<OpSRsqrt>(in, out, n, s, flags, st, v, g);
    case CR_SINF: return launch_variant<OpSTrig<TRIGK_SIN>>(in, out, n, s, flags, st, v, g);
    case CR_COSF: return launch_variant<OpSTrig<TRIGK_COS>>(in, out, n, s, flags, st, v, g);
    case CR_TANF: return launch_variant<OpSTrig<TRIGK_TAN>>(in, out, n, s, flags, st, v, g);
    case CR_SINCOSF: return launch_sincos<SinCosSplit>(in, out, n, s, flags, st, g);
    case CR_ASINF: return launch_variant<OpSAtan<ATANK_ASIN>>(in, out, n, s, flags, st, v, g);
    case CR_ACOSF: return launch_variant<OpSAtan<ATANK_ACOS>>(in, out, n, s, flags, st, v, g);
    case CR_ATANF: return launch_variant<OpSAtan<ATANK_ATAN>>(in, out, n, s, flags, st, v, g);
    case CR_SINHF: return launch_variant<OpSHyp<HYPK_SINH>>(in, out, n, s, flags, st, v, g);
    case CR_COSHF: return launch_variant<OpSHyp<HYPK_COSH>>(in, out, n, s, flags, st, v, g);
    case CR_TANHF: return launch_variant<OpSHyp<HYPK_TANH>>(in, out, n, s, flags, st, v, g);
  }
  return CR_E_IMPL;
}

int dispatch_f32(int f, const float* in, float* out, size_t n, hipStream_t s, unsigned flags,
                 DevStats* st, int v, int g) {
  switch (f) {
    case CR_EXPF: return launch_variant<OpExp<EXPK_E>>(in, out, n, s, flags, st, v, g);
    case CR_EXP2F: return launch_variant<OpExp<EXPK_2>>(in, out, n, s, flags, st, v, g);
    case CR_EXP10F: return launch_variant<OpExp<EXPK_10>>(in, out, n, s, flags, st, v, g);
    case CR_EXPM1F: return launch_variant<OpExp<EXPK_EM1>>(in, out, n, s, flags, st, v, g);
    case CR_LOGF: return launch_variant<OpLog<LOGK_E>>(in, out, n, s, flags, st, v, g);
    case CR_LOG2F: return launch_variant<OpLog<LOGK_2>>(in, out, n, s, flags, st, v, g);
    case CR_LOG10F: return launch_variant<OpLog<LOGK_10>>(in, out, n, s, flags, st, v, g);
    case CR_LOG1PF: return launch_variant<OpLog<LOGK_1P>>(in, out, n, s, flags, st, v, g);
    case CR_RSQRTF: return launch_variant<OpRsqrt>(in, out, n, s, flags, st, v, g);
    case CR_SINF: return launch_variant<OpTrig<TRIGK_SIN>>(in, out, n, s, flags, st, v, g);
    case CR_COSF: return launch_variant<OpTrig<TRIGK_COS>>(in, out, n, s, flags, st, v, g);
    case CR_TANF: return launch_variant<OpTrig<TRIGK_TAN>>(in, out, n, s, flags, st, v, g);
    case CR_SINCOSF: return launch_sincos<SinCosF64>(in, out, n, s, flags, st, g);
    case CR_ASINF: return launch_variant<OpAtan<ATANK_ASIN>>(in, out, n, s, flags, st, v, g);
    case CR_ACOSF: return launch_variant<OpAtan<ATANK_ACOS>>(in, out, n, s, flags, st, v, g);
    case CR_ATANF: return launch_variant<OpAtan<ATANK_ATAN>>(in, out, n, s, flags, st, v, g);
    case CR_SINHF: return launch_variant<OpHyp<HYPK_SINH>>(in, out, n, s, flags, st, v, g);
    case CR_COSHF: return launch_variant<OpHyp<HYPK_COSH>>(in, out, n, s, flags, st, v, g);
    case CR_TANHF: return launch_variant<OpHyp<HYPK_TANH>>(in, out, n, s, flags, st, v, g);
  }
  return CR_E_FUNC;
}


// Directed rounding modes: one kernel per (function, mode), in the default shape.
template <class Op, int RM>
int launch_dir(const float* in, float* out, size_t n, hipStream_t s, unsigned flags, DevStats* st,
               int grid) {
  return launch_map_f32<OpDir<Op, RM>, 2, 1, 0>(in, out, n, s, flags, st, grid);
}

template <int RM>
int dispatch_f32_dir(int f, const float* in, float* out, size_t n, hipStream_t s,
                     unsigned flags, DevStats* st, int g) {
  switch (f) {
    case CR_EXPF: return launch_dir<OpExp<EXPK_E>, RM>(in, out, n, s, flags, st, g);
    case CR_EXP2F: return launch_dir<OpExp<EXPK_2>, RM>(in, out, n, s, flags, st, g);
    case CR_EXP10F: return launch_dir<OpExp<EXPK_10>, RM>(in, out, n, s, flags, st, g);
    case CR_EXPM1F: return launch_dir<OpExp<EXPK_EM1>, RM>(in, out, n, s, flags, st, g);
    case CR_LOGF: return launch_dir<OpLog<LOGK_E>, RM>(in, out, n, s, flags, st, g);
    case CR_LOG2F: return launch_dir<OpLog<LOGK_2>, RM>(in, out, n, s, flags, st, g);
    case CR_LOG10F: return launch_dir<OpLog<LOGK_10>, RM>(in, out, n, s, flags, st, g);
    case CR_LOG1PF: return launch_dir<OpLog<LOGK_1P>, RM>(in, out, n, s, flags, st, g);
    case CR_RSQRTF: return launch_dir<OpRsqrt, RM>(in, out, n, s, flags, st, g);
    case CR_SINF: return launch_dir<OpTrig<TRIGK_SIN>, RM>(in, out, n, s, flags, st, g);
    case CR_COSF: return launch_dir<OpTrig<TRIGK_COS>, RM>(in, out, n, s, flags, st, g);
    case CR_TANF: return launch_dir<OpTrig<TRIGK_TAN>, RM>(in, out, n, s, flags, st, g);
    case CR_ASINF: return launch_dir<OpAtan<ATANK_ASIN>, RM>(in, out, n, s, flags, st, g);
    case CR_ACOSF: return launch_dir<OpAtan<ATANK_ACOS>, RM>(in, out, n, s, flags, st, g);
    case CR_ATANF: return launch_dir<OpAtan<ATANK_ATAN>, RM>(in, out, n, s, flags, st, g);
    case CR_SINHF: return launch_dir<OpHyp<HYPK_SINH>, RM>(in, out, n, s, flags, st, g);
    case CR_COSHF: return launch_dir<OpHyp<HYPK_COSH>, RM>(in, out, n, s, flags, st, g);
    case CR_TANHF: return launch_dir<OpHyp<HYPK_TANH>, RM>(in, out, n, s, flags, st, g);
    case CR_SINCOSF:
      return launch_sincos<SinCosDir<SinCosF64, RM>>(in, out, n, s, flags, st, g);
  }
  return CR_E_FUNC;
}

int dispatch_dir(int mode, int f, const float* in, float* out, size_t n, hipStream_t s,
                 unsigned flags, DevStats* st, int g) {
  switch (mode) {
    case RM_RZ: return dispatch_f32_dir<RM_RZ>(f, in, out, n, s, flags, st, g);
    case RM_RU: return dispatch_f32_dir<RM_RU>(f, in, out, n, s, flags, st, g);
    case RM_RD: return dispatch_f32_dir<RM_RD>(f, in, out, n, s, flags, st, g);
  }
  return CR_E_IMPL;
}

// ------------------------------------------------------------ tuning table
// One launch configuration per (implementation, function): a k_map_f32
// variant and the persistent grid in workgroups per compute unit.  Index 0 of
// the first dimension is the binary64-internal implementation (and AUTO), 1
// the split one; functions 0..18, then the ids of EXTRA_FUNCS.
constexpr int EXTRA_FUNCS[] = {CR_EXP, CR_LOG, CR_EXP2, CR_CEXPF, CR_CLOGF, CR_CSINF};
constexpr int NFUNC_IDX = CR_NUM_F32 + (int)(sizeof(EXTRA_FUNCS) / sizeof(EXTRA_FUNCS[0]));
std::atomic<int> g_cfg_variant[2][NFUNC_IDX];  // the variant + 1, 0: not set
std::atomic<int> g_cfg_bpc[2][NFUNC_IDX];  // 0: the default

int fidx(int f) {
  if (f < CR_NUM_F32) return f;
  for (int i = 0; i < NFUNC_IDX - CR_NUM_F32; i++)
    if (EXTRA_FUNCS[i] == f) return CR_NUM_F32 + i;
  return 0;  // not reached: callers validate f first
}
int iidx(int impl) { return impl == CR_IMPL_SPLIT_F32 ? 1 : 0; }
// sincos and the complex functions have one kernel shape (variant 0 only),
// the binary64 functions NVARIANT64
int num_variants_of(int f) {
  return (f == CR_SINCOSF || func_complex(f)) ? 1 : f >= 64 ? NVARIANT64 : NVARIANT;
}

int eval_cfg(int func_id, int impl, unsigned flags, const void* in, void* out, size_t n,
             hipStream_t s, int variant, int bpc) {
  DevState* ds = nullptr;
  int dev = 0;
  int rc = get_state(&ds, &dev);
  if (rc) return rc;
  DevStats* const st = ds->stats;
  const int g = num_cus() * (bpc > 0 ? bpc : default_bpc());
  const int mode = (int)((flags & CR_FLAG_ROUND_MASK) >> CR_FLAG_ROUND_SHIFT);
  if (mode != RM_RN)
    rc = dispatch_dir(mode, func_id, (const float*)in, (float*)out, n, s, flags, st, g);
  else if (func_id < CR_NUM_F32 && impl == CR_IMPL_SPLIT_F32)
    rc = dispatch_f32_split(func_id, (const float*)in, (float*)out, n, s, flags, st, variant, g);
  else if (func_id < CR_NUM_F32)
    rc = dispatch_f32(func_id, (const float*)in, (float*)out, n, s, flags, st, variant, g);
  else if (func_id == CR_EXP)
    rc = launch_variant64<OpExp64>((const double*)in, (double*)out, n, s, flags, st, variant, g);
  else if (func_id == CR_EXP2)
    rc = launch_variant64<OpExp2_64>((const double*)in, (double*)out, n, s, flags, st, variant, g);
  else if (func_id == CR_LOG && impl == CR_IMPL_LOG128)
    rc = launch_variant64<OpLog128>((const double*)in, (double*)out, n, s, flags, st, variant, g);
  else if (func_id == CR_CEXPF)
    rc = launch_complex<CExpF>((const float*)in, (float*)out, n, s, flags, st, g);
  else if (func_id == CR_CLOGF)
    rc = launch_complex<CLogF>((const float*)in, (float*)out, n, s, flags, st, g);
  else if (func_id == CR_CSINF)
    rc = launch_complex<CSinF>((const float*)in, (float*)out, n, s, flags, st, g);
  else
    rc = launch_variant64<OpLog64>((const double*)in, (double*)out, n, s, flags, st, variant, g);
  if (rc == CR_OK) g_elems[dev] += n;
  return rc;
}

const char* const FUNC_NAMES[NFUNC_IDX] = {
    "expf", "exp2f", "exp10f", "expm1f", "logf", "log2f", "log10f", "log1pf", "rsqrtf",
    "sinf", "cosf", "sincosf", "tanf", "asinf", "acosf", "atanf", "sinhf", "coshf", "tanhf",
    "exp", "log", "exp2", "cexpf", "clogf", "csinf"};

int func_of_idx(int i) { return i < CR_NUM_F32 ? i : EXTRA_FUNCS[i - CR_NUM_F32]; }

// ------------------------------------------------------------ batch plans

// A batch on the host: the requests with elements, sorted by (implementation,
// function), and the request of every tile.
struct BatchTables {
  std::vector<BReq> reqs;
  std::vector<unsigned> tile_req;
  int split_req = 0, split_tile = 0;  // where the binary32-only ones begin
  int tile = TILE;                    // elements per tile
  long long elems = 0;
};

// The functions in the order a batch evaluates them within an implementation: the
// most expensive element first, so that the last workgroups are short ones.
constexpr int BATCH_ORDER[CR_NUM_F32] = {
    CR_SINCOSF, CR_TANF,  CR_ACOSF, CR_ASINF,  CR_SINF,   CR_COSF,  CR_ATANF,
    CR_SINHF,   CR_TANHF, CR_COSHF, CR_LOG1PF, CR_EXPM1F, CR_LOGF,  CR_LOG10F,
    CR_LOG2F,   CR_EXP2F, CR_EXP10F, CR_EXPF,  CR_RSQRTF};

// Workgroups per compute unit of the batch kernels, per implementation
// (binary64-internal, binary32-only): a tuned setting (cr_tune_batch_set, the
// "batch" lines of the tuning file).  The graph of a large plan runs up to four
// per-function kernels at a time with this many each (2, 4, 8: 636, 588, 592 us on
// 3.07e8 elements); the one kernel over all functions gets BATCH_GRID_SCALE times as
// many, of which four fit at a time: the rest start as others end, which evens out
// the functions' different costs (a scale of 1, 4, 8: 48, 41, 38 us on 12.4e6).
constexpr int BATCH_BPC_DEFAULT = 4, BATCH_GRID_SCALE = 8;
std::atomic<int> g_batch_bpc[2] = {BATCH_BPC_DEFAULT, BATCH_BPC_DEFAULT};

// Validate requests and build the tables.
int build_tables_unguarded(const cr_request* reqs, int32_t num, BatchTables& T) {
  if (num < 0) return CR_E_SIZE;
  if (num > 0 && !reqs) return CR_E_NULL;
  for (int i = 0; i < num; i++) {
    const cr_request& r = reqs[i];
    if (r.func_id < 0 || r.func_id >= CR_NUM_F32) return CR_E_FUNC;
    if (r.impl != CR_IMPL_AUTO && r.impl != CR_IMPL_F64_INTERNAL && r.impl != CR_IMPL_SPLIT_F32)
      return CR_E_IMPL;
    if (r.n < 0 || r.n >= ((int64_t)1 << 31)) return CR_E_SIZE;
    if (r.n == 0) continue;
    if (!r.in || !r.out) return CR_E_NULL;
    uintptr_t a = (uintptr_t)r.in, b = (uintptr_t)r.out;
    if ((a & 3) || (b & 3)) return CR_E_ALIGN;
    size_t nout = r.func_id == CR_SINCOSF ? 2 * (size_t)r.n : (size_t)r.n;
    bool same = a == b && nout == (size_t)r.n;
    if (!same && a < b + nout * 4 && b < a + (size_t)r.n * 4) return CR_E_OVERLAP;
    if (!cr_available(r.func_id, r.impl)) return CR_E_IMPL;
    T.elems += r.n;
  }
  int rank[CR_NUM_F32];
  for (int k = 0; k < CR_NUM_F32; k++) rank[BATCH_ORDER[k]] = k;
  std::vector<std::pair<int, int>> order;  // (rank, index in the caller's array)
  for (int i = 0; i < num; i++)
    if (reqs[i].n > 0)
      order.push_back({rank[reqs[i].func_id] +
                           (reqs[i].impl == CR_IMPL_SPLIT_F32 ? CR_NUM_F32 : 0), i});
  std::sort(order.begin(), order.end());
  // A batch that leaves the chip short of workgroups is cut finer, up to 8 tiles per
  // compute unit.  Finer still costs more in look-ups than it gains: at up to 32 tiles
  // per compute unit 12.4e6 elements took 42 us instead of 38, 3.2e6 19 instead of 16.
  for (T.tile = TILE / 4; T.tile < TILE && T.elems / T.tile > 8LL * num_cus(); T.tile *= 2) {
  }
  long long ntiles = 0;
  for (const auto& o : order) ntiles += (reqs[o.second].n + T.tile - 1) / T.tile;
  if (ntiles > ((long long)1 << 30)) return CR_E_SIZE;
  T.reqs.reserve(order.size());
  T.tile_req.reserve((size_t)ntiles);
  for (const auto& o : order) {
    const cr_request& r = reqs[o.second];
    const bool split = o.first >= CR_NUM_F32;
    if (!split) {
      T.split_req++;
      T.split_tile += (int)((r.n + T.tile - 1) / T.tile);
    }
    const unsigned ri = (unsigned)T.reqs.size();
    T.reqs.push_back({(const float*)r.in, (float*)r.out, (unsigned)r.n,
                      (unsigned)T.tile_req.size(), r.func_id + (split ? BSPLIT : 0), o.second});
    T.tile_req.insert(T.tile_req.end(), (size_t)((r.n + T.tile - 1) / T.tile), ri);
  }
  return CR_OK;
}

int build_tables(const cr_request* reqs, int32_t num, BatchTables& T) {
  try {
    return build_tables_unguarded(reqs, num, T);
  } catch (const std::bad_alloc&) {
    return CR_E_NOMEM;
  }
}

// Tiles per workgroup for a launch of nt tiles.
int batch_per(long long nt, bool split) {
  const long long grid =
      (long long)num_cus() * BATCH_GRID_SCALE * g_batch_bpc[split ? 1 : 0].load();
  return (int)((nt + grid - 1) / grid);
}

// The batch from tables in device memory: one kernel per implementation present.
hipError_t launch_batch(const BReq* reqs, const unsigned* tile_req, const BatchTables& T,
                        const int (&per)[2], DevStats* st, unsigned flags, hipStream_t s) {
  const int nt = (int)T.tile_req.size();
  if (T.split_tile > 0)
    hipLaunchKernelGGL(k_batch<false>, dim3((T.split_tile + per[0] - 1) / per[0]), dim3(BLOCK), 0,
                       s, (BReqTab)reqs, (BTileTab)tile_req, 0, T.split_tile, per[0], T.tile, st,
                       flags);
  if (nt > T.split_tile)
    hipLaunchKernelGGL(k_batch<true>, dim3((nt - T.split_tile + per[1] - 1) / per[1]), dim3(BLOCK),
                       0, s, (BReqTab)reqs, (BTileTab)tile_req, T.split_tile, nt, per[1], T.tile,
                       st, flags);
  return hipGetLastError();
}

// One kernel per function present, on the streams in turn.
template <class E>
void launch_tiles(const BReq* r, const unsigned* tr, int t0, int t1, int grid, int tile,
                  DevStats* st, unsigned flags, hipStream_t s) {
  hipLaunchKernelGGL(k_tiles<E>, dim3(grid), dim3(BLOCK), 0, s, (BReqTab)r, (BTileTab)tr, t0, t1,
                     tile, st, flags);
}
int launch_functions(const BReq* r, const unsigned* tr, const BatchTables& T, DevStats* st,
                     unsigned flags, hipStream_t* streams, int nstreams) {
  const int n = (int)T.reqs.size(), nt = (int)T.tile_req.size();
  int si = 0;
  for (int r0 = 0, r1; r0 < n; r0 = r1) {
    const int key = T.reqs[r0].key;
    for (r1 = r0; r1 < n && T.reqs[r1].key == key;) r1++;
    const int t0 = (int)T.reqs[r0].tile0, t1 = r1 < n ? (int)T.reqs[r1].tile0 : nt;
    const int g = (int)std::min<long long>(
        t1 - t0, (long long)num_cus() * g_batch_bpc[key >= BSPLIT ? 1 : 0].load());
    hipStream_t s = streams[si++ % nstreams];
    switch (key) {
#define CR_CASE(id, ...)                                               \
  case id:                                                             \
    launch_tiles<__VA_ARGS__>(r, tr, t0, t1, g, T.tile, st, flags, s); \
    break
      CR_CASE(CR_EXPF, BOne<OpExp<EXPK_E>>);
      CR_CASE(CR_EXP2F, BOne<OpExp<EXPK_2>>);
      CR_CASE(CR_EXP10F, BOne<OpExp<EXPK_10>>);
      CR_CASE(CR_EXPM1F, BOne<OpExp<EXPK_EM1>>);
      CR_CASE(CR_LOGF, BOne<OpLog<LOGK_E>>);
      CR_CASE(CR_LOG2F, BOne<OpLog<LOGK_2>>);
      CR_CASE(CR_LOG10F, BOne<OpLog<LOGK_10>>);
      CR_CASE(CR_LOG1PF, BOne<OpLog<LOGK_1P>>);
      CR_CASE(CR_RSQRTF, BOne<OpRsqrt>);
      CR_CASE(CR_SINF, BOne<OpTrig<TRIGK_SIN>>);
      CR_CASE(CR_COSF, BOne<OpTrig<TRIGK_COS>>);
      CR_CASE(CR_SINCOSF, BTwo<SinCosF64>);
      CR_CASE(CR_TANF, BOne<OpTrig<TRIGK_TAN>>);
      CR_CASE(CR_ASINF, BOne<OpAtan<ATANK_ASIN>>);
      CR_CASE(CR_ACOSF, BOne<OpAtan<ATANK_ACOS>>);
      CR_CASE(CR_ATANF, BOne<OpAtan<ATANK_ATAN>>);
      CR_CASE(CR_SINHF, BOne<OpHyp<HYPK_SINH>>);
      CR_CASE(CR_COSHF, BOne<OpHyp<HYPK_COSH>>);
      CR_CASE(CR_TANHF, BOne<OpHyp<HYPK_TANH>>);
      CR_CASE(BSPLIT + CR_EXPF, BOne<OpSExp<EXPK_E>>);
      CR_CASE(BSPLIT + CR_EXP2F, BOne<OpSExp<EXPK_2>>);
      CR_CASE(BSPLIT + CR_EXP10F, BOne<OpSExp<EXPK_10>>);
      CR_CASE(BSPLIT + CR_EXPM1F, BOne<OpSExp<EXPK_EM1>>);
      CR_CASE(BSPLIT + CR_LOGF, BOne<OpSLog<LOGK_E>>);
      CR_CASE(BSPLIT + CR_LOG2F, BOne<OpSLog<LOGK_2>>);
      CR_CASE(BSPLIT + CR_LOG10F, BOne<OpSLog<LOGK_10>>);
      CR_CASE(BSPLIT + CR_LOG1PF, BOne<OpSLog<LOGK_1P>>);
      CR_CASE(BSPLIT + CR_RSQRTF, BOne<OpSRsqrt>);
      CR_CASE(BSPLIT + CR_SINF, BOne<OpSTrig<TRIGK_SIN>>);
      CR_CASE(BSPLIT + CR_COSF, BOne<OpSTrig<TRIGK_COS>>);
      CR_CASE(BSPLIT + CR_SINCOSF, BTwo<SinCosSplit>);
      CR_CASE(BSPLIT + CR_TANF, BOne<OpSTrig<TRIGK_TAN>>);
      CR_CASE(BSPLIT + CR_ASINF, BOne<OpSAtan<ATANK_ASIN>>);
      CR_CASE(BSPLIT + CR_ACOSF, BOne<OpSAtan<ATANK_ACOS>>);
      CR_CASE(BSPLIT + CR_ATANF, BOne<OpSAtan<ATANK_ATAN>>);
      CR_CASE(BSPLIT + CR_SINHF, BOne<OpSHyp<HYPK_SINH>>);
      CR_CASE(BSPLIT + CR_COSHF, BOne<OpSHyp<HYPK_COSH>>);
      CR_CASE(BSPLIT + CR_TANHF, BOne<OpSHyp<HYPK_TANH>>);
#undef CR_CASE
      default: return CR_E_FUNC;
    }
  }
  return CR_OK;
}

// Plans of more elements than this run one kernel per function (at most 8 waves per
// SIMD instead of the 4 that the registers of the most demanding function leave the
// one kernel), captured in a graph on four parallel branches, whose 125 us of launch
// work then overlaps the kernels: 3.07e8 elements 588 us against about 630 by the one
// kernel, 1.14e8 256 against 255, 5.6e7 158 against 125-143.
constexpr long long GRAPH_ELEMS = 1LL << 26;

// The graph of a plan's per-function kernels: private streams at default priority,
// a fork from the origin stream and a join back to it, so that one kernel's tail
// overlaps the next kernel's start.
hipError_t capture_functions(const BReq* r, const unsigned* tr, const BatchTables& T, DevStats* st,
                             unsigned flags, hipGraphExec_t* exec) {
  constexpr int NBRANCH = 4;
  hipStream_t cs = nullptr, side[NBRANCH] = {};
  hipEvent_t fork = nullptr, join[NBRANCH] = {};
  hipGraph_t g = nullptr;
  hipError_t e = hipStreamCreateWithFlags(&cs, hipStreamNonBlocking);
  for (int b = 0; b < NBRANCH && e == hipSuccess; b++) {
    e = hipStreamCreateWithFlags(&side[b], hipStreamNonBlocking);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&join[b], hipEventDisableTiming);
  }
  if (e == hipSuccess) e = hipEventCreateWithFlags(&fork, hipEventDisableTiming);
  if (e == hipSuccess) e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
  if (e == hipSuccess) {
    hipError_t ec = hipEventRecord(fork, cs);
    for (int b = 0; b < NBRANCH && ec == hipSuccess; b++) ec = hipStreamWaitEvent(side[b], fork, 0);
    int rc = ec == hipSuccess ? launch_functions(r, tr, T, st, flags, side, NBRANCH) : CR_OK;
    for (int b = 0; b < NBRANCH && ec == hipSuccess; b++) {
      ec = hipEventRecord(join[b], side[b]);
      if (ec == hipSuccess) ec = hipStreamWaitEvent(cs, join[b], 0);
    }
    hipError_t e2 = hipStreamEndCapture(cs, &g);
    e = hipGetLastError();
    if (e == hipSuccess) e = ec;
    if (e == hipSuccess) e = e2;
    if (e == hipSuccess && rc != CR_OK) e = hipErrorInvalidValue;
  }
  if (e == hipSuccess) e = hipGraphInstantiate(exec, g, nullptr, nullptr, 0);
  if (g) (void)hipGraphDestroy(g);
  if (fork) (void)hipEventDestroy(fork);
  for (int b = 0; b < NBRANCH; b++) {
    if (join[b]) (void)hipEventDestroy(join[b]);
    if (side[b]) (void)hipStreamDestroy(side[b]);
  }
  if (cs) (void)hipStreamDestroy(cs);
  return e;
}

// The batch from kernel arguments, BARG requests of one implementation a launch.
int args_launches(const BatchTables& T) {
  return (T.split_req + BARG - 1) / BARG + ((int)T.reqs.size() - T.split_req + BARG - 1) / BARG;
}
hipError_t launch_batch_args(const BatchTables& T, DevStats* st, unsigned flags, hipStream_t s) {
  BArgs a;
  for (int r0 = 0, n = (int)T.reqs.size(); r0 < n;) {
    const bool split = r0 >= T.split_req;
    const int r1 = std::min(r0 + BARG, split ? n : T.split_req);
    const unsigned base = T.reqs[r0].tile0;
    const int nt = (int)((r1 < n ? T.reqs[r1].tile0 : (unsigned)T.tile_req.size()) - base);
    for (int k = 0; k < 128; k++) {
      a.tile0[k] = k < r1 - r0 ? T.reqs[r0 + k].tile0 - base : 0xffffffffu;
      if (k < r1 - r0) {
        a.req[k] = T.reqs[r0 + k];
        a.req[k].tile0 -= base;
      }
    }
    const int per = batch_per(nt, split);
    if (split)
      hipLaunchKernelGGL(k_batch_args<true>, dim3((nt + per - 1) / per), dim3(BLOCK), 0, s, a, nt,
                         per, T.tile, st, flags);
    else
      hipLaunchKernelGGL(k_batch_args<false>, dim3((nt + per - 1) / per), dim3(BLOCK), 0, s, a, nt,
                         per, T.tile, st, flags);
    r0 = r1;
  }
  return hipGetLastError();
}

bool capturing(hipStream_t s) {
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &cs) == hipSuccess) return cs != hipStreamCaptureStatusNone;
  (void)hipGetLastError();  // what is wrong with the stream shows in the call that uses it
  return false;
}

// Whether a batch goes by kernel arguments: a launch costs about 4.5 us here, the
// allocation and copy of the tables and the wait for it about 35 us more than that
// (200 requests, three launches: 18 us; 512 requests by tables: 44 us), so up to
// ARGS_LAUNCHES launches.  They can be captured like any launch; the tables cannot
// (the call waits for their copy), so a larger batch is refused on a stream that is
// being captured before anything is enqueued there.
constexpr int ARGS_LAUNCHES = 4;
hipError_t batch_route(const BatchTables& T, hipStream_t s, bool& args) {
  args = args_launches(T) <= ARGS_LAUNCHES;
  if (args) return hipSuccess;
  return capturing(s) ? hipErrorStreamCaptureUnsupported : hipSuccess;
}

}  // namespace

struct cr_batch_plan {
  int device;
  BReq* d_reqs;
  unsigned* d_tile_req;
  BatchTables tables;
  DevStats* stats;
  int per[2];  // tiles per workgroup, binary64-internal and binary32-only
  unsigned flags;
  hipGraphExec_t exec;  // large plans: the per-function kernels
  hipEvent_t done;
  bool launched;
};

extern "C" {

int cr_available(int func_id, int impl);

int cr_eval_ex(int func_id, int impl, unsigned flags, const void* in, void* out, size_t n,
               void* stream) {
  if (!func_valid(func_id)) return CR_E_FUNC;
  if (!impl_valid(impl)) return CR_E_IMPL;
  if (n == 0) return CR_OK;
  if (!in || !out) return CR_E_NULL;
  const size_t es = elem_bytes(func_id), al = func_complex(func_id) ? 4 : es;
  const size_t nout = func_id == CR_SINCOSF ? 2 * n : n;
  if (n > ((size_t)1 << 60)) return CR_E_SIZE;
  uintptr_t a = (uintptr_t)in, b = (uintptr_t)out;
  if ((a % al) || (b % al)) return CR_E_ALIGN;
  bool same = a == b && nout == n;
  if (!same && a < b + nout * es && b < a + n * es) return CR_E_OVERLAP;
  if (!cr_available(func_id, impl)) return CR_E_IMPL;
  if ((flags & CR_FLAG_ROUND_MASK) &&
      (func_id >= CR_NUM_F32 || impl == CR_IMPL_SPLIT_F32 || impl == CR_IMPL_LOG128))
    return CR_E_IMPL;  // directed modes: the binary32 functions, binary64-internal
  const int ii = iidx(impl), fi = fidx(func_id);
  return eval_cfg(func_id, impl, flags, in, out, n, (hipStream_t)stream,
                  g_cfg_variant[ii][fi].load() - 1, g_cfg_bpc[ii][fi].load());
}

// ------------------------------------------------------------------ tuning
int cr_tune_num_variants(void) { return NVARIANT; }

int cr_tune_variant_info(int variant, int* elems_per_thread, int* prefetch, int* table_in_lds) {
  if (variant < 0 || variant >= NVARIANT) return CR_E_TUNE;
  if (elems_per_thread) *elems_per_thread = 4 * VARIANTS[variant][0];
  if (prefetch) *prefetch = VARIANTS[variant][1];
  if (table_in_lds) *table_in_lds = VARIANTS[variant][2] ? 0 : 1;
  return CR_OK;
}

static int tune_check(int func_id, int impl, const cr_tune_cfg* cfg) {
  if (!func_valid(func_id)) return CR_E_FUNC;
  if (!impl_valid(impl)) return CR_E_IMPL;
  if (!cfg) return CR_E_NULL;
  if (cfg->variant < 0 || cfg->variant >= num_variants_of(func_id)) return CR_E_TUNE;
  if (cfg->blocks_per_cu < 0 || cfg->blocks_per_cu > 64) return CR_E_TUNE;
  return CR_OK;
}

int cr_tune_get(int func_id, int impl, cr_tune_cfg* cfg) {
  if (!func_valid(func_id)) return CR_E_FUNC;
  if (!impl_valid(impl)) return CR_E_IMPL;
  if (!cfg) return CR_E_NULL;
  const int ii = iidx(impl), fi = fidx(func_id);
  cfg->variant = std::max(g_cfg_variant[ii][fi].load() - 1, 0);
  int b = g_cfg_bpc[ii][fi].load();
  cfg->blocks_per_cu = b > 0 ? b : default_bpc();
  return CR_OK;
}

int cr_tune_set(int func_id, int impl, const cr_tune_cfg* cfg) {
  int rc = tune_check(func_id, impl, cfg);
  if (rc) return rc;
  const int ii = iidx(impl), fi = fidx(func_id);
  g_cfg_variant[ii][fi] = cfg->variant + 1;
  g_cfg_bpc[ii][fi] = cfg->blocks_per_cu;
  return CR_OK;
}

int cr_tune_reset(void) {
  for (int i = 0; i < 2; i++) {
    for (int f = 0; f < NFUNC_IDX; f++) {
      g_cfg_variant[i][f] = 0;
      g_cfg_bpc[i][f] = 0;
    }
    g_batch_bpc[i] = BATCH_BPC_DEFAULT;
  }
  return CR_OK;
}

int cr_tune_batch_get(int impl, int32_t* blocks_per_cu) {
  if (!impl_valid(impl) || impl == CR_IMPL_LOG128) return CR_E_IMPL;
  if (!blocks_per_cu) return CR_E_NULL;
  *blocks_per_cu = g_batch_bpc[iidx(impl)].load();
  return CR_OK;
}

int cr_tune_batch_set(int impl, int32_t blocks_per_cu) {
  if (!impl_valid(impl) || impl == CR_IMPL_LOG128) return CR_E_IMPL;
  if (blocks_per_cu < 1 || blocks_per_cu > 64) return CR_E_TUNE;
  g_batch_bpc[iidx(impl)] = blocks_per_cu;
  return CR_OK;
}

int cr_tune_save(const char* path) {
  if (!path) return CR_E_NULL;
  FILE* fp = fopen(path, "w");
  if (!fp) return CR_E_TUNE;
  fprintf(fp, "# libcr launch configurations: function implementation variant blocks_per_cu\n");
  for (int i = 0; i < 2; i++)
    for (int f = 0; f < NFUNC_IDX; f++) {
      int b = g_cfg_bpc[i][f].load();
      fprintf(fp, "%s %s %d %d\n", FUNC_NAMES[f], i ? "split" : "f64",
              std::max(g_cfg_variant[i][f].load() - 1, 0), b > 0 ? b : default_bpc());
    }
  for (int i = 0; i < 2; i++)
    fprintf(fp, "batch %s 0 %d\n", i ? "split" : "f64", g_batch_bpc[i].load());
  int bad = ferror(fp);
  if (fclose(fp) != 0 || bad) return CR_E_TUNE;
  return CR_OK;
}

int cr_tune_load(const char* path) {
  if (!path) return CR_E_NULL;
  FILE* fp = fopen(path, "r");
  if (!fp) return CR_E_TUNE;
  struct Entry { int impl, func, variant, bpc; };
  std::vector<Entry> es;
  char line[512];
  int rc = CR_OK;
  while (fgets(line, sizeof line, fp)) {
    char* p = line;
    while (*p == ' ' || *p == '\t') p++;
    if (*p == '#' || *p == '\n' || *p == '\r' || *p == 0) continue;
    char fname[64], iname[16];
    int v = -1, b = -1;
    if (sscanf(p, "%63s %15s %d %d", fname, iname, &v, &b) != 4) {
      rc = CR_E_TUNE;
      break;
    }
    int f = -1;
    for (int k = 0; k < NFUNC_IDX; k++)
      if (!strcmp(fname, FUNC_NAMES[k])) f = func_of_idx(k);
    int impl = !strcmp(iname, "f64") ? CR_IMPL_F64_INTERNAL
               : !strcmp(iname, "split") ? CR_IMPL_SPLIT_F32 : -1;
    if (!strcmp(fname, "batch")) {  // the batch kernels' grid: variant 0 only
      if (impl < 0 || v != 0 || b < 1 || b > 64) {
        rc = CR_E_TUNE;
        break;
      }
      es.push_back({impl, -1, v, b});
      continue;
    }
    cr_tune_cfg c = {v, b};
    if (f < 0 || impl < 0 || tune_check(f, impl, &c) != CR_OK) {
      rc = CR_E_TUNE;
      break;
    }
    es.push_back({impl, f, v, b});
  }
  fclose(fp);
  if (rc) return rc;  // nothing applied from a malformed file
  for (const Entry& e : es) {
    if (e.func < 0) {
      g_batch_bpc[iidx(e.impl)] = e.bpc;
      continue;
    }
    g_cfg_variant[iidx(e.impl)][fidx(e.func)] = e.variant + 1;
    g_cfg_bpc[iidx(e.impl)][fidx(e.func)] = e.bpc;
  }
  return CR_OK;
}

int cr_autotune(int func_id, int impl, const void* in, void* out, size_t n, int reps,
                void* stream, double* best_gelem_s) {
  if (!func_valid(func_id)) return CR_E_FUNC;
  if (!impl_valid(impl)) return CR_E_IMPL;
  if (n == 0 || !in || !out) return CR_E_NULL;
  const size_t es = elem_bytes(func_id), al = func_complex(func_id) ? 4 : es;
  const size_t nout = func_id == CR_SINCOSF ? 2 * n : n;
  if (n > ((size_t)1 << 60)) return CR_E_SIZE;
  uintptr_t a = (uintptr_t)in, b = (uintptr_t)out;
  if ((a % al) || (b % al)) return CR_E_ALIGN;
  bool same = a == b && nout == n;
  if (!same && a < b + nout * es && b < a + n * es) return CR_E_OVERLAP;
  if (!cr_available(func_id, impl)) return CR_E_IMPL;
  if (reps <= 0) reps = 10;
  hipStream_t s = (hipStream_t)stream;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  hipError_t e = hipEventCreate(&e0);
  if (e == hipSuccess) e = hipEventCreate(&e1);
  if (e != hipSuccess) {
    if (e0) (void)hipEventDestroy(e0);
    return hip_fail(e);
  }
  static const int BPCS[] = {2, 4, 8, 16, 32};
  constexpr int NB = sizeof(BPCS) / sizeof(BPCS[0]);
  const int nv = num_variants_of(func_id);
  // time reps launches of one configuration (after one untimed launch)
  auto time_cfg = [&](int v, int bpc, float& ms) -> int {
    int r0 = eval_cfg(func_id, impl, 0u, in, out, n, s, v, bpc);
    if (r0) return r0;
    hipError_t he = hipEventRecord(e0, s);
    for (int r = 0; r < reps && he == hipSuccess && r0 == CR_OK; r++)
      r0 = eval_cfg(func_id, impl, 0u, in, out, n, s, v, bpc);
    if (r0) return r0;
    if (he == hipSuccess) he = hipEventRecord(e1, s);
    if (he == hipSuccess) he = hipEventSynchronize(e1);
    if (he == hipSuccess) he = hipEventElapsedTime(&ms, e0, e1);
    return he == hipSuccess ? CR_OK : hip_fail(he);
  };
  // Let the clocks settle under this load (about 100 ms of it) before
  // timing: the first milliseconds of work run at lower clocks and would
  // favour whichever configuration is timed last.
  int rc = CR_OK;
  for (float busy = 0.0f; busy < 100.0f && rc == CR_OK;) {
    float ms = 0.0f;
    rc = time_cfg(0, 0, ms);
    busy += ms > 0.0f ? ms : 100.0f;
  }
  // three passes over the space, alternating in order; the median counts
  constexpr int NPASS = 3;
  std::vector<float> times((size_t)nv * NB * NPASS, 0.0f);
  for (int pass = 0; pass < NPASS && rc == CR_OK; pass++) {
    for (int c = 0; c < nv * NB && rc == CR_OK; c++) {
      const int idx = (pass & 1) ? nv * NB - 1 - c : c;
      float ms = 0.0f;
      rc = time_cfg(idx / NB, BPCS[idx % NB], ms);
      times[(size_t)idx * NPASS + pass] = ms;
    }
  }
  std::vector<float> best_of(nv * NB, 0.0f);
  for (int idx = 0; idx < nv * NB && rc == CR_OK; idx++) {
    float* t = &times[(size_t)idx * NPASS];
    std::sort(t, t + NPASS);
    best_of[idx] = t[NPASS / 2];
  }
  float best_ms = 0.0f;
  int best_v = 0, best_b = 0;
  for (int idx = 0; idx < nv * NB && rc == CR_OK; idx++) {
    if (best_ms == 0.0f || best_of[idx] < best_ms) {
      best_ms = best_of[idx];
      best_v = idx / NB;
      best_b = BPCS[idx % NB];
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (rc) return rc;
  const int ii = iidx(impl), fi = fidx(func_id);
  g_cfg_variant[ii][fi] = best_v + 1;
  g_cfg_bpc[ii][fi] = best_b;
  if (best_gelem_s) *best_gelem_s = best_ms > 0 ? (double)n * reps / (best_ms * 1e-3) / 1e9 : 0.0;
  return CR_OK;
}

int cr_available(int func_id, int impl) {
  if (!func_valid(func_id)) return 0;
  if (impl == CR_IMPL_SPLIT_F32) return split_built(func_id) ? 1 : 0;
  if (impl == CR_IMPL_LOG128) return func_id == CR_LOG ? 1 : 0;
  if (impl != CR_IMPL_AUTO && impl != CR_IMPL_F64_INTERNAL) return 0;
  return func_built(func_id) ? 1 : 0;
}

int cr_eval(int func_id, const void* in, void* out, size_t n, void* stream) {
  return cr_eval_ex(func_id, CR_IMPL_AUTO, 0u, in, out, n, stream);
}

int cr_dft(const float* x, int64_t n, const float* w, int64_t m, double* X, unsigned flags,
           void* stream) {
  if (n < 0 || m < 0 || n > ((int64_t)1 << 24) || m > ((int64_t)1 << 31)) return CR_E_SIZE;
  if (m == 0) return CR_OK;
  if (!w || !X || (n > 0 && !x)) return CR_E_NULL;
  if (((uintptr_t)x % 4) || ((uintptr_t)w % 4) || ((uintptr_t)X % 16)) return CR_E_ALIGN;
  const uintptr_t xo = (uintptr_t)X, xe = xo + (uintptr_t)m * 16;
  if ((n > 0 && (uintptr_t)x < xe && xo < (uintptr_t)x + (uintptr_t)n * 4) ||
      ((uintptr_t)w < xe && xo < (uintptr_t)w + (uintptr_t)m * 4))
    return CR_E_OVERLAP;
  DevStats* st = nullptr;
  int rc = get_stats(&st);
  if (rc) return rc;
  hipStream_t s = (hipStream_t)stream;
  // samples per block: enough blocks to fill the chip (8 per CU) but at least
  // 8 samples per thread
  const long long target = (long long)num_cus() * 8;
  long long S = (target + m - 1) / m;
  const long long smax = (n + BLOCK * 8 - 1) / (BLOCK * 8);
  if (S > smax) S = smax;
  // up to 64 terms a thread in one slice take less than the allocation of a workspace
  // and a second kernel (18 us of host work), whatever the number of outputs.  A call,
  // one slice at n = 2^14: 14.6 us for 1 output, 17.1 for 64, 42.8 for 1024; several
  // slices at n = 20000: 27.4, 27.1, 54.4 (at n = 2^14, with the sine and cosine of
  // before: 27.0, 26.0, 75.2).
  if (S < 1 || n <= 64 * BLOCK) S = 1;
  long long slice = (n + S - 1) / S;
  slice = (slice + BLOCK - 1) / BLOCK * BLOCK;
  if (slice < BLOCK) slice = BLOCK;
  S = n > 0 ? (n + slice - 1) / slice : 1;
  // one slice: the kernel writes the result itself, without a workspace
  double4* part = nullptr;
  hipError_t e = hipSuccess;
  if (S > 1) e = hipMallocAsync((void**)&part, (size_t)m * S * sizeof(double4), s);
  if (e != hipSuccess) return e == hipErrorOutOfMemory ? CR_E_NOMEM : hip_fail(e);
  double2* Xd = reinterpret_cast<double2*>(X);
  auto kernel = S > 1 ? k_dft<false> : k_dft<true>;
  for (long long k0 = 0; k0 < m; k0 += 65535) {  // grid.y is at most 65535
    const long long mk = m - k0 < 65535 ? m - k0 : 65535;
    hipLaunchKernelGGL(kernel, dim3((unsigned)S, (unsigned)mk), dim3(BLOCK), 0, s, x, (int)n,
                       w + k0, (int)slice, part ? part + k0 * S : nullptr, Xd + k0, (int)S, st,
                       flags, k0);
  }
  if (S > 1)
    hipLaunchKernelGGL(k_dft_finish, dim3((unsigned)((m + BLOCK / 64 - 1) / (BLOCK / 64))),
                       dim3(BLOCK), 0, s, part, (int)S, (long long)m, Xd);
  e = hipGetLastError();
  hipError_t e2 = part ? hipFreeAsync(part, s) : hipSuccess;
  if (e != hipSuccess) return hip_fail(e);
  if (e2 != hipSuccess) return hip_fail(e2);
  int dev = 0;
  (void)hipGetDevice(&dev);
  g_elems[dev] += (unsigned long long)n * (unsigned long long)m;
  return CR_OK;
}


int cr_batch_plan_destroy(cr_batch_plan* plan) {
  if (!plan) return CR_OK;
  if (plan->launched && plan->done) (void)hipEventSynchronize(plan->done);
  if (plan->exec) (void)hipGraphExecDestroy(plan->exec);
  if (plan->done) (void)hipEventDestroy(plan->done);
  if (plan->d_reqs) (void)hipFree(plan->d_reqs);
  if (plan->d_tile_req) (void)hipFree(plan->d_tile_req);
  delete plan;
  return CR_OK;
}

int cr_batch_plan_create(const cr_request* reqs, int32_t num, unsigned flags,
                         cr_batch_plan** plan) {
  if (!plan) return CR_E_NULL;
  *plan = nullptr;
  if (flags & CR_FLAG_ROUND_MASK) return CR_E_IMPL;  // batches round to nearest
  BatchTables T;
  int rc = build_tables(reqs, num, T);
  if (rc) return rc;
  DevStats* st = nullptr;
  rc = get_stats(&st);
  if (rc) return rc;
  cr_batch_plan* p = new cr_batch_plan();
  (void)hipGetDevice(&p->device);
  p->flags = flags;
  p->stats = st;
  p->tables = std::move(T);
  const std::vector<BReq>& hr = p->tables.reqs;
  const std::vector<unsigned>& ht = p->tables.tile_req;
  p->per[0] = std::max(1, batch_per(p->tables.split_tile, false));
  p->per[1] = std::max(1, batch_per((long long)ht.size() - p->tables.split_tile, true));
  hipError_t e = hipSuccess;
  if (!hr.empty()) e = hipMalloc(&p->d_reqs, hr.size() * sizeof(BReq));
  if (e == hipSuccess && !ht.empty()) e = hipMalloc(&p->d_tile_req, ht.size() * sizeof(unsigned));
  if (e != hipSuccess) {
    t_last_hip = (int)e;
    cr_batch_plan_destroy(p);
    return CR_E_NOMEM;
  }
  if (!hr.empty()) e = hipMemcpy(p->d_reqs, hr.data(), hr.size() * sizeof(BReq), hipMemcpyHostToDevice);
  if (e == hipSuccess && !ht.empty())
    e = hipMemcpy(p->d_tile_req, ht.data(), ht.size() * sizeof(unsigned), hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipEventCreateWithFlags(&p->done, hipEventDisableTiming);
  if (e == hipSuccess && p->tables.elems > GRAPH_ELEMS)
    e = capture_functions(p->d_reqs, p->d_tile_req, p->tables, st, flags, &p->exec);
  if (e != hipSuccess) {
    t_last_hip = (int)e;
    cr_batch_plan_destroy(p);
    return CR_E_HIP;
  }
  *plan = p;
  return CR_OK;
}

int cr_batch_plan_launch(cr_batch_plan* plan, void* stream) {
  if (!plan) return CR_E_NULL;
  hipStream_t s = (hipStream_t)stream;
  if (!plan->tables.reqs.empty()) {
    // Into a caller's capture go the kernels themselves (a graph launch leaves
    // nothing there) and no event: `done` stands for the launches that run now.
    const bool cap = capturing(s);
    hipError_t e = hipSuccess;
    if (plan->exec && !cap)
      e = hipGraphLaunch(plan->exec, s);
    else
      e = launch_batch(plan->d_reqs, plan->d_tile_req, plan->tables, plan->per, plan->stats,
                       plan->flags, s);
    if (e == hipSuccess && !cap) e = hipEventRecord(plan->done, s);
    if (e != hipSuccess) return hip_fail(e);
    if (!cap) plan->launched = true;
    g_elems[plan->device] += plan->tables.elems;
  }
  return CR_OK;
}

// The batch by kernel arguments or, for larger ones, by tables copied to device
// memory at dr and dt; the host vectors are freed on return, so the call waits until
// the copies have read them.
static int run_batch(const BatchTables& T, bool args, BReq* dr, unsigned* dt, DevStats* st,
                     hipStream_t s) {
  hipError_t e = hipSuccess;
  if (args) {
    e = launch_batch_args(T, st, 0u, s);
  } else {
    const int per[2] = {std::max(1, batch_per(T.split_tile, false)),
                        std::max(1, batch_per((long long)T.tile_req.size() - T.split_tile, true))};
    e = hipMemcpyAsync(dr, T.reqs.data(), T.reqs.size() * sizeof(BReq), hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
      e = hipMemcpyAsync(dt, T.tile_req.data(), T.tile_req.size() * sizeof(unsigned),
                         hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e == hipSuccess) e = launch_batch(dr, dt, T, per, st, 0u, s);
  }
  if (e != hipSuccess) return hip_fail(e);
  int dev = 0;
  (void)hipGetDevice(&dev);
  g_elems[dev] += T.elems;
  return CR_OK;
}

int cr_eval_batch(const cr_request* reqs, int32_t num, void* stream) {
  BatchTables T;
  int rc = build_tables(reqs, num, T);
  if (rc) return rc;
  if (T.reqs.empty()) return CR_OK;
  DevStats* st = nullptr;
  rc = get_stats(&st);
  if (rc) return rc;
  hipStream_t s = (hipStream_t)stream;
  bool args = false;
  hipError_t e = batch_route(T, s, args);
  if (e != hipSuccess) return hip_fail(e);
  if (args) return run_batch(T, true, nullptr, nullptr, st, s);
  // one stream-ordered allocation for both tables
  const size_t rb = (T.reqs.size() * sizeof(BReq) + 255) / 256 * 256;
  unsigned char* d = nullptr;
  e = hipMallocAsync((void**)&d, rb + T.tile_req.size() * sizeof(unsigned), s);
  if (e != hipSuccess) {
    t_last_hip = (int)e;
    return CR_E_NOMEM;
  }
  rc = run_batch(T, false, (BReq*)d, (unsigned*)(d + rb), st, s);
  (void)hipFreeAsync(d, s);
  return rc;
}

int cr_eval_batch_noalloc(const cr_request* reqs, int32_t num, void* stream) {
  if (num > CR_NOALLOC_MAX_REQUESTS) return CR_E_SCRATCH;
  BatchTables T;
  int rc = build_tables(reqs, num, T);
  if (rc) return rc;
  if (T.reqs.empty()) return CR_OK;
  // the limit counts tiles of 4096 elements, whatever tiles the batch is cut into
  size_t tiles = 0;
  for (const BReq& r : T.reqs) tiles += ((size_t)r.n + TILE - 1) / TILE;
  if (tiles > (size_t)CR_NOALLOC_MAX_TILES || T.tile_req.size() > (size_t)CR_NOALLOC_MAX_TILES)
    return CR_E_SCRATCH;
  DevState* ds = nullptr;
  rc = get_state(&ds);
  if (rc) return rc;
  hipStream_t s = (hipStream_t)stream;
  bool args = false;
  const hipError_t e = batch_route(T, s, args);
  if (e != hipSuccess) return hip_fail(e);
  // stream-ordered after earlier work on s (including an earlier call's kernels
  // still reading the tables)
  return run_batch(T, args, reinterpret_cast<BReq*>(ds->scratch),
                   reinterpret_cast<unsigned*>(ds->scratch + NOALLOC_REQ_BYTES), ds->stats, s);
}

int cr_stats_reset(void* stream) {
  DevStats* st = nullptr;
  int rc = get_stats(&st);
  if (rc) return rc;
  hipLaunchKernelGGL(k_zero_stats, dim3(1), dim3(256), 0, (hipStream_t)stream, st);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e);
  int dev = 0;
  (void)hipGetDevice(&dev);
  g_elems[dev] = 0;
  return CR_OK;
}

int cr_stats_read(void* stream, cr_stats* out) {
  if (!out) return CR_E_NULL;
  DevStats* st = nullptr;
  int rc = get_stats(&st);
  if (rc) return rc;
  DevStats* h = new DevStats;
  hipError_t e = hipMemcpyAsync(h, st, sizeof(DevStats), hipMemcpyDeviceToHost,
                                (hipStream_t)stream);
  if (e == hipSuccess) e = hipStreamSynchronize((hipStream_t)stream);
  if (e != hipSuccess) {
    delete h;
    return hip_fail(e);
  }
  int dev = 0;
  (void)hipGetDevice(&dev);
  out->elems = g_elems[dev];
  out->fallback_lanes = out->fallback_waves = 0;
  for (int i = 0; i < NSLOT; i++) {
    out->fallback_lanes += h->slot[i].fallback_lanes;
    out->fallback_waves += h->slot[i].fallback_waves;
  }
  out->escapes = h->escapes;
  for (int i = 0; i < 16; i++) out->escape_index[i] = h->escape_index[i];
  delete h;
  return CR_OK;
}

const char* cr_status_str(int status) {
  switch (status) {
    case CR_OK: return "ok";
    case CR_E_FUNC: return "unknown function id";
    case CR_E_NULL: return "null pointer";
    case CR_E_OVERLAP: return "input and output overlap";
    case CR_E_ALIGN: return "pointer not aligned to its element size";
    case CR_E_IMPL: return "implementation not available";
    case CR_E_HIP: return "HIP runtime error";
    case CR_E_NOMEM: return "device allocation failed";
    case CR_E_SIZE: return "size too large";
    case CR_E_TUNE: return "invalid launch configuration or tuning file";
    case CR_E_SCRATCH: return "batch exceeds the static scratch of cr_eval_batch_noalloc";
  }
  return "unknown status";
}

int cr_last_hip_error(void) { return t_last_hip; }

}  // extern "C"
