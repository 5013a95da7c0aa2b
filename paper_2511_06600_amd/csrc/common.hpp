// Internal helpers shared by the HIP translation units of libhyperef.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <cstdio>
#include <string>

#include "hyperef.h"

namespace hef {

// ---------------------------------------------------------------- errors
void set_error(const char *fmt, ...);
const char *last_error();

#define HEF_HIP(call)                                                        \
  do {                                                                       \
    hipError_t _e = (call);                                                  \
    if (_e != hipSuccess) {                                                  \
      ::hef::set_error("%s failed: %s (%s:%d)", #call, hipGetErrorString(_e), \
                       __FILE__, __LINE__);                                  \
      return HEF_ERR_DEVICE;                                                 \
    }                                                                        \
  } while (0)

#define HEF_TRY(expr)                  \
  do {                                 \
    hef_status _s = (expr);            \
    if (_s != HEF_OK) return _s;       \
  } while (0)

#define HEF_LAUNCH_CHECK() HEF_HIP(hipGetLastError())

// A workspace carve that ran past the caller's workspace.
#define HEF_WS_CHECK(arena)                                                       \
  do {                                                                            \
    if ((arena).overflow) {                                                       \
      ::hef::set_error("workspace overflow in %s (%s:%d)", __func__, __FILE__, __LINE__); \
      return HEF_ERR_WORKSPACE_TOO_SMALL;                                         \
    }                                                                             \
  } while (0)

// ------------------------------------------------------------- workspace
// Bump allocator over the caller's workspace.  With base == nullptr it only
// measures, so the planner and the runtime carve the workspace identically.
struct Arena {
  char *base = nullptr;
  size_t cap = 0;
  size_t off = 0;
  bool overflow = false;

  template <class T>
  T *take(size_t count) {
    size_t bytes = count * sizeof(T);
    size_t start = (off + 255) & ~size_t(255);
    off = start + bytes;
    if (base == nullptr) return nullptr;
    if (off > cap) {
      overflow = true;
      return nullptr;
    }
    return reinterpret_cast<T *>(base + start);
  }
  size_t mark() const { return off; }
  void reset(size_t m) { off = m; }
};

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// The Krylov pool before orthonormalisation is stored in a row-octet layout:
// rows in groups of 8, each column of a group contiguous, i.e. element
// (r, c) of an n x K pool at ((r >> 3) * K + c) * 8 + (r & 7), with n
// padded to oct_rows(n) (padding rows are zero).
inline int64_t oct_rows(int64_t n) { return (n + 7) / 8 * 8; }

// Orders the LDS accesses of one wave: what a lane wrote before the call is
// seen by the wave's other lanes after it.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Lane l's value of v on every lane (l the same on all lanes: a scalar
// broadcast, no LDS round trip).
__device__ __forceinline__ double readlane_f64(double v, int l) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane(uint32_t(u), l);
  const uint32_t hi = __builtin_amdgcn_readlane(uint32_t(u >> 32), l);
  return __builtin_bit_cast(double, (uint64_t(hi) << 32) | lo);
}

// A Cholesky pivot: root = sqrt(d) and inv, its reciprocal to within an ulp,
// for d within 1e-200 .. 1e200.  A kept pivot exceeds tau^2 times its Gram
// diagonal, a sum of squares of float32 values (1e-90 .. 1e90), or with tau = 0
// is what their roundings leave of it, 1e-16 of it or so.  Goldschmidt steps
// from an approximate reciprocal square root y (relative error 2^-20 or less),
// with two residual corrections of the root; over that range root equals
// sqrt(d) to the bit.  The chain is 13 operations; sqrt() and a division by it
// are about 35 with their range checks.
struct Pivot {
  double root, inv;
};
__host__ __device__ __forceinline__ Pivot pivot_from(double d, double y) {
  double g = d * y, h = 0.5 * y;
  const double r = __builtin_fma(-h, g, 0.5);
  g = __builtin_fma(g, r, g);
  h = __builtin_fma(h, r, h);
  g = __builtin_fma(__builtin_fma(-g, g, d), h, g);
  g = __builtin_fma(__builtin_fma(-g, g, d), h, g);
  double i = h + h;
  i = __builtin_fma(__builtin_fma(-g, i, 1.0), i, i);
  return {g, i};
}
// (from the hardware's reciprocal square root)
__device__ __forceinline__ Pivot pivot_of(double d) {
  return pivot_from(d, __builtin_amdgcn_rsq(d));
}
// x / p.root by a quotient within an ulp or two, its exact residual and one
// fused correction (Markstein): equal to the division, or an ulp off in the
// few cases where inv is not the nearest to 1 / root.
__host__ __device__ __forceinline__ double div_pivot(double x, const Pivot &p) {
  const double q = x * p.inv;
  return __builtin_fma(__builtin_fma(-q, p.root, x), p.inv, q);
}

// acc[i] + x[i](lane 0) + x[i](lane 1) + ... + x[i](lane cnt - 1), added in that
// order (cnt the same on all lanes): N sequential sums whose terms a wave loaded
// side by side.
template <int N>
__device__ __forceinline__ void ordered_sums(double (&acc)[N], const double (&x)[N], int cnt) {
  if (cnt == 64) {  // (lane numbers known: no loop between the additions)
#pragma unroll
    for (int l = 0; l < 64; ++l)
#pragma unroll
      for (int i = 0; i < N; ++i) acc[i] = acc[i] + readlane_f64(x[i], l);
    return;
  }
  for (int l = 0; l < cnt; ++l)
#pragma unroll
    for (int i = 0; i < N; ++i) acc[i] = acc[i] + readlane_f64(x[i], l);
}

// Map a launched block index to a logical one so that each of the 8 XCDs of
// an MI355X (which receive blocks round-robin) walks a contiguous range of
// logical blocks; neighbouring work then shares its XCD's L2.
__device__ __forceinline__ int64_t xcd_block(int64_t bid, int64_t nblocks) {
  constexpr int64_t kXcd = 8;
  int64_t per = nblocks / kXcd;
  int64_t rem = nblocks % kXcd;
  int64_t x = bid % kXcd;
  int64_t i = bid / kXcd;
  // XCDs 0..rem-1 own per+1 blocks, the rest own per.
  int64_t start = x * per + (x < rem ? x : rem);
  int64_t cnt = per + (x < rem ? 1 : 0);
  return i < cnt ? start + i : bid;  // i < cnt always holds for a full grid
}

// Level-independent sizes of one hypergraph level.
struct Level {
  int32_t n = 0, m = 0;
  int64_t nnz = 0;
  const int32_t *eptr = nullptr;
  const int32_t *pins = nullptr;
  const float *w = nullptr;  // nullptr = unit weights
};

}  // namespace hef

namespace hef {

// ------------------------------------------------------------ stage timing
// Optional per-stage kernel timing (hef_timing_enable): HIP events recorded
// on the launch stream around each stage's kernels.  Off by default; when
// off a TimedScope does nothing.
enum Stage : int {
  kStStructure = 0,
  kStSpmmCsr,
  kStSpmmCsc,
  kStLanczosGram,
  kStLanczosSolve,
  kStLanczosApply,
  kStOrthGram,
  kStOrthChol,
  kStOrthApply,
  kStScoreQ,
  kStScoreR,
  kStClusterUpdate,
  kStClusterContract,
  kStClusterLocal,
  kStClusterRebuild,
  kStAdjoint,
  kStStart,
  kStSpmmPrep,
  kStLanczosReduce,
  kStOrthReduce,
  kStScoreReduce,
  kStClusterBest,
  kStQuality,
  kStRating,
  kStSpmmStep,  // the fused SpMM (prep, CSR and CSC) as one span; off unless selected
  kStageCount
};

bool timing_on(int stage);
void timing_push(int stage, hipEvent_t a, hipEvent_t b);

struct TimedScope {
  int stage;
  hipStream_t s;
  hipEvent_t a = nullptr, b = nullptr;
  TimedScope(int st, hipStream_t stream) : stage(st), s(stream) {
    if (timing_on(st)) {
      if (hipEventCreate(&a) == hipSuccess && hipEventCreate(&b) == hipSuccess)
        (void)hipEventRecord(a, s);
      else
        a = b = nullptr;
    }
  }
  ~TimedScope() {
    if (a && b) {
      (void)hipEventRecord(b, s);
      timing_push(stage, a, b);
    }
  }
};

}  // namespace hef
