// Resistance ratios (Eqs. (9), (13), (14); Alg. 1).
//
// For every hyperedge e and pool column i the two most distant pins along
// chi^(i) are its largest and smallest entries, so the numerator of Eq. (13)
// is s_e^(i) = (max_{p in e} chi_p^(i) - min_{p in e} chi_p^(i))^2.
// A first pass takes the extremes of the long hyperedges (k_score_long).
// Pass 1 forms Q_H(chi^(i)) = sum_e w_e s_e^(i) (Eq. (9)) and stores the
// m x K numerators s (float32, row e contiguous); pass 2 streams them back
// to form R_e = max_i s_e^(i) / Q_H(chi^(i)) (Eq. (14)).  Streaming s costs
// 8 K bytes per hyperedge; regathering the pool rows cost about 4 K bytes per
// pin, mostly missed in L2.
//
// A group of LPR lanes handles one hyperedge, each lane CPL consecutive
// columns of the gathered rows; a workgroup walks a contiguous range of
// hyperedges (XCD-contiguous), so neighbouring hyperedges share pool rows
// in L2.  Sums are float64 in a fixed order.
#include <cfloat>
#include <type_traits>

#include "krylov.hpp"
#include "prims.hpp"
#include "score.hpp"

namespace hef {
namespace {

constexpr int kThreads = 256;
constexpr int kEdgesPerBlk = 128;

// Pool values of one type: float64 for the float64 debug basis, else float
// (bfloat16 widens exactly).
template <int PT>
using PoolVal = typename std::conditional<PT == kPoolF64, double, float>::type;

template <int CPL, int PT>
__device__ __forceinline__ void load_cols(const void *pool, int64_t p, int K, int c0,
                                          PoolVal<PT> (&v)[CPL]) {
  if constexpr (PT == kPoolF64) {
    const double *row = reinterpret_cast<const double *>(pool) + p * K + c0;
    if ((K & 1) == 0 && c0 + CPL <= K) {
#pragma unroll
      for (int q = 0; q < CPL; q += 2) {
        const double2 t = *reinterpret_cast<const double2 *>(row + q);
        v[q] = t.x; v[q + 1] = t.y;
      }
    } else {
#pragma unroll
      for (int q = 0; q < CPL; ++q) v[q] = (c0 + q < K) ? row[q] : 0.0;
    }
  } else if (PT == kPoolF32) {
    const float *row = reinterpret_cast<const float *>(pool) + p * K + c0;
    if ((K & 3) == 0 && c0 + CPL <= K) {
#pragma unroll
      for (int q = 0; q < CPL; q += 4) {
        const float4 t = *reinterpret_cast<const float4 *>(row + q);
        v[q] = t.x; v[q + 1] = t.y; v[q + 2] = t.z; v[q + 3] = t.w;
      }
    } else {
#pragma unroll
      for (int q = 0; q < CPL; ++q) v[q] = (c0 + q < K) ? row[q] : 0.0f;
    }
  } else {
    const uint16_t *row = reinterpret_cast<const uint16_t *>(pool) + p * K + c0;
    if ((K & 3) == 0 && c0 + CPL <= K) {
#pragma unroll
      for (int q = 0; q < CPL; q += 4) {
        const uint2 t = *reinterpret_cast<const uint2 *>(row + q);
        v[q] = __uint_as_float(t.x << 16);
        v[q + 1] = __uint_as_float(t.x & 0xFFFF0000u);
        v[q + 2] = __uint_as_float(t.y << 16);
        v[q + 3] = __uint_as_float(t.y & 0xFFFF0000u);
      }
    } else {
#pragma unroll
      for (int q = 0; q < CPL; ++q)
        v[q] = (c0 + q < K) ? __uint_as_float(uint32_t(row[q]) << 16) : 0.0f;
    }
  }
}

// Spread of hyperedge [a, b) of pins over this lane's columns.  Pins go in
// chunks of 4 (ids first, then rows, so the loads overlap); a chunk past the
// end repeats the last pin, which leaves max and min unchanged.
__device__ __forceinline__ float vmax(float a, float b) { return fmaxf(a, b); }
__device__ __forceinline__ float vmin(float a, float b) { return fminf(a, b); }
__device__ __forceinline__ double vmax(double a, double b) { return fmax(a, b); }
__device__ __forceinline__ double vmin(double a, double b) { return fmin(a, b); }

template <int CPL, int PT>
__device__ __forceinline__ void edge_spread(const int32_t *__restrict__ pins, const void *pool,
                                            int K, int c0, int32_t a, int32_t b,
                                            double (&s)[CPL]) {
  using T = PoolVal<PT>;
  constexpr T kBig = PT == kPoolF64 ? T(DBL_MAX) : T(FLT_MAX);
  T mx[CPL], mn[CPL];
#pragma unroll
  for (int q = 0; q < CPL; ++q) { mx[q] = -kBig; mn[q] = kBig; }
  for (int32_t j0 = a; j0 < b; j0 += 4) {
    int32_t pp[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) pp[u] = pins[j0 + u < b ? j0 + u : b - 1];
    T v[4][CPL];
#pragma unroll
    for (int u = 0; u < 4; ++u) load_cols<CPL, PT>(pool, pp[u], K, c0, v[u]);
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int q = 0; q < CPL; ++q) { mx[q] = vmax(mx[q], v[u][q]); mn[q] = vmin(mn[q], v[u][q]); }
  }
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    const double d = double(mx[q]) - double(mn[q]);
    s[q] = d * d;
  }
}

// Pool values of columns c0.. (exact: they are pool values).
template <int CPL, int PT>
__device__ __forceinline__ void store_cols(void *pool, int64_t row, int K, int c0,
                                           const PoolVal<PT> (&v)[CPL]) {
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    if (c0 + q >= K) continue;
    if constexpr (PT == kPoolF64)
      reinterpret_cast<double *>(pool)[row * K + c0 + q] = v[q];
    else if constexpr (PT == kPoolF32)
      reinterpret_cast<float *>(pool)[row * K + c0 + q] = v[q];
    else
      reinterpret_cast<uint16_t *>(pool)[row * K + c0 + q] =
          uint16_t(__float_as_uint(v[q]) >> 16);
  }
}

// Largest and smallest pool values of every long hyperedge (of more than
// long_from(longseg) pins), a workgroup per hyperedge of the list: as many of
// its groups of LPR lanes as it has fours of pins take 4 at a time, then their
// extremes meet in LDS, by halves down to 16 groups.  Row 2 i of `ext`
// receives the largest, row 2 i + 1 the smallest values, i = (first pin
// position) / longseg, which no two such hyperedges share.  Maxima do not
// depend on the order, so the ratios keep their bits.  The longest hyperedge's
// chain bounds it at small sizes, the gathers at large ones: 26 us at 20k nodes,
// K = 464, 43 at 200k, K = 160, 337 at 2M, K = 480 (206 with the bfloat16 pool).
// With the groups' extremes taken in one after the other, all of them for a
// hyperedge of any length, 50000 hyperedges of 40 pins at K = 24 took 727 us,
// seven times a lane group each.
constexpr int kLongThreads = 1024;
constexpr int kLongLast = 16;

// The line where many hyperedges are long (long_from): 128 pins, but none with
// lane groups of 32 lanes or more, of which a workgroup has 32 at most.  us, an
// estimate with a workgroup for every one / above 64 / above 128 pins: 50000
// hyperedges of 40 pins, K = 24, 1618 / 982 / 984, K = 160, 2946 / 2870 / 2864;
// 20000 of 100 pins, K = 24, 1172 / 1025 / 937, K = 160, 2810 / 2821 / 2953; 2M
// nodes, bfloat16, K = 480 (15k hyperedges above 32 pins), 28579 / 28695 / -.
__device__ __forceinline__ int score_many(int lanes) { return lanes >= 32 ? 0 : 128; }

// (held to 64 VGPRs but for the float64 pool: two workgroups a CU, 206 us
// against 308 at 2M nodes, K = 480, bfloat16)
template <int CPL, int PT>
__global__ void __launch_bounds__(kLongThreads)
__attribute__((amdgpu_waves_per_eu(PT == kPoolF64 ? 4 : 8, 8)))
k_score_long(const int32_t *__restrict__ list, const int32_t *__restrict__ count,
             const int32_t *__restrict__ eptr, const int32_t *__restrict__ pins,
             const void *__restrict__ pool, int K, int LPR, int longseg, void *__restrict__ ext) {
  using T = PoolVal<PT>;
  constexpr T kBig = PT == kPoolF64 ? T(DBL_MAX) : T(FLT_MAX);
  __shared__ T smx[kLongThreads * CPL], smn[kLongThreads * CPL];
  const int tid = threadIdx.x;
  const int ngrp = kLongThreads / LPR;
  const int grp = tid / LPR;
  const int c0 = (tid % LPR) * CPL;
  const int W = LPR * CPL;  // columns of a group's LDS row
  const int32_t cnt = *count;
  const int from = long_from(longseg, score_many(LPR), cnt);
  for (int32_t bi = blockIdx.x; bi < cnt; bi += gridDim.x) {
    const int32_t e = list[bi];
    const int32_t a = eptr[e], b = eptr[e + 1];
    if (b - a <= from) continue;  // (the same on every thread)
    const int use = b - a < 4 * ngrp ? (b - a + 3) / 4 : ngrp;  // groups with pins
    T mx[CPL], mn[CPL];
#pragma unroll
    for (int q = 0; q < CPL; ++q) { mx[q] = -kBig; mn[q] = kBig; }
    if (c0 < K) {
      for (int64_t j0 = a + 4 * grp; j0 < b; j0 += 4 * ngrp) {
        int32_t pp[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) pp[u] = pins[j0 + u < b ? j0 + u : b - 1];
        T v[4][CPL];
#pragma unroll
        for (int u = 0; u < 4; ++u) load_cols<CPL, PT>(pool, pp[u], K, c0, v[u]);
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int q = 0; q < CPL; ++q) {
            mx[q] = vmax(mx[q], v[u][q]);
            mn[q] = vmin(mn[q], v[u][q]);
          }
      }
    }
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      smx[grp * W + c0 + q] = mx[q];
      smn[grp * W + c0 + q] = mn[q];
    }
    __syncthreads();
    // groups [0, half) take in [half, 2 half) down to kLongLast groups, whose
    // extremes the first takes in (a barrier costs more than the reads it saves)
    int left = use;
#pragma unroll 1
    for (int half = kLongThreads / 2; half >= kLongLast; half /= 2) {
      if (half >= left) continue;
      if (grp < half && grp + half < left) {
#pragma unroll
        for (int q = 0; q < CPL; ++q) {
          mx[q] = vmax(mx[q], smx[(grp + half) * W + c0 + q]);
          mn[q] = vmin(mn[q], smn[(grp + half) * W + c0 + q]);
          smx[grp * W + c0 + q] = mx[q];
          smn[grp * W + c0 + q] = mn[q];
        }
      }
      left = half;
      __syncthreads();
    }
    if (grp == 0 && c0 < K) {
#pragma unroll 1
      for (int g = 1; g < left; ++g)
#pragma unroll
        for (int q = 0; q < CPL; ++q) {
          mx[q] = vmax(mx[q], smx[g * W + c0 + q]);
          mn[q] = vmin(mn[q], smn[g * W + c0 + q]);
        }
      const int64_t row = 2 * int64_t(a / longseg);
      store_cols<CPL, PT>(ext, row, K, c0, mx);
      store_cols<CPL, PT>(ext, row + 1, K, c0, mn);
    }
    __syncthreads();
  }
}

// A workgroup takes kEdgesPerBlk consecutive hyperedges [e0, e1); group grp
// (LPR lanes, ngrp groups) takes e0 + grp + ngrp k, in rounds of LPR: lane j
// of the group fetches the pin range of the round's j-th hyperedge up front.
// Hyperedges of more than long_from(longseg) pins take their extremes from `ext`
// (k_score_long): one group walking 2000 pins is a chain of 500 dependent
// gathers, 0.2 to 0.4 ms whatever the size of the launch.  Measured with
// that chain / without (this pass plus k_score_long): 20k nodes, K = 464,
// 204 / 92 us; 200k nodes, K = 160, 410 / 174 us; 2M nodes, K = 480,
// 3.85 / 3.62 ms.
template <int CPL, int PT>
__global__ void __launch_bounds__(kThreads)
k_score_qh(const int32_t *__restrict__ eptr, const int32_t *__restrict__ pins,
           const float *__restrict__ w, const void *__restrict__ pool, int K, int LPR,
           int64_t m, double *__restrict__ partial, float *__restrict__ sbuf, int longseg,
           const int32_t *__restrict__ n_big, const void *__restrict__ ext) {
  __shared__ double comb[kThreads * CPL];
  const int from = long_from(longseg, score_many(LPR), *n_big);
  const int tid = threadIdx.x;
  const int ngrp = kThreads / LPR;
  const int grp = tid / LPR;
  const int sub = tid % LPR;
  const int c0 = sub * CPL;
  const int64_t blk = xcd_block(blockIdx.x, gridDim.x);
  const int64_t e0 = blk * kEdgesPerBlk;
  const int64_t e1 = e0 + kEdgesPerBlk < m ? e0 + kEdgesPerBlk : m;
  double acc[CPL];
#pragma unroll
  for (int q = 0; q < CPL; ++q) acc[q] = 0.0;
  for (int k0 = 0; k0 < kEdgesPerBlk / ngrp && e0 + grp + int64_t(ngrp) * k0 < e1; k0 += LPR) {
    int32_t ea = 0, eb = 0;
    float ew = 0.0f;
    {
      const int64_t e = e0 + grp + int64_t(ngrp) * (k0 + sub);
      if (e < e1) {
        ea = eptr[e];
        eb = eptr[e + 1];
        ew = w ? w[e] : 1.0f;
      }
    }
    for (int k = 0; k < LPR && e0 + grp + int64_t(ngrp) * (k0 + k) < e1; ++k) {
      const int32_t a = __shfl(ea, k, LPR), b = __shfl(eb, k, LPR);
      const double we = double(__shfl(ew, k, LPR));
      if (c0 < K) {
        double s[CPL];
        if (b - a > from) {
          PoolVal<PT> mx[CPL], mn[CPL];
          const int64_t row = 2 * int64_t(a / longseg);
          load_cols<CPL, PT>(ext, row, K, c0, mx);
          load_cols<CPL, PT>(ext, row + 1, K, c0, mn);
#pragma unroll
          for (int q = 0; q < CPL; ++q) {
            const double d = double(mx[q]) - double(mn[q]);
            s[q] = d * d;
          }
        } else {
          edge_spread<CPL, PT>(pins, pool, K, c0, a, b, s);
        }
#pragma unroll
        for (int q = 0; q < CPL; ++q) acc[q] = fma(we, s[q], acc[q]);
        float *out = sbuf + (e0 + grp + int64_t(ngrp) * (k0 + k)) * K + c0;
        if (c0 + CPL <= K && (K & 3) == 0) {
#pragma unroll
          for (int q = 0; q < CPL; q += 4)
            *reinterpret_cast<float4 *>(out + q) =
                make_float4(float(s[q]), float(s[q + 1]), float(s[q + 2]), float(s[q + 3]));
        } else {
#pragma unroll
          for (int q = 0; q < CPL; ++q)
            if (c0 + q < K) out[q] = float(s[q]);
        }
      }
    }
  }
  // the groups' sums, added in group order
#pragma unroll
  for (int q = 0; q < CPL; ++q) comb[grp * LPR * CPL + c0 + q] = acc[q];
  __syncthreads();
  for (int c = tid; c < K; c += kThreads) {
    double t = comb[c];
    for (int g = 1; g < ngrp; ++g) t = t + comb[g * LPR * CPL + c];
    partial[blk * K + c] = t;
  }
}

// k_score_qh for few hyperedges: the same workgroups of kEdgesPerBlk
// hyperedges, whose sums must keep their order, would leave most of the chip
// idle, each group walking LPR / 2 hyperedges one after another.  Four times
// the threads take them: group gid handles hyperedge number 4 t + gid / ngrp of
// the old group gid % ngrp in round t, its spreads go to LDS, and the old
// groups' sums are formed there in their old order.  A round waits for its
// longest hyperedge, so this pays while the launch fills the chip at most once:
// 512 workgroups of 4 columns a lane, 256 of 8.  us, k_score_qh / this:
//   hyperedges     5k         21k        42k        65k        126k
//   K = 20      28 / 18    30 / 17    32 / 20    40 / 23    42 / 44
//   K = 160     59 / 41    61 / 42    73 / 55    77 / 60    95 / 106
//   K = 464     78 / 64    85 / 67   113 / 125  124 / 151  224 / 296
template <int CPL>
constexpr int kFewBlocks = 2048 / CPL;
constexpr int kFewThreads = 1024;

template <int CPL, int PT>
__global__ void __launch_bounds__(kFewThreads)
k_score_qh_few(const int32_t *__restrict__ eptr, const int32_t *__restrict__ pins,
               const float *__restrict__ w, const void *__restrict__ pool, int K, int LPR,
               int64_t m, double *__restrict__ partial, float *__restrict__ sbuf, int longseg,
               const int32_t *__restrict__ n_big, const void *__restrict__ ext) {
  const int from = long_from(longseg, score_many(LPR), *n_big);
  constexpr int R = kFewThreads / kThreads;
  constexpr int NA = kThreads * CPL / kFewThreads;  // sums per thread
  static_assert(NA * kFewThreads == kThreads * CPL, "whole sums per thread");
  __shared__ double sp[kFewThreads * CPL];
  __shared__ float sw[kFewThreads];
  const int tid = threadIdx.x;
  const int ngrp = kThreads / LPR, W = LPR * CPL;
  const int gid = tid / LPR, g = gid % ngrp, r = gid / ngrp;
  const int c0 = (tid % LPR) * CPL;
  const int per = kEdgesPerBlk / ngrp;  // hyperedges of an old group
  const int64_t blk = xcd_block(blockIdx.x, gridDim.x);
  const int64_t e0 = blk * kEdgesPerBlk;
  const int64_t e1 = e0 + kEdgesPerBlk < m ? e0 + kEdgesPerBlk : m;
  double acc[NA];
#pragma unroll
  for (int i = 0; i < NA; ++i) acc[i] = 0.0;
  int32_t na = 0, nb = 0;  // the next round's pins and weight
  float nw = 0.0f;
  auto fetch = [&](int k) {
    const int64_t e = e0 + g + int64_t(ngrp) * k;
    na = nb = 0;
    if (k < per && e < e1) {
      na = eptr[e];
      nb = eptr[e + 1];
      nw = w ? w[e] : 1.0f;
    }
  };
  fetch(r);
  for (int k0 = 0; k0 < per && e0 + int64_t(ngrp) * k0 < e1; k0 += R) {
    const int32_t a = na, b = nb;
    const float we = nw;
    const int64_t e = e0 + g + int64_t(ngrp) * (k0 + r);
    fetch(k0 + R + r);
    if (a < b && c0 < K) {
      double s[CPL];
      if (b - a > from) {
        PoolVal<PT> mx[CPL], mn[CPL];
        const int64_t row = 2 * int64_t(a / longseg);
        load_cols<CPL, PT>(ext, row, K, c0, mx);
        load_cols<CPL, PT>(ext, row + 1, K, c0, mn);
#pragma unroll
        for (int q = 0; q < CPL; ++q) {
          const double d = double(mx[q]) - double(mn[q]);
          s[q] = d * d;
        }
      } else {
        edge_spread<CPL, PT>(pins, pool, K, c0, a, b, s);
      }
#pragma unroll
      for (int q = 0; q < CPL; ++q) sp[gid * W + c0 + q] = s[q];
      float *out = sbuf + e * K + c0;
      if (c0 + CPL <= K && (K & 3) == 0) {
#pragma unroll
        for (int q = 0; q < CPL; q += 4)
          *reinterpret_cast<float4 *>(out + q) =
              make_float4(float(s[q]), float(s[q + 1]), float(s[q + 2]), float(s[q + 3]));
      } else {
#pragma unroll
        for (int q = 0; q < CPL; ++q)
          if (c0 + q < K) out[q] = float(s[q]);
      }
    }
    if (c0 == 0) sw[gid] = we;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const int at = tid + kFewThreads * i, og = at / W, c = at % W;
      if (c >= K) continue;
#pragma unroll
      for (int q = 0; q < R; ++q)
        if (k0 + q < per && e0 + og + int64_t(ngrp) * (k0 + q) < e1)
          acc[i] = fma(double(sw[q * ngrp + og]), sp[(q * ngrp + og) * W + c], acc[i]);
    }
    __syncthreads();
  }
  // the groups' sums, added in group order
#pragma unroll
  for (int i = 0; i < NA; ++i) sp[tid + kFewThreads * i] = acc[i];
  __syncthreads();
  for (int c = tid; c < K; c += kFewThreads) {
    double t = sp[c];
    for (int og = 1; og < ngrp; ++og) t = t + sp[og * W + c];
    partial[blk * K + c] = t;
  }
}

// R_e = max_i s_e^(i) / Q_H^(i) from the stored numerators: LPR lanes per
// hyperedge, CPL columns each (ties in the maximum are irrelevant: only the
// value is kept).
template <int CPL>
__global__ void __launch_bounds__(kThreads)
k_score_r(const float *__restrict__ sbuf, int K, int LPR, int64_t m,
          const double *__restrict__ qh, float *__restrict__ R) {
  const int tid = threadIdx.x;
  const int ngrp = kThreads / LPR;
  const int grp = tid / LPR;
  const int sub = tid % LPR;
  const int c0 = sub * CPL;
  double inv[CPL];
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    const double qv = (c0 + q < K) ? qh[c0 + q] : 0.0;
    inv[q] = qv > 0.0 ? 1.0 / qv : 0.0;
  }
  const int64_t e0 = int64_t(xcd_block(blockIdx.x, gridDim.x)) * kEdgesPerBlk;
  const int64_t e1 = e0 + kEdgesPerBlk < m ? e0 + kEdgesPerBlk : m;
  for (int64_t e = e0 + grp; e < e1; e += ngrp) {
    double best = 0.0;
    if (c0 < K) {
      const float *row = sbuf + e * K + c0;
      float v[CPL];
      if (c0 + CPL <= K && (K & 3) == 0) {
#pragma unroll
        for (int q = 0; q < CPL; q += 4) {
          const float4 t = *reinterpret_cast<const float4 *>(row + q);
          v[q] = t.x; v[q + 1] = t.y; v[q + 2] = t.z; v[q + 3] = t.w;
        }
      } else {
#pragma unroll
        for (int q = 0; q < CPL; ++q) v[q] = c0 + q < K ? row[q] : 0.0f;
      }
#pragma unroll
      for (int q = 0; q < CPL; ++q) best = fmax(best, double(v[q]) * inv[q]);
    }
    for (int off = LPR / 2; off > 0; off >>= 1) best = fmax(best, __shfl_xor(best, off, LPR));
    if (sub == 0) R[e] = float(best);
  }
}

// At least kThreads / kEdgesPerBlk lanes, so that a workgroup has no more
// groups than hyperedges: with one lane a group (K <= CPL) its 256 groups
// would share 128 hyperedges, and the groups' loops, which run
// kEdgesPerBlk / ngrp times, would visit none.
int lanes_for(int K, int CPL) {
  int need = (K + CPL - 1) / CPL;
  int l = kThreads / kEdgesPerBlk;
  while (l < need) l <<= 1;
  return l;
}

template <int CPL, int PT>
hef_status score_t(const Level &L, const Structure &st, const void *pool, int K, double *qh,
                   float *R, double *partial, float *sbuf, int64_t nblk, int longseg, void *ext,
                   hipStream_t s) {
  const int LPR = lanes_for(K, CPL);
  {
  TimedScope ts(kStScoreQ, s);
  const int nlong = int(std::min<int64_t>(L.nnz / longseg, 2048));
  if (nlong > 0)
    k_score_long<CPL, PT><<<nlong, kLongThreads, 0, s>>>(st.big_e, st.n_big, L.eptr, L.pins,
                                                         pool, K, LPR, longseg, ext);
  if (nblk <= kFewBlocks<CPL>)
    k_score_qh_few<CPL, PT><<<nblk, kFewThreads, 0, s>>>(L.eptr, L.pins, L.w, pool, K, LPR, L.m,
                                                         partial, sbuf, longseg, st.n_big, ext);
  else
    k_score_qh<CPL, PT><<<nblk, kThreads, 0, s>>>(L.eptr, L.pins, L.w, pool, K, LPR, L.m, partial,
                                                  sbuf, longseg, st.n_big, ext);
  HEF_LAUNCH_CHECK();
  }
  {
  TimedScope ts(kStScoreReduce, s);
  HEF_TRY(reduce_cols_f64(partial, nblk, K, qh, s));
  }
  TimedScope ts(kStScoreR, s);
  k_score_r<CPL><<<nblk, kThreads, 0, s>>>(sbuf, K, LPR, L.m, qh, R);
  HEF_LAUNCH_CHECK();
  return HEF_OK;
}

}  // namespace

size_t score_ws_bytes(int64_t m, int K) {
  Arena a;
  a.take<double>(cdiv(std::max<int64_t>(m, 1), kEdgesPerBlk) * K);
  a.take<float>(std::max<int64_t>(m, 1) * K);
  return a.mark();
}

hef_status score_pool(const Level &L, const Structure &st, const void *pool, int pool_type, int K,
                      double *qh, float *R, void *ext, Arena &ws, hipStream_t s, float *keep_s) {
  if (K > 512) return HEF_ERR_UNSUPPORTED;
  if (L.m == 0) return HEF_OK;
  const int64_t nblk = cdiv(L.m, kEdgesPerBlk);
  const size_t mk = ws.mark();
  double *partial = ws.take<double>(nblk * K);
  float *sbuf = keep_s ? keep_s : ws.take<float>(int64_t(L.m) * K);
  HEF_WS_CHECK(ws);
  // the shortest hyperedge taken as long: more than kSmallSeg pins (those of
  // the structure's list), or more where nnz / longseg + 1 pairs of rows
  // would not fit ext's oct_rows(n) rows
  int64_t longseg = kSmallSeg;
  while (2 * (L.nnz / longseg + 1) > oct_rows(L.n)) longseg *= 2;
  hef_status rc;
  const bool wide = K > 256;
  if (pool_type == kPoolF32)
    rc = wide ? score_t<8, kPoolF32>(L, st, pool, K, qh, R, partial, sbuf, nblk, int(longseg), ext, s)
              : score_t<4, kPoolF32>(L, st, pool, K, qh, R, partial, sbuf, nblk, int(longseg), ext, s);
  else if (pool_type == kPoolF64)
    rc = wide ? score_t<8, kPoolF64>(L, st, pool, K, qh, R, partial, sbuf, nblk, int(longseg), ext, s)
              : score_t<4, kPoolF64>(L, st, pool, K, qh, R, partial, sbuf, nblk, int(longseg), ext, s);
  else
    rc = wide ? score_t<8, kPoolBF16>(L, st, pool, K, qh, R, partial, sbuf, nblk, int(longseg), ext, s)
              : score_t<4, kPoolBF16>(L, st, pool, K, qh, R, partial, sbuf, nblk, int(longseg), ext, s);
  ws.reset(mk);
  return rc;
}

}  // namespace hef
