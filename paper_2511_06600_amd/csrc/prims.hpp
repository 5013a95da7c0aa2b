// Device primitives used by several stages: exclusive scan, stable LSD radix
// sort of (key, value) pairs, stream compaction.  All are deterministic.
#pragma once

#include <array>

#include "common.hpp"

namespace hef {

// Workspace bytes for a scan over `n` elements (three of them together).
size_t scan_ws_bytes(int64_t n);
// out[i] = sum_{j<i} in[j]; out[n] = total (out has n+1 entries).
// `in` and `out` may alias.
hef_status exclusive_scan_i32(const int32_t *in, int32_t *out, int64_t n,
                              Arena &ws, hipStream_t s);

// Three scans of n items each in the launches of one; out[i] holds n entries
// and totals[i] the sum (consecutive, so that one copy reads them).
hef_status exclusive_scan3_i32(const std::array<const int32_t *, 3> &in,
                               const std::array<int32_t *, 3> &out, int32_t *totals, int64_t n,
                               Arena &ws, hipStream_t s);

// Workspace bytes for radix_sort_pairs over `n` items (about 2 n bytes up to
// 2^20 items, n / 2 above; n / 4 with `lean`, which keeps to large tiles and
// 8-bit digits): with n just above 2^20 less than with n just below, so a
// workspace that also sorts fewer items is sized by radix_ws_upto.
size_t radix_ws_bytes(int64_t n, bool lean = false);
// Workspace bytes for sorts of any number of items up to n.
size_t radix_ws_upto(int64_t n);
// Stable LSD radix sort of n (key, value) pairs by the low `bits` bits of
// the keys, 8 or 9 bits a pass: src -> out, with tmp as the other ping-pong buffer
// (both n items; the last pass writes out, so nothing is copied at the end).
// src may be buffers of its own (left as they are), or the buffers that the
// first pass does not write: out when the number of passes is even, tmp when
// it is odd (radix_src picks them).
hef_status radix_sort_pairs(const uint32_t *src_k, const uint32_t *src_v, uint32_t *tmp_k,
                            uint32_t *tmp_v, uint32_t *out_k, uint32_t *out_v, int64_t n,
                            int bits, Arena &ws, hipStream_t s, bool lean = false);
inline int radix_passes(int bits, bool lean = false) {
  return lean ? (bits + 7) / 8 : (bits + 8) / 9;
}
template <class T>
inline T radix_src(int bits, T tmp, T out, bool lean = false) {
  return radix_passes(bits, lean) % 2 == 0 ? out : tmp;
}

// idx_out[0..count) = ascending indices i < n with flag[i] = 1 (flags are 0
// or 1), pos[i] = the number of set flags before i; *count_dev = count.
hef_status scan_compact_flags(const int32_t *flag, int32_t *pos, int32_t *idx_out,
                              int32_t *count_dev, int64_t n, Arena &ws, hipStream_t s);

// out[c] = sum_r in[r * ncols + c] (float64) in a fixed order that does not
// depend on timing: 32 row lanes per column each sum every 32nd row (eight
// interleaved accumulators), then a fixed tree over the lanes.
hef_status reduce_cols_f64(const double *in, int64_t nrows, int64_t ncols, double *out,
                           hipStream_t s);
// Two independent reduce_cols_f64 (same ncols) in one launch.
hef_status reduce_cols_f64_pair(const double *in0, int64_t nrows0, double *out0,
                                const double *in1, int64_t nrows1, double *out1, int64_t ncols,
                                hipStream_t s);

// The column sums above for a workgroup of 256 QG threads on 8 columns: thread
// (column, row lane l < 32, part < QG) adds the rows l + 32 (8 i + q) of its
// 8 / QG accumulators q, i ascending, eight loads in flight; the accumulators
// are added pairwise and the row lanes by halves, so every QG gives the same
// bits.  `ok`: the thread's column c is inside.  The sums are returned on
// threads 0 .. 7.
template <int QG>
struct ColSum {
  static constexpr int kLds = 32 * 9 * QG;
  static constexpr int kQ = 8 / QG;  // accumulators per thread
  static __device__ __forceinline__ double run(const double *__restrict__ in, int64_t nrows,
                                               int64_t ncols, int64_t c, bool ok, double *red) {
    constexpr int kI = QG;  // row groups per round
    const int cl = threadIdx.x & 7, rl = (threadIdx.x >> 3) & 31, part = threadIdx.x >> 8;
    double acc[kQ] = {};
    if (ok) {
      for (int64_t r = rl + 32 * kQ * part; r < nrows; r += 256 * kI) {
        double t[kI][kQ];
#pragma unroll
        for (int i = 0; i < kI; ++i)
#pragma unroll
          for (int q = 0; q < kQ; ++q) {
            const int64_t rr = r + 256 * i + 32 * q;
            t[i][q] = in[(rr < nrows ? rr : r) * ncols + c];
          }
#pragma unroll
        for (int i = 0; i < kI; ++i)
#pragma unroll
          for (int q = 0; q < kQ; ++q)
            if (r + 256 * i + 32 * q < nrows) acc[q] += t[i][q];
      }
    }
    double v = 0.0;
    if constexpr (QG == 1) v = ((acc[0] + acc[1]) + (acc[2] + acc[3])) +
                               ((acc[4] + acc[5]) + (acc[6] + acc[7]));
    else v = acc[0] + acc[1];
    static_assert(QG == 1 || QG == 4, "parts");
    red[(part * 32 + rl) * 9 + cl] = v;
    __syncthreads();
    double x = 0.0;
    if (threadIdx.x < 64) {
      // lane (column, k < 8) takes row lanes k, k + 8, k + 16, k + 24
      double y[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int at = ((threadIdx.x >> 3) + 8 * k) * 9 + cl;
        if constexpr (QG == 1) y[k] = red[at];
        else y[k] = (red[at] + red[32 * 9 + at]) + (red[2 * 32 * 9 + at] + red[3 * 32 * 9 + at]);
      }
      x = (y[0] + y[2]) + (y[1] + y[3]);
#pragma unroll
      for (int off = 32; off >= 8; off >>= 1) x += __shfl_down(x, off, 64);
    }
    return x;
  }
};

// Zeroes `bytes` bytes at p on stream s with a fill kernel rather than
// hipMemsetAsync, so that a caller capturing the stream into a HIP graph
// records kernel nodes only.
hef_status zero_async(void *p, size_t bytes, hipStream_t s);

inline int bits_for(int64_t maxval) {
  int b = 1;
  while (b < 32 && (int64_t(1) << b) <= maxval) ++b;
  return b;
}

// A wave takes 64 consecutive hyperedges, lane l the hyperedge e0 + l, whose
// pins [a0, an) are contiguous: the lanes then walk that range side by side
// (coalesced), each finding the hyperedge of its position by a search over
// the lanes' starts.  One thread per hyperedge walking its own pins is a
// serial chain of |e| dependent steps: with a 2000-pin hyperedge the
// validation took 150 us at 756k pins, and 205 us at 7.9M.
__device__ __forceinline__ int lane_of_pos(int32_t start, int32_t j, int cnt) {
  int lo = 0, hi = cnt;  // last lane < cnt whose start is <= j
#pragma unroll
  for (int s = 0; s < 6; ++s) {
    const int mid = (lo + hi) >> 1;
    const int32_t sm = __shfl(start, mid, 64);
    const bool up = hi - lo > 1 && sm <= j;
    lo = up ? mid : lo;
    hi = (hi - lo > 1 && !up) ? mid : hi;
  }
  return lo;
}

// Such a wave walks at most kSpan positions.  Where 64 hyperedges have more,
// the rest goes to waves of its own, span_extra(nnz) of them ahead of the
// others: extra wave x takes what lies in positions [(x + 1) kSpan,
// (x + 2) kSpan) of the 64 hyperedges that hold the first of these positions,
// past their first kSpan pins (the rest of any later 64 starts behind them).
// With short hyperedges only, an extra wave ends after its search.  200
// hyperedges of 5000 pins, four waves' work otherwise: the validation 2600 us
// to 38 us, the labels of a partition 3070 us to 44 us.
constexpr int kSpan = 4096;
inline int64_t span_extra(int64_t nnz) { return nnz > 0 ? (nnz - 1) / kSpan : 0; }
// Workgroups of 256 threads of a walk over m hyperedges.
inline int64_t span_blocks(int64_t m, int64_t nnz) {
  return cdiv(span_extra(nnz) + cdiv(m, 64), 4);
}

struct PinSpan {
  int64_t e0;   // first of the 64 hyperedges (m or more: no such wave)
  int64_t pos;  // first position of an extra wave's span, -1 for the others
  // the span's part [lo, hi) of the 64 hyperedges' positions [j0, j1)
  __device__ __forceinline__ int64_t lo(int64_t j0) const {
    return pos < 0 ? j0 : pos > j0 + kSpan ? pos : j0 + kSpan;
  }
  __device__ __forceinline__ int64_t hi(int64_t j0, int64_t j1) const {
    const int64_t end = (pos < 0 ? j0 : pos) + kSpan;
    return end < j1 ? end : j1;
  }
};

// This wave among the waves of its launch, in a scalar register.
__device__ __forceinline__ int64_t wave_index() {
  return int64_t(blockIdx.x) * (blockDim.x >> 6) +
         __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
}

// The span of a wave (eptr need not be valid: only its entries 0, 64, ... are
// read, and the search ends whatever they hold).
__device__ __forceinline__ PinSpan pin_span(const int32_t *__restrict__ eptr, int64_t m,
                                            int64_t wave, int64_t extra) {
  if (wave >= extra) return {64 * (wave - extra), -1};
  const int64_t pos = (wave + 1) * kSpan;
  int64_t lo = 0, hi = (m + 63) / 64;
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (eptr[64 * mid] <= pos) lo = mid; else hi = mid;
  }
  return {64 * lo, pos};
}

}  // namespace hef
