// Resistance-based vertex-pair rating (Section III-E, Eq. (17)): for every
// node p and every node q sharing a hyperedge with it,
//   r(p, q) = sum over hyperedges e holding both of  w(e) / (R_e - shift),
// the rating function of Eq. (7) with the hyperedge cardinality term
// replaced by the effective resistance R_e.  Reading of the printed
// denominator: with shift = 0 the whole cardinality term |e| - 1 of Eq. (7)
// becomes R_e, so heavy hyperedges of low resistance rate high, as the text
// asks; shift = 1 gives the printed R_e - 1 literally (negative for every
// hyperedge with w(e) >= 1, since R_e <= 1/w(e)).  A hyperedge whose
// denominator is exactly 0 adds nothing.  Output per node: the neighbour of
// largest rating (ties to the smallest id) and that rating, or -1 and 0 for
// a node without neighbours.
//
// Layout (deterministic: no floating-point atomics, every sum in ascending
// hyperedge order).  A group of lanes takes one node p and keeps a hash table
// q -> r(p, q) in LDS.  It walks p's hyperedges in ascending order; within a
// hyperedge the q are distinct, so its lanes add to distinct entries and
// each entry receives its terms in ascending hyperedge order.  The table's
// largest entry (ties to the smallest q) is p's result: nothing is sorted
// and no (p, q, e) triple is stored.  bound(p) = sum over the hyperedges of
// p of (|e| - 1), at least the number of distinct q, selects the group:
//   up to 64     16 lanes, 128 entries   (16 nodes per workgroup);
//   up to 512    a wave, 1024 entries    (single-wave workgroups);
//   above        256 threads, 4096 entries, in passes over hash classes of
//                the q when they do not fit at once (k_rate_big);
//   above, in kHubDeg or more hyperedges: waves of 1024 entries, each for its
//                share of the hash classes (rate_unit).
// Earlier every triple was emitted and sorted by q, then by p (six radix
// passes per million triples), and one thread per node walked its triples
// through two indirections: 9.9 ms for the 16M triples of a 200k-node
// netlist, the node walk itself bound by the longest node's serial chain.  Now
// 0.6 ms: bound by the latency of the segment and pin loads of the middle and
// big classes.
#include <cmath>

#include "prims.hpp"
#include "rating.hpp"
#include "structure.hpp"

namespace hef {
namespace {

constexpr int kRT = 256;
constexpr int kRateSmall = 64, kRateMid = 512;  // largest bound(p) of a class
constexpr int kRateNG = 16;                     // nodes per workgroup of k_rate_small
constexpr int kRateBigT = 4096;                 // table of the big class
constexpr int kRateFill = kRateBigT * 3 / 4;    // entries a pass aims at

// A node of many hyperedges (a hub) is the work of several waves.  Each walks
// all of the node's hyperedges, in order and without a barrier, and keeps the q
// of its own hash classes.  One workgroup that takes the classes one after the
// other, with a barrier behind every hyperedge, is quadratic in the node's
// degree: 6.0 / 58.8 / 861 ms a call with one node of the 200k in 3000 / 10000 /
// 40000 hyperedges of 4 pins, now 1.3 / 3.5 / 13.5.  From 256 hyperedges on
// the waves are faster even with one class (one node in 300 hyperedges, 447
// and 403 us).
constexpr int kHubDeg = 256;
constexpr int kUnitT = kRateBigT / (kRT / 64);  // a wave's table
constexpr int kUnitBits = 10;
constexpr int kUnitFill = kUnitT * 3 / 4;       // entries a class aims at
constexpr int kUnitEdges = 16;                  // least hyperedges of a node per wave
static_assert(1 << kUnitBits == kUnitT, "table size");

// Unit u of 1 << lu of hub p: the classes [u, u + 1) << (cb - lu) of 1 << cb;
// `first` is the place of the hub's unit 0.
struct RateUnit {
  int32_t p, first, u, lu_cb;
};
// The units' results, and how many of a hub's units have stored theirs (at the
// hub's first place).
struct RateHubs {
  int32_t *n_units;
  RateUnit *unit;
  int32_t *q, *done;
  unsigned long long *r;
};

// flag |= 1 if an R value is not finite
__global__ void k_rate_check(const float *__restrict__ R, int64_t m, int32_t *__restrict__ flag) {
  const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e < m && !isfinite(R[e])) atomicOr(flag, 1);
}

// Multiplication by an odd constant is a bijection of the 32-bit integers:
// its top bits index a table, other bits split the q into classes.
__device__ __forceinline__ uint32_t rate_hash(int32_t q) { return uint32_t(q) * 2654435769u; }

// The entry of q in a table of T keys (-1: free), claimed if absent; -1 when
// the table is full.
template <int T>
__device__ __forceinline__ int rate_slot(int32_t *key, int32_t q) {
  uint32_t h = rate_hash(q) >> (32 - __builtin_ctz(T));
  for (int t = 0; t < T; ++t) {
    int32_t k = key[h];
    if (k == -1) k = atomicCAS(&key[h], -1, q);
    if (k == -1 || k == q) return int(h);
    h = (h + 1) & (T - 1);
  }
  return -1;
}

// w(e) / (R_e - shift), 0 for a zero denominator
__device__ __forceinline__ double rate_term(const float *w, const float *R, double shift,
                                            int32_t e) {
  const double den = double(R[e]) - shift;
  return den != 0.0 ? double(w ? w[e] : 1.0f) / den : 0.0;
}

struct RateBest {
  int32_t q;
  double r;
  __device__ __forceinline__ void take(int32_t oq, double orr) {
    if (oq >= 0 && (q < 0 || orr > r || (orr == r && oq < q))) {
      q = oq;
      r = orr;
    }
  }
};

// The class of q among 1 << cb: the hash bits right below the BITS that index
// the table (cb = 0: one class).
template <int BITS>
__device__ __forceinline__ uint32_t rate_class(int32_t q, int cb) {
  return (rate_hash(q) << BITS) >> 1 >> (31 - cb);
}

// The best of a node's q (CLS: of class c among 1 << cb) by G lanes of one
// wave, the same on all of them.  Without CLS the q fit the table.  *full is set
// (to the same on all lanes) where they do not; the result is then of no use.
template <int G, int T, bool CLS>
__device__ __forceinline__ RateBest
rate_walk(int32_t p, int32_t v0, int32_t deg, int gl, const int32_t *__restrict__ eids,
          const int32_t *__restrict__ eptr, const int32_t *__restrict__ pins,
          const float *__restrict__ w, const float *__restrict__ R, double shift, int32_t *key,
          double *acc, uint32_t c, int cb, bool *full) {
  bool over = false;
  for (int i = gl; i < T; i += G) {
    key[i] = -1;
    acc[i] = 0.0;
  }
  wave_sync();
  for (int32_t t0 = 0; t0 < deg; t0 += G) {
    // G hyperedges' segments and terms at once, then one hyperedge at a time
    int32_t ea = 0, eb = 0;
    double et = 0.0;
    if (t0 + gl < deg) {
      const int32_t e = eids[v0 + t0 + gl];
      ea = eptr[e];
      eb = eptr[e + 1];
      et = rate_term(w, R, shift, e);
    }
    // (the first G pins of the next hyperedge load during the current one; p
    // stands for no pin)
    const int nt = deg - t0 < G ? int(deg - t0) : G;
    int32_t a = __shfl(ea, 0, G), b = __shfl(eb, 0, G);
    int32_t qn = a + gl < b ? pins[a + gl] : p;
    for (int t = 0; t < nt; ++t) {
      const double term = __shfl(et, t, G);
      const int32_t b0 = b;
      int64_t j = int64_t(a) + gl;
      int32_t q = qn;
      if (t + 1 < nt) {
        a = __shfl(ea, t + 1, G);
        b = __shfl(eb, t + 1, G);
        qn = a + gl < b ? pins[a + gl] : p;
      }
      while (j < b0) {
        const int32_t q1 = j + G < b0 ? pins[j + G] : p;
        if (q != p && (!CLS || rate_class<__builtin_ctz(T)>(q, cb) == c)) {
          const int h = rate_slot<T>(key, q);
          if (h >= 0) acc[h] += term;
          else over = true;
        }
        q = q1;
        j += G;
      }
      wave_sync();
    }
    if (CLS && __ballot(over)) break;
  }
  RateBest bst{-1, 0.0};
  if (CLS) {
    static_assert(!CLS || G == 64, "a whole wave");
    *full = __ballot(over) != 0;
    if (*full) return bst;
  }
  for (int i = gl; i < T; i += G) bst.take(key[i], acc[i]);
#pragma unroll
  for (int off = G / 2; off > 0; off >>= 1) {
    const int32_t oq = __shfl_xor(bst.q, off, G);
    const double orr = __shfl_xor(bst.r, off, G);
    bst.take(oq, orr);
  }
  return bst;
}

__device__ __forceinline__ void rate_store(int32_t p, const RateBest &b,
                                           int32_t *__restrict__ best,
                                           double *__restrict__ rating) {
  best[p] = b.q;
  rating[p] = b.q < 0 ? 0.0 : b.r;
}

// One node of the classes that fit their table: G lanes of one wave.
// bound is the same on all G lanes and at most T / 2.
template <int G, int T>
__device__ __forceinline__ void
rate_node(int32_t p, int32_t v0, int32_t deg, int gl, const int32_t *__restrict__ eids,
          const int32_t *__restrict__ eptr, const int32_t *__restrict__ pins,
          const float *__restrict__ w, const float *__restrict__ R, double shift, int32_t *key,
          double *acc, int32_t *__restrict__ best, double *__restrict__ rating) {
  const RateBest b = rate_walk<G, T, false>(p, v0, deg, gl, eids, eptr, pins, w, R, shift, key,
                                            acc, 0u, 0, nullptr);
  if (gl == 0) rate_store(p, b, best, rating);
}

// One unit of a hub, by a wave: the best q of its classes.  A class that fills
// the table is halved, and so are those after it; the hash is a bijection, so
// this ends.  The wave that stores the last of the hub's results takes the
// best of them.
__device__ void rate_unit(const RateHubs &H, int32_t i, int lane, const int32_t *__restrict__ vptr,
                          const int32_t *__restrict__ eids, const int32_t *__restrict__ eptr,
                          const int32_t *__restrict__ pins, const float *__restrict__ w,
                          const float *__restrict__ R, double shift, int32_t *key, double *acc,
                          int32_t *__restrict__ best, double *__restrict__ rating) {
  const RateUnit x = H.unit[i];
  const int lu = x.lu_cb >> 8;
  int cb = x.lu_cb & 255;
  const int32_t v0 = vptr[x.p], deg = vptr[x.p + 1] - v0;
  RateBest bst{-1, 0.0};
  uint32_t c = uint32_t(x.u) << (cb - lu), end = uint32_t(x.u + 1) << (cb - lu);
  while (c < end) {
    bool full = false;
    const RateBest b = rate_walk<64, kUnitT, true>(x.p, v0, deg, lane, eids, eptr, pins, w, R,
                                                   shift, key, acc, c, cb, &full);
    wave_sync();
    if (full) {
      ++cb;
      c *= 2;
      end *= 2;
      continue;
    }
    bst.take(b.q, b.r);
    ++c;
  }
  int32_t before = 0;
  if (lane == 0) {
    __hip_atomic_store(&H.q[i], bst.q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&H.r[i], __builtin_bit_cast(unsigned long long, bst.r), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    before = __hip_atomic_fetch_add(&H.done[x.first], 1, __ATOMIC_ACQ_REL,
                                    __HIP_MEMORY_SCOPE_AGENT);
  }
  before = __builtin_amdgcn_readfirstlane(before);
  if (before != (1 << lu) - 1) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  RateBest all{-1, 0.0};
  for (int k = lane; k < 1 << lu; k += 64) {
    const int32_t q = __hip_atomic_load(&H.q[x.first + k], __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long r = __hip_atomic_load(&H.r[x.first + k], __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT);
    all.take(q, __builtin_bit_cast(double, r));
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const int32_t oq = __shfl_xor(all.q, off, 64);
    const double orr = __shfl_xor(all.r, off, 64);
    all.take(oq, orr);
  }
  if (lane == 0) rate_store(x.p, all, best, rating);
}

// Every node: bound(p), then the node itself (small class), its units (hub) or
// its place in the workgroup's own slice of a list: mid[NG blk ..] and
// big[NG blk ..], their lengths in counts[2 blk], counts[2 blk + 1].  (One counter per list served
// 60k nodes of a 200k-node netlist one after the other: 473 us, now
// 96 us.)
__global__ void __launch_bounds__(kRT)
k_rate_small(const int32_t *__restrict__ vptr, const int32_t *__restrict__ eids,
             const int32_t *__restrict__ eptr, const int32_t *__restrict__ pins,
             const float *__restrict__ w, const float *__restrict__ R, double shift, int32_t n,
             int32_t *__restrict__ mid, int32_t *__restrict__ big, int32_t *__restrict__ counts,
             const RateHubs H, int32_t *__restrict__ best, double *__restrict__ rating) {
  constexpr int G = 16, T = 2 * kRateSmall, NG = kRateNG;
  static_assert(NG * G == kRT, "lanes");
  __shared__ int32_t key[NG][T];
  __shared__ double acc[NG][T];
  __shared__ int32_t cls[NG];  // 0 small, 1 middle, 2 big, 3 hub
  const int gi = threadIdx.x / G, gl = threadIdx.x % G;
  const int64_t p0 = int64_t(blockIdx.x) * NG, p = p0 + gi;
  const int32_t v0 = p < n ? vptr[p] : 0, deg = p < n ? vptr[p + 1] - v0 : 0;
  int32_t bound = 0;
  for (int32_t t = gl; t < deg; t += G) {
    const int32_t e = eids[v0 + t];
    bound += eptr[e + 1] - eptr[e] - 1;
  }
#pragma unroll
  for (int off = G / 2; off > 0; off >>= 1) bound += __shfl_xor(bound, off, G);
  const bool hub = bound > kRateMid && deg >= kHubDeg;
  if (gl == 0) cls[gi] = bound <= kRateSmall ? 0 : bound <= kRateMid ? 1 : hub ? 3 : 2;
  if (hub) {
    const int32_t most = bound < n - 1 ? bound : n - 1;  // distinct q
    int cb = 0, lu = 0;
    while (cb < 32 - kUnitBits && (most >> cb) > kUnitFill) ++cb;
    while (lu < cb && (deg >> (lu + 1)) >= kUnitEdges) ++lu;
    int32_t first = 0;
    if (gl == 0) {
      first = atomicAdd(H.n_units, 1 << lu);
      H.done[first] = 0;
    }
    first = __shfl(first, 0, G);
    for (int32_t u = gl; u < 1 << lu; u += G)
      H.unit[first + u] = RateUnit{int32_t(p), first, u, (lu << 8) | cb};
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    int32_t *list = threadIdx.x == 0 ? mid : big;
    int32_t c = 0;
    for (int q = 0; q < NG; ++q)
      if (cls[q] == int(threadIdx.x) + 1) list[p0 + c++] = int32_t(p0 + q);
    counts[2 * int64_t(blockIdx.x) + threadIdx.x] = c;
  }
  if (p >= n || bound > kRateSmall) return;
  rate_node<G, T>(int32_t(p), v0, deg, gl, eids, eptr, pins, w, R, shift, key[gi], acc[gi], best,
                  rating);
}

// kMidSplit single-wave workgroups share a slice, so that a table is given
// back as soon as its wave is done.
constexpr int kMidSplit = 4;

__global__ void __launch_bounds__(64)
k_rate_mid(const int32_t *__restrict__ list, const int32_t *__restrict__ counts,
           const int32_t *__restrict__ vptr, const int32_t *__restrict__ eids,
           const int32_t *__restrict__ eptr, const int32_t *__restrict__ pins,
           const float *__restrict__ w, const float *__restrict__ R, double shift,
           int32_t *__restrict__ best, double *__restrict__ rating) {
  constexpr int T = 2 * kRateMid;
  __shared__ int32_t key[T];
  __shared__ double acc[T];
  const int64_t slice = blockIdx.x / kMidSplit;
  const int32_t cnt = counts[2 * slice];
  for (int32_t i = blockIdx.x % kMidSplit; i < cnt; i += kMidSplit) {
    const int32_t p = list[slice * kRateNG + i];
    const int32_t v0 = vptr[p], deg = vptr[p + 1] - v0;
    rate_node<64, T>(p, v0, deg, int(threadIdx.x), eids, eptr, pins, w, R, shift, key, acc, best,
                     rating);
    wave_sync();
  }
}

// The units of the hubs, a wave each; then a workgroup per node of the big
// class.  The q are split into 2^cb classes by bits of their
// hash below the table's; pass c takes class c.  cb starts so that a pass
// meets about kRateFill distinct q at most and grows by one, restarting the
// class sweep, whenever a table fills up; the hash is a bijection, so the
// classes separate any set of q and the sweep ends.
__global__ void __launch_bounds__(kRT)
k_rate_big(const int32_t *__restrict__ list, const int32_t *__restrict__ counts,
           const int32_t *__restrict__ vptr, const int32_t *__restrict__ eids,
           const int32_t *__restrict__ eptr, const int32_t *__restrict__ pins,
           const float *__restrict__ w, const float *__restrict__ R, double shift, int32_t n,
           int32_t nslice, const RateHubs H, int32_t *__restrict__ best,
           double *__restrict__ rating) {
  constexpr int T = kRateBigT;
  constexpr int kTableBits = 12;  // the hash bits that index the table
  static_assert(1 << kTableBits == T, "table size");
  __shared__ int32_t key[T];
  __shared__ double acc[T];
  __shared__ int32_t full;
  __shared__ int32_t rq[kRT / 64];
  __shared__ double rr[kRT / 64];
  __shared__ long long bsum;
  __shared__ int32_t ea[kRT], eb[kRT];  // a batch of the node's hyperedges
  __shared__ double et[kRT];
  const int tid = threadIdx.x;
  {
    const int wv = tid >> 6;
    const int32_t nu = *H.n_units;
    for (int32_t i = int32_t(wave_index()); i < nu; i += gridDim.x * (kRT / 64))
      rate_unit(H, i, tid & 63, vptr, eids, eptr, pins, w, R, shift, key + wv * kUnitT,
                acc + wv * kUnitT, best, rating);
    __syncthreads();
  }
  // (slice, entry) pairs in turn: workgroup b takes slots b, b + grid, ... of
  // the nslice x kRateNG slots (the big nodes of one slice go to different
  // workgroups); kRT slots are looked up together, those past a slice's
  // length are skipped
  __shared__ int32_t found[kRT];
  __shared__ int32_t nfound;
  const int64_t slots = int64_t(nslice) * kRateNG;
  for (int64_t i0 = blockIdx.x; i0 < slots; i0 += int64_t(gridDim.x) * kRT) {
  if (tid == 0) nfound = 0;
  __syncthreads();
  {
    const int64_t i = i0 + int64_t(tid) * gridDim.x;
    const int64_t slice = i % nslice, entry = i / nslice;
    if (i < slots && entry < counts[2 * slice + 1])
      found[atomicAdd(&nfound, 1)] = list[slice * kRateNG + entry];
  }
  __syncthreads();
  const int nf = nfound;
  for (int f = 0; f < nf; ++f) {
    const int32_t p = found[f];
    const int32_t v0 = vptr[p], deg = vptr[p + 1] - v0;
    if (tid == 0) bsum = 0;
    __syncthreads();
    long long my = 0;
    for (int32_t t = tid; t < deg; t += kRT) {
      const int32_t e = eids[v0 + t];
      my += eptr[e + 1] - eptr[e] - 1;
    }
    atomicAdd(reinterpret_cast<unsigned long long *>(&bsum), (unsigned long long)my);
    __syncthreads();
    const int64_t most = bsum < n - 1 ? int64_t(bsum) : int64_t(n - 1);  // distinct q
    int cb = 0;
    while (cb < 32 - kTableBits && (most >> cb) > kRateFill) ++cb;
    RateBest bst{-1, 0.0};
    for (uint32_t c = 0; c < (1u << cb);) {
      for (int k = tid; k < T; k += kRT) {
        key[k] = -1;
        acc[k] = 0.0;
      }
      if (tid == 0) full = 0;
      __syncthreads();
      for (int32_t t0 = 0; t0 < deg; t0 += kRT) {
        // kRT hyperedges' segments and terms side by side, then one at a time
        const int nt = deg - t0 < kRT ? int(deg - t0) : kRT;
        if (tid < nt) {
          const int32_t e = eids[v0 + t0 + tid];
          ea[tid] = eptr[e];
          eb[tid] = eptr[e + 1];
          et[tid] = rate_term(w, R, shift, e);
        }
        __syncthreads();
        for (int t = 0; t < nt; ++t) {
          const int32_t a = ea[t], b = eb[t];
          const double term = et[t];
          for (int64_t j = a + tid; j < b; j += 4 * kRT) {
            int32_t q[4];  // four pins' loads together; p stands for no pin
#pragma unroll
            for (int u = 0; u < 4; ++u) q[u] = j + u * kRT < b ? pins[j + u * kRT] : p;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              if (q[u] != p && rate_class<kTableBits>(q[u], cb) == c) {
                const int h = rate_slot<T>(key, q[u]);
                if (h >= 0) acc[h] += term;
                else full = 1;
              }
            }
          }
          __syncthreads();
        }
      }
      if (full) {  // (the same on every thread)
        // halve the classes and start over
        ++cb;
        c = 0;
        bst = RateBest{-1, 0.0};
        __syncthreads();
        continue;
      }
      for (int k = tid; k < T; k += kRT) bst.take(key[k], acc[k]);
      __syncthreads();
      ++c;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const int32_t oq = __shfl_xor(bst.q, off, 64);
      const double orr = __shfl_xor(bst.r, off, 64);
      bst.take(oq, orr);
    }
    if ((tid & 63) == 0) {
      rq[tid >> 6] = bst.q;
      rr[tid >> 6] = bst.r;
    }
    __syncthreads();
    if (tid == 0) {
      for (int k = 1; k < kRT / 64; ++k) bst.take(rq[k], rr[k]);
      best[p] = bst.q;
      rating[p] = bst.q < 0 ? 0.0 : bst.r;
    }
    __syncthreads();
  }
  }
}

inline unsigned gr(int64_t n) { return unsigned(std::max<int64_t>(1, cdiv(n, kRT))); }

}  // namespace

size_t rating_bytes(int64_t n, int64_t m, int64_t nnz) {
  Arena a;
  Structure st;
  structure_carve(a, n, m, nnz, st);
  a.take<int32_t>(4);
  a.take<int32_t>(n + kRateNG);  // the lists of the middle and the big class
  a.take<int32_t>(n + kRateNG);
  a.take<int32_t>(2 * cdiv(n, kRateNG) + 2);
  return a.mark() + structure_build_ws(n, m, nnz) + 4096;
}

hef_status rating_run(const Level &L, const float *R, float shift, int32_t *best, double *rating,
                      void *ws, size_t ws_bytes, hipStream_t s) {
  const int64_t n = L.n, m = L.m, nnz = L.nnz;
  Arena a;
  a.base = static_cast<char *>(ws);
  a.cap = ws_bytes;
  Structure st;
  structure_carve(a, n, m, nnz, st);
  int32_t *flags = a.take<int32_t>(4);
  int32_t *mid = a.take<int32_t>(n + kRateNG), *big = a.take<int32_t>(n + kRateNG);
  int32_t *counts = a.take<int32_t>(2 * cdiv(n, kRateNG) + 2);
  HEF_WS_CHECK(a);
  int32_t bad = 0;
  HEF_TRY(validate_device(L, flags, &bad, s, 2));
  if (bad) {
    set_error("invalid hypergraph (code %d)", bad);
    return HEF_ERR_INVALID_HYPERGRAPH;
  }
  if (m > 0) {  // (flags[0] is still 0)
    k_rate_check<<<gr(m), kRT, 0, s>>>(R, m, flags);
    HEF_LAUNCH_CHECK();
    int32_t f = 0;
    HEF_HIP(hipMemcpyAsync(&f, flags, sizeof(int32_t), hipMemcpyDeviceToHost, s));
    HEF_HIP(hipStreamSynchronize(s));
    if (f) {
      set_error("a resistance is not finite");
      return HEF_ERR_INVALID_ARGUMENT;
    }
  }
  if (n == 0) return HEF_OK;
  TimedScope ts(kStRating, s);
  HEF_TRY(structure_build(L, st, a, s));
  const double sh = double(shift);
  // (the lists' lengths stay on the device; a hub has at most a unit per
  // kUnitEdges hyperedges, and the structure's scratch is free again)
  const int64_t units = nnz / kUnitEdges + 1;
  RateHubs H;
  H.n_units = flags + 1;
  H.unit = a.take<RateUnit>(units);
  H.q = a.take<int32_t>(units);
  H.done = a.take<int32_t>(units);
  H.r = a.take<unsigned long long>(units);
  HEF_WS_CHECK(a);
  const unsigned nslice = unsigned(cdiv(n, kRateNG));
  k_rate_small<<<nslice, kRT, 0, s>>>(st.vptr, st.eids, L.eptr, L.pins, L.w, R, sh, int32_t(n),
                                      mid, big, counts, H, best, rating);
  HEF_LAUNCH_CHECK();
  k_rate_mid<<<nslice * kMidSplit, 64, 0, s>>>(mid, counts, st.vptr, st.eids, L.eptr, L.pins, L.w, R, sh,
                                    best, rating);
  HEF_LAUNCH_CHECK();
  k_rate_big<<<std::min<unsigned>(nslice * kRateNG, 4096u), kRT, 0, s>>>(
      big, counts, st.vptr, st.eids, L.eptr, L.pins, L.w, R, sh, int32_t(n), int32_t(nslice), H,
      best, rating);
  HEF_LAUNCH_CHECK();
  HEF_HIP(hipStreamSynchronize(s));
  return HEF_OK;
}

}  // namespace hef
