// One level's structure: validation, CSC incidence, expansion scales and the
// lists of long segments (Section III-A, star and clique expansions; the
// normalised adjacency of each is applied implicitly by the SpMM kernels).
#include <cmath>

#include "prims.hpp"
#include "structure.hpp"

namespace hef {
namespace {

__global__ void __launch_bounds__(256)
k_validate(const int32_t *__restrict__ eptr, const int32_t *__restrict__ pins,
           const float *__restrict__ w, int32_t n, int32_t m, int64_t nnz, int64_t extra,
           int32_t *__restrict__ flag) {
  const int lane = threadIdx.x & 63;
  const PinSpan sp = pin_span(eptr, m, wave_index(), extra);
  const int64_t e0 = sp.e0, e = e0 + lane;
  if (e0 >= m) return;
  const int cnt = m - e0 < 64 ? int(m - e0) : 64;
  // an extra wave past its hyperedges' pins (wherever they claim to lie)
  if (sp.pos >= 0 && sp.lo(eptr[e0]) >= eptr[e0 + cnt]) return;
  const bool on = lane < cnt;
  int bad = 0;
  const int64_t a = on ? eptr[e] : 0, b = on ? eptr[e + 1] : 2;
  if (on) {
    if (e == 0 && a != 0) bad |= 1;
    if (e == m - 1 && b != nnz) bad |= 1;
    if (a < 0 || b > nnz || b - a < 2) bad |= 2;
    if (w) {
      const float x = w[e];
      if (!(x > 0.0f) || !isfinite(x)) bad |= 8;
    }
  }
  if (__ballot(bad & 3) == 0) {
    // every segment of the wave lies in [0, nnz) and starts where the one
    // before it ends
    const int32_t a32 = int32_t(a);
    const int32_t j0 = __shfl(a32, 0, 64);
    const int32_t j1 = int32_t(sp.hi(j0, __shfl(int32_t(b), cnt - 1, 64)));
    for (int64_t jb = sp.lo(j0); jb < j1; jb += 64) {
      const bool in = jb + lane < j1;
      const int32_t j = in ? int32_t(jb + lane) : j1 - 1;
      const int32_t p = in ? pins[j] : 0;
      const int32_t q = in && j > j0 ? pins[j - 1] : -1;
      const int32_t start = __shfl(a32, lane_of_pos(a32, j, cnt), 64);
      if (in && (p < 0 || p >= n || (j != start && p <= q))) bad |= 4;
    }
  } else if (sp.pos < 0 && on && !(bad & 3)) {
    int32_t prev = -1;
    for (int64_t j = a; j < b; ++j) {
      const int32_t p = pins[j];
      if (p < 0 || p >= n || p <= prev) {
        bad |= 4;
        break;
      }
      prev = p;
    }
  }
  if (bad) atomicOr(flag, bad);
}

// eid[j] = the hyperedge of pin position j (same walk: 36 us to about 12 us at
// 756k pins with a 2000-pin hyperedge among them, 544 us to 30 us for 200
// hyperedges of 5000 pins); also clears the list lengths of the long segments
// for the kernels after it.
__global__ void __launch_bounds__(256)
k_edge_ids(const int32_t *__restrict__ eptr, uint32_t *__restrict__ eid, int32_t m, int64_t extra,
           int32_t *__restrict__ n_big) {
  if (blockIdx.x == 0 && threadIdx.x < 2) n_big[threadIdx.x] = 0;
  const int lane = threadIdx.x & 63;
  const PinSpan sp = pin_span(eptr, m, wave_index(), extra);
  const int64_t e0 = sp.e0;
  if (e0 >= m) return;
  const int cnt = m - e0 < 64 ? int(m - e0) : 64;
  const int64_t jlo = sp.lo(eptr[e0]);
  const int32_t j1 = int32_t(sp.hi(eptr[e0], eptr[e0 + cnt]));
  if (jlo >= j1) return;
  const int32_t a = lane < cnt ? eptr[e0 + lane] : 0;
  for (int64_t jb = jlo; jb < j1; jb += 64) {
    const bool in = jb + lane < j1;
    const int32_t j = in ? int32_t(jb + lane) : j1 - 1;
    const int k = lane_of_pos(a, j, cnt);
    if (in) eid[j] = uint32_t(e0 + k);
  }
}

// vptr[v] = first position of a key >= v in the sorted pin keys (v <= n):
// position j writes the nodes in (key[j-1], key[j]] (key[-1] = -1,
// key[nnz] = n).
__global__ void k_seg_bounds(const uint32_t *__restrict__ key, int64_t nnz, int32_t n,
                             int32_t *__restrict__ vptr) {
  const int64_t j = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (j > nnz) return;
  const int64_t cur = j < nnz ? int64_t(key[j]) : int64_t(n);
  const int64_t prev = j > 0 ? int64_t(key[j - 1]) : -1;
  for (int64_t v = prev + 1; v <= cur; ++v) vptr[v] = int32_t(j);
}

// Appends the ids of a workgroup's threads with `take` to list[0 .. *count),
// one reservation per workgroup.  The long-segment lists need no order: every
// entry is handled by itself.  (Flags, their scan and a compaction are three
// launches per list.)
__device__ __forceinline__ void append_ids(bool take, int32_t id, int32_t *__restrict__ list,
                                           int32_t *__restrict__ count) {
  __shared__ int32_t n, base;
  if (threadIdx.x == 0) n = 0;
  __syncthreads();
  const int32_t at = take ? atomicAdd(&n, 1) : 0;
  __syncthreads();
  if (threadIdx.x == 0 && n > 0) base = atomicAdd(count, n);
  __syncthreads();
  if (take) list[base + at] = id;
}

// Per hyperedge: alpha_e = sqrt(w_e)/|e|, beta_e = w_e/(|e|(|e|-1)); lists
// the long ones; the float64 terms w_e/|e| and beta_e of the node sums.
__global__ void k_edge_scales(const int32_t *__restrict__ eptr, const float *__restrict__ w,
                              float *__restrict__ alpha, float *__restrict__ beta,
                              int32_t *__restrict__ big, int32_t *__restrict__ n_big,
                              double *__restrict__ tdb, double *__restrict__ tcb, int32_t m) {
  const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const int32_t sz = e < m ? eptr[e + 1] - eptr[e] : 0;
  append_ids(sz > kSmallSeg, int32_t(e), big, n_big);
  if (e >= m) return;
  const double we = w ? double(w[e]) : 1.0;
  const double k = double(sz);
  alpha[e] = float(sqrt(we) / k);
  beta[e] = float(we / (k * (k - 1.0)));
  tdb[e] = we / k;
  tcb[e] = we / (k * (k - 1.0));
}

// Per node, over its hyperedges in ascending order, in float64:
// d_b = sum w_e/|e|, cb = sum beta_e; s = d_b^-1/2, gam = s^2 cb.  A thread
// takes a node, eight loads at a time; a wave's nodes of more than kWaveSeg
// hyperedges are taken by the whole wave one after the other while they are
// few (wave_takes).
// Average over the three levels of a coarsening from 20k / 200k / 2M nodes:
// 19 / 26 / 144 us; four loads at a time without the wave 20 / 27 / 174 us
// (and 1 us more per eight hyperedges of the largest hub); the wave always, 23
// / 30 / 157 us, and from kSmallSeg on 61 / 81 / 189 us.
__global__ void __launch_bounds__(256)
k_node_scales(const int32_t *__restrict__ vptr, const int32_t *__restrict__ eids,
              const double *__restrict__ tdb, const double *__restrict__ tcb,
              float *__restrict__ s_out, float *__restrict__ gam, int32_t *__restrict__ big,
              int32_t *__restrict__ n_big, int32_t n) {
  const int64_t u = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const int lane = threadIdx.x & 63;
  const int32_t a = u < n ? vptr[u] : 0, b = u < n ? vptr[u + 1] : 0;
  append_ids(b - a > kSmallSeg, int32_t(u), big, n_big);
  const int32_t len = b - a > kWaveSeg ? b - a : 0;
  const bool lng = wave_takes(len) && len > 0;
  double db = 0.0, cb = 0.0;
  if (!lng) {
    // eight incidences' loads ahead of their sums, which run in order
    for (int32_t j = a; j < b; j += 8) {
      int32_t e[8];
      double td[8], tc[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) e[q] = eids[j + q < b ? j + q : b - 1];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        td[q] = tdb[e[q]];
        tc[q] = tcb[e[q]];
      }
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (j + q < b) {
          db += td[q];
          cb += tc[q];
        }
    }
  }
  for (uint64_t left = __ballot(lng); left != 0; left &= left - 1) {
    const int l = __ffsll(static_cast<long long>(left)) - 1;
    const int32_t la = __builtin_amdgcn_readlane(a, l), lb = __builtin_amdgcn_readlane(b, l);
    double sum[2] = {0.0, 0.0};
    for (int32_t j = la; j < lb; j += 64) {
      const int cnt = lb - j < 64 ? lb - j : 64;
      const int32_t e = eids[lane < cnt ? j + lane : lb - 1];
      const double t[2] = {tdb[e], tcb[e]};
      ordered_sums(sum, t, cnt);
    }
    if (lane == l) {
      db = sum[0];
      cb = sum[1];
    }
  }
  if (u >= n) return;
  const double sv = db > 0.0 ? 1.0 / sqrt(db) : 0.0;
  s_out[u] = float(sv);
  gam[u] = float(sv * sv * cb);
}

}  // namespace

void structure_carve(Arena &a, int64_t n, int64_t m, int64_t nnz, Structure &st) {
  st.vptr = a.take<int32_t>(n + 1);
  st.eids = a.take<int32_t>(nnz);
  st.s = a.take<float>(n);
  st.gam = a.take<float>(n);
  st.alpha = a.take<float>(m);
  st.beta = a.take<float>(m);
  st.big_e = a.take<int32_t>(m + 1);
  st.big_v = a.take<int32_t>(n + 1);
  st.n_big = a.take<int32_t>(2);
}

// Scratch of the build: the sort's buffers, then in their place the arrays
// of the scales and lists.
struct SortWs {
  uint32_t *tmp_k, *tmp_v, *out_k;
};
struct ScaleWs {
  double *tdb, *tcb;  // per-hyperedge terms of the node sums
};
static void carve_sort(Arena &a, int64_t nnz, SortWs &w) {
  w.tmp_k = a.take<uint32_t>(nnz);
  w.tmp_v = a.take<uint32_t>(nnz);
  w.out_k = a.take<uint32_t>(nnz);
}
static void carve_scale(Arena &a, int64_t m, ScaleWs &w) {
  w.tdb = a.take<double>(std::max<int64_t>(m, 1));
  w.tcb = a.take<double>(std::max<int64_t>(m, 1));
}

// The sort's histograms take up to 2 nnz bytes, nnz / 4 in the lean form;
// hypergraphs of very long hyperedges take the lean form, so that this scratch
// stays within 12 nnz + nnz / 4 + 16 m + 8 max(n, m) bytes and everything that
// fitted the static scratch still does.
static int64_t most_full(int64_t n, int64_t m) {  // pins up to which it is not lean
  return std::max<int64_t>(0, (4 * (16 * m + 8 * std::max(n, m)) - 32768) / 7);
}
static bool lean_sort(int64_t n, int64_t m, int64_t nnz) { return nnz > most_full(n, m); }

static size_t sort_bytes(int64_t nnz, size_t radix) {
  Arena a;
  SortWs w;
  carve_sort(a, nnz, w);
  return a.mark() + radix;
}

size_t structure_build_need(int64_t n, int64_t m, int64_t nnz) {
  Arena c;
  ScaleWs w;
  carve_scale(c, m, w);
  return std::max(sort_bytes(nnz, radix_ws_bytes(nnz, lean_sort(n, m, nnz))), c.mark()) + 4096;
}

size_t structure_build_ws(int64_t n, int64_t m, int64_t nnz) {
  const int64_t full = std::min(nnz, most_full(n, m));
  return std::max(structure_build_need(n, m, nnz), sort_bytes(full, radix_ws_upto(full)) + 4096);
}

hef_status validate_device(const Level &L, int32_t *flag_dev, int32_t *bad_host,
                           hipStream_t s, int clear) {
  HEF_TRY(zero_async(flag_dev, clear * sizeof(int32_t), s));
  if (L.m > 0)
    k_validate<<<span_blocks(L.m, L.nnz), 256, 0, s>>>(L.eptr, L.pins, L.w, L.n, L.m, L.nnz,
                                                      span_extra(L.nnz), flag_dev);
  HEF_LAUNCH_CHECK();
  HEF_HIP(hipMemcpyAsync(bad_host, flag_dev, sizeof(int32_t), hipMemcpyDeviceToHost, s));
  HEF_HIP(hipStreamSynchronize(s));
  return HEF_OK;
}

hef_status structure_build(const Level &L, Structure &st, Arena &ws, hipStream_t s) {
  const int64_t n = L.n, m = L.m, nnz = L.nnz;
  TimedScope ts(kStStructure, s);
  const size_t mk = ws.mark();
  // eids: stable sort of (pin, edge) by pin; input is in edge order, so
  // each node's hyperedges come out ascending.  vptr from the sorted pins.
  if (nnz > 0) {
    SortWs w;
    carve_sort(ws, nnz, w);
    HEF_WS_CHECK(ws);
    const int bits = bits_for(n > 0 ? n - 1 : 0);
    uint32_t *eids = reinterpret_cast<uint32_t *>(st.eids);
    uint32_t *ids = radix_src(bits, w.tmp_v, eids, lean_sort(n, m, nnz));
    k_edge_ids<<<span_blocks(m, nnz), 256, 0, s>>>(L.eptr, ids, int32_t(m), span_extra(nnz),
                                                  st.n_big);
    HEF_LAUNCH_CHECK();
    HEF_TRY(radix_sort_pairs(reinterpret_cast<const uint32_t *>(L.pins), ids, w.tmp_k, w.tmp_v,
                             w.out_k, eids, nnz, bits, ws, s, lean_sort(n, m, nnz)));
    k_seg_bounds<<<cdiv(nnz + 1, 256), 256, 0, s>>>(w.out_k, nnz, int32_t(n), st.vptr);
    HEF_LAUNCH_CHECK();
  } else {
    HEF_TRY(zero_async(st.vptr, (n + 1) * sizeof(int32_t), s));
    HEF_TRY(zero_async(st.n_big, 2 * sizeof(int32_t), s));
  }
  ws.reset(mk);  // (the stream orders the reuse)

  // scales and big-segment lists
  ScaleWs w;
  carve_scale(ws, m, w);
  HEF_WS_CHECK(ws);
  if (m > 0) {
    k_edge_scales<<<cdiv(m, 256), 256, 0, s>>>(L.eptr, L.w, st.alpha, st.beta, st.big_e, st.n_big,
                                               w.tdb, w.tcb, int32_t(m));
    HEF_LAUNCH_CHECK();
  }
  if (n > 0) {
    k_node_scales<<<cdiv(n, 256), 256, 0, s>>>(st.vptr, st.eids, w.tdb, w.tcb, st.s, st.gam,
                                              st.big_v, st.n_big + 1, int32_t(n));
    HEF_LAUNCH_CHECK();
  }
  ws.reset(mk);
  return HEF_OK;
}

}  // namespace hef
