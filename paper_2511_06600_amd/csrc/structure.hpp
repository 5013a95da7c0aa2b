// Per-level structure and scales of the implicit star and clique expansions.
#pragma once

#include "common.hpp"

namespace hef {

// Segments longer than this go to the wave-per-segment kernels.
constexpr int kSmallSeg = 32;
// Sequential sums over a segment longer than this may be taken by the whole wave
// (64 terms loaded side by side, added in order); up to here a thread with
// eight loads in flight is faster.  A lane's chain takes about 75 ns a term, the
// wave's 25 ns a term of all its long segments together, so the wave takes them
// while their terms are at most three times the longest's.  Nodes of 5000
// hyperedges, 1 / 3 / 64 of them in a wave: 126 / 372 / 630 us (a thread each
// 286 / 377 / 818, the wave always 1600 for 64).
constexpr int kWaveSeg = 256;
constexpr int kWaveRatio = 3;
// Whether the wave takes its lanes' long segments (len on the lanes that have
// one, 0 on the others), the same on every lane.
__device__ __forceinline__ bool wave_takes(int32_t len) {
  if (__ballot(len > 0) == 0) return false;
  int64_t sum = len;
  int32_t most = len;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    sum += __shfl_xor(sum, off, 64);
    const int32_t o = __shfl_xor(most, off, 64);
    most = o > most ? o : most;
  }
  return sum <= kWaveRatio * int64_t(most);
}

// The passes that give a long hyperedge a workgroup of 1024 threads (the ratios
// and their adjoint) take those of more than kSmallSeg pins while these are
// few, and where there are more than kFewLong those of more than `many`.  512
// such workgroups run at a time, a few us each, so 2048 hyperedges are four
// turns, about a lane group's chain over 128 pins, while thousands of lane
// groups run at once.
constexpr int kFewLong = 2048;
__device__ __forceinline__ int long_from(int least, int many, int32_t n_big) {
  return n_big > kFewLong && least < many ? many : least;
}

struct Structure {
  // CSC incidence (node -> hyperedges), hyperedges ascending per node.
  int32_t *vptr = nullptr;  // [n+1]
  int32_t *eids = nullptr;  // [nnz]
  // Expansion scales (float32, computed in float64):
  //   s[u]     = d_b(u)^-1/2, d_b(u) = sum_{e ∋ u} w_e/|e|  (0 if d_b = 0)
  //   gam[u]   = s[u]^2 * sum_{e ∋ u} beta_e  (clique self-term)
  //   alpha[e] = sqrt(w_e)/|e|  (star edge factor, d_b(e) = w_e)
  //   beta[e]  = w_e/(|e|(|e|-1))  (half the clique pair weight c_e)
  float *s = nullptr, *gam = nullptr, *alpha = nullptr, *beta = nullptr;
  // Hyperedges / nodes whose segment exceeds kSmallSeg (in no set order), and
  // counts.
  int32_t *big_e = nullptr, *big_v = nullptr;
  int32_t *n_big = nullptr;  // [2]: big edges, big nodes
};

// Workspace of a Structure plus the temporaries to build it.
void structure_carve(Arena &a, int64_t n, int64_t m, int64_t nnz, Structure &st);
// Scratch of structure_build at these sizes (with which it need not grow: see
// radix_ws_bytes), and the scratch that serves any sizes up to these.
size_t structure_build_need(int64_t n, int64_t m, int64_t nnz);
size_t structure_build_ws(int64_t n, int64_t m, int64_t nnz);

// Device validation of a CSR hypergraph; *bad_host != 0 if invalid.  Clears
// flag_dev[0 .. clear) and uses flag_dev[0].
hef_status validate_device(const Level &L, int32_t *flag_dev, int32_t *bad_host,
                           hipStream_t s, int clear = 1);

// Builds CSC, scales and big-segment lists for one level.
hef_status structure_build(const Level &L, Structure &st, Arena &ws, hipStream_t s);

}  // namespace hef
