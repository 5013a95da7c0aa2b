// Deterministic device primitives: exclusive scan, stable LSD radix sort,
// stream compaction.
#include "prims.hpp"

namespace hef {
namespace {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanThreads * kScanItems;

// Inclusive scan of one value per thread over a workgroup of NT threads;
// wtot holds one entry per wave.  Ends with every thread past the barriers.
template <int NT>
__device__ __forceinline__ int32_t block_inclusive(int32_t x, int tid, int32_t *wtot) {
  const int lane = tid & 63, wv = tid >> 6;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int32_t o = __shfl_up(x, off, 64);
    if (lane >= off) x += o;
  }
  if (lane == 63) wtot[wv] = x;
  __syncthreads();
  int32_t add = 0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w)
    if (w < wv) add += wtot[w];
  __syncthreads();
  return x + add;
}

// Up to three arrays of one length per launch (blockIdx.y).
struct Scan3 {
  const int32_t *in[3];
  int32_t *out[3], *sums[3], *total[3];
};

__global__ void __launch_bounds__(kScanThreads)
k_scan_tiles(const Scan3 S, int64_t n) {
  const int32_t *in = S.in[blockIdx.y];
  int32_t *out = S.out[blockIdx.y], *tile_sums = S.sums[blockIdx.y];
  __shared__ int32_t sh[kScanThreads];
  const int tid = threadIdx.x;
  const int64_t base = int64_t(blockIdx.x) * kScanTile + int64_t(tid) * kScanItems;
  int32_t v[kScanItems];
  int32_t sum = 0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    int32_t t = (base + i < n) ? in[base + i] : 0;
    v[i] = sum;
    sum += t;
  }
  sh[tid] = sum;
  __syncthreads();
  for (int off = 1; off < kScanThreads; off <<= 1) {
    int32_t x = tid >= off ? sh[tid - off] : 0;
    __syncthreads();
    sh[tid] += x;
    __syncthreads();
  }
  const int32_t excl = sh[tid] - sum;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i)
    if (base + i < n) out[base + i] = v[i] + excl;
  if (tid == kScanThreads - 1) tile_sums[blockIdx.x] = sh[tid];
}

// One block scans the tile sums in place (exclusive) and writes the total.
__global__ void __launch_bounds__(1024)
k_scan_sums(int32_t *sums, int64_t ntiles, int32_t *total) {
  __shared__ int32_t sh[1024];
  __shared__ int32_t carry;
  const int tid = threadIdx.x;
  if (tid == 0) carry = 0;
  __syncthreads();
  for (int64_t c0 = 0; c0 < ntiles; c0 += 1024) {
    int64_t i = c0 + tid;
    int32_t v = i < ntiles ? sums[i] : 0;
    sh[tid] = v;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
      int32_t x = tid >= off ? sh[tid - off] : 0;
      __syncthreads();
      sh[tid] += x;
      __syncthreads();
    }
    if (i < ntiles) sums[i] = carry + sh[tid] - v;
    __syncthreads();
    if (tid == 1023) carry += sh[1023];
    __syncthreads();
  }
  if (tid == 0) *total = carry;
}

__global__ void __launch_bounds__(kScanThreads)
k_scan_add(int32_t *out, const int32_t *tile_off, int64_t n) {
  const int64_t base = int64_t(blockIdx.x) * kScanTile;
  const int32_t add = tile_off[blockIdx.x];
  for (int i = threadIdx.x; i < kScanTile; i += kScanThreads) {
    int64_t j = base + i;
    if (j < n) out[j] += add;
  }
}

// Adds to every item of tile t the sum of the tiles before it, a block
// reduction over tile_sums[0, t) (integer sums, so the order does not
// matter); the last tile's block also writes the total to out[n].  Up to
// kFinishTiles tiles this replaces the two kernels above: re-reading the
// earlier sums (at most kFinishTiles^2 / 2 reads, from L2) costs less than a
// launch.
// COMPACT: the items were flags; also idx[position] = i for every set flag.
constexpr int64_t kFinishTiles = 2048;
template <bool COMPACT>
__global__ void __launch_bounds__(kScanThreads)
k_scan_finish(const Scan3 S, int64_t n, int64_t ntiles, int32_t *idx) {
  int32_t *out = S.out[blockIdx.y];
  const int32_t *tile_sums = S.sums[blockIdx.y], *flag = S.in[blockIdx.y];
  __shared__ int32_t red[kScanThreads / 64];
  const int tid = threadIdx.x;
  const int64_t t = blockIdx.x;
  int32_t acc = 0;
  for (int64_t j = tid; j < t; j += kScanThreads) acc += tile_sums[j];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off);
  if ((tid & 63) == 0) red[tid >> 6] = acc;
  __syncthreads();
  int32_t add = 0;
#pragma unroll
  for (int w = 0; w < kScanThreads / 64; ++w) add += red[w];
  const int64_t base = t * kScanTile;
  for (int i = tid; i < kScanTile; i += kScanThreads) {
    const int64_t q = base + i;
    if (q < n) {
      const int32_t at = out[q] + add;
      out[q] = at;
      if constexpr (COMPACT)
        if (flag[q]) idx[at] = int32_t(q);
    }
  }
  if (t == ntiles - 1 && tid == 0) *S.total[blockIdx.y] = add + tile_sums[t];
}

// Scan (COMPACT: compaction of flags, as above) of at most kScanOne items in
// one workgroup and one launch; two launches cost more than the second
// workgroups would bring at these sizes.
constexpr int kScanOneThreads = 1024;
constexpr int kScanOneItems = 16;
constexpr int kScanOne = kScanOneThreads * kScanOneItems;
template <bool COMPACT>
__global__ void __launch_bounds__(kScanOneThreads)
k_scan_one(const Scan3 S, int n, int32_t *idx) {
  const int32_t *in = S.in[blockIdx.x];
  int32_t *out = S.out[blockIdx.x], *total = S.total[blockIdx.x];
  __shared__ int32_t wtot[kScanOneThreads / 64];
  // the items pass through LDS both ways: coalesced in global memory, a run
  // of 16 per thread in between (a pad word per 32, so that runs 16 apart
  // start on different banks)
  __shared__ int32_t buf[kScanOne + kScanOne / 32];
  const int tid = threadIdx.x;
  const int base = tid * kScanOneItems;
#pragma unroll
  for (int i = 0; i < kScanOneItems; ++i) {
    const int j = i * kScanOneThreads + tid;
    if (i * kScanOneThreads < n) buf[j + (j >> 5)] = j < n ? in[j] : 0;
  }
  __syncthreads();
  int32_t v[kScanOneItems];
#pragma unroll
  for (int i = 0; i < kScanOneItems; ++i) {
    const int j = base + i;
    v[i] = j < n ? buf[j + (j >> 5)] : 0;
    if (COMPACT) v[i] = v[i] != 0;
  }
  int32_t sum = 0;
#pragma unroll
  for (int i = 0; i < kScanOneItems; ++i) sum += v[i];
  const int32_t incl = block_inclusive<kScanOneThreads>(sum, tid, wtot);
  int32_t at = incl - sum;
#pragma unroll
  for (int i = 0; i < kScanOneItems; ++i) {
    const int j = base + i;
    if constexpr (COMPACT)
      if (v[i]) idx[at] = j;
    buf[j + (j >> 5)] = at;
    at += v[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kScanOneItems; ++i) {
    const int j = i * kScanOneThreads + tid;
    if (j < n) out[j] = buf[j + (j >> 5)];
  }
  if (tid == kScanOneThreads - 1) *total = incl;
}

// Digits of 8 bits, or of 9 where that saves a pass (9, 17, 18 or 25 to 27
// bits: the ids of 65k to 262k nodes, for one).  A pass over 7.9M pairs takes
// 57 us (histogram and scatter) with 8 bits and 71 us with 9, so three passes
// of 8 bits cost more than two of 9, and 9 is no gain where the count is equal.
inline int radix_bits(int bits) { return radix_passes(bits) < (bits + 7) / 8 ? 9 : 8; }
constexpr int kRadixThreads = 256;
constexpr int kRadixWaves = kRadixThreads / 64;
// Items per workgroup of a pass: 4096, or 1024 up to kRadixSmallN items.
// With 4096 a sort of a few hundred thousand items fills a fraction of the
// 256 CUs (15 to 20 us a pass at 70k to 760k items, 6 to 9 with 1024); from
// about a million items on the chip is full either way and the larger tile
// writes longer runs per digit.
constexpr int kRadixRounds = 16;
constexpr int kRadixRoundsSmall = 4;
constexpr int64_t kRadixSmallN = int64_t(1) << 20;
constexpr int kRadixTile = kRadixThreads * kRadixRounds;
constexpr int kRadixTileSmall = kRadixThreads * kRadixRoundsSmall;

inline int64_t radix_tile(int64_t n, bool lean) {
  return n <= kRadixSmallN && !lean ? kRadixTileSmall : kRadixTile;
}

template <int ROUNDS, int BITS>
__global__ void __launch_bounds__(kRadixThreads)
k_radix_hist(const uint32_t *__restrict__ keys, int64_t n, int shift, int32_t *__restrict__ hist,
             int nblocks) {
  constexpr int kBins = 1 << BITS;
  __shared__ int32_t cnt[kBins];
  const int tid = threadIdx.x;
#pragma unroll
  for (int b = tid; b < kBins; b += kRadixThreads) cnt[b] = 0;
  __syncthreads();
  const int64_t base = int64_t(blockIdx.x) * (kRadixThreads * ROUNDS);
#pragma unroll 4
  for (int r = 0; r < ROUNDS; ++r) {
    int64_t i = base + int64_t(r) * kRadixThreads + tid;
    if (i < n) atomicAdd(&cnt[(keys[i] >> shift) & (kBins - 1)], 1);
  }
  __syncthreads();
#pragma unroll
  for (int b = tid; b < kBins; b += kRadixThreads) hist[int64_t(b) * nblocks + blockIdx.x] = cnt[b];
}

// The histogram scan folded into the scatter: when the histogram has at most
// kRadixScanTiles scan tiles, it is scanned within tiles only (k_scan_tiles)
// and each scatter block adds the tile prefixes itself, from an exclusive
// scan of the tile sums in LDS (each thread takes a run of kTileRun sums).
constexpr int kTileRun = 8;
constexpr int kRadixScanTiles = kRadixThreads * kTileRun;

// Ranks of a wave's ROUNDS x 64 consecutive items among the items of the same
// digit before them in the wave; cnt[d] (the wave's own row of LDS counters,
// zero on entry) ends as the wave's count of digit d.  Only this wave touches
// cnt, so the rounds need no barrier.  Items past `left` take no part.
template <int ROUNDS, int BITS>
__device__ __forceinline__ void wave_ranks(const uint32_t (&k)[ROUNDS], int shift, int64_t left,
                                           int lane, int32_t *cnt, int32_t (&rank)[ROUNDS]) {
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const bool valid = 64 * r + lane < left;
    const uint32_t d = (k[r] >> shift) & ((1 << BITS) - 1);
    uint64_t peer = __ballot(valid);
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
      const bool bit = (d >> b) & 1u;
      const uint64_t bb = __ballot(bit);
      peer &= bit ? bb : ~bb;
    }
    const int before = __popcll(peer & lt);
    const int32_t c = valid ? cnt[d] : 0;
    wave_sync();
    if (valid && before == 0) cnt[d] = c + __popcll(peer);
    wave_sync();
    rank[r] = c + before;
  }
}

// One pass's scatter.  Wave w ranks its own ROUNDS * 64 consecutive items of
// the tile, the digits' counts are scanned over the waves and the digits, and
// the tile is put in digit order in LDS, so that the stores to global memory
// go out in runs of one digit (16 items on average at 4096 a tile) instead of
// one by one.  Bound by the launch and its load latency at small sizes, by
// the read and write of the items at large ones: 8 bits of 7.9M pairs in 40
// to 45 us (126 MB moved) against 100 us for the earlier pass, which ranked
// round by round behind four barriers each.
// offs holds the exclusive scan of the histogram (digit-major), or with
// tile_sums given its scan within scan tiles, to which the block adds the
// sum of the scan tiles before each entry's.
template <int ROUNDS, int BITS>
__global__ void __launch_bounds__(kRadixThreads)
k_radix_scatter(const uint32_t *__restrict__ kin, const uint32_t *__restrict__ vin,
                uint32_t *__restrict__ kout, uint32_t *__restrict__ vout, int64_t n, int shift,
                const int32_t *__restrict__ offs, int nblocks,
                const int32_t *__restrict__ tile_sums, int ntiles) {
  constexpr int TILE = kRadixThreads * ROUNDS;
  constexpr int kBins = 1 << BITS;
  constexpr int BPT = kBins / kRadixThreads;  // bins per thread (neighbours)
  __shared__ int32_t gbase[kBins];              // global position of the tile's first item per digit
  __shared__ int32_t lbase[kBins];              // its position within the tile
  __shared__ int32_t wcnt[kRadixWaves][kBins];  // per wave: counts, then offsets within the digit
  __shared__ int32_t wtot[kRadixWaves];
  // the reordered tile; before that, the scan-tile prefixes
  __shared__ uint32_t pool[2 * TILE > kRadixScanTiles ? 2 * TILE : kRadixScanTiles];
  uint32_t *sk = pool, *sv = pool + TILE;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wv = tid >> 6;
  const int64_t base = int64_t(blockIdx.x) * TILE;
  const int64_t wbase = base + int64_t(wv) * (64 * ROUNDS);
  uint32_t k[ROUNDS], v[ROUNDS];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int64_t i = wbase + 64 * r + lane;
    k[r] = i < n ? kin[i] : 0u;
    v[r] = i < n ? vin[i] : 0u;
  }
  int64_t hidx[BPT];
  int32_t gb[BPT];
#pragma unroll
  for (int b = 0; b < BPT; ++b) {
    hidx[b] = int64_t(tid * BPT + b) * nblocks + blockIdx.x;
    gb[b] = offs[hidx[b]];
  }
  if (tile_sums) {
    // the sum of the scan tiles before each hidx's: a run of kTileRun per thread,
    // scanned over the block
    int32_t run[kTileRun];
    int32_t tot = 0;
#pragma unroll
    for (int q = 0; q < kTileRun; ++q) {
      const int t = tid * kTileRun + q;
      run[q] = tot;
      tot += t < ntiles ? tile_sums[t] : 0;
    }
    const int32_t before = block_inclusive<kRadixThreads>(tot, tid, wtot) - tot;
#pragma unroll
    for (int q = 0; q < kTileRun; ++q) pool[tid * kTileRun + q] = uint32_t(before + run[q]);
    __syncthreads();
#pragma unroll
    for (int b = 0; b < BPT; ++b) gb[b] += int32_t(pool[hidx[b] / kScanTile]);
  }
#pragma unroll
  for (int b = 0; b < BPT; ++b) {
    gbase[tid * BPT + b] = gb[b];
#pragma unroll
    for (int w = 0; w < kRadixWaves; ++w) wcnt[w][tid * BPT + b] = 0;
  }
  __syncthreads();
  int32_t rank[ROUNDS];
  wave_ranks<ROUNDS, BITS>(k, shift, n - wbase, lane, wcnt[wv], rank);
  __syncthreads();
  int32_t tot[BPT], sum = 0;
#pragma unroll
  for (int b = 0; b < BPT; ++b) {
    tot[b] = 0;
#pragma unroll
    for (int w = 0; w < kRadixWaves; ++w) {
      const int32_t c = wcnt[w][tid * BPT + b];
      wcnt[w][tid * BPT + b] = tot[b];
      tot[b] += c;
    }
    sum += tot[b];
  }
  int32_t at = block_inclusive<kRadixThreads>(sum, tid, wtot) - sum;
#pragma unroll
  for (int b = 0; b < BPT; ++b) {
    lbase[tid * BPT + b] = at;
    at += tot[b];
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    if (wbase + 64 * r + lane < n) {
      const uint32_t d = (k[r] >> shift) & (kBins - 1);
      const int32_t to = lbase[d] + wcnt[wv][d] + rank[r];
      sk[to] = k[r];
      sv[to] = v[r];
    }
  }
  __syncthreads();
  const int cnt = n - base < TILE ? int(n - base) : TILE;
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int i = r * kRadixThreads + tid;
    if (i < cnt) {
      const uint32_t key = sk[i];
      const uint32_t d = (key >> shift) & (kBins - 1);
      const int32_t pos = gbase[d] + (i - lbase[d]);
      kout[pos] = key;
      vout[pos] = sv[i];
    }
  }
}

// All passes of a sort of at most 1024 * ROUNDS items in one workgroup: the
// items stay in registers and pass through LDS once per pass.  Replaces
// three launches per pass (about 4 us each when the chip is otherwise idle):
// two passes over 7k items 18 us.  At 16 items a thread two passes took 42 us,
// more than the six launches, so the line lies at 8.
constexpr int kOneThreads = 1024;
constexpr int kOneWaves = kOneThreads / 64;
constexpr int kOneRounds = 8;

template <int ROUNDS, int BITS>
__global__ void __launch_bounds__(kOneThreads)
k_radix_one(const uint32_t *kin, const uint32_t *vin, uint32_t *kout, uint32_t *vout, int n,
            int passes) {
  constexpr int kBins = 1 << BITS;
  __shared__ uint32_t buf[kOneThreads * ROUNDS];
  __shared__ int32_t wcnt[kOneWaves][kBins];
  __shared__ int32_t lbase[kBins];
  __shared__ int32_t wtot[kOneWaves];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wv = tid >> 6;
  const int wbase = wv * (64 * ROUNDS);
  uint32_t k[ROUNDS], v[ROUNDS];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int i = wbase + 64 * r + lane;
    k[r] = i < n ? kin[i] : 0u;
    v[r] = i < n ? vin[i] : 0u;
  }
  for (int p = 0; p < passes; ++p) {
    const int shift = p * BITS;
    for (int i = tid; i < kOneWaves * kBins; i += kOneThreads) (&wcnt[0][0])[i] = 0;
    __syncthreads();
    int32_t rank[ROUNDS];
    wave_ranks<ROUNDS, BITS>(k, shift, n - wbase, lane, wcnt[wv], rank);
    __syncthreads();
    int32_t tot = 0;
    if (tid < kBins) {
#pragma unroll
      for (int w = 0; w < kOneWaves; ++w) {
        const int32_t c = wcnt[w][tid];
        wcnt[w][tid] = tot;
        tot += c;
      }
    }
    const int32_t incl = block_inclusive<kOneThreads>(tot, tid, wtot);
    if (tid < kBins) lbase[tid] = incl - tot;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      const uint32_t d = (k[r] >> shift) & (kBins - 1);
      rank[r] += lbase[d] + wcnt[wv][d];
      if (wbase + 64 * r + lane < n) buf[rank[r]] = k[r];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) k[r] = buf[wbase + 64 * r + lane];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r)
      if (wbase + 64 * r + lane < n) buf[rank[r]] = v[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) v[r] = buf[wbase + 64 * r + lane];
    __syncthreads();
  }
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int i = wbase + 64 * r + lane;
    if (i < n) {
      kout[i] = k[r];
      vout[i] = v[r];
    }
  }
}

__global__ void k_compact(const int32_t *flag, const int32_t *pos, int32_t *idx_out, int64_t n) {
  int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n && flag[i]) idx_out[pos[i]] = int32_t(i);
}

template <int QG>
__global__ void __launch_bounds__(256 * QG)
k_reduce_cols(const double *__restrict__ in0, int64_t nrows0, double *__restrict__ out0,
              const double *__restrict__ in1, int64_t nrows1, double *__restrict__ out1,
              int64_t nbc, int64_t ncols) {
  __shared__ double red[ColSum<QG>::kLds];
  // workgroups [0, nbc) reduce side 0, the rest side 1
  const bool second = int64_t(blockIdx.x) >= nbc;
  const double *__restrict__ in = second ? in1 : in0;
  const int64_t nrows = second ? nrows1 : nrows0;
  double *__restrict__ out = second ? out1 : out0;
  const int64_t c = (int64_t(blockIdx.x) - (second ? nbc : 0)) * 8 + (threadIdx.x & 7);
  const double t = ColSum<QG>::run(in, nrows, ncols, c, c < ncols, red);
  if (threadIdx.x < 8 && c < ncols) out[c] = t;
}

// 4-byte words when the pointer and the size allow it, else bytes.
__global__ void k_zero_words(uint32_t *p, int64_t n) {
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
       i += int64_t(gridDim.x) * blockDim.x)
    p[i] = 0u;
}

__global__ void k_zero_bytes(uint8_t *p, int64_t n) {
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
       i += int64_t(gridDim.x) * blockDim.x)
    p[i] = 0u;
}

}  // namespace

hef_status zero_async(void *p, size_t bytes, hipStream_t s) {
  if (bytes == 0) return HEF_OK;
  const bool words = ((reinterpret_cast<uintptr_t>(p) | bytes) & 3) == 0;
  const int64_t n = int64_t(words ? bytes / 4 : bytes);
  const int64_t nb = std::min<int64_t>(cdiv(n, 256), 4096);
  if (words)
    k_zero_words<<<nb, 256, 0, s>>>(static_cast<uint32_t *>(p), n);
  else
    k_zero_bytes<<<nb, 256, 0, s>>>(static_cast<uint8_t *>(p), n);
  HEF_LAUNCH_CHECK();
  return HEF_OK;
}

// With few columns there are few workgroups (8 columns each), and the rows
// are split over four times the threads; from kWideCols columns on the
// workgroups fill the chip and hold few rows each.  200k nodes, b = 4: the
// 1.6k x 48 step products of the adjoint 10.7 -> 4.8 us, the Lanczos Gram's
// 0.9k x 144 partials (k_gram_reduce) 5.4 -> 4.0 us; 2M nodes, b = 8: the
// Gram's 1k x 576 partials 7.1 -> 4.8 us, the 17k x 480 Q_H partials 48 -> 45
// us (60 workgroups: bound by their number).
constexpr int64_t kWideCols = 8192;

hef_status reduce_cols_f64_pair(const double *in0, int64_t nrows0, double *out0,
                                const double *in1, int64_t nrows1, double *out1, int64_t ncols,
                                hipStream_t s) {
  if (ncols <= 0) return HEF_OK;
  const int64_t nbc = cdiv(ncols, 8), nb = out1 ? 2 * nbc : nbc;
  if (ncols < kWideCols)
    k_reduce_cols<4><<<nb, 1024, 0, s>>>(in0, nrows0, out0, in1, nrows1, out1, nbc, ncols);
  else
    k_reduce_cols<1><<<nb, 256, 0, s>>>(in0, nrows0, out0, in1, nrows1, out1, nbc, ncols);
  HEF_LAUNCH_CHECK();
  return HEF_OK;
}

hef_status reduce_cols_f64(const double *in, int64_t nrows, int64_t ncols, double *out,
                           hipStream_t s) {
  return reduce_cols_f64_pair(in, nrows, out, nullptr, 0, nullptr, ncols, s);
}

size_t scan_ws_bytes(int64_t n) {
  Arena a;
  for (int i = 0; i < 3; ++i) a.take<int32_t>(cdiv(n, kScanTile) + 1);
  return a.mark();
}

namespace {

// Exclusive scans of `count` arrays of n items each; with idx (count = 1) also
// the compaction.  More tiles than kFinishTiles take the separate scan of the
// tile sums, an array at a time.
hef_status scan_run(Scan3 S, int count, int64_t n, int32_t *idx, Arena &ws, hipStream_t s) {
  if (n <= kScanOne) {
    if (idx)
      k_scan_one<true><<<count, kScanOneThreads, 0, s>>>(S, int(n), idx);
    else
      k_scan_one<false><<<count, kScanOneThreads, 0, s>>>(S, int(n), nullptr);
    HEF_LAUNCH_CHECK();
    return HEF_OK;
  }
  const int64_t ntiles = cdiv(n, kScanTile);
  const size_t mk = ws.mark();
  for (int i = 0; i < count; ++i) S.sums[i] = ws.take<int32_t>(ntiles + 1);
  HEF_WS_CHECK(ws);
  const dim3 grid(static_cast<unsigned>(ntiles), static_cast<unsigned>(count));
  k_scan_tiles<<<grid, kScanThreads, 0, s>>>(S, n);
  if (ntiles <= kFinishTiles) {
    if (idx)
      k_scan_finish<true><<<grid, kScanThreads, 0, s>>>(S, n, ntiles, idx);
    else
      k_scan_finish<false><<<grid, kScanThreads, 0, s>>>(S, n, ntiles, nullptr);
  } else {
    for (int i = 0; i < count; ++i) {
      k_scan_sums<<<1, 1024, 0, s>>>(S.sums[i], ntiles, S.total[i]);
      k_scan_add<<<ntiles, kScanThreads, 0, s>>>(S.out[i], S.sums[i], n);
    }
    if (idx) k_compact<<<cdiv(n, 256), 256, 0, s>>>(S.in[0], S.out[0], idx, n);
  }
  HEF_LAUNCH_CHECK();
  ws.reset(mk);
  return HEF_OK;
}

}  // namespace

hef_status exclusive_scan_i32(const int32_t *in, int32_t *out, int64_t n, Arena &ws,
                              hipStream_t s) {
  if (n == 0) return zero_async(out, sizeof(int32_t), s);
  Scan3 S{};
  S.in[0] = in;
  S.out[0] = out;
  S.total[0] = out + n;
  return scan_run(S, 1, n, nullptr, ws, s);
}

hef_status exclusive_scan3_i32(const std::array<const int32_t *, 3> &in,
                               const std::array<int32_t *, 3> &out, int32_t *totals, int64_t n,
                               Arena &ws, hipStream_t s) {
  if (n == 0) return zero_async(totals, 3 * sizeof(int32_t), s);
  Scan3 S{};
  for (int i = 0; i < 3; ++i) {
    S.in[i] = in[i];
    S.out[i] = out[i];
    S.total[i] = totals + i;
  }
  return scan_run(S, 3, n, nullptr, ws, s);
}

size_t radix_ws_bytes(int64_t n, bool lean) {
  const int64_t nb = cdiv(n, radix_tile(n, lean)), bins = lean ? 256 : 512;
  Arena a;
  a.take<int32_t>(nb * bins + 1);
  return a.mark() + scan_ws_bytes(nb * bins) + 512;
}

size_t radix_ws_upto(int64_t n) {
  return std::max(radix_ws_bytes(n), radix_ws_bytes(std::min(n, kRadixSmallN)));
}

namespace {

template <int ROUNDS, int BITS>
hef_status radix_pass(const uint32_t *ka, const uint32_t *va, uint32_t *kb, uint32_t *vb,
                      int64_t n, int64_t nb, int shift, int32_t *hist, int32_t *tsum,
                      int64_t htiles, Arena &ws, hipStream_t s) {
  constexpr int kBins = 1 << BITS;
  k_radix_hist<ROUNDS, BITS><<<nb, kRadixThreads, 0, s>>>(ka, n, shift, hist, int(nb));
  if (tsum) {
    Scan3 S{};
    S.in[0] = hist;
    S.out[0] = hist;
    S.sums[0] = tsum;
    k_scan_tiles<<<htiles, kScanThreads, 0, s>>>(S, nb * kBins);
  } else {
    HEF_TRY(exclusive_scan_i32(hist, hist, nb * kBins, ws, s));
  }
  k_radix_scatter<ROUNDS, BITS><<<nb, kRadixThreads, 0, s>>>(ka, va, kb, vb, n, shift, hist,
                                                            int(nb), tsum, int(htiles));
  HEF_LAUNCH_CHECK();
  return HEF_OK;
}

template <int BITS>
hef_status radix_run(const uint32_t *src_k, const uint32_t *src_v, uint32_t *tmp_k,
                     uint32_t *tmp_v, uint32_t *out_k, uint32_t *out_v, int64_t n, int passes,
                     bool lean, Arena &ws, hipStream_t s) {
  if (n <= kOneThreads * kOneRounds) {
    if (n <= kOneThreads * 4)
      k_radix_one<4, BITS><<<1, kOneThreads, 0, s>>>(src_k, src_v, out_k, out_v, int(n), passes);
    else
      k_radix_one<kOneRounds, BITS><<<1, kOneThreads, 0, s>>>(src_k, src_v, out_k, out_v, int(n),
                                                              passes);
    HEF_LAUNCH_CHECK();
    return HEF_OK;
  }
  const bool small = radix_tile(n, lean) == kRadixTileSmall;
  const int64_t nb = cdiv(n, radix_tile(n, lean)), entries = nb << BITS;
  const size_t mk = ws.mark();
  int32_t *hist = ws.take<int32_t>(entries + 1);
  HEF_WS_CHECK(ws);
  // the histogram's scan tiles: when there are at most kRadixScanTiles
  // (n up to 64M keys, 32M with 9 bits) the scatter adds their prefixes itself
  const int64_t htiles = cdiv(entries, kScanTile);
  int32_t *tsum = htiles <= kRadixScanTiles ? ws.take<int32_t>(htiles) : nullptr;
  HEF_WS_CHECK(ws);
  const uint32_t *ka = src_k, *va = src_v;
  for (int p = 0; p < passes; ++p) {
    // the last pass writes out, the ones before alternate
    const bool to_out = ((passes - 1 - p) & 1) == 0;
    uint32_t *kb = to_out ? out_k : tmp_k, *vb = to_out ? out_v : tmp_v;
    if (small)
      HEF_TRY((radix_pass<kRadixRoundsSmall, BITS>(ka, va, kb, vb, n, nb, p * BITS, hist, tsum,
                                                   htiles, ws, s)));
    else
      HEF_TRY((radix_pass<kRadixRounds, BITS>(ka, va, kb, vb, n, nb, p * BITS, hist, tsum, htiles,
                                              ws, s)));
    ka = kb;
    va = vb;
  }
  ws.reset(mk);
  return HEF_OK;
}

}  // namespace

hef_status radix_sort_pairs(const uint32_t *src_k, const uint32_t *src_v, uint32_t *tmp_k,
                            uint32_t *tmp_v, uint32_t *out_k, uint32_t *out_v, int64_t n,
                            int bits, Arena &ws, hipStream_t s, bool lean) {
  if (n == 0) return HEF_OK;
  const int passes = radix_passes(bits, lean);
  if (!lean && radix_bits(bits) == 9)
    return radix_run<9>(src_k, src_v, tmp_k, tmp_v, out_k, out_v, n, passes, lean, ws, s);
  return radix_run<8>(src_k, src_v, tmp_k, tmp_v, out_k, out_v, n, passes, lean, ws, s);
}

hef_status scan_compact_flags(const int32_t *flag, int32_t *pos, int32_t *idx_out,
                              int32_t *count_dev, int64_t n, Arena &ws, hipStream_t s) {
  if (n == 0) return zero_async(count_dev, sizeof(int32_t), s);
  Scan3 S{};
  S.in[0] = flag;
  S.out[0] = pos;
  S.total[0] = count_dev;
  return scan_run(S, 1, n, idx_out, ws, s);
}

}  // namespace hef
