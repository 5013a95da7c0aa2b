// Block Krylov bases of both expansions (Eq. (12), Alg. 1).
//
// Per expansion, b start vectors and k steps of the block three-term
// recurrence: Y = A V_j, then V_{j+1} is the Gram-Schmidt of Y against
// [V_{j-1}, V_j] and within itself.  The Gram-Schmidt is carried out in the
// Gram metric of M = [V_{j-1} | V_j | Y]: G = M^T M is accumulated in FP32
// register blocks over row chunks and summed across chunks in float64, its
// Cholesky factor R (float64) gives V_{j+1} = M R^-1[:, Y columns].  A
// column whose Gram-Schmidt residual falls below tau times its length is a
// breakdown and becomes zero.  V_0 = X R^-1 starts the sequence and is not
// part of the pool; V_1..V_k are (star: node rows only).
#include <cmath>

#include "krylov.hpp"
#include "prims.hpp"

namespace hef {
namespace {

constexpr int kGramBlocks = 1024;  // workgroups of the Gram partial pass

// Register staging of one Gram slab of M = [v0 | v1 | y] (SLAB rows).
// LDS row stride (floats) of a Gram slab of C = 3B columns.  The products
// read, per half-wave, 6-column blocks of about four consecutive rows; at
// B = 8 a stride of C + 1 = 25 maps some of those (row, block) pairs to one
// bank (measured: a third of the kernel's cycles in bank conflicts), C + 4 =
// 28 spreads them (7 % faster, same values).
template <int B>
__host__ __device__ constexpr int gram_ld() { return B == 8 ? 3 * B + 4 : 3 * B + 1; }

template <int B, int SLAB>
struct GramSlab {
  static constexpr int C = 3 * B;
  static constexpr int LD = gram_ld<B>();
  static constexpr int Q = B >= 4 ? B / 4 : 1;  // float4 per row per array
  static constexpr int TOT = B >= 4 ? SLAB * 3 * Q : SLAB * C;
  static constexpr int NPT = (TOT + 255) / 256;
  static __device__ __forceinline__ void fetch(float4 (&pre)[NPT], int tid, int64_t base,
                                               int64_t r1, const float *v0, const float *v1,
                                               const float *y) {
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
      const int e = tid + 256 * i;
      float4 t = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      if (e < TOT) {
        if constexpr (B >= 4) {
          const int a = e / (SLAB * Q);
          const int rem = e % (SLAB * Q);
          const int r = rem / Q, q = rem % Q;
          const int64_t row = base + r;
          const float *src = a == 0 ? v0 : (a == 1 ? v1 : y);
          if (row < r1 && src) t = *reinterpret_cast<const float4 *>(src + row * B + 4 * q);
        } else {
          const int r = e / C, c = e % C;
          const int64_t row = base + r;
          if (row < r1) {
            if (c < B) t.x = v0 ? v0[row * B + c] : 0.0f;
            else if (c < 2 * B) t.x = v1 ? v1[row * B + c - B] : 0.0f;
            else t.x = y[row * B + c - 2 * B];
          }
        }
      }
      pre[i] = t;
    }
  }
  static __device__ __forceinline__ void stash(const float4 (&pre)[NPT], int tid, float *sh) {
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
      const int e = tid + 256 * i;
      if (e < TOT) {
        if constexpr (B >= 4) {
          const int a = e / (SLAB * Q);
          const int rem = e % (SLAB * Q);
          const int r = rem / Q, q = rem % Q;
          float *d = sh + r * LD + a * B + 4 * q;
          d[0] = pre[i].x; d[1] = pre[i].y; d[2] = pre[i].z; d[3] = pre[i].w;
        } else {
          const int r = e / C, c = e % C;
          sh[r * LD + c] = pre[i].x;
        }
      }
    }
  }
};

// Gram partials of M = [v0 | v1 | y] (rows x C, C = 3B), FP32 register
// blocks: the C x C Gram is cut into S x S blocks, one thread per block on or
// above the diagonal; a workgroup stages 64-row slabs in LDS and its RG row
// groups split each slab's rows.  Per-thread FP32 sums (a few hundred rows)
// are combined in float64 in row-group order; partial[blk][C*C].  The next
// slab is loaded into registers while the current one is consumed.
// Operands of one expansion's Gram.  A launch covers two expansions:
// workgroups [0, nb0) take side 0, the rest side 1.
struct GramSide {
  const float *v0, *v1, *y;
  int64_t rows, rows_per_blk;
  double *partial;
};
struct GramPair {
  GramSide s[2];
  int nb0;
};

template <int B>
__global__ void __launch_bounds__(256)
k_lgram(const GramPair P) {
  const bool second = int(blockIdx.x) >= P.nb0;
  const int bid = int(blockIdx.x) - (second ? P.nb0 : 0);
  const float *__restrict__ v0 = second ? P.s[1].v0 : P.s[0].v0;
  const float *__restrict__ v1 = second ? P.s[1].v1 : P.s[0].v1;
  const float *__restrict__ y = second ? P.s[1].y : P.s[0].y;
  const int64_t rows = second ? P.s[1].rows : P.s[0].rows;
  const int64_t rows_per_blk = second ? P.s[1].rows_per_blk : P.s[0].rows_per_blk;
  double *__restrict__ partial = second ? P.s[1].partial : P.s[0].partial;
  constexpr int C = 3 * B;
  constexpr int S = (C % 6 == 0) ? 6 : 3;
  constexpr int NB = C / S;
  constexpr int NT = NB * (NB + 1) / 2;
  constexpr int RG = 256 / NT;
  constexpr int SLAB = 128;
  constexpr int LD = gram_ld<B>();
  // slab buffer, reused for the row groups' sums at the end
  constexpr int SH = SLAB * LD > RG * NT * S * S ? SLAB * LD : RG * NT * S * S;
  __shared__ float sh[SH];
  const int tid = threadIdx.x;
  const int g = tid / NT;
  const int blk = tid % NT;
  const bool active = g < RG;
  int bi = 0, bj = 0;
  {
    int q = blk;
    for (int a = 0; a < NB; ++a) {
      if (q < NB - a) { bi = a; bj = a + q; break; }
      q -= NB - a;
    }
  }
  float acc[S][S];
#pragma unroll
  for (int a = 0; a < S; ++a)
#pragma unroll
    for (int b = 0; b < S; ++b) acc[a][b] = 0.0f;
  const int64_t r0 = int64_t(bid) * rows_per_blk;
  const int64_t r1 = r0 + rows_per_blk < rows ? r0 + rows_per_blk : rows;
  // the next slab is fetched into registers while the current one is used
  using SL = GramSlab<B, SLAB>;
  float4 pre[SL::NPT];
  if (r0 < r1) SL::fetch(pre, tid, r0, r1, v0, v1, y);
  for (int64_t base = r0; base < r1; base += SLAB) {
    __syncthreads();
    SL::stash(pre, tid, sh);
    __syncthreads();
    if (base + SLAB < r1) SL::fetch(pre, tid, base + SLAB, r1, v0, v1, y);
    if (active) {
      for (int r = g; r < SLAB; r += RG) {
        float xa[S], xb[S];
#pragma unroll
        for (int a = 0; a < S; ++a) xa[a] = sh[r * LD + bi * S + a];
#pragma unroll
        for (int b = 0; b < S; ++b) xb[b] = sh[r * LD + bj * S + b];
#pragma unroll
        for (int a = 0; a < S; ++a)
#pragma unroll
          for (int b = 0; b < S; ++b) acc[a][b] = fmaf(xa[a], xb[b], acc[a][b]);
      }
    }
  }
  // every row group's sums go to LDS (the slab buffer is free now); each
  // entry is then summed over the row groups in ascending order, in float64
  __syncthreads();
  float *red = sh;
  if (active) {
#pragma unroll
    for (int a = 0; a < S; ++a)
#pragma unroll
      for (int b = 0; b < S; ++b) red[(g * NT + blk) * S * S + a * S + b] = acc[a][b];
  }
  __syncthreads();
  for (int e = tid; e < C * C; e += 256) {
    const int i = e / C, j = e % C;
    const int ri = i / S, rj = j / S;
    double t = 0.0;
    if (ri <= rj) {
      int id = rj - ri;
      for (int a = 0; a < ri; ++a) id += NB - a;
      const int off = id * S * S + (i % S) * S + (j % S);
      for (int gg = 0; gg < RG; ++gg) t += double(red[gg * NT * S * S + off]);
    }
    partial[int64_t(bid) * C * C + e] = t;
  }
}

// G = the column sums of the partials (float64, ColSum's order), written for
// the entries in blocks on or above the diagonal and mirrored into the blocks
// below it.  Two expansions per launch: workgroups [0, nbh) reduce (in0,
// nrows0) into G0, the rest (in1, nrows1) into G1.
__global__ void __launch_bounds__(1024)
k_gram_reduce(const double *__restrict__ in0, int64_t nrows0, double *__restrict__ G0,
              const double *__restrict__ in1, int64_t nrows1, double *__restrict__ G1, int nbh,
              int C, int S) {
  __shared__ double red[ColSum<4>::kLds];
  const bool second = int(blockIdx.x) >= nbh;
  const double *__restrict__ in = second ? in1 : in0;
  const int64_t nrows = second ? nrows1 : nrows0;
  double *__restrict__ G = second ? G1 : G0;
  const int c = (int(blockIdx.x) - (second ? nbh : 0)) * 8 + int(threadIdx.x & 7);
  const int i = c / C, j = c % C;
  const bool upper = c < C * C && i / S <= j / S;
  const double t = ColSum<4>::run(in, nrows, int64_t(C) * C, c, upper, red);
  if (threadIdx.x < 8 && upper) {
    G[int64_t(i) * C + j] = t;
    if (i / S < j / S) G[int64_t(j) * C + i] = t;
  }
}

// Cholesky of G with column dropping, then the Y-block columns of R^-1.
// Bound by its chain of 2 C pivots and the in-order sums of the back
// substitution: C = 24 in 8.6 us and C = 12 in 3.9 us with pivot_of, 14.0 and
// 6.0 with sqrt(), divisions and a branch per column.
// One wave per expansion; lane t holds row t of the C x C Gram (registers),
// so the factorisation needs no barriers: column k's pivot and the entries
// L_jk reach the other lanes by readlane.  Column c is dropped when its reference
// length is 0 or its Schur pivot d_c <= tau^2 * G_cc.  L goes to LDS; lane c
// then forms column c of R^-1 = L^-T by back substitution.
template <int C>
__device__ __forceinline__ void lsolve_wave(const double *G, int B, double tau, double *T,
                                            double *Rf, double *Ls) {
  const int t = threadIdx.x & 63;
  double a[C], l[C];
#pragma unroll
  for (int j = 0; j < C; ++j) {
    a[j] = t < C ? G[t * C + j] : 0.0;
    l[j] = 0.0;
  }
  double gref = 0.0;
#pragma unroll
  for (int j = 0; j < C; ++j)
    if (j == t) gref = a[j];
  // straight-line steps: a dropped column's multiples are zero, which leaves
  // the later columns as they are, so that the next pivot's root is under way
  // during a step's updates
  uint64_t keep = 0;
  Pivot pv[C];
#pragma unroll
  for (int k = 0; k < C; ++k) {
    const double d = readlane_f64(a[k], k);
    const double ref = readlane_f64(gref, k);
    const bool kk = ref > 0.0 && d > tau * tau * ref;
    keep |= kk ? uint64_t(1) << k : 0;
    pv[k] = pivot_of(kk ? d : 1.0);
    const double below = t > k ? div_pivot(a[k], pv[k]) : 0.0;
    const double lk = kk ? (t == k ? pv[k].root : below) : 0.0;
    l[k] = lk;
    // (also the entries right of lane t's diagonal, which are never read:
    // an unpredicated update; lk is zero on the rows above the pivot)
#pragma unroll
    for (int j = k + 1; j < C; ++j) {
      const double ljk = readlane_f64(lk, j);
      a[j] -= lk * ljk;
    }
  }
  if (t < C) {
#pragma unroll
    for (int j = 0; j < C; ++j) Ls[t * C + j] = l[j];
  }
  wave_sync();
  // column c of R^-1 (R = L^T): L^T x = e_c, rows c, c-1, ..., 0
  const int c = t;
  const bool kc = c < C && ((keep >> c) & 1);
  double x[C];
#pragma unroll
  for (int i = C - 1; i >= 0; --i) {
    double acc = 0.0;
#pragma unroll
    for (int q = i + 1; q < C; ++q) acc += Ls[q * C + i] * x[q];
    const bool ki = (keep >> i) & 1;
    const double v = div_pivot(i == c ? 1.0 : -acc, pv[i]);
    x[i] = kc && ki && i <= c ? v : 0.0;
  }
  if (c >= 2 * B && c < C) {
#pragma unroll
    for (int i = 0; i < C; ++i) T[i * B + (c - 2 * B)] = x[i];
  }
  // optionally the whole R^-1 (row-major C x C), zero rows/columns for drops
  if (Rf && c < C) {
#pragma unroll
    for (int i = 0; i < C; ++i) Rf[i * C + c] = x[i];
  }
}

template <int C>
__global__ void __launch_bounds__(64)
k_lsolve(const double *__restrict__ Gall, int B, double tau, double *__restrict__ Tall,
         double *__restrict__ Rall) {
  __shared__ double Ls[C * C];
  lsolve_wave<C>(Gall + blockIdx.x * C * C, B, tau, Tall + blockIdx.x * C * B,
                 Rall ? Rall + blockIdx.x * C * C : nullptr, Ls);
}

// The reduce of the Gram partials and the solve in one launch, a workgroup
// per expansion (mask bit x: expansion x takes part): for C <= 6 (b <= 2) the
// partials are at most 1024 x 36 values, and the second launch of the step
// costs more than the workgroups it brings (2k nodes, b = 1: 2.6 + 2.2 us and
// a launch -> 2.8; 20k, b = 2: 4.6 + 3.3 and a launch -> 5.8).  The sums
// are ColSum's, as in k_gram_reduce.
template <int C, int S>
__global__ void __launch_bounds__(1024)
k_lreduce_solve(const double *__restrict__ in0, int64_t nrows0, const double *__restrict__ in1,
                int64_t nrows1, int mask, int B, double tau, double *__restrict__ Tall,
                double *__restrict__ Rall) {
  constexpr int NG = (C * C + 7) / 8;  // groups of 8 columns, all loaded together
  __shared__ double red[NG][4][32][9];
  __shared__ double G[C * C], Ls[C * C];
  const int x = blockIdx.x;
  if (!((mask >> x) & 1)) return;
  const double *__restrict__ in = x ? in1 : in0;
  const int64_t nrows = x ? nrows1 : nrows0;
  const int cl = threadIdx.x & 7, rl = (threadIdx.x >> 3) & 31, part = threadIdx.x >> 8;
  double acc[NG][2] = {};
  for (int64_t r = rl + 64 * part; r < nrows; r += 256) {
    double t[NG][2];
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int c = 8 * g + cl < C * C ? 8 * g + cl : C * C - 1;
        t[g][q] = in[(r + 32 * q < nrows ? r + 32 * q : r) * (C * C) + c];
      }
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int q = 0; q < 2; ++q)
        if (r + 32 * q < nrows) acc[g][q] += t[g][q];
  }
#pragma unroll
  for (int g = 0; g < NG; ++g) red[g][part][rl][cl] = acc[g][0] + acc[g][1];
  __syncthreads();
  // wave g finishes group g: lane (column, k < 8) takes row lanes k + 8 i
  const int g = threadIdx.x >> 6;
  if (g < NG) {
    const int k = (threadIdx.x >> 3) & 7;
    double y[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      y[i] = (red[g][0][k + 8 * i][cl] + red[g][1][k + 8 * i][cl]) +
             (red[g][2][k + 8 * i][cl] + red[g][3][k + 8 * i][cl]);
    double t = (y[0] + y[2]) + (y[1] + y[3]);
#pragma unroll
    for (int off = 32; off >= 8; off >>= 1) t += __shfl_down(t, off, 64);
    const int c = 8 * g + cl;
    const int i = c / C, j = c % C;
    if (k == 0 && c < C * C && i / S <= j / S) {
      G[i * C + j] = t;
      if (i / S < j / S) G[j * C + i] = t;
    }
  }
  __syncthreads();
  if (threadIdx.x < 64)
    lsolve_wave<C>(G, B, tau, Tall + x * C * B, Rall ? Rall + x * C * C : nullptr, Ls);
}

// the solve for C = 3B columns (B in {1, 2, 4, 8, 16})
hef_status lsolve_launch(const double *G, int B, double tau, double *T, double *R,
                         hipStream_t s) {
  switch (B) {
    case 1: k_lsolve<3><<<2, 64, 0, s>>>(G, B, tau, T, R); break;
    case 2: k_lsolve<6><<<2, 64, 0, s>>>(G, B, tau, T, R); break;
    case 4: k_lsolve<12><<<2, 64, 0, s>>>(G, B, tau, T, R); break;
    case 8: k_lsolve<24><<<2, 64, 0, s>>>(G, B, tau, T, R); break;
    case 16: k_lsolve<48><<<2, 64, 0, s>>>(G, B, tau, T, R); break;
    default: return HEF_ERR_UNSUPPORTED;
  }
  HEF_LAUNCH_CHECK();
  return HEF_OK;
}

__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return uint16_t(u >> 16);
}

// V_next = [v0 | v1 | y] T in float64 arithmetic.  A workgroup stages its
// rows of the three inputs in LDS with coalesced float4 loads, one thread per
// row (two for B = 16) forms the outputs, which leave through LDS as
// coalesced stores.  The first pool_rows rows also go to the pool (row-octet
// layout, float32, bfloat16 or, for the float64 debug basis, float64) at
// column col0.
template <int CH>
__device__ __forceinline__ void ld(const float *p, float (&v)[CH]) {
  if constexpr (CH == 4) {
    const float4 t = *reinterpret_cast<const float4 *>(p);
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  } else if constexpr (CH == 2) {
    const float2 t = *reinterpret_cast<const float2 *>(p);
    v[0] = t.x; v[1] = t.y;
  } else {
    v[0] = *p;
  }
}

// Operands of one expansion's apply.  A launch covers two expansions:
// logical workgroups [0, nb0) take side 0, the rest side 1.
struct ApplySide {
  const float *v0, *v1, *y;
  const double *T;
  float *vn;
  int64_t rows;
  int col0;
};
struct ApplyPair {
  ApplySide s[2];
  int64_t nb0;
};

// The 8 rows of one (octet, column) of the pool, as float32, bfloat16 or, for
// the float64 debug basis, float64.
__device__ __forceinline__ void pool_store8(void *pool, int pool_type, int64_t off,
                                            const float (&v)[8]) {
  if (pool_type == kPoolF32) {
    float4 *pp = reinterpret_cast<float4 *>(reinterpret_cast<float *>(pool) + off);
    pp[0] = make_float4(v[0], v[1], v[2], v[3]);
    pp[1] = make_float4(v[4], v[5], v[6], v[7]);
  } else if (pool_type == kPoolF64) {
    double2 *pp = reinterpret_cast<double2 *>(reinterpret_cast<double *>(pool) + off);
#pragma unroll
    for (int q = 0; q < 4; ++q) pp[q] = make_double2(double(v[2 * q]), double(v[2 * q + 1]));
  } else {
    uint32_t wv[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      wv[q] = uint32_t(f2bf(v[2 * q])) | (uint32_t(f2bf(v[2 * q + 1])) << 16);
    *reinterpret_cast<uint4 *>(reinterpret_cast<uint16_t *>(pool) + off) =
        make_uint4(wv[0], wv[1], wv[2], wv[3]);
  }
}

template <int B>
__global__ void __launch_bounds__(256)
k_lapply(const ApplyPair P, void *__restrict__ pool, int pool_type, int64_t pool_rows, int K) {
  constexpr int C = 3 * B;
  constexpr int RB = B <= 8 ? 256 : 128;  // rows per workgroup
  constexpr int NSPL = 256 / RB;          // threads per row
  constexpr int OPT = B / NSPL;           // outputs per thread
  constexpr int LDR = B + 1;              // LDS row stride (odd: no bank conflicts)
  __shared__ double Ts[C * B];
  __shared__ float sm[3][RB * LDR];
  const int tid = threadIdx.x;
  const int64_t lb = xcd_block(blockIdx.x, gridDim.x);
  const bool second = lb >= P.nb0;
  const float *__restrict__ v0 = second ? P.s[1].v0 : P.s[0].v0;
  const float *__restrict__ v1 = second ? P.s[1].v1 : P.s[0].v1;
  const float *__restrict__ y = second ? P.s[1].y : P.s[0].y;
  const double *__restrict__ Tm = second ? P.s[1].T : P.s[0].T;
  float *__restrict__ vn = second ? P.s[1].vn : P.s[0].vn;
  const int64_t rows = second ? P.s[1].rows : P.s[0].rows;
  const int col0 = second ? P.s[1].col0 : P.s[0].col0;
  const int64_t row0 = (lb - (second ? P.nb0 : 0)) * RB;
  const int nrow = int(rows - row0 < RB ? rows - row0 : RB);
  const float *src[3] = {v0, v1, y};
  // coalesced loads of the workgroup's rows into LDS, all of a thread's
  // loads issued before the first is stored
  if constexpr (B >= 4) {
    constexpr int NL = (RB * B / 4 + 255) / 256;  // float4 per thread and array
    float4 t[3][NL];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int u = 0; u < NL; ++u) {
        const int i = tid + 256 * u;
        t[a][u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (src[a] != nullptr && i < nrow * B / 4)
          t[a][u] = reinterpret_cast<const float4 *>(src[a] + row0 * B)[i];
      }
    for (int e = tid; e < C * B; e += 256) Ts[e] = Tm[e];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int u = 0; u < NL; ++u) {
        const int i = tid + 256 * u;
        if (src[a] != nullptr && i < nrow * B / 4) {
          float *d = &sm[a][(4 * i / B) * LDR + (4 * i) % B];
          d[0] = t[a][u].x; d[1] = t[a][u].y; d[2] = t[a][u].z; d[3] = t[a][u].w;
        }
      }
  } else {
    for (int e = tid; e < C * B; e += 256) Ts[e] = Tm[e];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      if (src[a] == nullptr) continue;
      const float *base = src[a] + row0 * B;
      for (int i = tid; i < nrow * B; i += 256) sm[a][(i / B) * LDR + i % B] = base[i];
    }
  }
  __syncthreads();
  const int r = tid / NSPL, h = tid % NSPL;
  float of[OPT];
  {
    double out[OPT];
#pragma unroll
    for (int c = 0; c < OPT; ++c) out[c] = 0.0;
    if (r < nrow) {
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        if (src[a] == nullptr) continue;
#pragma unroll
        for (int u = 0; u < B; ++u) {
          const double md = double(sm[a][r * LDR + u]);
          const double *trow = Ts + (a * B + u) * B + h * OPT;
#pragma unroll
          for (int c = 0; c < OPT; ++c) out[c] = fma(md, trow[c], out[c]);
        }
      }
    }
#pragma unroll
    for (int c = 0; c < OPT; ++c) of[c] = float(out[c]);
  }
  __syncthreads();
  if (r < nrow) {
#pragma unroll
    for (int c = 0; c < OPT; ++c) sm[0][r * LDR + h * OPT + c] = of[c];
  }
  __syncthreads();
  // coalesced stores of the new rows, then the pool columns
  float *vbase = vn + row0 * B;
  if constexpr (B >= 4) {
    for (int i = tid; i < nrow * B / 4; i += 256) {
      const float *d = &sm[0][(4 * i / B) * LDR + (4 * i) % B];
      reinterpret_cast<float4 *>(vbase)[i] = make_float4(d[0], d[1], d[2], d[3]);
    }
  } else {
    for (int i = tid; i < nrow * B; i += 256) vbase[i] = sm[0][(i / B) * LDR + i % B];
  }
  if (pool) {
    // pool rows in the row-octet layout: per (octet, column) 8 consecutive
    // values; rows at or past pool_rows are zero (row0 is a multiple of 8)
    const int noct = (nrow + 7) / 8;
    for (int i = tid; i < noct * B; i += 256) {
      const int o = i / B, c = i % B;
      const int64_t gr0 = row0 + 8 * o;
      if (gr0 >= pool_rows) continue;
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        v[u] = (8 * o + u < nrow && gr0 + u < pool_rows) ? sm[0][(8 * o + u) * LDR + c] : 0.0f;
      const int64_t off = ((gr0 >> 3) * K + col0 + c) * 8;
      pool_store8(pool, pool_type, off, v);
    }
  }
}

// k_lapply for both expansions when the product with A comes next: a
// workgroup takes RB / 2 node rows of both expansions, or RB hyperedge rows
// of the star expansion, and the node workgroups also write the next
// product's gather rows U[p] = [s_p x_V[p] | s_p x_c[p]] (spmm.hip).  A node
// row's halves meet in one workgroup, so U leaves in whole 128-byte lines
// (from separate workgroups per expansion every line was written in two
// parts, and the apply took 302 us instead of 157 at 2M nodes, b = 8).  The
// prep pass, which read both blocks again, and its launch are gone.  A thread
// holds its row of the inputs in registers and only the new rows pass through
// LDS (the pool's octets, coalesced stores); with the inputs staged in LDS as
// in k_lapply the kernel took 237 us.  Per step, apply + prep -> this kernel:
// 2M nodes, b = 8, 159 + 41 -> 190 us (5.5 TB/s over its 1.05 GB: the copy
// rate); 200k, b = 4, 9.6 + 3.7 -> 11.9 us; 20k, b = 8, 5.2 + 2.9 -> 7.8 us;
// 2k, b = 1, 4.0 + 2.2 -> 3.5 us.  Same operations per row, same bits.
template <int B>
__global__ void __launch_bounds__(256)
k_lapply_u(const ApplyPair P, int64_t n, int64_t nbn, const float *__restrict__ scale,
           float *__restrict__ U, void *__restrict__ pool, int pool_type, int K) {
  static_assert(B <= 8, "one thread per row");
  constexpr int RB = 256;     // rows per workgroup (both sides counted)
  constexpr int RN = RB / 2;  // node rows per side
  constexpr int LDR = B + 1;  // LDS row stride (odd: no bank conflicts)
  constexpr int CH = B < 4 ? B : 4;
  __shared__ float sm[RB * LDR];
  __shared__ float sc[RN];
  const int tid = threadIdx.x;
  // node workgroups and hyperedge workgroups each spread over the XCDs
  const bool nodes = int64_t(blockIdx.x) < nbn;
  const int64_t lb = nodes ? xcd_block(blockIdx.x, nbn)
                           : xcd_block(int64_t(blockIdx.x) - nbn, int64_t(gridDim.x) - nbn);
  const int64_t row0 = nodes ? lb * RN : n + lb * RB;
  const int64_t rend = nodes ? n : P.s[0].rows;
  const int cap = nodes ? RN : RB;
  const int nrow = int(rend - row0 < cap ? rend - row0 : cap);
  const int sides = nodes ? 2 : 1;
  if (nodes && tid < nrow) sc[tid] = scale[row0 + tid];
  // (a wave's rows lie on one side, so its T is uniform: scalar loads)
  const int side = __builtin_amdgcn_readfirstlane(nodes ? tid / RN : 0);
  const int rr = nodes ? tid % RN : tid;
  const ApplySide &S = side ? P.s[1] : P.s[0];
  // a thread reads its row of the three inputs straight into registers
  float x[3][B];
  const int64_t row = row0 + (rr < nrow ? rr : nrow - 1);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float *src = a == 0 ? S.v0 : a == 1 ? S.v1 : S.y;
#pragma unroll
    for (int u = 0; u < B; ++u) x[a][u] = 0.0f;
    if (src != nullptr) {
#pragma unroll
      for (int u = 0; u < B; u += CH) {
        float t[CH];
        ld<CH>(src + row * B + u, t);
#pragma unroll
        for (int c = 0; c < CH; ++c) x[a][u + c] = t[c];
      }
    }
  }
  {
    double out[B];
#pragma unroll
    for (int c = 0; c < B; ++c) out[c] = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      if ((a == 0 && S.v0 == nullptr) || (a == 1 && S.v1 == nullptr)) continue;
#pragma unroll
      for (int u = 0; u < B; ++u) {
        const double md = double(x[a][u]);
        const double *trow = S.T + (a * B + u) * B;
#pragma unroll
        for (int c = 0; c < B; ++c) out[c] = fma(md, trow[c], out[c]);
      }
    }
#pragma unroll
    for (int c = 0; c < B; ++c) sm[tid * LDR + c] = float(out[c]);
  }
  __syncthreads();
  // coalesced stores of the new rows, the gather rows, the pool columns
  for (int q = 0; q < sides; ++q) {
    float *vbase = (q ? P.s[1].vn : P.s[0].vn) + row0 * B;
    const float *o = sm + q * RN * LDR;
    if constexpr (B >= 4) {
      for (int i = tid; i < nrow * B / 4; i += 256) {
        const float *d = o + (4 * i / B) * LDR + (4 * i) % B;
        reinterpret_cast<float4 *>(vbase)[i] = make_float4(d[0], d[1], d[2], d[3]);
      }
    } else {
      for (int i = tid; i < nrow * B; i += 256) vbase[i] = o[(i / B) * LDR + i % B];
    }
  }
  if (!nodes) return;
  if (U) {
    float *ub = U + row0 * 2 * B;
    if constexpr (B >= 4) {
      for (int i = tid; i < nrow * B / 2; i += 256) {
        const int q = i / (B / 2), f = 4 * (i % (B / 2));  // row, first column of 2 B
        const float *d = sm + ((f / B) * RN + q) * LDR + f % B;
        const float g = sc[q];
        reinterpret_cast<float4 *>(ub)[i] =
            make_float4(d[0] * g, d[1] * g, d[2] * g, d[3] * g);
      }
    } else {
      for (int i = tid; i < nrow * 2 * B; i += 256) {
        const int q = i / (2 * B), f = i % (2 * B);
        ub[i] = sm[((f / B) * RN + q) * LDR + f % B] * sc[q];
      }
    }
  }
  if (pool) {
    // row-octet layout: per (octet, column) 8 consecutive values; rows past n
    // are zero (row0 is a multiple of 8)
    const int noct = (nrow + 7) / 8;
    for (int i = tid; i < 2 * noct * B; i += 256) {
      const int q = i / (noct * B), k = i % (noct * B);
      const int o = k / B, c = k % B;
      const float *d = sm + q * RN * LDR + c;
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = 8 * o + u < nrow ? d[(8 * o + u) * LDR] : 0.0f;
      const int col = (q ? P.s[1].col0 : P.s[0].col0) + c;
      pool_store8(pool, pool_type, (((row0 >> 3) + o) * K + col) * 8, v);
    }
  }
}

__host__ __device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
  uint64_t z = x + 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// N(0,1) element i of stream (seed, level, expansion): splitmix64 counter and
// Box-Muller, float64.  Two streams in one launch: elements [0, n0) are the
// first's, the others the second's.
__global__ void k_start(uint64_t h0, int64_t n0, float *__restrict__ out0, uint64_t h1, int64_t n1,
                        float *__restrict__ out1) {
  int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n0 + n1) return;
  const bool second = i >= n0;
  if (second) i -= n0;
  const uint64_t h = second ? h1 : h0;
  const uint64_t a = splitmix64(h + 2ull * uint64_t(i));
  const uint64_t c = splitmix64(h + 2ull * uint64_t(i) + 1ull);
  const double u1 = (double((a >> 11)) + 1.0) * 0x1.0p-53;
  const double u2 = double(c >> 11) * 0x1.0p-53;
  (second ? out1 : out0)[i] = float(sqrt(-2.0 * log(u1)) * cos(2.0 * M_PI * u2));
}

uint64_t stream_hash(uint64_t seed, int level, int expansion) {
  return splitmix64(splitmix64(seed) + 2ull * uint64_t(level) + uint64_t(expansion));
}

hef_status start_launch(uint64_t h0, int64_t n0, float *out0, uint64_t h1, int64_t n1, float *out1,
                        hipStream_t s) {
  if (n0 + n1 == 0) return HEF_OK;
  TimedScope ts(kStStart, s);
  k_start<<<cdiv(n0 + n1, 256), 256, 0, s>>>(h0, n0, out0, h1, n1, out1);
  HEF_LAUNCH_CHECK();
  return HEF_OK;
}

// Sides with zero rows launch nothing.
template <int B>
hef_status apply_t(const ApplySide &a, const ApplySide &b, void *pool, int pool_type,
                   int64_t pool_rows, int K, hipStream_t s) {
  constexpr int RB = B <= 8 ? 256 : 128;
  ApplyPair P;
  P.s[0] = a;
  P.s[1] = b;
  P.nb0 = cdiv(a.rows, RB);
  const int64_t nblk = P.nb0 + cdiv(b.rows, RB);
  if (nblk == 0) return HEF_OK;
  TimedScope ts(kStLanczosApply, s);
  k_lapply<B><<<nblk, 256, 0, s>>>(P, pool, pool_type, pool_rows, K);
  HEF_LAUNCH_CHECK();
  return HEF_OK;
}

// Both expansions of n node rows (a: star with n + m rows, b: clique) with
// the next product's gather rows.
template <int B>
hef_status apply_u_t(const ApplySide &a, const ApplySide &b, const float *scale, float *U,
                     void *pool, int pool_type, int K, hipStream_t s) {
  ApplyPair P;
  P.s[0] = a;
  P.s[1] = b;
  P.nb0 = 0;
  const int64_t n = b.rows, nbn = cdiv(n, 128);
  const int64_t nblk = nbn + cdiv(a.rows - n, 256);
  if (nblk == 0) return HEF_OK;
  TimedScope ts(kStLanczosApply, s);
  k_lapply_u<B><<<nblk, 256, 0, s>>>(P, n, nbn, scale, U, pool, pool_type, K);
  HEF_LAUNCH_CHECK();
  return HEF_OK;
}

hef_status lapply_u(int B, const ApplySide &a, const ApplySide &b, const float *scale, float *U,
                    void *pool, int pool_type, int K, hipStream_t s) {
  switch (B) {
    case 1: return apply_u_t<1>(a, b, scale, U, pool, pool_type, K, s);
    case 2: return apply_u_t<2>(a, b, scale, U, pool, pool_type, K, s);
    case 4: return apply_u_t<4>(a, b, scale, U, pool, pool_type, K, s);
    case 8: return apply_u_t<8>(a, b, scale, U, pool, pool_type, K, s);
    default: return HEF_ERR_UNSUPPORTED;
  }
}

hef_status lapply2(int B, const ApplySide &a, const ApplySide &b, void *pool, int pool_type,
                   int64_t pool_rows, int K, hipStream_t s) {
  switch (B) {
    case 1: return apply_t<1>(a, b, pool, pool_type, pool_rows, K, s);
    case 2: return apply_t<2>(a, b, pool, pool_type, pool_rows, K, s);
    case 4: return apply_t<4>(a, b, pool, pool_type, pool_rows, K, s);
    case 8: return apply_t<8>(a, b, pool, pool_type, pool_rows, K, s);
    case 16: return apply_t<16>(a, b, pool, pool_type, pool_rows, K, s);
    default: return HEF_ERR_UNSUPPORTED;
  }
}

// The Grams of up to two expansions (a side with y == nullptr is skipped),
// each over its own rows, and the solves of both: T = R^-1[:, y columns] and
// (if given) all of R^-1.
hef_status lgram_solve(int B, const float *v0a, const float *v1a, const float *ya, int64_t rowsa,
                       double *partiala, double *Ga, const float *v0b, const float *v1b,
                       const float *yb, int64_t rowsb, double *partialb, double *Gb, double tau,
                       double *T, double *R, hipStream_t s) {
  double *const G = Ga;  // (Ga and Gb are consecutive C x C matrices)
  const int C = 3 * B;
  const int S = (C % 6 == 0) ? 6 : 3;
  GramPair P;
  int nb[2] = {0, 0};
  const float *v0[2] = {v0a, v0b}, *v1[2] = {v1a, v1b}, *y[2] = {ya, yb};
  const int64_t rows[2] = {rowsa, rowsb};
  double *part[2] = {partiala, partialb};
  for (int i = 0; i < 2; ++i) {
    const int64_t per = std::max<int64_t>(64, cdiv(cdiv(rows[i], kGramBlocks), 64) * 64);
    nb[i] = y[i] ? int(std::max<int64_t>(1, cdiv(rows[i], per))) : 0;
    P.s[i] = GramSide{v0[i], v1[i], y[i], rows[i], per, part[i]};
  }
  P.nb0 = nb[0];
  const int nblk = nb[0] + nb[1];
  if (nblk == 0) return HEF_OK;
  {
  TimedScope ts(kStLanczosGram, s);
  switch (B) {
    case 1: k_lgram<1><<<nblk, 256, 0, s>>>(P); break;
    case 2: k_lgram<2><<<nblk, 256, 0, s>>>(P); break;
    case 4: k_lgram<4><<<nblk, 256, 0, s>>>(P); break;
    case 8: k_lgram<8><<<nblk, 256, 0, s>>>(P); break;
    case 16: k_lgram<16><<<nblk, 256, 0, s>>>(P); break;
    default: return HEF_ERR_UNSUPPORTED;
  }
  HEF_LAUNCH_CHECK();
  }
  if (C <= 6) {
    TimedScope ts(kStLanczosSolve, s);
    const int mask = (nb[0] > 0 ? 1 : 0) | (nb[1] > 0 ? 2 : 0);
    if (C == 3)
      k_lreduce_solve<3, 3><<<2, 1024, 0, s>>>(partiala, nb[0], partialb, nb[1], mask, B, tau, T, R);
    else
      k_lreduce_solve<6, 6><<<2, 1024, 0, s>>>(partiala, nb[0], partialb, nb[1], mask, B, tau, T, R);
    HEF_LAUNCH_CHECK();
    return HEF_OK;
  }
  {
  TimedScope ts(kStLanczosReduce, s);
  const int nbh = int(cdiv(int64_t(C) * C, 8));
  if (nb[0] > 0 && nb[1] > 0)
    k_gram_reduce<<<2 * nbh, 1024, 0, s>>>(partiala, nb[0], Ga, partialb, nb[1], Gb, nbh, C, S);
  else if (nb[0] > 0)
    k_gram_reduce<<<nbh, 1024, 0, s>>>(partiala, nb[0], Ga, nullptr, 0, nullptr, nbh, C, S);
  else
    k_gram_reduce<<<nbh, 1024, 0, s>>>(partialb, nb[1], Gb, nullptr, 0, nullptr, nbh, C, S);
  HEF_LAUNCH_CHECK();
  }
  TimedScope ts(kStLanczosSolve, s);
  return lsolve_launch(G, B, tau, T, R, s);
}

}  // namespace

hef_status lanczos_apply_pair(int B, const float *v0a, const float *v1a, const float *ya,
                              const double *Ta, float *vna, int64_t rowsa, const float *v0b,
                              const float *v1b, const float *yb, const double *Tb, float *vnb,
                              int64_t rowsb, int K, hipStream_t s) {
  const ApplySide a{v0a, v1a, ya, Ta, vna, rowsa, 0};
  const ApplySide b{v0b, v1b, yb, Tb, vnb, rowsb, 0};
  return lapply2(B, a, b, nullptr, 0, 0, K, s);
}

size_t krylov_ws_bytes(int64_t n, int64_t m, int B) {
  Arena a;
  for (int i = 0; i < 4; ++i) a.take<float>((n + m) * B);
  for (int i = 0; i < 4; ++i) a.take<float>(n * B);
  a.take<float>(spmm_scratch_floats(n, m, B));
  a.take<double>(size_t(2) * kGramBlocks * 9 * B * B);
  a.take<double>(2 * 48 * 48);
  a.take<double>(2 * 48 * 16);
  return a.mark();
}

hef_status start_block(uint64_t seed, int level, int expansion, int64_t rows, int B,
                       float *out, hipStream_t s) {
  return start_launch(stream_hash(seed, level, expansion), rows * B, out, 0, 0, nullptr, s);
}

hef_status start_blocks(uint64_t seed, int level, int64_t n, int64_t m, int B,
                        const float **star, const float **clique, float *xs, float *xc,
                        hipStream_t s) {
  const bool ds = star && !*star, dc = clique && !*clique;
  HEF_TRY(start_launch(stream_hash(seed, level, 0), ds ? (n + m) * B : 0, xs,
                       stream_hash(seed, level, 1), dc ? n * B : 0, xc, s));
  if (ds) *star = xs;
  if (dc) *clique = xc;
  return HEF_OK;
}

hef_status start_blocks(uint64_t seed, int level, int64_t n, int64_t m, int B,
                        const float **star, const float **clique, Arena &ws, hipStream_t s) {
  float *xs = star && !*star ? ws.take<float>((n + m) * B) : nullptr;
  float *xc = clique && !*clique ? ws.take<float>(n * B) : nullptr;
  HEF_WS_CHECK(ws);
  return start_blocks(seed, level, n, m, B, star, clique, xs, xc, s);
}

hef_status krylov_pool(const Level &L, const Structure &st, int B, int k, double tau,
                       const float *start_star, const float *start_clique, bool use_star,
                       bool use_clique, KrylovOut &out, Arena &ws, hipStream_t s,
                       const KrylovTape *tape) {
  const int64_t n = L.n, m = L.m;
  const int64_t Ns = n + m;
  const size_t mk = ws.mark();
  float *sb[4], *cb[4];
  for (int i = 0; i < 4; ++i) sb[i] = ws.take<float>(Ns * B);
  for (int i = 0; i < 4; ++i) cb[i] = ws.take<float>(n * B);
  float *tb = ws.take<float>(spmm_scratch_floats(n, m, B));
  double *partial = ws.take<double>(size_t(2) * kGramBlocks * 9 * B * B);
  double *G = ws.take<double>(2 * 48 * 48);
  double *Tm = ws.take<double>(2 * 48 * 16);
  HEF_WS_CHECK(ws);
  const int C = 3 * B;
  double *Gs = G, *Gc = G + C * C;
  double *ps = partial, *pc = partial + size_t(kGramBlocks) * 9 * B * B;
  // (the solve reads both expansions' Grams)
  if (!(use_star && use_clique)) HEF_TRY(zero_async(G, 2 * 48 * 48 * sizeof(double), s));
  // per-step T (and R^-1 for the adjoint)
  auto t_of = [&](int j) { return tape ? tape->T + size_t(j) * 2 * C * B : Tm; };
  auto r_of = [&](int j) { return tape ? tape->Rinv + size_t(j) * 2 * C * C : nullptr; };
  const int seg = tape ? (tape->seg > 0 && tape->seg < k ? tape->seg : k) : 0;
  // checkpoint slot j/seg <- (V_{j-1}, V_j) at the start of each segment
  auto checkpoint = [&](int j, const float *vs_prev, const float *vs, const float *vc_prev,
                        const float *vc) -> hef_status {
    if (!tape || j % seg != 0 || j >= k) return HEF_OK;
    const size_t slot = size_t(j / seg);
    if (use_star) {
      float *d = tape->ck_star + slot * 2 * Ns * B;
      if (vs_prev) HEF_HIP(hipMemcpyAsync(d, vs_prev, Ns * B * sizeof(float), hipMemcpyDeviceToDevice, s));
      else HEF_TRY(zero_async(d, Ns * B * sizeof(float), s));
      HEF_HIP(hipMemcpyAsync(d + Ns * B, vs, Ns * B * sizeof(float), hipMemcpyDeviceToDevice, s));
    }
    if (use_clique) {
      float *d = tape->ck_clique + slot * 2 * n * B;
      if (vc_prev) HEF_HIP(hipMemcpyAsync(d, vc_prev, n * B * sizeof(float), hipMemcpyDeviceToDevice, s));
      else HEF_TRY(zero_async(d, n * B * sizeof(float), s));
      HEF_HIP(hipMemcpyAsync(d + n * B, vc, n * B * sizeof(float), hipMemcpyDeviceToDevice, s));
    }
    return HEF_OK;
  };

  // the rolling buffers: prev, cur, y, next (as pointers: with a full tape
  // Y_j and V_j live in the tape's step buffers instead)
  const bool full = tape && seg == k && tape->y_s;
  const size_t scr = spmm_scratch_floats(n, m, B);
  const int K = out.K;
  const int64_t bk = int64_t(B) * k;
  // step j's SpMM scratch; with both expansions the apply before the step
  // fills its gather rows U
  // (b = 16 keeps the prep pass: k_lapply_u would hold 48 inputs a row and,
  // at 174 registers, 2 waves per SIMD)
  const bool both = use_star && use_clique && B <= 8;
  auto t_scr = [&](int j) { return full ? tape->t + size_t(j - 1) * scr : tb; };
  auto u_of = [&](int j) { return t_scr(j) + spmm_u_offset(m, B); };
  // V_0 = X R^-1 (no pool write).  The start blocks are read where they are,
  // or copied when a caller's are not aligned for 16-byte loads.
  const float *ys = start_star, *yc = start_clique;
  if (use_star && (reinterpret_cast<uintptr_t>(start_star) & 15)) {
    HEF_HIP(hipMemcpyAsync(sb[2], start_star, Ns * B * sizeof(float), hipMemcpyDeviceToDevice, s));
    ys = sb[2];
  }
  if (use_clique && (reinterpret_cast<uintptr_t>(start_clique) & 15)) {
    HEF_HIP(hipMemcpyAsync(cb[2], start_clique, n * B * sizeof(float), hipMemcpyDeviceToDevice, s));
    yc = cb[2];
  }
  HEF_TRY(lgram_solve(B, nullptr, nullptr, use_star ? ys : nullptr, Ns, ps, Gs, nullptr, nullptr,
                      use_clique ? yc : nullptr, n, pc, Gc, tau, t_of(0), r_of(0), s));
  {
    const ApplySide as{nullptr, nullptr, ys, t_of(0), sb[3], use_star ? Ns : 0, 0};
    const ApplySide ac{nullptr, nullptr, yc, t_of(0) + C * B, cb[3], use_clique ? n : 0, 0};
    if (both)
      HEF_TRY(lapply_u(B, as, ac, st.s, u_of(1), nullptr, 0, K, s));
    else
      HEF_TRY(lapply2(B, as, ac, nullptr, 0, 0, K, s));
  }
  HEF_TRY(checkpoint(0, nullptr, sb[3], nullptr, cb[3]));
  float *sp = nullptr, *sc = sb[3], *cp = nullptr, *cc = cb[3];  // prev (absent), cur
  // the rolling buffer that is neither prev, cur nor y (non-full runs)
  auto spare = [&](float *const *buf, const float *p, const float *c, const float *y) {
    for (int i = 0; i < 4; ++i)
      if (buf[i] != p && buf[i] != c && buf[i] != y) return buf[i];
    return buf[0];
  };
  for (int j = 1; j <= k; ++j) {
    float *sy = full ? tape->y_s + size_t(j - 1) * Ns * B : sb[2];
    float *cy = full ? tape->y_c + size_t(j - 1) * n * B : cb[2];
    HEF_TRY(spmm_apply(L, st, B, use_star ? sc : nullptr, use_star ? sy : nullptr,
                       use_clique ? cc : nullptr, use_clique ? cy : nullptr, t_scr(j), s, both));
    double *Tj = t_of(j);
    HEF_TRY(lgram_solve(B, sp, sc, use_star ? sy : nullptr, Ns, ps, Gs, cp, cc,
                        use_clique ? cy : nullptr, n, pc, Gc, tau, Tj, r_of(j), s));
    // V_j: a tape step buffer (j < k, full tape) or the spare rolling buffer
    float *sn = (full && j < k) ? tape->v_s + size_t(j - 1) * Ns * B
                                : spare(sb, sp, sc, full ? sb[2] : sy);
    float *cn = (full && j < k) ? tape->v_c + size_t(j - 1) * n * B
                                : spare(cb, cp, cc, full ? cb[2] : cy);
    const int64_t col_s = (j - 1) * int64_t(B);
    const int64_t col_c = (use_star ? bk : 0) + (j - 1) * int64_t(B);
    {
      const ApplySide as{sp, sc, sy, Tj, sn, use_star ? Ns : 0, int(col_s)};
      const ApplySide ac{cp, cc, cy, Tj + C * B, cn, use_clique ? n : 0, int(col_c)};
      if (both)
        HEF_TRY(lapply_u(B, as, ac, st.s, j < k ? u_of(j + 1) : nullptr, out.pool, out.pool_type,
                         K, s));
      else
        HEF_TRY(lapply2(B, as, ac, out.pool, out.pool_type, n, K, s));
    }
    HEF_TRY(checkpoint(j, sc, sn, cc, cn));
    sp = sc;
    sc = sn;
    cp = cc;
    cc = cn;
  }
  ws.reset(mk);
  return HEF_OK;
}

}  // namespace hef
