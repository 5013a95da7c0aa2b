// Joint block orthonormalisation of the pool (Cholesky QR on matrix cores).
#pragma once

#include "common.hpp"

namespace hef {

size_t orth_ws_bytes(int64_t n, int K);

// Orthonormalises the Krylov pool (Alg. 1, the joint Gram-Schmidt
// of [star | clique]): G = V^T V (matrix-core tiles, float64 across row
// chunks), Cholesky G = R^T R in float64 with the drop rule (column j
// dropped when its Schur pivot <= tau^2 G_jj), Q = V R^-1.  `P` holds V in
// the row-octet layout (oct_rows(n) x K); Q goes to `out` (n x K row-major).
// `passes` = 2 repeats the factorisation on Q (keeping the first pass's
// drops), using P as scratch.  `keep_out` (device int32 [K], may be null)
// receives 1 for kept and 0 for dropped columns; `rinv_out` (device float64
// [Kp x Kp], Kp = K rounded up to 32, may be null) the last pass's R^-1
// (row-major, upper triangular, zero rows and columns for drops); `rho_out`
// (device float64 [K], may be null) the first pass's relative residuals
// rho_j = |R_jj| / ||V_j|| (0 for dropped columns).
hef_status orthonormalize_pool(void *P, void *out, int pool_type, int64_t n, int K, double tau,
                               int passes, int32_t *keep_out, Arena &ws, hipStream_t s,
                               double *rinv_out = nullptr, double *rho_out = nullptr);

// Test hook: G = X^T X (float64, K x K) of a row-major n x K float32 matrix,
// through the same matrix-core Gram kernels.
hef_status gram_f32(const float *X, int64_t n, int K, double *G, Arena &ws, hipStream_t s);

// G = sym(X^T W) (float64, K x K) of two row-major n x K float32 matrices, the
// lower triangle of X^T W mirrored, through the same kernels; scratch
// gram_cross_ws_bytes(n, K).
size_t gram_cross_ws_bytes(int64_t n, int K);
hef_status gram_cross_f32(const float *X, const float *W, int64_t n, int K, double *G, Arena &ws,
                          hipStream_t s);

// out (n x K) = X W1 + X2 W2 for general row-major float32 X, X2, a lower
// triangular W1 and a general W2 (K x K), given transposed (W1T[j][i] =
// W1[gemm2_k(i)][j], row stride Kp, zero outside K x K), on the matrix cores.
__host__ __device__ inline int gemm2_k(int i) {
  return (i & ~31) + 2 * (i & 15) + ((i >> 4) & 1);
}
hef_status gemm2_f32(const float *X, const float *W1T, const float *X2, const float *W2T,
                     int64_t n, int K, int Kp, float *out, hipStream_t s);

}  // namespace hef
