// Marginal covariances of the tracking Hessian (Sec. 3.1, Eq. 1 and 2) in
// FP64 on gfx950: the producer of the per-pixel depth variances Sigma_D that
// weight the depth loss (Eq. 4).
//
//   H_T     = C - E P^{-1} E^T                 (Schur complement, c x c)
//   H_T     = L L^T,  Sigma_T = (L L^T)^{-1}   (Cholesky, then L^{-T} L^{-1})
//   Sigma_d = 1/P_j + e_j^T Sigma_T e_j / P_j^2   (diagonal of Eq. 2)
//   Sigma_D = Sigma_d / d_j^4                  (first order, D = 1/d)
//
// c (6 per keyframe, at most 60) is small and p (pixels) large.  The three
// contractions (the Schur sum, X^T D^{-1} X and the quadratic forms) run on
// v_mfma_f64_16x16x4_f64: lane (g, i) = (lane/16, lane%16) gives A[i][k = g]
// and B[k = g][j = i] and holds rows 4 r + g of column i of the result.
// The window of 8 keyframes of 30 x 40 pixels (c = 48, p = 9600) is bound by
// the latency of its four launches and by the pivots of the factorisation,
// one after another.
#include "kernels.h"

namespace nsl {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ d4 mfma_f64(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

constexpr int kCovThreads = 256;
constexpr int kCovWaves = kCovThreads / kWave;
constexpr int kPixChunk = 256;  // pixels whose 1/sqrt(P) wait in LDS, a quarter of them a wave
constexpr int kMaxC = 60;       // largest c
constexpr int kPadC = 64;       // c rounded up to whole 16x16 tiles, at most

// The value of lane k (uniform) of the wave.
__device__ __forceinline__ double lane_value(double v, int k) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, k);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), k);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Tile t of the lower block triangle (rows of tiles: 0; 1, 2; 3, 4, 5; ...).
__device__ __forceinline__ void lower_tile(int t, int& m, int& n) {
  m = 0;
  while (t >= (m + 1) * (m + 2) / 2) ++m;
  n = t - m * (m + 1) / 2;
}

// partial[blk] = sum over the block's pixels of e_j e_j^T / P_j.  Workgroup
// (blk, tile): one 16x16 tile of the lower block triangle, whose four waves
// take a quarter of the pixels each (the transposed tile is written too).
// (110 -> 5 us at c = 48, p = 9600, against nine outputs a thread over pixels
// staged in LDS on 38 workgroups, two LDS reads a product.)
__global__ __launch_bounds__(kCovThreads) void schur_partial_kernel(const double* __restrict__ Et,
                                                                    const double* __restrict__ P, int c, int p,
                                                                    int per_block, double* __restrict__ partial) {
  __shared__ double inv[kPixChunk];
  __shared__ d4 sums[kCovWaves][kWave];
  const int j0 = (int)blockIdx.x * per_block, j1 = min(p, j0 + per_block);
  const int wave = (int)threadIdx.x / kWave, lane = lane_id(), g = lane >> 4, i = lane & 15;
  int m, n;
  lower_tile((int)blockIdx.y, m, n);
  const int row = 16 * m + i, col = 16 * n + i;
  d4 acc = {0.0, 0.0, 0.0, 0.0};
  for (int jc = j0; jc < j1; jc += kPixChunk) {
    const int np = min(kPixChunk, j1 - jc);
    __syncthreads();
    inv[threadIdx.x] = (int)threadIdx.x < np ? 1.0 / sqrt(P[jc + (int)threadIdx.x]) : 0.0;
    __syncthreads();
    constexpr int kSteps = kPixChunk / kCovWaves / 4;
    const int p0 = wave * (kPixChunk / kCovWaves) + g;
    double a[kSteps], b[kSteps];  // every load of the chunk in flight
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
      const bool on = p0 + 4 * s < np;
      const size_t at = (size_t)(jc + p0 + 4 * s) * c;
      a[s] = on && row < c ? Et[at + row] : 0.0;
      b[s] = on && col < c ? Et[at + col] : 0.0;
    }
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
      const double f = inv[p0 + 4 * s];
      acc = mfma_f64(a[s] * f, b[s] * f, acc);
    }
  }
  sums[wave][lane] = acc;
  __syncthreads();
  // wave w finishes result register w: row 16 m + 4 w + g
  double v = 0.0;
#pragma unroll
  for (int w = 0; w < kCovWaves; ++w) v += sums[w][lane][wave];
  const int r = 16 * m + 4 * wave + g;
  if (r >= c || col >= c) return;
  double* out = partial + (size_t)blockIdx.x * c * c;
  out[r * c + col] = v;
  out[col * c + r] = v;
}

// H = C - sum of partials (fixed order): a workgroup takes 16 elements, each
// of its 16 thread groups every 16th partial.
__global__ __launch_bounds__(256) void schur_reduce_kernel(const double* __restrict__ C,
                                                           const double* __restrict__ partial, int nblk, int cc,
                                                           double* __restrict__ H) {
  __shared__ double red[256];
  const int col = (int)threadIdx.x & 15, grp = (int)threadIdx.x >> 4, i = (int)blockIdx.x * 16 + col;
  double s = 0.0;
  if (i < cc) {
#pragma unroll 4
    for (int b = grp; b < nblk; b += 16) s += partial[(size_t)b * cc + i];
  }
  red[threadIdx.x] = s;
  __syncthreads();
  if (grp != 0 || i >= cc) return;
  s = 0.0;
#pragma unroll
  for (int k = 0; k < 16; ++k) s += red[16 * k + col];
  H[i] = C[i] - s;
}

// In place: H (c x c, symmetric positive definite; its lower triangle is
// read) -> Sigma_T = H^{-1} via H = L D L^T, that is the Cholesky factor
// without its square roots, and X = L^{-1}: Sigma_T = X^T D^{-1} X.
// status = 1 (and NaN output) if a pivot is not positive.
//
// One workgroup of 16 waves, each holding one 16x16 tile of the matrix as an
// MFMA result.  Four pivots a step: the four rows (register k0 / 4 % 4 of the
// tiles of one block row) go to wave 0, which eliminates them among themselves;
// one product of depth 4 a tile then eliminates every row below: the columns
// after the pivots become the next Schur complement, and those before and
// under them rows of X, in the place of what was eliminated.  The pivots, one
// division after another, bound it; row-at-a-time forms spent their time on
// broadcasts instead.  (c = 48: 143 us for a right-looking factorisation in LDS
// with three barriers a pivot and a forward substitution of one thread a
// column, 23 us one row at a time from registers, 16 us so.)
constexpr int kCholThreads = 1024;
__global__ __launch_bounds__(kCholThreads) void chol_inverse_kernel(double* __restrict__ H, int c,
                                                                    int* __restrict__ status) {
  __shared__ double raw[4][kPadC], left[4][kPadC], right[4][kPadC];
  __shared__ double X[kPadC][kPadC];
  __shared__ double dinv[kPadC];
  __shared__ int bad;
  constexpr int kWaves = kCholThreads / kWave;
  static_assert(kWaves * 256 == kPadC * kPadC, "one tile a wave");
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), j = lane_id();
  const int g = j >> 4, i = j & 15, tm = w >> 2, tn = w & 3;
  d4 acc;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = 16 * tm + 4 * r + g, col = 16 * tn + i;
    acc[r] = row < c && col < c ? H[max(row, col) * c + min(row, col)] : 0.0;
  }
  if (threadIdx.x == 0) bad = 0;
  for (int k0 = 0; k0 < c; k0 += 4) {
    const int tk = k0 >> 4, rk = (k0 >> 2) & 3;
    if (tm == tk) raw[g][16 * tn + i] = rk == 0 ? acc[0] : rk == 1 ? acc[1] : rk == 2 ? acc[2] : acc[3];
    __syncthreads();
    if (w == 0) {
      double x[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) x[t] = raw[t][j];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int k = k0 + t;
        const double d = lane_value(x[t], k);
        const bool in = k < c, ok = d > 0.0;
        const double r = in ? 1.0 / (ok ? d : 1.0) : 0.0;
        if (in && !ok) bad = 1;
        // row t against the rows after it: column k of those is eliminated,
        // and X[k][k] = 1 takes its place
        const double xt = j == k ? 1.0 : x[t];
#pragma unroll
        for (int u = t + 1; u < 4; ++u) {
          const double f = lane_value(x[t], k0 + u) * r;  // L[k0 + u][k]
          x[u] = fma(-f, xt, j == k ? 0.0 : x[u]);
        }
        const double b = !in || (j > k && j < k0 + 4) ? 0.0 : xt;
        right[t][j] = b;
        left[t][j] = j >= k0 + 4 ? -(x[t] * r) : 0.0;  // -L[j][k]
        X[k][j] = j <= k ? b : 0.0;
        if (j == 0) dinv[k] = r;
      }
    }
    __syncthreads();
    if (tn == tk && (i >> 2) == rk) acc = d4{0.0, 0.0, 0.0, 0.0};  // the eliminated columns
    acc = mfma_f64(left[g][16 * tm + i], right[g][16 * tn + i], acc);
  }
  const int tiles = (c + 15) / 16;
  if (w < tiles * (tiles + 1) / 2) {
    int m, n;
    lower_tile(w, m, n);
    d4 sum = {0.0, 0.0, 0.0, 0.0};
    for (int s = 0; s < (c + 3) / 4; ++s) {
      const int k = 4 * s + g;
      sum = mfma_f64(X[k][16 * m + i] * dinv[k], X[k][16 * n + i], sum);
    }
    const int col = 16 * n + i;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 16 * m + 4 * r + g;
      if (row >= c || col > row) continue;
      const double o = bad ? __longlong_as_double(0x7ff8000000000000ll) : sum[r];
      H[row * c + col] = o;
      H[col * c + row] = o;
    }
  }
  if (threadIdx.x == 0) *status = bad;
}

// Per pixel: sigma_d = 1/P + e^T Sigma_T e / P^2, depth_var = sigma_d / d^4.
// A wave takes 16 pixels: Y = Sigma_T E with the pixels as columns (Sigma_T in
// LDS, e in registers as the B operand of every product), whose result rows
// are the entries of e the same lane holds, so the dot product with e needs
// no move but the sum over the four lane groups.  (135 -> 5 us at c = 48, p = 9600, against one thread a pixel reading
// Sigma_T from LDS, whose reads of e were strided by c.)
__global__ __launch_bounds__(kCovThreads) void marginal_kernel(const double* __restrict__ Et,
                                                               const double* __restrict__ P,
                                                               const double* __restrict__ inv_depth,
                                                               const double* __restrict__ S, int c, int p,
                                                               double* __restrict__ sigma_d,
                                                               float* __restrict__ depth_var) {
  constexpr int kSteps = kPadC / 4;
  __shared__ double sh[kPadC][kPadC];
  const int wave = (int)threadIdx.x / kWave, lane = lane_id(), g = lane >> 4;
  const int j = ((int)blockIdx.x * kCovWaves + wave) * 16 + (lane & 15);
  double e[kSteps];
#pragma unroll
  for (int s = 0; s < kSteps; ++s) {
    const int b = 4 * s + g;
    e[s] = j < p && b < c ? Et[(size_t)j * c + b] : 0.0;
  }
  double st[kPadC / kCovWaves];  // this wave's rows of Sigma_T, the loads in flight together
#pragma unroll
  for (int r = 0; r < kPadC / kCovWaves; ++r) {
    const int a = wave + kCovWaves * r;
    st[r] = a < c && lane < c ? S[a * c + lane] : 0.0;
  }
#pragma unroll
  for (int r = 0; r < kPadC / kCovWaves; ++r) sh[wave + kCovWaves * r][lane] = st[r];
  __syncthreads();
  double q = 0.0;
#pragma unroll
  for (int m = 0; m < kPadC / 16; ++m) {
    if (16 * m >= c) continue;
    d4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < kSteps; ++s)
      if (4 * s < c) acc = mfma_f64(sh[4 * s + g][16 * m + (lane & 15)], e[s], acc);
#pragma unroll
    for (int r = 0; r < 4; ++r) q = fma(e[4 * m + r], acc[r], q);
  }
  q += __shfl_xor(q, 16, kWave);
  q += __shfl_xor(q, 32, kWave);
  if (g != 0 || j >= p) return;
  const double pi = 1.0 / P[j];
  const double sd = pi + pi * pi * q;
  if (sigma_d) sigma_d[j] = sd;
  if (depth_var) {
    const double d = inv_depth[j], d2 = d * d;
    depth_var[j] = (float)(sd / (d2 * d2));
  }
}

}  // namespace

size_t cov_partial_blocks(int p) { return (size_t)min(256, max(1, (p + 255) / 256)); }

hipError_t depth_covariance(int c, int p, const double* C, const double* Et, const double* P,
                            const double* inv_depth, double* sigma_T, double* sigma_d, float* depth_var,
                            int* status, double* partial, hipStream_t st) {
  const int nblk = (int)cov_partial_blocks(p);
  const int per_block = (p + nblk - 1) / nblk;
  const int cc = c * c, tiles = (c + 15) / 16;
  static_assert(kMaxC <= kPadC, "whole tiles");
  if (c > kMaxC) return hipErrorInvalidValue;
  hipLaunchKernelGGL(schur_partial_kernel, dim3(nblk, tiles * (tiles + 1) / 2), dim3(kCovThreads), 0, st, Et, P, c, p,
                     per_block, partial);
  hipLaunchKernelGGL(schur_reduce_kernel, dim3((cc + 15) / 16), dim3(256), 0, st, C, partial, nblk, cc, sigma_T);
  hipLaunchKernelGGL(chol_inverse_kernel, dim3(1), dim3(kCholThreads), 0, st, sigma_T, c, status);
  if (p > 0) {
    const int per = 16 * kCovWaves;  // pixels a workgroup
    hipLaunchKernelGGL(marginal_kernel, dim3((p + per - 1) / per), dim3(kCovThreads), 0, st, Et, P, inv_depth, sigma_T,
                       c, p, sigma_d, depth_var);
  }
  return hipGetLastError();
}

}  // namespace nsl
