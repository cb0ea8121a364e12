// Hash-grid field on gfx950: density/colour MLP forward, the recompute adjoint
// (MLP forward again, MLP backward with weight gradients and dL/de), and fused
// rendering.
//
// One wave evaluates 16 samples: lane (g, j) = (lane/16, lane%16) takes
// levels g, g+4, ... of sample j (given, or gathered here), which are exactly
// its B-operand slots of the first MFMA layer (net.h).  Nothing but sigma and
// colour leaves the forward kernel; the backward kernel computes every
// activation again instead of reading stored ones.
#include <algorithm>
#include <type_traits>

#include "bf16_ops.h"
#include "bins.h"
#include "field_common.h"
#include "march_common.h"

namespace nsl {

// ---------------------------------------------------------------------------
// MLP forward (activations kept for the adjoint)
// ---------------------------------------------------------------------------

template <class N>
struct Acts {
  float e[N::NSLOT];
  f4 h1[N::HD / 16];
  f4 o;
  float sh[4];
  f4 h3[N::HC / 16];
  f4 h4[N::HC / 16];
  f4 z;
};

template <class N>
__device__ __forceinline__ void mlp_fwd(const float* __restrict__ Af, int lane, Acts<N>& a) {
  auto w = [&](int j, int m, int s) { return Af[N::foff(j) + (m * N::fks(j) + s) * kWave + lane]; };
  constexpr f4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
  // layer 0: encoding -> h1
  {
    f4 acc[N::HD / 16];
#pragma unroll
    for (int m = 0; m < N::HD / 16; ++m) acc[m] = zero;
#pragma unroll
    for (int s = 0; s < N::fks(0); ++s)
#pragma unroll
      for (int m = 0; m < N::HD / 16; ++m) acc[m] = mfma4(w(0, m, s), a.e[s], acc[m]);
#pragma unroll
    for (int m = 0; m < N::HD / 16; ++m) a.h1[m] = relu4(acc[m]);
  }
  // layer 1: h1 -> o (geometry, 16)
  {
    f4 acc = zero;
#pragma unroll
    for (int s = 0; s < N::fks(1); ++s) acc = mfma4(w(1, 0, s), a.h1[s >> 2][s & 3], acc);
    a.o = acc;
  }
  // layer 2: [o, sh] -> h3
  {
    f4 acc[N::HC / 16];
#pragma unroll
    for (int m = 0; m < N::HC / 16; ++m) acc[m] = zero;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const float b = s < 4 ? a.o[s & 3] : a.sh[s & 3];
#pragma unroll
      for (int m = 0; m < N::HC / 16; ++m) acc[m] = mfma4(w(2, m, s), b, acc[m]);
    }
#pragma unroll
    for (int m = 0; m < N::HC / 16; ++m) a.h3[m] = relu4(acc[m]);
  }
  const f4* hl = a.h3;
  if constexpr (N::NCH == 2) {
    f4 acc[N::HC / 16];
#pragma unroll
    for (int m = 0; m < N::HC / 16; ++m) acc[m] = zero;
#pragma unroll
    for (int s = 0; s < N::HC / 4; ++s)
#pragma unroll
      for (int m = 0; m < N::HC / 16; ++m)
        acc[m] = mfma4(w(3, m, s), a.h3[s >> 2][s & 3], acc[m]);
#pragma unroll
    for (int m = 0; m < N::HC / 16; ++m) a.h4[m] = relu4(acc[m]);
    hl = a.h4;
  }
  // last layer -> z (rows 0..2 valid, held by lane group 0)
  {
    f4 acc = zero;
#pragma unroll
    for (int s = 0; s < N::HC / 4; ++s) acc = mfma4(w(N::NW - 1, 0, s), hl[s >> 2][s & 3], acc);
    a.z = acc;
  }
}

// ---------------------------------------------------------------------------
// Weight-operand preparation (once per step from the FP32 parameters)
// ---------------------------------------------------------------------------

template <class N>
__device__ __forceinline__ void prep_weight(const float* __restrict__ params, const WOffsets& wo,
                                            float* __restrict__ out, int idx) {
  if (idx >= N::FWD_FLOATS + N::BWD_FLOATS) return;
  float v = 0.0f;
  if (idx < N::FWD_FLOATS) {
    int j = 0;
    while (j + 1 < N::NW && idx >= N::foff(j + 1)) ++j;
    const int r = idx - N::foff(j);
    const int lane = r % kWave, ms = r / kWave;
    const int s = ms % N::fks(j), m = ms / N::fks(j);
    const int g = lane >> 4, i = lane & 15;
    const int row = fwd_in_feature<N>(j, s, g), col = 16 * m + i;
    if (row >= 0 && row < N::kin(j) && col < N::kout(j)) v = params[wo.off[j] + row * N::kout(j) + col];
  } else {
    const int b = idx - N::FWD_FLOATS;
    int j = 0;
    while (j + 1 < N::NW && b >= N::boff(j + 1)) ++j;
    const int r = b - N::boff(j);
    const int lane = r % kWave, ms = r / kWave;
    const int s = ms % N::bks(j), m = ms / N::bks(j);
    const int g = lane >> 4, i = lane & 15;
    const int row = bwd_row_feature<N>(j, m, i), col = bwd_k_feature<N>(j, s, g);
    if (row >= 0 && row < N::kin(j) && col < N::kout(j)) v = params[wo.off[j] + row * N::kout(j) + col];
  }
  out[idx] = v;
}

template <class N>
__global__ __launch_bounds__(256) void prep_weights_kernel(const float* __restrict__ params, WOffsets wo,
                                                           float* __restrict__ out) {
  prep_weight<N>(params, wo, out, (int)(blockIdx.x * 256 + threadIdx.x));
}

// The FP32 step's first launch: workgroups [0, ncount) set up the candidate
// rays and count their samples, the next nfill clear zero[0, nzero) and the
// rest lay out the weight operands; the first thread resets clear_flag (may be
// null).  As three launches, each waiting for the one before, 18.2 us at 4096 rays
// of the paper-scale map and 7.5 at 1024 of the tiny field; so 10.5 and 3.9.
template <class N>
__global__ __launch_bounds__(256) void prepare_count_kernel(const float* __restrict__ params, WOffsets wo,
                                                            float* __restrict__ out, float* __restrict__ zero,
                                                            int64_t nzero, int nfill, float* __restrict__ clear_flag,
                                                            KeyframeStore kf, MarchParams mp,
                                                            const uint32_t* __restrict__ ids, int n, RayBuffers rb,
                                                            int ncount) {
  if (clear_flag && blockIdx.x == 0 && threadIdx.x == 0) *clear_flag = 0.0f;
  const int b = (int)blockIdx.x - ncount;
  if (b < 0) {
    march_detail::rays_count_block(kf, mp, ids, n, rb, (int)blockIdx.x);
  } else if (b < nfill) {
    const int64_t i = ((int64_t)b * 256 + threadIdx.x) * 4;
    if (i + 4 <= nzero) {
      *reinterpret_cast<float4*>(zero + i) = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    } else {
      for (int64_t k = i; k < nzero; ++k) zero[k] = 0.0f;
    }
  } else {
    prep_weight<N>(params, wo, out, (b - nfill) * 256 + (int)threadIdx.x);
  }
}

// ---------------------------------------------------------------------------
// Forward: sigma and colour per sample
// ---------------------------------------------------------------------------

// Inputs of one sample for the MLP from the kept encoding: this lane's
// encoding slots and the ray direction (ray index ridx, fetched earlier).
template <class N>
__device__ __forceinline__ void fetch_kept(const SampleSrc& src, int g, int s, bool valid, uint32_t ridx,
                                           float e[N::NSLOT], float d[3]) {
  read_encoding<N>(static_cast<const float2*>(src.ecache), src.ecache_stride, g, s, valid, e);
  d[0] = 0.0f; d[1] = 0.0f; d[2] = 1.0f;
  if (valid) {
    if (src.t) {
      const float4 dd = src.rays[2 * ridx + 1];
      d[0] = dd.x; d[1] = dd.y; d[2] = dd.z;
    } else {
#pragma unroll
      for (int i = 0; i < 3; ++i) d[i] = src.dir[3 * s + i];
    }
  }
}

template <class N>
__device__ __forceinline__ void fwd_tile_out(const float* Af, int lane, int g, int s, bool valid, Acts<N>& act,
                                             const float d[3], float* __restrict__ sigma_out,
                                             float* __restrict__ rgb_out) {
  sh_lane<N>(d, g, act.sh);
  mlp_fwd<N>(Af, lane, act);
  if (g == 0 && valid) {
    sigma_out[s] = __expf(act.o[0]) ;
    rgb_out[3 * s + 0] = sigmoidf(act.z[0]);
    rgb_out[3 * s + 1] = sigmoidf(act.z[1]);
    rgb_out[3 * s + 2] = sigmoidf(act.z[2]);
  }
}

// Forward of 16-sample tiles, one per wave at a time, on a fixed grid (the
// weight operands are staged into LDS once per workgroup); with the kept
// encoding a wave fetches its next tile's inputs while it computes the
// current one (ray indices two tiles ahead).
constexpr int kFieldFwdGrid = 768;

// Workgroups past the MLP's (bp.nbins of them) run the table-gradient column
// scan (bins.h), which needs only the record counts of the encoding.
template <class N>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void field_fwd_kernel(FieldArgs a, SampleSrc src,
                                                        float* __restrict__ sigma_out,
                                                        float* __restrict__ rgb_out, BinPrep bp) {
  const int G = (int)gridDim.x - bp.nbins;  // the MLP's workgroups
  if ((int)blockIdx.x >= G) {
    colscan_bin(bp.rb, bp.nunits, (int)blockIdx.x - G);
    return;
  }
  __shared__ __attribute__((aligned(16))) float Af[N::FWD_FLOATS];
  copy_to_lds<256, sizeof(Af)>(Af, a.wprep);
  __syncthreads();
  const int S = src.n_dev ? (int)*src.n_dev : src.n;
  const int ntiles = (S + 15) / 16;
  const int lane = lane_id(), g = lane >> 4, jc = lane & 15;
  const int first = blockIdx.x * (blockDim.x / kWave) + (threadIdx.x / kWave);
  const int step = G * (blockDim.x / kWave);
  if (first >= ntiles) return;
  if (src.ecache) {
    auto rid = [&](int s) -> uint32_t { return src.t && s < S ? src.ray[s] : 0u; };
    float e[N::NSLOT], d[3];
    const int s0 = 16 * first + jc;
    fetch_kept<N>(src, g, s0, s0 < S, rid(s0), e, d);
    uint32_t rid1 = rid(s0 + 16 * step);
    for (int tile = first; tile < ntiles; tile += step) {
      const int s = 16 * tile + jc, s1 = s + 16 * step;
      float en[N::NSLOT], dn[3];
      fetch_kept<N>(src, g, s1, s1 < S, rid1, en, dn);
      rid1 = rid(s1 + 16 * step);
      Acts<N> act;
#pragma unroll
      for (int k = 0; k < N::NSLOT; ++k) act.e[k] = e[k];
      fwd_tile_out<N>(Af, lane, g, s, s < S, act, d, sigma_out, rgb_out);
#pragma unroll
      for (int k = 0; k < N::NSLOT; ++k) e[k] = en[k];
#pragma unroll
      for (int i = 0; i < 3; ++i) d[i] = dn[i];
    }
  } else {
    LaneLevels<N> ll;
    lane_levels<N>(a.lv, g, ll);
    for (int tile = first; tile < ntiles; tile += step) {
      const int s = 16 * tile + jc;
      const bool valid = s < S;
      Acts<N> act;
      float xn[3] = {0.5f, 0.5f, 0.5f}, d[3] = {0.0f, 0.0f, 1.0f};
      if (valid) load_sample(src, s, xn, d);
      encode<N>(a.table, a.lv.table_mask, ll, xn, act.e);
      fwd_tile_out<N>(Af, lane, g, s, valid, act, d, sigma_out, rgb_out);
    }
  }
}

// ---------------------------------------------------------------------------
// Backward
// ---------------------------------------------------------------------------

constexpr int kBwdStep = 16 * kFieldBwdWaves;  // samples of a workgroup's step
constexpr int kBwdRow = kBwdStep + 4;          // floats of a staged row (the pad steps rows through the LDS banks)

// Weight gradient of layer J, kin x kout in 16x16 tiles: the workgroup's waves
// own consecutive tiles, or with fewer tiles than waves share one, each taking
// its part of a step's samples.  Tile (m, n), lane (gk, i) holds
// dW[16m + 4gk + r][16n + i], in two sums so that products in a row are independent.
template <class N, int J>
struct OwnedDW {
  static constexpr int W = kFieldBwdWaves;
  static constexpr int MI = (N::kin(J) + 15) / 16, NJ = (N::kout(J) + 15) / 16, TILES = MI * NJ;
  static_assert(TILES % W == 0 || W % TILES == 0, "whole tiles a wave or whole waves a tile");
  static constexpr int SLOTS = TILES >= W ? TILES / W : 1, SPLIT = TILES >= W ? 1 : W / TILES;
  static constexpr int CHUNKS = W / SPLIT;  // 16-sample pieces of a step a wave takes
  f4 v[SLOTS][2];
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int k = 0; k < SLOTS; ++k) v[k][0] = v[k][1] = f4{0.0f, 0.0f, 0.0f, 0.0f};
  }
  static __device__ __forceinline__ int tile(int w, int k) { return SPLIT == 1 ? w * SLOTS + k : w % TILES; }
  __device__ __forceinline__ void chunk(const float* Xs, const float* Ys, int w, int lane, int c, int odd) {
    const int gk = lane >> 4, i = lane & 15;
#pragma unroll
    for (int k = 0; k < SLOTS; ++k) {
      const int t = tile(w, k), m = t / NJ, n = t % NJ;
      const f4 x = *reinterpret_cast<const f4*>(Xs + (16 * m + i) * kBwdRow + 16 * c + 4 * gk);
      const f4 y = *reinterpret_cast<const f4*>(Ys + (16 * n + i) * kBwdRow + 16 * c + 4 * gk);
#pragma unroll
      for (int q = 0; q < 4; ++q) v[k][odd] = mfma4(x[q], y[q], v[k][odd]);
    }
  }
  // += X^T dY over the step's first nt pieces of 16 samples, staged
  // [feature][sample]
  __device__ __forceinline__ void add(const float* Xs, const float* Ys, int w, int lane, int nt) {
    const int c0 = SPLIT == 1 ? 0 : w / TILES * CHUNKS;
    if (nt == W) {
#pragma unroll
      for (int c = 0; c < CHUNKS; ++c) chunk(Xs, Ys, w, lane, c0 + c, c & 1);
    } else {
#pragma unroll 1
      for (int c = c0; c < min(nt, c0 + CHUNKS); ++c) chunk(Xs, Ys, w, lane, c, 0);
    }
  }
  // The workgroup's sums to out (row-major kin x kout); waves that share a
  // tile meet in LDS.
  __device__ __forceinline__ void store(float* lds, float* __restrict__ out, int w, int lane) const {
    const int gk = lane >> 4, i = lane & 15;
    if constexpr (SPLIT > 1) {
      __syncthreads();
      *reinterpret_cast<f4*>(lds + (w * kWave + lane) * 4) = v[0][0] + v[0][1];
      __syncthreads();
      if (w >= TILES) return;
    }
#pragma unroll
    for (int k = 0; k < SLOTS; ++k) {
      const int t = tile(w, k), m = t / NJ, n = t % NJ, col = 16 * n + i;
      f4 sum = v[k][0] + v[k][1];
      if constexpr (SPLIT > 1) {
#pragma unroll
        for (int p = 1; p < SPLIT; ++p) sum += *reinterpret_cast<const f4*>(lds + ((w + p * TILES) * kWave + lane) * 4);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * m + 4 * gk + r;
        if (row < N::kin(J) && col < N::kout(J)) out[row * N::kout(J) + col] = sum[r];
      }
    }
  }
};

// Stage a D-layout activation block (tiles of 16 rows) from row S on.
template <int TILES>
__device__ __forceinline__ void stage_d(float* S, const f4* v, int g) {
#pragma unroll
  for (int m = 0; m < TILES; ++m)
#pragma unroll
    for (int r = 0; r < 4; ++r) S[(16 * m + 4 * g + r) * kBwdRow] = v[m][r];
}

// out[m] = sum over the k-steps s of W (tile m, step s; 64 floats each from A
// on) times x(s).
template <int MT, int KS, class X>
__device__ __forceinline__ void bwd_products(const float* A, int lane, const X& x, f4 (&out)[MT]) {
#pragma unroll
  for (int m = 0; m < MT; ++m) out[m] = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int s = 0; s < KS; ++s)
#pragma unroll
    for (int m = 0; m < MT; ++m) out[m] = mfma4(A[(m * KS + s) * kWave + lane], x(s), out[m]);
}

// acc where the ReLU output h is above zero, else 0.
template <int K>
__device__ __forceinline__ void relu_mask(f4 (&acc)[K], const f4 (&h)[K]) {
#pragma unroll
  for (int m = 0; m < K; ++m)
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[m][r] = h[m][r] > 0.0f ? acc[m][r] : 0.0f;
}

// Eight waves a workgroup, two a SIMD.  Each wave recomputes the forward and
// runs the input-gradient chain of 16 samples; the 128 samples of the
// workgroup's step are staged a layer at a time, and each wave adds the
// products of its own weight-gradient tiles over all of them.  It then holds
// six of the 40 tiles instead of all, which leaves the registers for a second wave
// on the SIMD: bound by the FP32 matrix instructions, and a lone wave idles them
// whenever it waits for its own operands (60% busy, also with two tiles of 16
// samples at a time).  At 262k samples of the 64-wide network 177 us with four
// waves that hold all tiles, 148 so, of which 98 are matrix cycles; at 49999 samples
// 51.8 and 42; the 32-wide network at 131072 samples 36.3 and 30.7.
template <class N>
__global__ __launch_bounds__(kFieldBwdWaves * kWave, 2) void field_bwd_kernel(FieldArgs a, SampleSrc src,
                                                           const float* __restrict__ dsigma,
                                                           const float* __restrict__ drgb, RecordBuffers rec,
                                                           float* __restrict__ dw_partial) {
  constexpr int kOps = N::FWD_FLOATS + N::BWD_FLOATS, H = N::HC / 16, D = N::HD / 16;
  __shared__ __attribute__((aligned(16))) float ops[kOps];
  __shared__ __attribute__((aligned(16))) float stage[(N::XROWS + N::YROWS) * kBwdRow];
  const float *Af = ops, *Ab = ops + N::FWD_FLOATS;
  copy_to_lds<kFieldBwdWaves * kWave, (int)sizeof(ops)>(ops, a.wprep);
  __syncthreads();

  const uint32_t S = src.n_dev ? *src.n_dev : (uint32_t)src.n;
  const int w = threadIdx.x / kWave;
  const int lane = lane_id(), g = lane >> 4, jc = lane & 15;
  const float *Xs = stage, *Ys = stage + N::XROWS * kBwdRow;
  float *Xw = stage + 16 * w + jc, *Yw = Xw + N::XROWS * kBwdRow;  // this lane's column
  LaneLevels<N> ll;
  if constexpr (kGathers<N>) lane_levels<N>(a.lv, g, ll);
  OwnedDW<N, 0> dw0;
  OwnedDW<N, 1> dw1;
  OwnedDW<N, 2> dw2;
  OwnedDW<N, N::NCH == 2 ? 3 : 2> dw3;  // second colour hidden layer (unused with one)
  OwnedDW<N, N::NW - 1> dwl;
  dw0.zero(); dw1.zero(); dw2.zero(); dwl.zero();
  if constexpr (N::NCH == 2) dw3.zero();

  // inputs of a tile: encoding slots, direction and (lane group 0) seeds; with
  // the encoding given, those of the next step are fetched while this one is
  // computed (ray indices two steps ahead)
  struct In {
    float e[N::NSLOT], d[3], ds, dr[3];
  };
  auto rid = [&](uint32_t s) -> uint32_t { return src.t && s < S ? src.ray[s] : 0u; };
  auto seeds = [&](uint32_t s, In& in) {
    in.ds = in.dr[0] = in.dr[1] = in.dr[2] = 0.0f;
    if (g != 0 || s >= S) return;
    in.ds = dsigma[s];
#pragma unroll
    for (int r = 0; r < 3; ++r) in.dr[r] = drgb[3 * (size_t)s + r];
  };
  const uint32_t stride = kBwdStep * gridDim.x;  // samples
  In in;
  uint32_t rid1 = 0u;
  const bool given = src.ecache;  // (with the larger networks always)
  if (given) {
    const uint32_t s0 = kBwdStep * blockIdx.x + 16 * w + jc;
    fetch_kept<N>(src, g, s0, s0 < S, rid(s0), in.e, in.d);
    seeds(s0, in);
    rid1 = rid(s0 + stride);
  }
  for (uint32_t p = kBwdStep * blockIdx.x; p < S; p += stride) {
    const uint32_t s = p + 16 * w + jc;
    const bool valid = s < S;
    const int nt = (int)min((uint32_t)kFieldBwdWaves, (S - p + 15) / 16);  // tiles of 16 samples in this step
    In next;
    if (given) {
      const uint32_t s1 = s + stride;
      fetch_kept<N>(src, g, s1, s1 < S, rid1, next.e, next.d);
      seeds(s1, next);
      rid1 = rid(s1 + stride);
    } else if constexpr (kGathers<N>) {
      float xn[3] = {0.5f, 0.5f, 0.5f};
      in.d[0] = in.d[1] = 0.0f;
      in.d[2] = 1.0f;
      if (valid) load_sample(src, s, xn, in.d);
      encode<N>(a.table, a.lv.table_mask, ll, xn, in.e);
      if (!valid) {
#pragma unroll
        for (int k = 0; k < N::NSLOT; ++k) in.e[k] = 0.0f;
      }
      seeds(s, in);
      next = in;
    } else {
      next = in;  // (never: but without a branch here the loop took 151 us instead of 147 at 262144 samples)
    }
    Acts<N> act;
#pragma unroll
    for (int k = 0; k < N::NSLOT; ++k) act.e[k] = in.e[k];
    sh_lane<N>(in.d, g, act.sh);
    mlp_fwd<N>(Af, lane, act);

    // seeds: dz = dc * c (1 - c) and dsigma, on lane group 0
    f4 dz = {0.0f, 0.0f, 0.0f, 0.0f};
    if (g == 0) {
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        const float c = sigmoidf(act.z[r]);
        dz[r] = in.dr[r] * c * (1.0f - c);
      }
    }
    // last layer: dh_last = W_last dz, masked
    const f4(&hl)[H] = N::NCH == 2 ? act.h4 : act.h3;
    f4 dhl[H];
    bwd_products<H, 3>(Ab + N::boff(N::NW - 1), lane, [&](int k) { return dz[k]; }, dhl);
    relu_mask(dhl, hl);
    // Between the two barriers of a layer, the weight-gradient products of
    // the step's samples and the next input-gradient product, which are independent.
    __syncthreads();
    stage_d<H>(Xw, hl, g);
    stage_d<1>(Yw, &dz, g);
    __syncthreads();
    dwl.add(Xs, Ys, w, lane, nt);
    f4 dh3[H];
    if constexpr (N::NCH == 2) {
      bwd_products<H, N::HC / 4>(Ab + N::boff(3), lane, [&](int k) { return dhl[k >> 2][k & 3]; }, dh3);
      relu_mask(dh3, act.h3);
      __syncthreads();
      stage_d<H>(Xw, act.h3, g);
      stage_d<H>(Yw, dhl, g);
      __syncthreads();
      dw3.add(Xs, Ys, w, lane, nt);
    } else {
#pragma unroll
      for (int m = 0; m < H; ++m) dh3[m] = dhl[m];
    }
    // colour input layer: d(geo) = W3[geo rows] dh3; dW3 with X = [o, sh]
    f4 dgeo[1];
    bwd_products<1, N::HC / 4>(Ab + N::boff(2), lane, [&](int k) { return dh3[k >> 2][k & 3]; }, dgeo);
    __syncthreads();
    stage_d<1>(Xw, &act.o, g);
#pragma unroll
    for (int r = 0; r < 4; ++r) Xw[(16 + 4 * g + r) * kBwdRow] = act.sh[r];
    stage_d<H>(Yw, dh3, g);
    __syncthreads();
    dw2.add(Xs, Ys, w, lane, nt);
    // density output: do = dgeo, do_0 += sigma * dsigma
    if (g == 0) dgeo[0][0] += __expf(act.o[0]) * in.ds;
    f4 dh1[D];
    bwd_products<D, 4>(Ab + N::boff(1), lane, [&](int k) { return dgeo[0][k]; }, dh1);
    relu_mask(dh1, act.h1);
    __syncthreads();
    stage_d<D>(Xw, act.h1, g);
    stage_d<1>(Yw, dgeo, g);
    __syncthreads();
    dw1.add(Xs, Ys, w, lane, nt);
    // encoding gradient: de = W1 dh1 (rows = this lane group's slots)
    constexpr int MT0 = N::bmt(0);
    f4 de[MT0];
    bwd_products<MT0, N::HD / 4>(Ab + N::boff(0), lane, [&](int k) { return dh1[k >> 2][k & 3]; }, de);
    // dL/de of this lane's levels g + 4q, level-major: the 16 lanes of a row
    // store 16 consecutive samples of one level
    if (valid) {
#pragma unroll
      for (int q = 0; q < N::LPL; ++q) {
        const int k0 = 2 * q, k1 = 2 * q + 1;
        rec.de[(size_t)(g + 4 * q) * rec.stride + s] = make_float2(de[k0 >> 2][k0 & 3], de[k1 >> 2][k1 & 3]);
      }
    }
    // dW1 with X = e (slots -> features; rows past the features feed no weight)
    __syncthreads();
#pragma unroll
    for (int k = 0; k < N::NSLOT; ++k) Xw[fwd_in_feature<N>(0, k, g) * kBwdRow] = act.e[k];
    stage_d<D>(Yw, dh1, g);
    __syncthreads();
    dw0.add(Xs, Ys, w, lane, nt);
    in = next;
  }
  float* out = dw_partial + (size_t)blockIdx.x * N::NWEIGHTS;
  dw0.store(stage, out + N::woff(0), w, lane);
  dw1.store(stage, out + N::woff(1), w, lane);
  dw2.store(stage, out + N::woff(2), w, lane);
  if constexpr (N::NCH == 2) dw3.store(stage, out + N::woff(3), w, lane);
  dwl.store(stage, out + N::woff(N::NW - 1), w, lane);
}

// Networks whose rendering runs on the BF16 matrix cores in three parts
// (bf16_ops.h): the 64-wide ones, whose FP32 products would take 2.6 ms of
// matrix cycles at 640x480 x 64 samples.  There 4.41 ms with FP32 products and
// 3.98 so, at 320x240 1.65 and 1.60, at 160x120 0.62 and 0.61; the errors of the
// outputs against 64 bits are the same with either.  (Training keeps FP32 products throughout: a
// table entry's gradient may be a small residue of its terms, and the optimiser
// divides it by its own size.)
template <class N>
constexpr bool kSplitNet = N::HD >= 64;

// The forward operands in three BF16 parts, each part laid out like the mixed
// precision's (split_mlp).
template <class N>
__device__ __forceinline__ void prep_split(const float* __restrict__ params, const WOffsets& wo,
                                           __bf16* __restrict__ out, int idx) {
  using M = Mixed<N>;
  if (idx >= M::FWD) return;
  int j = 0;
  while (j + 1 < N::NW && idx >= M::foff(j + 1)) ++j;
  const int r = idx - M::foff(j);
  const int u = r % 8, lane = (r / 8) % kWave, ms = r / M::BLK;
  const int s = ms % M::fks(j), m = ms / M::fks(j);
  const int row = mixed_fwd_feature<N>(j, s, lane >> 4, u), col = 16 * m + (lane & 15);
  float v = row >= 0 && row < N::kin(j) && col < N::kout(j) ? params[wo.off[j] + row * N::kout(j) + col] : 0.0f;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const __bf16 h = (__bf16)v;
    out[c * M::FWD + idx] = h;
    v -= (float)h;
  }
}

// The operands of the rendering, and (with dst) the request record, whose pose
// and intrinsics come from device memory: one launch.
template <class N>
__global__ __launch_bounds__(256) void render_prep_kernel(const float* __restrict__ params, WOffsets wo,
                                                          void* __restrict__ out, nsl_render_request r,
                                                          const float* __restrict__ pose,
                                                          const float* __restrict__ intr, nsl_render_request* dst) {
  const int idx = (int)(blockIdx.x * 256 + threadIdx.x);
  if constexpr (kSplitNet<N>)
    prep_split<N>(params, wo, static_cast<__bf16*>(out), idx);
  else
    prep_weight<N>(params, wo, static_cast<float*>(out), idx);
  if (!dst || blockIdx.x != gridDim.x - 1 || threadIdx.x != 255) return;
#pragma unroll
  for (int i = 0; i < 12; ++i) r.pose[i] = pose[i];
#pragma unroll
  for (int i = 0; i < 4; ++i) r.intr[i] = intr[i];
  *dst = r;
}

// One tile with FP32 products, its weights from the parameter vector: for
// columns that split_mlp cannot represent (values that are not finite).  The
// loops over a layer's tiles stay rolled: these tiles are rare, and the
// registers are the fast path's.
template <class N, int J>
__device__ __forceinline__ void fp32_layer(const float* __restrict__ params, const WOffsets& wo, int lane,
                                           const float (&x)[N::fks(J)], f4 (&out)[N::fmt(J)]) {
  const float* w = params + wo.off[J];
#pragma unroll 1
  for (int m = 0; m < N::fmt(J); ++m) {
    asm volatile("" : "+v"(lane));  // the addresses are formed here, not held in registers outside
    const int col = 16 * m + (lane & 15);
    f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int s = 0; s < N::fks(J); ++s) {
      const int row = fwd_in_feature<N>(J, s, lane >> 4);
      acc = mfma4(row >= 0 && col < N::kout(J) ? w[row * N::kout(J) + col] : 0.0f, x[s], acc);
      __builtin_amdgcn_sched_barrier(0);  // (one weight at a time)
    }
#pragma unroll
    for (int i = 0; i < N::fmt(J); ++i) out[i] = i == m ? acc : out[i];
  }
}
template <int K>
__device__ __forceinline__ void flat4(const f4 (&v)[K], bool relu, float (&x)[4 * K]) {
#pragma unroll
  for (int k = 0; k < 4 * K; ++k) x[k] = relu ? fmaxf(v[k >> 2][k & 3], 0.0f) : v[k >> 2][k & 3];
}
template <class N>
__device__ __forceinline__ void fp32_tile(const float* __restrict__ params, const WOffsets& wo, int lane,
                                          const float (&e)[N::NSLOT], f4 sh, f4& o, f4& z) {
  f4 h[N::HC / 16], r[1];
  float x[N::HC / 4];
  fp32_layer<N, 0>(params, wo, lane, e, h);
  flat4(h, true, x);
  fp32_layer<N, 1>(params, wo, lane, x, r);
  o = r[0];
  {
    const f4 c[2] = {o, sh};
    float xc[8];
    flat4(c, false, xc);
    fp32_layer<N, 2>(params, wo, lane, xc, h);
  }
  flat4(h, true, x);
  fp32_layer<N, 3>(params, wo, lane, x, h);
  flat4(h, true, x);
  fp32_layer<N, 4>(params, wo, lane, x, r);
  z = r[0];
}

// ---------------------------------------------------------------------------
// Fused rendering: a workgroup takes 16 pixels, the columns of the MFMA tiles,
// and its four waves consecutive samples of all 16 rays, 16 a round: wave w
// evaluates samples 16 q + 4 w + (0..3) of every ray, one tile each, and passes
// their densities and colours through LDS so that lane group g holds tile g's;
// then every lane composites one sample of one ray.  The waves exchange the optical depths
// of the round through LDS (one barrier a round), and the rays leave together,
// once the transmittance left for each is below stop_T.
//
// A group of fewer pixels (the edge of an image, a ragged tile, an image of one
// row) does not repeat them over the columns: with np pixels rounded up to a power
// of two P, a tile takes 16 / P consecutive samples of each, the waves share the
// tiles of a pass of 16 / P rounds, and the rounds are composited in their order,
// so that a pixel has the same bits whatever shares its workgroup.  At 64 samples
// one pixel took 64 us at paper scale as 16 equal columns, 20 so; 16384 pixels in
// one row 689 and 212 us.
//
// The gathers bound it.  Samples of one ray are several cells apart at the
// fine levels, so a tile of 16 samples of a ray touched four lines of the
// table per sample and level; 16 neighbouring pixels at one depth share most
// of them.  And the samples of 16 rays spread over four waves keep a small
// image (160x120: 1200 workgroups) from leaving one wave a SIMD to wait on its
// own loads.  Against one ray a wave at a time, its samples 16 a tile: 640x480
// pixels of 64 samples at paper scale 11.3 -> 4.3 ms, 160x120 of 32 samples
// with the tiny field 105 -> 45 us (compositing four tiles at once, on every
// lane instead of the 16 that hold a tile's outputs, 5.8 -> 4.3 ms of it).
//
// V* = sum w (t - d*)^2 is formed without a second pass, from the sums of w, w t
// and w t^2 in FP64: V* = sum w t^2 - d*^2 (2 - A).  The products of FP32 values
// are exact or rounded at 2^-53, so what cancels costs no FP32 digit: over rays of
// constant density, of 32 and 64 samples, the mean relative error of V* is that of
// the weights, 3.6e-8 and 4.5e-8, against 7.0e-8 and 7.2e-8 for a second pass in
// FP32 and 1.1e-7 and 1.0e-7 for a running weighted mean and squared deviation
// in FP32, in the same time (608 us for 160x120 x 64 samples at paper scale).
// ---------------------------------------------------------------------------
constexpr int kRenderWaves = 4;                 // waves of a group of 16 pixels
constexpr int kRenderRound = 4 * kRenderWaves;  // samples of a round
constexpr int kRenderThreads = kRenderWaves * kWave;

// Sums over some samples of w, w t and w t^2.
struct Moments {
  double A, D, S;
  __device__ __forceinline__ void add(float w, float t) {
    const double wt = (double)w * (double)t;
    A += (double)w;
    D += wt;
    S = fma(wt, (double)t, S);
  }
  __device__ __forceinline__ void add(const Moments& o) {
    A += o.A;
    D += o.D;
    S += o.S;
  }
  // sum w (t - d*)^2, which rounding may leave just below zero
  __device__ __forceinline__ double variance() const {
    const double v = fma(-D * D, 2.0 - A, S);
    return v < 0.0 ? 0.0 : v;
  }
};

// Workgroup -> pixels: with tiles, the workgroups 4 k .. 4 k + 3 take the quarters
// of tile k, 16 consecutive pixels each, in an order that turns with k: workgroups
// go round the XCDs and, within one, round its shader engines in a fixed order, so
// that with quarter k % 4 in workgroup k, the first quarters of tiles of at most 16
// pixels all met on a fourth of the CUs (1200 such tiles at paper scale 1.55 ms
// instead of 0.72, 19200 of one pixel 2.2 instead of 0.70).  Without tiles, the workgroup takes block b of request
// 0's image, side x side pixels (blocks_x blocks a row, nblocks in all).  The grid is
// two-dimensional because the largest images have more threads than one
// dimension of a launch may.
//
// One group of 16 pixels a workgroup, although the split operands (60 KB) then
// leave room for two workgroups a CU: two groups on one copy of them, sixteen
// waves a CU instead of eight, took 4.37 ms instead of 4.16 for 640x480 x 64
// samples of the paper-scale map and 1.86 instead of 1.70 for 320x240; what more
// waves gather at a time pushes the others' lines out of the caches.  (The tiny
// field's tables stay in the caches; eight waves a SIMD instead of the seven its
// registers would leave take 247 us for 252, eight requests of 2048 tiles.)
template <class N>
__global__ __launch_bounds__(kRenderThreads) __attribute__((amdgpu_waves_per_eu(N::HD >= 64 ? 2 : 8))) void render_kernel(
    LevelInfo lv, Aabb box, WOffsets wo, const nsl_render_request* __restrict__ reqs, int n_req,
    const nsl_render_tile* __restrict__ tiles, uint32_t nblocks, int blocks_x, int side, RenderParams rp) {
  typedef typename std::conditional<kSplitNet<N>, __bf16, float>::type Op;
  constexpr int kOps = kSplitNet<N> ? 3 * Mixed<N>::FWD : N::FWD_FLOATS;
  __shared__ __attribute__((aligned(16))) Op Af[kOps];
  __shared__ float4 tile_out[kRenderRound][16];  // (o_0, z) of sample 16 r + m: [m][column r P + pixel]
  __shared__ float tau_of[2][kRenderRound][16];
  __shared__ float sums[kRenderWaves][3][16];  // C
  __shared__ Moments moments[kRenderWaves][16];
  __shared__ float scale_of[16];
  __shared__ uint32_t px_of[16];
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
  const int lane = lane_id(), g = lane >> 4, jc = lane & 15;
  // consecutive workgroups go round the 8 XCDs: of each 512 blocks an XCD
  // takes 64 consecutive ones, as many as its CUs hold, whose lines it finds in its L2
  // (16 or 256 of them were up to 2% and 7% slower)
  uint32_t blk = blockIdx.y * gridDim.x + blockIdx.x;
  if (blk >= nblocks) return;
  if ((blk | 511u) < nblocks) blk = (blk & ~511u) | ((blk & 7u) << 6) | ((blk >> 3) & 63u);
  // its np pixels, pix of which this lane's column takes: np rounded up to P = 2^lg
  int req = 0, u, v, np, lg, pix;
  auto columns = [&] {
    lg = np > 1 ? 32 - __clz(np - 1) : 0;
    pix = jc & ((1 << lg) - 1);
  };
  if (tiles) {
    const uint32_t k = blk / 4, quarter = (blk - k / 2 - k / 8) & 3u;
    const nsl_render_tile tile = tiles[k];
    req = tile.request;
    if (req < 0 || req >= n_req) return;
    const int npix = reqs[req].H * reqs[req].W;
    const int first = max(tile.first_pixel, 0) + 16 * (int)quarter;
    const int last = min(tile.first_pixel + min(tile.n_pixels, NSL_RENDER_TILE), npix);
    if (first >= last) return;
    np = min(16, last - first);
    columns();
    const int px = first + min(pix, np - 1);
    v = px / reqs[req].W;
    u = px - v * reqs[req].W;
  } else {
    // bands of four rows of blocks, down and then along each, so that the 64
    // consecutive blocks an XCD works at are 64x16 pixels: rows of blocks
    // instead took 4.08 ms against 3.98, and at 320x240 1.70 against 1.60
    const int rows = (reqs[0].H + side - 1) / side, band = 4 * ((int)blk / (4 * blocks_x)), high = min(4, rows - band);
    const int i = (int)blk - band * blocks_x, bx = i / high, by = band + i - bx * high;
    const int w4 = min(side, reqs[0].W - side * bx);
    np = w4 * min(side, reqs[0].H - side * by);
    columns();
    const int at = min(pix, np - 1), y = w4 == 3 ? (at * 11) >> 5 : at >> (w4 / 2);  // at / w4
    u = side * bx + at - y * w4;
    v = side * by + y;
  }
  np = __builtin_amdgcn_readfirstlane(np);
  lg = __builtin_amdgcn_readfirstlane(lg);
  const nsl_render_request& rq = reqs[req];
  copy_to_lds<kRenderThreads, sizeof(Af)>(Af, rq.prepared);
  __syncthreads();
  LaneLevels<N> ll;
  lane_levels<N>(lv, g, ll);
  float o[3], d[3], s, shv[4];
  camera_ray(rq.pose, rq.intr, u, v, o, d, s);
  sh_lane<N>(d, g, shv);
  if (threadIdx.x < 16) {
    scale_of[jc] = s;
    px_of[jc] = (uint32_t)(v * rq.W + u);
  }
  auto t_of = [&](int j) {
#pragma clang fp contract(off)
    return rp.t_near + ((float)j + 0.5f) * rp.dt;
  };
  float carry = 0.0f, C0 = 0.0f, C1 = 0.0f, C2 = 0.0f;
  Moments mo{0.0, 0.0, 0.0};
  bool done = pix >= np;                    // this lane's ray has stopped
  const int mine = 4 * wave + g;            // this lane's sample of a round
  // the passes over the rays' samples: one round each where a group has all
  // columns (kFull), else 2^per
  auto passes = [&](auto full) {
    constexpr bool kFull = decltype(full)::value;
    const int r = kFull ? 0 : jc >> lg, per = kFull ? 0 : 4 - lg;
    const int span = kRenderRound << per;
    auto from_round = [&](auto x, int i) { return __shfl(x, (lane & 48) | (i << lg) | pix, kWave); };
    for (int base = 0, q = 0; base < rp.n_samples; base += span, ++q) {
      const int left = min(rp.n_samples - base, span), nr = (left + kRenderRound - 1) / kRenderRound;
      const int ntile = (left + (1 << per) - 1) >> per;
      for (int k = 0; k < 4; ++k) {
        const int ti = kFull ? 4 * wave + k : wave + kRenderWaves * k;
        if (ti >= ntile) break;
        const int jl = (ti << per) + r;       // this column's sample of the pass
        const float tk = t_of(base + jl);
        float xn[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) xn[i] = normalise_axis(pos_axis(o[i], d[i], tk), box.lo[i], box.inv[i]);
        f4 oo, zz;
        if constexpr (kSplitNet<N>) {
          float e[1][N::NSLOT];
          encode<N>(rq.params, lv.table_mask, ll, xn, e[0]);
          const f4 sh[1] = {f4{shv[0], shv[1], shv[2], shv[3]}};
          f4 o1[1], z1[1];
          split_mlp<N, 1>(Af, lane, e, sh, o1, z1);
          oo = o1[0];
          zz = z1[0];
          const bool bad = g == 0 && !all_finite(oo[0], zz);
          if (__ballot(bad) != 0ull) {  // those columns alone: a pixel's bits do not depend on the others
            f4 o2, z2;
            fp32_tile<N>(rq.params, wo, lane, e[0], sh[0], o2, z2);
            oo = bad ? o2 : oo;
            zz = bad ? z2 : zz;
          }
        } else {
          Acts<N> act;
          encode<N>(rq.params, lv.table_mask, ll, xn, act.e);
#pragma unroll
          for (int i = 0; i < 4; ++i) act.sh[i] = shv[i];
          mlp_fwd<N>(Af, lane, act);
          oo = act.o;
          zz = act.z;
        }
        // lanes of row 0 hold the column's density and colour
        const int row = kFull ? ti : jl & (kRenderRound - 1), col = kFull ? jc : ((jl / kRenderRound) << lg) | pix;
        if (g == 0) tile_out[row][col] = make_float4(oo[0], zz[0], zz[1], zz[2]);
      }
      if constexpr (kFull)
        wave_lds_fence();  // a wave composites its own tiles
      else
        __syncthreads();
      const int j = base + kRenderRound * r + mine;
      const bool valid = j < rp.n_samples;
      const float t = t_of(j);
      float(*tw)[16] = tau_of[q & 1];
      const float4 oz = tile_out[mine][jc];
      const float tau = valid ? expf(oz.x) * rp.dt : 0.0f;
      tw[mine][jc] = tau;
      __syncthreads();
      // optical depth of the round before this sample, and of all of it, by
      // sums of four (in order, sixteen roundings would reach T)
      float sum4[kRenderWaves], before = 0.0f;
#pragma unroll
      for (int w = 0; w < kRenderWaves; ++w) {
        const float t0 = tw[4 * w][jc], t1 = tw[4 * w + 1][jc], t2 = tw[4 * w + 2][jc], t3 = tw[4 * w + 3][jc];
        sum4[w] = (t0 + t1) + (t2 + t3);
        if (w == wave) before = (g > 0 ? t0 : 0.0f) + (g > 1 ? t1 : 0.0f) + (g > 2 ? t2 : 0.0f);
      }
      const float half = sum4[0] + sum4[1];
      before += wave > 2 ? half + sum4[2] : wave > 1 ? half : wave > 0 ? sum4[0] : 0.0f;
      const float round = half + (sum4[2] + sum4[3]);
      float start = carry;  // the optical depth before this lane's round
      if constexpr (kFull) {
        carry += round;
      } else {
        for (int i = 0; i < nr; ++i) {
          if (r == i) start = carry;
          carry += from_round(round, i);
        }
      }
      const float T0 = expf(-(start + before));
      const bool on = valid && !done && !(rp.stop_T > 0.0f && (T0 < rp.stop_T || (!kFull && expf(-start) < rp.stop_T)));
      auto add = [&] {
        const float w = T0 * -expm1f(-tau);
        C0 = fmaf(w, sigmoidf(oz.y), C0);
        C1 = fmaf(w, sigmoidf(oz.z), C1);
        C2 = fmaf(w, sigmoidf(oz.w), C2);
        mo.add(w, t);
      };
      if constexpr (kFull) {
        if (on) add();
      } else {  // round after round, as the rays of a full group
        for (int i = 0; i < nr; ++i) {
          if (on && r == i) add();
          C0 = from_round(C0, i);
          C1 = from_round(C1, i);
          C2 = from_round(C2, i);
          mo = Moments{from_round(mo.A, i), from_round(mo.D, i), from_round(mo.S, i)};
        }
      }
      if (rp.stop_T > 0.0f) {
        done |= expf(-carry) < rp.stop_T;
        if (__ballot(!done) == 0ull) break;  // every wave holds the same sums
      }
    }
  };
  // (in this order: full groups first took 0.4% longer, a launch of eight requests
  // of the tiny field 215.9 us for 215.0)
  if (np <= 8)
    passes(std::false_type{});
  else
    passes(std::true_type{});
  // (the lane's place again, from nothing: held over the loop it would spill, and
  // the reload costs a memory latency)
  int lane2;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane2));
  const int g2 = lane2 >> 4, jc2 = lane2 & 15;
#pragma unroll
  for (int x = 16; x <= 32; x <<= 1) {
    C0 += __shfl_xor(C0, x, kWave);
    C1 += __shfl_xor(C1, x, kWave);
    C2 += __shfl_xor(C2, x, kWave);
    mo.add(Moments{__shfl_xor(mo.A, x, kWave), __shfl_xor(mo.D, x, kWave), __shfl_xor(mo.S, x, kWave)});
  }
  if (g2 == 0) {
    sums[wave][0][jc2] = C0;
    sums[wave][1][jc2] = C1;
    sums[wave][2][jc2] = C2;
    moments[wave][jc2] = mo;
  }
  __syncthreads();
  if (wave != 0 || g2 != 0 || jc2 >= np) return;
  C0 = C1 = C2 = 0.0f;
  mo = Moments{0.0, 0.0, 0.0};
#pragma unroll
  for (int w = 0; w < kRenderWaves; ++w) {
    const float(*p)[16] = sums[w];
    C0 += p[0][jc2];
    C1 += p[1][jc2];
    C2 += p[2][jc2];
    mo.add(moments[w][jc2]);
  }
  const size_t px = px_of[jc2];
  s = scale_of[jc2];
  rq.rgb[3 * px] = C0;
  rq.rgb[3 * px + 1] = C1;
  rq.rgb[3 * px + 2] = C2;
  rq.depth_z[px] = (float)mo.D / s;
  rq.var_z[px] = (float)mo.variance() / (s * s);
  if (rq.opacity) rq.opacity[px] = (float)mo.A;
}

// ---------------------------------------------------------------------------
// Host launchers
// ---------------------------------------------------------------------------

template <class N>
static hipError_t launch_prep(const float* params, const WOffsets& wo, float* out, hipStream_t st) {
  const int n = N::FWD_FLOATS + N::BWD_FLOATS;
  hipLaunchKernelGGL(prep_weights_kernel<N>, dim3((n + 255) / 256), dim3(256), 0, st, params, wo, out);
  return hipGetLastError();
}

template <class N>
static hipError_t launch_render_prep(const float* params, const WOffsets& wo, void* out, const nsl_render_request* r,
                                     const float* pose, const float* intr, nsl_render_request* dst, hipStream_t st) {
  int n = N::FWD_FLOATS + N::BWD_FLOATS;
  if constexpr (kSplitNet<N>) {
    n = Mixed<N>::FWD;
    static_assert(3 * sizeof(__bf16) * Mixed<N>::FWD <= sizeof(float) * (N::FWD_FLOATS + N::BWD_FLOATS),
                  "they fit the space of the FP32 operands");
  }
  hipLaunchKernelGGL(render_prep_kernel<N>, dim3((n + 255) / 256), dim3(256), 0, st, params, wo, out,
                     r ? *r : nsl_render_request{}, pose, intr, dst);
  return hipGetLastError();
}

hipError_t render_prep(int shape, const float* params, const WOffsets& wo, void* out, const nsl_render_request* r,
                       const float* pose, const float* intr, nsl_render_request* dst, hipStream_t st) {
  return shape == kShapeTiny ? launch_render_prep<NetTiny>(params, wo, out, r, pose, intr, dst, st)
                             : launch_render_prep<NetFull>(params, wo, out, r, pose, intr, dst, st);
}

template <class N>
static hipError_t launch_prep_count(const float* params, const WOffsets& wo, float* out, float* zero, int64_t nzero,
                                    float* clear_flag, const KeyframeStore& kf, const MarchParams& mp,
                                    const uint32_t* ids, int n, const RayBuffers& rb, hipStream_t st) {
  const int ncount = (int)count_block_count(mp, n), nfill = (int)((nzero + 1023) / 1024);
  const int nprep = (N::FWD_FLOATS + N::BWD_FLOATS + 255) / 256;
  hipLaunchKernelGGL(prepare_count_kernel<N>, dim3(ncount + nfill + nprep), dim3(256), 0, st, params, wo, out, zero,
                     nzero, nfill, clear_flag, kf, mp, ids, n, rb, ncount);
  return hipGetLastError();
}

hipError_t field_prep_count(int shape, const float* params, const WOffsets& wo, float* out, float* zero, int64_t nzero,
                            float* clear_flag, const KeyframeStore& kf, const MarchParams& mp, const uint32_t* ids,
                            int n, const RayBuffers& rb, hipStream_t st) {
  return shape == kShapeTiny
             ? launch_prep_count<NetTiny>(params, wo, out, zero, nzero, clear_flag, kf, mp, ids, n, rb, st)
             : launch_prep_count<NetFull>(params, wo, out, zero, nzero, clear_flag, kf, mp, ids, n, rb, st);
}

template <class N>
static hipError_t launch_fwd(const FieldArgs& a, const SampleSrc& src, int max_samples,
                             float* sigma, float* rgb, hipStream_t st, const BinPrep* bp) {
  const int tiles = (max_samples + 15) / 16;
  const int grid = (tiles + 3) / 4 < kFieldFwdGrid ? (tiles + 3) / 4 : kFieldFwdGrid;
  const BinPrep none{};
  const BinPrep& b = bp ? *bp : none;
  if (grid + b.nbins > 0)
    hipLaunchKernelGGL(field_fwd_kernel<N>, dim3(grid + b.nbins), dim3(256), 0, st, a, src, sigma, rgb, b);
  return hipGetLastError();
}

template <class N>
static hipError_t launch_bwd(const FieldArgs& a, const SampleSrc& src, int nblocks,
                             const float* dsigma, const float* drgb, const RecordBuffers& rec,
                             float* partial, const WOffsets& wo, float* grads, hipStream_t st) {
  if (!kGathers<N> && !src.ecache) return hipErrorInvalidValue;
  hipLaunchKernelGGL(field_bwd_kernel<N>, dim3(nblocks), dim3(kFieldBwdWaves * kWave), 0, st, a, src, dsigma, drgb,
                     rec, partial);
  return hipGetLastError();
}

// Images of at most this many 4x4 blocks, which leave half of the chip without a
// workgroup or more, go by 2x2 blocks: at paper scale, 64 samples, 4x4 pixels
// 27 us instead of 135, 16x16 37 instead of 124, 32x32 60 instead of 121.
constexpr int kRenderFewBlocks = 128;
template <class N>
static hipError_t launch_render(const LevelInfo& lv, const Aabb& box, const WOffsets& wo,
                                const nsl_render_request* reqs, int n_req, const nsl_render_tile* tiles, int n_tiles,
                                int H, int W, const RenderParams& rp, hipStream_t st) {
  static_assert(NSL_RENDER_TILE == 64, "four groups of 16 pixels a tile");
  auto across = [](int n, int side) { return ((int64_t)n + side - 1) / side; };
  const int side = across(W, 4) * across(H, 4) <= kRenderFewBlocks ? 2 : 4;
  const int64_t bx = across(W, side), nblocks = tiles ? (int64_t)n_tiles * 4 : bx * across(H, side);
  if (nblocks <= 0) return hipSuccess;
  const int64_t gx = std::min<int64_t>(nblocks, 1 << 20);
  hipLaunchKernelGGL(render_kernel<N>, dim3((unsigned)gx, (unsigned)((nblocks + gx - 1) / gx)),
                     dim3(kRenderThreads), 0, st, lv, box, wo, reqs, n_req, tiles, (uint32_t)nblocks, (int)bx, side, rp);
  return hipGetLastError();
}

hipError_t render_tiles(int shape, const LevelInfo& lv, const Aabb& box, const WOffsets& wo,
                        const nsl_render_request* reqs, int n_req, const nsl_render_tile* tiles, int n_tiles,
                        const RenderParams& rp, hipStream_t st) {
  return shape == kShapeTiny ? launch_render<NetTiny>(lv, box, wo, reqs, n_req, tiles, n_tiles, 0, 0, rp, st)
                             : launch_render<NetFull>(lv, box, wo, reqs, n_req, tiles, n_tiles, 0, 0, rp, st);
}

hipError_t render_one(int shape, const LevelInfo& lv, const Aabb& box, const WOffsets& wo,
                      const nsl_render_request* req, int H, int W, const RenderParams& rp, hipStream_t st) {
  return shape == kShapeTiny ? launch_render<NetTiny>(lv, box, wo, req, 1, nullptr, 0, H, W, rp, st)
                             : launch_render<NetFull>(lv, box, wo, req, 1, nullptr, 0, H, W, rp, st);
}

hipError_t field_encode(int shape, const FieldArgs& a, const SampleSrc& src, int max_samples, uint32_t* hist,
                        const BinLevels& bl, int64_t entries, hipStream_t st) {
  return shape == kShapeTiny
             ? launch_encode<NetTiny, float, float2>(a.lv, a.table, src, max_samples, hist, bl, entries, st)
             : launch_encode<NetFull, float, float2>(a.lv, a.table, src, max_samples, hist, bl, entries, st);
}

__global__ __launch_bounds__(256) void loss_sum_kernel(LossSum ls) {
  __shared__ float lds[kSumScratchFloats];
  loss_sum_block(ls, lds);
}

hipError_t loss_sum(const LossSum& ls, hipStream_t st) {
  hipLaunchKernelGGL(loss_sum_kernel, dim3(1), dim3(256), 0, st, ls);
  return hipGetLastError();
}

hipError_t field_dw_reduce(int shape, const float* partial, int nblocks, const WOffsets& wo, float* grads,
                           float* overflow, const LossSum* ls, hipStream_t st) {
  return shape == kShapeTiny ? launch_dw_reduce<NetTiny>(partial, nblocks, wo, grads, overflow, ls, st)
                             : launch_dw_reduce<NetFull>(partial, nblocks, wo, grads, overflow, ls, st);
}

size_t field_prep_floats(int shape) {
  return shape == kShapeTiny ? NetTiny::FWD_FLOATS + NetTiny::BWD_FLOATS
                             : NetFull::FWD_FLOATS + NetFull::BWD_FLOATS;
}
size_t field_nweights(int shape) {
  return shape == kShapeTiny ? NetTiny::NWEIGHTS : NetFull::NWEIGHTS;
}

hipError_t field_prep(int shape, const float* params, const WOffsets& wo, float* out, hipStream_t st) {
  return shape == kShapeTiny ? launch_prep<NetTiny>(params, wo, out, st)
                             : launch_prep<NetFull>(params, wo, out, st);
}

hipError_t field_forward(int shape, const FieldArgs& a, const SampleSrc& src, int max_samples,
                         float* sigma, float* rgb, hipStream_t st, const BinPrep* bp) {
  return shape == kShapeTiny ? launch_fwd<NetTiny>(a, src, max_samples, sigma, rgb, st, bp)
                             : launch_fwd<NetFull>(a, src, max_samples, sigma, rgb, st, bp);
}

hipError_t field_backward(int shape, const FieldArgs& a, const SampleSrc& src, int nblocks,
                          const float* dsigma, const float* drgb, const RecordBuffers& rec,
                          float* partial, const WOffsets& wo, float* grads, hipStream_t st) {
  return shape == kShapeTiny
             ? launch_bwd<NetTiny>(a, src, nblocks, dsigma, drgb, rec, partial, wo, grads, st)
             : launch_bwd<NetFull>(a, src, nblocks, dsigma, drgb, rec, partial, wo, grads, st);
}

}  // namespace nsl
