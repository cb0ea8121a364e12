// Mixed-precision hash-grid field on gfx950: FP16 tables, BF16 weights and
// activations on v_mfma_f32_16x16x32_bf16 with FP32 accumulation (weight
// gradients too, with samples on the contraction axis), FP32 trilinear blending, FP32 table-gradient accumulation.
//
// Operand layouts follow the FP32 kernels (features as rows, 16 samples as
// columns): a 16x16x32 k-step takes 8 consecutive k-slots per lane group,
// filled from two 16-row output tiles of the previous layer (rows 4g..4g+3
// of each), and the weights are laid out for that permutation.
#include "bf16_ops.h"
#include "bins.h"
#include "field_common.h"
#include "march_common.h"

namespace nsl {

typedef short s4 __attribute__((ext_vector_type(4)));
typedef short s8 __attribute__((ext_vector_type(8)));

// Output feature consumed by backward k-slot (s, g, u) of layer j; -1 = pad.
template <class N>
__host__ __device__ constexpr int mixed_bwd_kfeature(int j, int s, int g, int u) {
  if (j == N::NW - 1 || j == 1) return u < 4 ? 4 * g + u : -1;
  return 32 * s + 16 * (u >> 2) + 4 * g + (u & 3);
}

// Element idx of the BF16 operand arrays (forward, then backward).
template <class N>
__device__ __forceinline__ void prep_operand(const float* __restrict__ params, const WOffsets& wo,
                                             __bf16* __restrict__ out, int idx) {
  using M = Mixed<N>;
  if (idx >= M::FWD + M::BWD) return;
  float v = 0.0f;
  const bool fwd = idx < M::FWD;
  const int r0 = fwd ? idx : idx - M::FWD;
  int j = 0;
  if (fwd) {
    while (j + 1 < N::NW && r0 >= M::foff(j + 1)) ++j;
  } else {
    while (j + 1 < N::NW && r0 >= M::boff(j + 1)) ++j;
  }
  const int r = r0 - (fwd ? M::foff(j) : M::boff(j));
  const int u = r % 8, lane = (r / 8) % kWave, ms = r / M::BLK;
  const int ks = fwd ? M::fks(j) : M::bks(j);
  const int s = ms % ks, m = ms / ks;
  const int g = lane >> 4, i = lane & 15;
  int row, col;
  if (fwd) {
    row = mixed_fwd_feature<N>(j, s, g, u);
    col = 16 * m + i;
  } else {
    row = bwd_row_feature<N>(j, m, i);
    col = mixed_bwd_kfeature<N>(j, s, g, u);
  }
  if (row >= 0 && col >= 0 && row < N::kin(j) && col < N::kout(j)) v = params[wo.off[j] + row * N::kout(j) + col];
  out[idx] = (__bf16)v;
}

// FP16 copy of the FP32 table (tf floats), eight values [i, i + 8) per
// thread; with g set, the same pass clears the gradient vector from tf
// rounded down to a multiple of 8 up to total.
__device__ __forceinline__ void table_to_half(const float* __restrict__ t, _Float16* __restrict__ h, int64_t tf,
                                              float* __restrict__ g, int64_t total, int64_t i) {
  typedef _Float16 h8 __attribute__((ext_vector_type(8)));
  if (i + 8 <= tf) {
    const float4 a = reinterpret_cast<const float4*>(t + i)[0];
    const float4 b = reinterpret_cast<const float4*>(t + i)[1];
    const h8 o = {(_Float16)a.x, (_Float16)a.y, (_Float16)a.z, (_Float16)a.w,
                  (_Float16)b.x, (_Float16)b.y, (_Float16)b.z, (_Float16)b.w};
    *reinterpret_cast<h8*>(h + i) = o;
  } else {
    for (int64_t k = i; k < tf; ++k) h[k] = (_Float16)t[k];
  }
  if (g && i >= (tf & ~(int64_t)7)) {
    if (i + 8 <= total) {
      reinterpret_cast<float4*>(g + i)[0] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      reinterpret_cast<float4*>(g + i)[1] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    } else {
      for (int64_t k = i; k < total; ++k) g[k] = 0.0f;
    }
  }
}

// One launch prepares a mixed-precision step: workgroups [0, tblocks) copy
// the table to FP16 (and clear the gradient tail), the rest lay out the BF16
// weight operands; clear_flag (may be null), the loss-scale overflow flag, is
// reset by the first thread.  Workgroup b of the preparation.
template <class N>
__device__ __forceinline__ void prepare_block(const float* __restrict__ params, const WOffsets& wo,
                                              __bf16* __restrict__ ops, _Float16* __restrict__ t16, int64_t tf,
                                              float* __restrict__ g, int64_t total, int tblocks,
                                              float* __restrict__ clear_flag, int b) {
  if (clear_flag && b == 0 && threadIdx.x == 0) *clear_flag = 0.0f;
  if (b < tblocks)
    table_to_half(params, t16, tf, g, total, ((int64_t)b * 256 + threadIdx.x) * 8);
  else
    prep_operand<N>(params, wo, ops, (b - tblocks) * 256 + (int)threadIdx.x);
}

template <class N>
__global__ __launch_bounds__(256) void mixed_prepare_kernel(const float* __restrict__ params, WOffsets wo,
                                                            __bf16* __restrict__ ops, _Float16* __restrict__ t16,
                                                            int64_t tf, float* __restrict__ g, int64_t total,
                                                            int tblocks, float* __restrict__ clear_flag) {
  prepare_block<N>(params, wo, ops, t16, tf, g, total, tblocks, clear_flag, (int)blockIdx.x);
}

// The step's first launch: workgroups [0, ncount) set up the candidate rays
// and count their samples, the rest prepare the step as above.  The two are
// independent, so the latency-bound marching overlaps the streaming table
// copy instead of following it.
template <class N>
__global__ __launch_bounds__(256) void mixed_prepare_count_kernel(
    const float* __restrict__ params, WOffsets wo, __bf16* __restrict__ ops, _Float16* __restrict__ t16, int64_t tf,
    float* __restrict__ g, int64_t total, int tblocks, float* __restrict__ clear_flag, KeyframeStore kf,
    MarchParams mp, const uint32_t* __restrict__ ids, int n, RayBuffers rb, int ncount) {
  if ((int)blockIdx.x < ncount) {
    march_detail::rays_count_block(kf, mp, ids, n, rb, (int)blockIdx.x);
    return;
  }
  prepare_block<N>(params, wo, ops, t16, tf, g, total, tblocks, clear_flag, (int)blockIdx.x - ncount);
}

// ---------------------------------------------------------------------------
// Pieces shared by the forward and backward kernels: the activations of a
// tile (kept by the backward as the BF16 operands the next layer consumed),
// its inputs, and the forward of T tiles interleaved layer by layer.
// ---------------------------------------------------------------------------

template <class N>
struct PActs {
  bf8 e;                   // layer-0 operand: encoding slots (zero beyond NSLOT)
  bf8 h1[N::HD / 32];      // ReLU outputs of layer 0, as layer-1 operands
  f4 o;                    // geometry output, FP32
  bf8 osh;                 // layer-2 operand: geometry rows 4g.., SH 4g..
  bf8 h3[N::HC / 32];
  bf8 h4[N::HC / 32];      // second colour hidden layer (NCH == 2)
  f4 z;                    // colour logits (rows 0..2 in lane group 0)
};

// Inputs of one tile: encoding slots, view direction, upstream gradients.
template <class N>
struct TileIn {
  uint32_t e[N::LPL];      // BF16 pairs of levels g + 4q
  float d[3];
  float ds, dr[3];
};

// acc[r] where the ReLU output (element 4*half + r of p) is positive, else 0.
typedef short s16x2 __attribute__((ext_vector_type(2)));

// ReLU of eight BF16 values on their bits: a BF16 value is below zero exactly
// when its bit pattern is negative as a 16-bit integer (and -0 becomes +0).
// Rounding keeps the sign, so this equals rounding the FP32 ReLU.
__device__ __forceinline__ bf8 relu8(bf8 v) {
  uint4 u = __builtin_bit_cast(uint4, v);
  const s16x2 z = {0, 0};
  u.x = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s16x2, u.x), z));
  u.y = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s16x2, u.y), z));
  u.z = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s16x2, u.z), z));
  u.w = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s16x2, u.w), z));
  return __builtin_bit_cast(bf8, u);
}

// The BF16 gradient g where the ReLU output p (bits of a value >= +0) is
// above zero, else 0: the same values as masking in FP32 and rounding after.
// (two packed 16-bit instructions: keep = min(p, 1), g * keep; written out
// because the compiler otherwise selects each half apart, after converting
// each value on its own)
__device__ __forceinline__ uint32_t relu_mask2(uint32_t g, uint32_t p) {
  uint32_t keep, r;
  asm("v_pk_min_u16 %0, %1, %2" : "=v"(keep) : "v"(p), "v"(0x00010001u));
  asm("v_pk_mul_lo_u16 %0, %1, %2" : "=v"(r) : "v"(g), "v"(keep));
  return r;
}
__device__ __forceinline__ bf8 relu_mask8(bf8 g, bf8 p) {
  uint4 a = __builtin_bit_cast(uint4, g);
  const uint4 b = __builtin_bit_cast(uint4, p);
  a.x = relu_mask2(a.x, b.x);
  a.y = relu_mask2(a.y, b.y);
  a.z = relu_mask2(a.z, b.z);
  a.w = relu_mask2(a.w, b.w);
  return __builtin_bit_cast(bf8, a);
}


// Sigmoid through the hardware reciprocal (1 ulp) rather than an IEEE
// division: in the backward the colour gradient it enters is rounded to BF16
// right after, and in the forward it is far below the BF16 network's error.
__device__ __forceinline__ float sigmoid_rcp(float z) { return __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }

template <class N, bool KEEP>
__device__ __forceinline__ void fetch_tile(const SampleSrc& src, const _Float16* __restrict__ table,
                                           const LevelInfo& lv, const LaneLevels<N>& ll,
                                           const float* __restrict__ dsigma, const float* __restrict__ drgb, int s,
                                           bool valid, int g, uint32_t ridx, TileIn<N>& in) {
  in.d[0] = 0.0f; in.d[1] = 0.0f; in.d[2] = 1.0f;
  if constexpr (KEEP) {
    const uint32_t* ec = static_cast<const uint32_t*>(src.ecache);
#pragma unroll
    for (int q = 0; q < N::LPL; ++q) in.e[q] = valid ? ec[(size_t)(g + 4 * q) * src.ecache_stride + s] : 0u;
    if (valid) {
      if (src.t) {
        const float4 dd = src.rays[2 * ridx + 1];
        in.d[0] = dd.x; in.d[1] = dd.y; in.d[2] = dd.z;
      } else {
#pragma unroll
        for (int i = 0; i < 3; ++i) in.d[i] = src.dir[3 * s + i];
      }
    }
  } else {
    float xn[3] = {0.5f, 0.5f, 0.5f};
    if (valid) load_sample(src, s, xn, in.d);
    float e[N::NSLOT];
    encode<N>(table, lv.table_mask, ll, xn, e);
#pragma unroll
    for (int q = 0; q < N::LPL; ++q) in.e[q] = valid ? bf16_pair(e[2 * q], e[2 * q + 1]) : 0u;
  }
  in.ds = 0.0f;
  in.dr[0] = in.dr[1] = in.dr[2] = 0.0f;
  if (dsigma && g == 0 && valid) {
    in.ds = dsigma[s];
#pragma unroll
    for (int r = 0; r < 3; ++r) in.dr[r] = drgb[3 * s + r];
  }
}

template <class N>
__device__ __forceinline__ uint32_t ray_of(const SampleSrc& src, int s, int S) {
  return src.t && s < S ? src.ray[s] : 0u;
}

// Forward of T tiles, interleaved layer by layer.
template <class N, int T>
__device__ __forceinline__ void fwd_tiles(const __bf16* __restrict__ Af, int lane, const f4 (&sh)[T],
                                          PActs<N> (&a)[T]) {
  using M = Mixed<N>;
  constexpr f4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
  auto wf = [&](int j, int k) { return lds_bf8<N>(Af + M::foff(j), k, lane); };
  {
    f4 h[T][N::HD / 16];
#pragma unroll
    for (int m = 0; m < N::HD / 16; ++m)
#pragma unroll
      for (int t = 0; t < T; ++t) h[t][m] = mfma32(wf(0, m), a[t].e, zero);
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int s = 0; s < N::HD / 32; ++s) a[t].h1[s] = relu8(pack8(h[t][2 * s], h[t][2 * s + 1]));
  }
  {
    f4 acc[T];
#pragma unroll
    for (int t = 0; t < T; ++t) acc[t] = zero;
#pragma unroll
    for (int s = 0; s < N::HD / 32; ++s)
#pragma unroll
      for (int t = 0; t < T; ++t) acc[t] = mfma32(wf(1, s), a[t].h1[s], acc[t]);
#pragma unroll
    for (int t = 0; t < T; ++t) {
      a[t].o = acc[t];
      a[t].osh = pack8(acc[t], sh[t]);
    }
  }
  {
    f4 h[T][N::HC / 16];
#pragma unroll
    for (int m = 0; m < N::HC / 16; ++m)
#pragma unroll
      for (int t = 0; t < T; ++t) h[t][m] = mfma32(wf(2, m), a[t].osh, zero);
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int s = 0; s < N::HC / 32; ++s) a[t].h3[s] = relu8(pack8(h[t][2 * s], h[t][2 * s + 1]));
  }
  if constexpr (N::NCH == 2) {
    f4 acc[T][N::HC / 16];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int m = 0; m < N::HC / 16; ++m) acc[t][m] = zero;
#pragma unroll
    for (int s = 0; s < N::HC / 32; ++s)
#pragma unroll
      for (int m = 0; m < N::HC / 16; ++m)
#pragma unroll
        for (int t = 0; t < T; ++t) acc[t][m] = mfma32(wf(3, m * (N::HC / 32) + s), a[t].h3[s], acc[t][m]);
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int s = 0; s < N::HC / 32; ++s) a[t].h4[s] = relu8(pack8(acc[t][2 * s], acc[t][2 * s + 1]));
  }
  {
    f4 acc[T];
#pragma unroll
    for (int t = 0; t < T; ++t) acc[t] = zero;
#pragma unroll
    for (int s = 0; s < N::HC / 32; ++s)
#pragma unroll
      for (int t = 0; t < T; ++t) acc[t] = mfma32(wf(N::NW - 1, s), N::NCH == 2 ? a[t].h4[s] : a[t].h3[s], acc[t]);
#pragma unroll
    for (int t = 0; t < T; ++t) a[t].z = acc[t];
  }
}

// Layer-0 operand (encoding slots, zero beyond NSLOT) and SH coefficients of
// one tile.
template <class N>
__device__ __forceinline__ void tile_operands(const TileIn<N>& in, int g, PActs<N>& a, f4& sh) {
  uint32_t w[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) w[q] = q < N::LPL ? in.e[q < N::LPL ? q : 0] : 0u;
  a.e = __builtin_bit_cast(bf8, make_uint4(w[0], w[1], w[2], w[3]));
  float shv[4];
  sh_lane<N>(in.d, g, shv);
  sh = f4{shv[0], shv[1], shv[2], shv[3]};
}

// ---------------------------------------------------------------------------
// Backward.  A workgroup of kBwdWaves waves takes steps of 16 samples a wave.
// Each wave runs the forward recompute and the input-gradient chain of its 16
// samples; the step's samples are staged into LDS two or one layers at a time
// (three groups a step), and each wave adds the products of its share of the group's
// weight-gradient tiles over all of them, so that it holds a few tiles
// instead of all.
//
// A sample's staged values lie next to each other, in the order in which the
// lanes hold them (one 16-byte store of a lane for 32 features), and the
// products' operands, which run along the samples, come from LDS reads that
// transpose 4 x 16 values a 16-lane row.
// ---------------------------------------------------------------------------
constexpr int kBwdWaves = 16;
constexpr int kStepSamples = 16 * kBwdWaves;  // samples of a workgroup step

// Staging groups: the layers whose weight-gradient products follow one
// barrier together (the colour layers; the geometry-feature layer and the
// second density layer; the first density layer).  Within a group each layer
// has its X columns (32 per k-step of its forward product) and then its dY
// columns (16 where the layer has at most 16 outputs), layers in backward order.
template <class N>
struct StageCols {
  static constexpr int xc(int j) { return 32 * Mixed<N>::fks(j); }
  static constexpr int yc(int j) { return j == 1 || j == N::NW - 1 ? 16 : N::kout(j); }
  static constexpr int group(int j) { return j >= 3 || j == N::NW - 1 ? 0 : j >= 1 ? 1 : 2; }
  static constexpr int x(int j) {
    int o = 0;
    for (int i = N::NW - 1; i > j; --i)
      if (group(i) == group(j)) o += xc(i) + yc(i);
    return o;
  }
  static constexpr int y(int j) { return x(j) + xc(j); }
  static constexpr int cols(int gr) {
    int o = 0;
    for (int i = 0; i < N::NW; ++i)
      if (group(i) == gr) o += xc(i) + yc(i);
    return o;
  }
  // BF16 values of a staged sample: an odd number of 32-byte pieces, so that
  // eight samples' pieces lie in different LDS banks
  static constexpr int COLS = N::cmax(cols(0), N::cmax(cols(1), cols(2)));
  static constexpr int ROW = COLS / 16 % 2 ? COLS : COLS + 16;
};

// Four rows (from p, this lane's 8-byte quarter of one) of 16 columns,
// transposed: lane i of a 16-lane row gets the four values of column i.
__device__ __forceinline__ s4 read_transposed(const __bf16* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) s4*)(reinterpret_cast<const s4*>(p)));
}

// Weight gradient of layer J in 16x16 tiles: the workgroup's waves own one
// each, or with fewer tiles than waves share one, each taking its part of a
// step's samples.  Tile (m, n), lane (gk, i): rows 16m + 4gk + r of the staged X
// columns, column 16n + i of the dY ones.
template <class N, int J>
struct OwnedDW16 {
  using SC = StageCols<N>;
  static constexpr int W = kBwdWaves, NJ = SC::yc(J) / 16, TILES = SC::xc(J) / 16 * NJ;
  static_assert(W % TILES == 0, "whole waves a tile");
  static constexpr int SPLIT = W / TILES, CHUNKS = kStepSamples / 32 / SPLIT;  // 32 samples a product
  static_assert(CHUNKS >= 1, "a product a wave");
  f4 v;
  __device__ __forceinline__ void zero() { v = f4{0.0f, 0.0f, 0.0f, 0.0f}; }
  __device__ __forceinline__ void chunk(const __bf16* x, const __bf16* y, int c) {
    constexpr int R = SC::ROW;
    auto rd = [&](const __bf16* p) {
      const s4 lo = read_transposed(p + 32 * c * R), hi = read_transposed(p + (32 * c + 16) * R);
      return __builtin_bit_cast(bf8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    v = mfma32(rd(x), rd(y), v);
  }
  // v += X^T dY over the step's first nc pieces of 32 samples
  __device__ __forceinline__ void add(const __bf16* stage, int w, int lane, int nc) {
    const int t = w % TILES, c0 = w / TILES * CHUNKS;
    const __bf16* row = stage + (lane >> 2) * SC::ROW + 4 * (lane & 3);
    const __bf16 *x = row + SC::x(J) + 16 * (t / NJ), *y = row + SC::y(J) + 16 * (t % NJ);
    if (nc == kStepSamples / 32) {
#pragma unroll
      for (int c = 0; c < CHUNKS; ++c) chunk(x, y, c0 + c);
    } else {
#pragma unroll 1
      for (int c = c0; c < min(nc, c0 + CHUNKS); ++c) chunk(x, y, c);
    }
  }
  // The workgroup's sums to out (row-major kin x kout); waves that share a
  // tile meet in LDS.
  __device__ __forceinline__ void store(float* lds, float* __restrict__ out, int w, int lane) const {
    f4 sum = v;
    if constexpr (SPLIT > 1) {
      __syncthreads();
      *reinterpret_cast<f4*>(lds + (w * kWave + lane) * 4) = v;
      __syncthreads();
      if (w >= TILES) return;
#pragma unroll
      for (int p = 1; p < SPLIT; ++p) sum += *reinterpret_cast<const f4*>(lds + ((w + p * TILES) * kWave + lane) * 4);
    }
    const int t = w % TILES, cy = 16 * (t % NJ) + (lane & 15);
    const int col = NJ == 1 ? cy : mixed_fwd_feature<N>(1, cy >> 5, (cy >> 3) & 3, cy & 7);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int cx = 16 * (t / NJ) + 4 * (lane >> 4) + r;
      const int row = mixed_fwd_feature<N>(J, cx >> 5, (cx >> 3) & 3, cx & 7);
      if (row >= 0 && row < N::kin(J) && col < N::kout(J)) out[row * N::kout(J) + col] = sum[r];
    }
  }
};

template <class N>
struct OwnAll {
  OwnedDW16<N, 0> w0;
  OwnedDW16<N, 1> w1;
  OwnedDW16<N, 2> w2;
  OwnedDW16<N, N::NCH == 2 ? 3 : 2> w3;  // second colour hidden layer (unused with one)
  OwnedDW16<N, N::NW - 1> wl;
};

// This lane's values of columns c on of its sample (S: the sample's row plus
// the lane group's place): 32 columns a bf8, or 16 (its first half).
template <int K>
__device__ __forceinline__ void stage32(__bf16* S, const bf8 (&a)[K], int g) {
#pragma unroll
  for (int k = 0; k < K; ++k) *reinterpret_cast<bf8*>(S + 32 * k + 8 * g) = a[k];
}
__device__ __forceinline__ void stage16(__bf16* S, const bf8& a, int g) {
  const s8 v = __builtin_bit_cast(s8, a);
  *reinterpret_cast<s4*>(S + 4 * g) = __builtin_shufflevector(v, v, 0, 1, 2, 3);
}

// Forward recompute, backward chain and dL/de of this wave's tile, with the
// workgroup's weight-gradient products of each staging group in between.
// fetch (of the next step's inputs into in) is called where the colour layers'
// activations are no longer held.
template <class N, class Fetch>
__device__ __forceinline__ void bwd_tile(const __bf16* __restrict__ Af, const __bf16* __restrict__ Ab, __bf16* stage,
                                         const TileIn<N>& in, int s, bool valid, int nc, const RecordBuffers& rec,
                                         OwnAll<N>& dw, int w, int lane, const Fetch& fetch) {
  using M = Mixed<N>;
  using SC = StageCols<N>;
  constexpr f4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
  constexpr int H = N::HC / 32, D = N::HD / 32;
  const int g = lane >> 4;
  __bf16* mine = stage + (16 * w + (lane & 15)) * SC::ROW;  // this lane's sample
  PActs<N> a[1];
  f4 sh[1];
  tile_operands<N>(in, g, a[0], sh[0]);
  fwd_tiles<N, 1>(Af, lane, sh, a);

  f4 dz = zero;
  if (g == 0) {
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      const float cc = sigmoid_rcp(a[0].z[r]);
      dz[r] = in.dr[r] * cc * (1.0f - cc);
    }
  }
  // W (m, k) of a layer's input-gradient product
  auto w_of = [&](int j, int m, int k) { return lds_bf8<N>(Ab + M::boff(j), m * M::bks(j) + k, lane); };
  // the hidden-layer gradients are used only as BF16 (MFMA operands and
  // staged values), so they are rounded once and masked on their bits
  const bf8(&hl)[H] = N::NCH == 2 ? a[0].h4 : a[0].h3;
  bf8 dhl[H];
  const bf8 dzp = pack8(dz, zero);
  {
    f4 raw[2 * H];
#pragma unroll
    for (int m = 0; m < 2 * H; ++m) raw[m] = mfma32(w_of(N::NW - 1, m, 0), dzp, zero);
#pragma unroll
    for (int k = 0; k < H; ++k) dhl[k] = relu_mask8(pack8(raw[2 * k], raw[2 * k + 1]), hl[k]);
  }
  // colour layers: the last one, then (with two) the second hidden one
  __syncthreads();  // the step before has been added
  stage32(mine + SC::x(N::NW - 1), hl, g);
  stage16(mine + SC::y(N::NW - 1), dzp, g);
  if constexpr (N::NCH == 2) {
    stage32(mine + SC::x(3), a[0].h3, g);
    stage32(mine + SC::y(3), dhl, g);
  }
  __syncthreads();
  dw.wl.add(stage, w, lane, nc);
  if constexpr (N::NCH == 2) dw.w3.add(stage, w, lane, nc);
  bf8 dh3[H];
  if constexpr (N::NCH == 2) {
    f4 acc[2 * H];
#pragma unroll
    for (int m = 0; m < 2 * H; ++m) acc[m] = zero;
#pragma unroll
    for (int k = 0; k < H; ++k)
#pragma unroll
      for (int m = 0; m < 2 * H; ++m) acc[m] = mfma32(w_of(3, m, k), dhl[k], acc[m]);
#pragma unroll
    for (int k = 0; k < H; ++k) dh3[k] = relu_mask8(pack8(acc[2 * k], acc[2 * k + 1]), a[0].h3[k]);
  } else {
#pragma unroll
    for (int k = 0; k < H; ++k) dh3[k] = dhl[k];
  }
  // first colour layer (gradient of the geometry features), second density layer
  f4 dgeo = zero;
#pragma unroll
  for (int k = 0; k < H; ++k) dgeo = mfma32(w_of(2, 0, k), dh3[k], dgeo);
  if (g == 0) dgeo[0] += __expf(a[0].o[0]) * in.ds;  // rounded to BF16 next
  bf8 dh1[D];
  const bf8 dgp = pack8(dgeo, zero);
  {
    f4 raw[2 * D];
#pragma unroll
    for (int m = 0; m < 2 * D; ++m) raw[m] = mfma32(w_of(1, m, 0), dgp, zero);
#pragma unroll
    for (int k = 0; k < D; ++k) dh1[k] = relu_mask8(pack8(raw[2 * k], raw[2 * k + 1]), a[0].h1[k]);
  }
  __syncthreads();
  *reinterpret_cast<bf8*>(mine + SC::x(2) + 8 * g) = a[0].osh;
  stage32(mine + SC::y(2), dh3, g);
  stage32(mine + SC::x(1), a[0].h1, g);
  stage16(mine + SC::y(1), dgp, g);
  fetch();
  __syncthreads();
  dw.w2.add(stage, w, lane, nc);
  dw.w1.add(stage, w, lane, nc);
  // first density layer: dL/de, as BF16 pairs (the table-gradient records it
  // feeds are BF16 too)
  constexpr int MT0 = N::bmt(0);
  f4 de[MT0];
#pragma unroll
  for (int m = 0; m < MT0; ++m) de[m] = zero;
#pragma unroll
  for (int k = 0; k < D; ++k)
#pragma unroll
    for (int m = 0; m < MT0; ++m) de[m] = mfma32(w_of(0, m, k), dh1[k], de[m]);
  if (valid) {
#pragma unroll
    for (int q = 0; q < N::LPL; ++q) {
      const int k0 = 2 * q, k1 = 2 * q + 1;
      reinterpret_cast<uint32_t*>(rec.de)[(size_t)(g + 4 * q) * rec.stride + s] =
          bf16_pair(de[k0 >> 2][k0 & 3], de[k1 >> 2][k1 & 3]);
    }
  }
  __syncthreads();
  *reinterpret_cast<bf8*>(mine + SC::x(0) + 8 * g) = a[0].e;
  stage32(mine + SC::y(0), dh1, g);
  __syncthreads();
  dw.w0.add(stage, w, lane, nc);
}

// Sixteen waves, four a SIMD.  The matrix instructions are a fifth of the
// time; a wave waits at each step of its serial chain (operands from LDS, product, rounding,
// barriers), so what counts is how many waves share a SIMD and how few LDS accesses
// a tile takes.  At 262k samples of the 64-wide network 46.8 us with eight
// waves of up to 256 registers, two-byte stores to [feature][sample] rows and
// the weights read a layer ahead, 38.6 so; at 100003 samples 26.4 and 21.6; the
// 32-wide network at 1M samples 75.7 and 54.7.  Of the 64-wide network's 128 registers
// two values spill (12 bytes of scratch a lane).  (Eight waves with two
// tiles each and 32x32 products, which halve the LDS reads: 48.1, 26.8, 75.0.)
template <class N>
__global__ __launch_bounds__(kBwdWaves * kWave) void mixed_bwd8_kernel(
    LevelInfo lv, const _Float16* __restrict__ table, const __bf16* __restrict__ prep, SampleSrc src,
    const float* __restrict__ dsigma, const float* __restrict__ drgb, RecordBuffers rec,
    float* __restrict__ dw_partial) {
  using M = Mixed<N>;
  __shared__ __attribute__((aligned(16))) __bf16 ops[M::FWD + M::BWD];
  __shared__ __attribute__((aligned(16))) __bf16 stage[kStepSamples * StageCols<N>::ROW];
  static_assert(sizeof(stage) >= kBwdWaves * kWave * sizeof(f4), "the sums' last step reuses it");
  const __bf16 *Af = ops, *Ab = ops + M::FWD;
  copy_to_lds<kBwdWaves * kWave, sizeof(ops)>(ops, prep);
  __syncthreads();

  const int S = src.n_dev ? (int)*src.n_dev : src.n;
  const int w = threadIdx.x / kWave, lane = lane_id(), g = lane >> 4, jc = lane & 15;
  OwnAll<N> dw;
  dw.w0.zero(); dw.w1.zero(); dw.w2.zero(); dw.wl.zero();
  if constexpr (N::NCH == 2) dw.w3.zero();
  LaneLevels<N> ll;
  lane_levels<N>(lv, g, ll);
  const int nsteps = (S + kStepSamples - 1) / kStepSamples, step = gridDim.x;
  const int off = 16 * w + jc;
  // pieces of 32 samples in step p
  auto pieces = [&](int p) { return min(kStepSamples / 32, (S - kStepSamples * p + 31) / 32); };
  TileIn<N> in;
  if (!kGathers<N> || src.ecache) {
    uint32_t rid = ray_of<N>(src, kStepSamples * (int)blockIdx.x + off, S);
    auto fetch = [&](int p) {  // the inputs of step p, and the ray index of the one after
      const int s = kStepSamples * p + off;
      fetch_tile<N, true>(src, table, lv, ll, dsigma, drgb, s, s < S, g, rid, in);
      rid = ray_of<N>(src, s + kStepSamples * step, S);
    };
    fetch(blockIdx.x);
    for (int p = blockIdx.x; p < nsteps; p += step) {
      const int s = kStepSamples * p + off;
      bwd_tile<N>(Af, Ab, stage, in, s, s < S, pieces(p), rec, dw, w, lane, [&] { fetch(p + step); });
    }
  } else if constexpr (kGathers<N>) {
    for (int p = blockIdx.x; p < nsteps; p += step) {
      const int s = kStepSamples * p + off;
      fetch_tile<N, false>(src, table, lv, ll, dsigma, drgb, s, s < S, g, 0u, in);
      bwd_tile<N>(Af, Ab, stage, in, s, s < S, pieces(p), rec, dw, w, lane, [] {});
    }
  }
  float* sums = reinterpret_cast<float*>(stage);
  float* out = dw_partial + (size_t)blockIdx.x * N::NWEIGHTS;
  dw.w0.store(sums, out + N::woff(0), w, lane);
  dw.w1.store(sums, out + N::woff(1), w, lane);
  dw.w2.store(sums, out + N::woff(2), w, lane);
  if constexpr (N::NCH == 2) dw.w3.store(sums, out + N::woff(3), w, lane);
  dw.wl.store(sums, out + N::woff(N::NW - 1), w, lane);
}

// Forward: density and colour of 16-sample tiles, one tile per wave at a
// time (four waves per SIMD stay resident, which hides latency better than
// pairing tiles here; the register budget is held to four waves, without
// which the compiler takes 136 registers, three waves, and the fixed grid
// needs a second round).  The grid is a fixed number of workgroups, so the
// weight operands are staged into LDS once per workgroup rather than once per
// four tiles; with the kept encoding, a wave fetches its next tile's inputs
// while it computes the current one (ray indices two tiles ahead).
template <class N>
constexpr int kMixedFwdGrid = N::HD >= 64 ? 1024 : 2048;  // four or eight waves a SIMD

template <class N>
__device__ __forceinline__ void fwd_store(const PActs<N>& a, int g, int s, bool valid, float* __restrict__ sigma_out,
                                          float* __restrict__ rgb_out) {
  if (g == 0 && valid) {
    sigma_out[s] = expf(a.o[0]);
    rgb_out[3 * s + 0] = sigmoid_rcp(a.z[0]);
    rgb_out[3 * s + 1] = sigmoid_rcp(a.z[1]);
    rgb_out[3 * s + 2] = sigmoid_rcp(a.z[2]);
  }
}

//
// Workgroups past the MLP's (bp.nbins of them) run the table-gradient column
// scan (bins.h), which needs only the record counts of the encoding.
template <class N>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void mixed_fwd_kernel(
    LevelInfo lv, const _Float16* __restrict__ table, const __bf16* __restrict__ prep, SampleSrc src,
    float* __restrict__ sigma_out, float* __restrict__ rgb_out, BinPrep bp) {
  using M = Mixed<N>;
  const int G = (int)gridDim.x - bp.nbins;  // the MLP's workgroups
  if ((int)blockIdx.x >= G) {
    colscan_bin(bp.rb, bp.nunits, (int)blockIdx.x - G);
    return;
  }
  __shared__ __attribute__((aligned(16))) __bf16 Af[M::FWD];
  copy_to_lds<256, sizeof(Af)>(Af, prep);
  __syncthreads();
  const int S = src.n_dev ? (int)*src.n_dev : src.n;
  const int ntiles = (S + 15) / 16;
  const int lane = lane_id(), g = lane >> 4, jc = lane & 15;
  const int first = blockIdx.x * (blockDim.x / kWave) + (threadIdx.x / kWave);
  const int step = G * (blockDim.x / kWave);
  if (first >= ntiles) return;
  LaneLevels<N> ll;
  lane_levels<N>(lv, g, ll);
  if (src.ecache) {
    TileIn<N> cur;
    const int s0 = 16 * first + jc;
    fetch_tile<N, true>(src, table, lv, ll, nullptr, nullptr, s0, s0 < S, g, ray_of<N>(src, s0, S), cur);
    uint32_t rid1 = ray_of<N>(src, 16 * (first + step) + jc, S);
    for (int tile = first; tile < ntiles; tile += step) {
      const int s = 16 * tile + jc, s1 = s + 16 * step;
      TileIn<N> nxt;
      fetch_tile<N, true>(src, table, lv, ll, nullptr, nullptr, s1, s1 < S, g, rid1, nxt);
      rid1 = ray_of<N>(src, s1 + 16 * step, S);
      PActs<N> a[1];
      f4 sh[1];
      tile_operands<N>(cur, g, a[0], sh[0]);
      fwd_tiles<N, 1>(Af, lane, sh, a);
      fwd_store<N>(a[0], g, s, s < S, sigma_out, rgb_out);
      cur = nxt;
    }
  } else {
    for (int tile = first; tile < ntiles; tile += step) {
      const int s = 16 * tile + jc;
      TileIn<N> in;
      fetch_tile<N, false>(src, table, lv, ll, nullptr, nullptr, s, s < S, g, 0u, in);
      PActs<N> a[1];
      f4 sh[1];
      tile_operands<N>(in, g, a[0], sh[0]);
      fwd_tiles<N, 1>(Af, lane, sh, a);
      fwd_store<N>(a[0], g, s, s < S, sigma_out, rgb_out);
    }
  }
}

// Forward of many samples without a given encoding, for the networks of 16
// levels: a wave takes 64 samples and gathers level after level, one sample a
// lane, so that all waves are at about the same level and its 2 MB stay in
// each XCD's L2 (mixed_fwd_kernel gathers all levels of 16 samples at once, 24 MB
// of tables).  Bound by the misses all the same, and by the lines a CU's
// loads take in.  From kWalkMin samples on it is the faster one: a call of 100003
// random samples 86.6 -> 71.5 us (the kernel 71.4 -> 64.8), 200000 160 -> 140, 40000
// 39.1 -> 33.9, but 20000 25.9 -> 27.2 and 5000 13.9 -> 20.3, since a wave then
// waits for 16 levels in turn.  And with tables of more than an L2's 4 MB: of
// 100003 samples along rays, levels of 2^17 entries take 51 us either way, of 2^18 61.7 -> 57.4,
// but of 2^16 32.4 -> 41.7 and of 2^10 18.7 -> 29.4 (random samples: 2^16 40 -> 46,
// 2^10 18.6 -> 29.9).
// (Two or four waves a workgroup, or two or four levels' loads in flight, were
// slower up to 100000.)
constexpr int kWalkMin = 32768;
constexpr int64_t kWalkTable = 4 << 20;
template <class N>
__global__ __launch_bounds__(kWave) void mixed_fwd_walk_kernel(
    LevelInfo lv, const _Float16* __restrict__ table, const __bf16* __restrict__ prep, SampleSrc src,
    float* __restrict__ sigma_out, float* __restrict__ rgb_out) {
  using M = Mixed<N>;
  __shared__ __attribute__((aligned(16))) __bf16 Af[M::FWD];
  __shared__ uint32_t enc[N::L][kWave];
  copy_to_lds<kWave, sizeof(Af)>(Af, prep);
  __syncthreads();
  const int S = src.n_dev ? (int)*src.n_dev : src.n;
  const int lane = lane_id(), g = lane >> 4, jc = lane & 15;
  for (int64_t first = (int64_t)blockIdx.x * kWave; first < S; first += (int64_t)gridDim.x * kWave) {
    const int s0 = (int)first, left = S - s0;
    float xn[3] = {0.5f, 0.5f, 0.5f};
    if (lane < left) load_position(src, s0 + lane, xn);
#pragma unroll 1
    for (int l = 0; l < N::L; ++l) {
      Corner8 c;
      corners(xn[0], xn[1], xn[2], lv.res[l], (lv.dense_bits >> l) & 1u, lv.table_mask, lv.offset[l], c);
      const float2 e = blend_corners<true>(table, c);
      enc[l][lane] = lane < left ? bf16_pair(e.x, e.y) : 0u;
    }
    wave_lds_fence();
#pragma unroll 1
    for (int t = 0; t < kWave / 16; ++t) {
      if (16 * t >= left) break;
      const bool valid = 16 * t + jc < left;
      const int st = s0 + 16 * t + jc;
      TileIn<N> in;
      in.d[0] = 0.0f; in.d[1] = 0.0f; in.d[2] = 1.0f;
      if (valid) load_direction(src, st, in.d);
#pragma unroll
      for (int q = 0; q < N::LPL; ++q) in.e[q] = enc[g + 4 * q][16 * t + jc];
      PActs<N> a[1];
      f4 sh[1];
      tile_operands<N>(in, g, a[0], sh[0]);
      fwd_tiles<N, 1>(Af, lane, sh, a);
      fwd_store<N>(a[0], g, st, valid, sigma_out, rgb_out);
    }
    wave_lds_fence();
  }
}

// ---------------------------------------------------------------------------
// Host launchers.  Shadow buffer: BF16 operands (forward, then backward),
// padded to 256 bytes, then the FP16 table (same entry layout as FP32).
// ---------------------------------------------------------------------------

template <class N>
constexpr size_t mixed_ops_bytes() {
  return ((size_t)(Mixed<N>::FWD + Mixed<N>::BWD) * 2 + 255) / 256 * 256;
}

size_t mixed_shadow_bytes(int shape, int64_t table_floats) {
  const size_t ops = shape == kShapeTiny ? mixed_ops_bytes<NetTiny>() : mixed_ops_bytes<NetFull>();
  return ops + ((size_t)table_floats * 2 + 255) / 256 * 256;
}

// With kf set, the same launch also sets up the n candidate rays and counts
// their samples.
template <class N>
static hipError_t prep_impl(const float* params, const WOffsets& wo, int64_t table_floats, void* shadow,
                            float* zero_grads, int64_t total, float* clear_flag, const KeyframeStore* kf,
                            const MarchParams* mp, const uint32_t* ids, int n, const RayBuffers* rb,
                            hipStream_t st) {
  using M = Mixed<N>;
  const int nops = M::FWD + M::BWD;
  _Float16* t16 = reinterpret_cast<_Float16*>(static_cast<char*>(shadow) + mixed_ops_bytes<N>());
  const int64_t span = zero_grads && total > table_floats ? total : table_floats;
  const int tblocks = (int)((span + 2047) / 2048);
  const int oblocks = (nops + 255) / 256;
  if (kf) {
    const int ncount = (int)count_block_count(*mp, n);
    hipLaunchKernelGGL(mixed_prepare_count_kernel<N>, dim3(ncount + tblocks + oblocks), dim3(256), 0, st, params,
                       wo, static_cast<__bf16*>(shadow), t16, table_floats, zero_grads, total, tblocks, clear_flag,
                       *kf, *mp, ids, n, *rb, ncount);
  } else {
    hipLaunchKernelGGL(mixed_prepare_kernel<N>, dim3(tblocks + oblocks), dim3(256), 0, st, params, wo,
                       static_cast<__bf16*>(shadow), t16, table_floats, zero_grads, total, tblocks, clear_flag);
  }
  return hipGetLastError();
}

template <class N>
static hipError_t fwd_impl(const LevelInfo& lv, const void* shadow, const SampleSrc& src, int max_samples,
                           float* sigma, float* rgb, hipStream_t st, const BinPrep* bp) {
  const int tiles = (max_samples + 15) / 16;
  const __bf16* ops = static_cast<const __bf16*>(shadow);
  const _Float16* t16 = reinterpret_cast<const _Float16*>(static_cast<const char*>(shadow) + mixed_ops_bytes<N>());
  const int grid = std::min((tiles + 3) / 4, kMixedFwdGrid<N>);
  const BinPrep none{};
  const BinPrep& b = bp ? *bp : none;
  if constexpr (!kGathers<N>) {
    const int last = lv.levels - 1;
    const int64_t m = lv.res[last] + 1;  // (the last level's entries: of a dense one its vertices)
    const int64_t entries = lv.offset[last] + ((lv.dense_bits >> last) & 1u ? m * m * m : (int64_t)lv.table_mask + 1);
    if (!src.ecache && b.nbins == 0 && max_samples >= kWalkMin && entries * 4 > kWalkTable) {
      hipLaunchKernelGGL(mixed_fwd_walk_kernel<N>, dim3(min(1 << 20, (max_samples - 1) / kWave + 1)), dim3(kWave), 0, st,
                         lv, t16, ops, src, sigma, rgb);
      return hipGetLastError();
    }
  }
  if (grid + b.nbins > 0)
    hipLaunchKernelGGL(mixed_fwd_kernel<N>, dim3(grid + b.nbins), dim3(256), 0, st, lv, t16, ops, src, sigma, rgb,
                       b);
  return hipGetLastError();
}

template <class N>
static hipError_t bwd_impl(const LevelInfo& lv, const void* shadow, const SampleSrc& src, int nblocks,
                           const float* dsigma, const float* drgb, const RecordBuffers& rec, float* partial,
                           const WOffsets& wo, float* grads, hipStream_t st) {
  if (!kGathers<N> && !src.ecache) return hipErrorInvalidValue;
  const __bf16* ops = static_cast<const __bf16*>(shadow);
  const _Float16* t16 = reinterpret_cast<const _Float16*>(static_cast<const char*>(shadow) + mixed_ops_bytes<N>());
  hipLaunchKernelGGL(mixed_bwd8_kernel<N>, dim3(nblocks), dim3(kBwdWaves * kWave), 0, st, lv, t16, ops, src,
                     dsigma, drgb, rec, partial);
  return hipGetLastError();
}

template <class N>
static hipError_t encode_impl(const LevelInfo& lv, const void* shadow, const SampleSrc& src, int max_samples,
                              uint32_t* hist, const BinLevels& bl, int64_t entries, hipStream_t st) {
  const _Float16* t16 = reinterpret_cast<const _Float16*>(static_cast<const char*>(shadow) + mixed_ops_bytes<N>());
  return launch_encode<N, _Float16, uint32_t>(lv, t16, src, max_samples, hist, bl, entries, st);
}
hipError_t mixed_encode(int shape, const LevelInfo& lv, const void* shadow, const SampleSrc& src, int max_samples,
                        uint32_t* hist, const BinLevels& bl, int64_t entries, hipStream_t st) {
  return shape == kShapeTiny ? encode_impl<NetTiny>(lv, shadow, src, max_samples, hist, bl, entries, st)
                             : encode_impl<NetFull>(lv, shadow, src, max_samples, hist, bl, entries, st);
}

hipError_t mixed_prepare(int shape, const float* params, const WOffsets& wo, int64_t table_floats, void* shadow,
                         float* zero_grads, int64_t total, float* clear_flag, hipStream_t st) {
  return shape == kShapeTiny ? prep_impl<NetTiny>(params, wo, table_floats, shadow, zero_grads, total, clear_flag,
                                                   nullptr, nullptr, nullptr, 0, nullptr, st)
                             : prep_impl<NetFull>(params, wo, table_floats, shadow, zero_grads, total, clear_flag,
                                                   nullptr, nullptr, nullptr, 0, nullptr, st);
}

hipError_t mixed_prepare_count(int shape, const float* params, const WOffsets& wo, int64_t table_floats,
                               void* shadow, float* zero_grads, int64_t total, float* clear_flag,
                               const KeyframeStore& kf, const MarchParams& mp, const uint32_t* ids, int n,
                               const RayBuffers& rb, hipStream_t st) {
  return shape == kShapeTiny ? prep_impl<NetTiny>(params, wo, table_floats, shadow, zero_grads, total, clear_flag,
                                                   &kf, &mp, ids, n, &rb, st)
                             : prep_impl<NetFull>(params, wo, table_floats, shadow, zero_grads, total, clear_flag,
                                                   &kf, &mp, ids, n, &rb, st);
}

hipError_t mixed_forward(int shape, const LevelInfo& lv, const void* shadow, const SampleSrc& src, int max_samples,
                         float* sigma, float* rgb, hipStream_t st, const BinPrep* bp) {
  return shape == kShapeTiny ? fwd_impl<NetTiny>(lv, shadow, src, max_samples, sigma, rgb, st, bp)
                             : fwd_impl<NetFull>(lv, shadow, src, max_samples, sigma, rgb, st, bp);
}

hipError_t mixed_backward(int shape, const LevelInfo& lv, const void* shadow, const SampleSrc& src, int nblocks,
                          const float* dsigma, const float* drgb, const RecordBuffers& rec, float* partial,
                          const WOffsets& wo, float* grads, hipStream_t st) {
  return shape == kShapeTiny
             ? bwd_impl<NetTiny>(lv, shadow, src, nblocks, dsigma, drgb, rec, partial, wo, grads, st)
             : bwd_impl<NetFull>(lv, shadow, src, nblocks, dsigma, drgb, rec, partial, wo, grads, st);
}

}  // namespace nsl
