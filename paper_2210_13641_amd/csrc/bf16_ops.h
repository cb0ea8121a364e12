// BF16 operands of v_mfma_f32_16x16x32_bf16: layout, conversion and LDS reads,
// shared by the mixed-precision kernels and by the FP32 networks that run on
// the BF16 matrix cores in three parts.
#pragma once
#include "net.h"

namespace nsl {

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ f4 mfma32(bf8 a, bf8 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

typedef __bf16 bf2 __attribute__((ext_vector_type(2)));

// Two floats as BF16 (round to nearest even), a in the low half; one
// v_cvt_pk_bf16_f32.
__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {
  const bf2 v = {(__bf16)a, (__bf16)b};
  return __builtin_bit_cast(uint32_t, v);
}

__device__ __forceinline__ bf8 pack8(f4 lo, f4 hi) {
  return __builtin_bit_cast(bf8, make_uint4(bf16_pair(lo[0], lo[1]), bf16_pair(lo[2], lo[3]),
                                            bf16_pair(hi[0], hi[1]), bf16_pair(hi[2], hi[3])));
}

// Layout of the BF16 operands (one block = 64 lanes x 8 values per (m, k-step)).
template <class N>
struct Mixed {
  static_assert(N::HD % 32 == 0 && N::HC % 32 == 0, "hidden widths must be multiples of 32");
  static constexpr int BLK = kWave * 8;
  static constexpr int fks(int j) { return j == 0 || j == 2 ? 1 : j == 1 ? N::HD / 32 : N::HC / 32; }
  static constexpr int fsize(int j) { return fks(j) * N::fmt(j) * BLK; }
  static constexpr int foff(int j) {
    int o = 0;
    for (int i = 0; i < j; ++i) o += fsize(i);
    return o;
  }
  static constexpr int FWD = foff(N::NW);
  static constexpr int bks(int j) { return j == N::NW - 1 || j == 1 ? 1 : j == 0 ? N::HD / 32 : N::HC / 32; }
  static constexpr int bsize(int j) { return bks(j) * N::bmt(j) * BLK; }
  static constexpr int boff(int j) {
    int o = 0;
    for (int i = 0; i < j; ++i) o += bsize(i);
    return o;
  }
  static constexpr int BWD = boff(N::NW);
};

// Input feature of forward k-slot (s, lane group g, value u) of layer j; -1 = pad.
template <class N>
__host__ __device__ constexpr int mixed_fwd_feature(int j, int s, int g, int u) {
  if (j == 0) return u < N::NSLOT ? 2 * (g + 4 * (u >> 1)) + (u & 1) : -1;
  if (j == 2) {
    if (u < 4) return 4 * g + u;
    const int k = 4 * g + (u - 4);
    return k < N::NSH ? N::GEO + k : -1;
  }
  return 32 * s + 16 * (u >> 2) + 4 * g + (u & 3);
}

template <class N>
__device__ __forceinline__ bf8 lds_bf8(const __bf16* A, int block, int lane) {
  return *reinterpret_cast<const bf8*>(A + (size_t)block * Mixed<N>::BLK + lane * 8);
}

// ---------------------------------------------------------------------------
// FP32 products on the BF16 matrix cores, in the three-part form of Henry, Tang
// and Heinecke ("Leveraging the bfloat16 artificial intelligence datatype for
// higher-precision computations", 2019).  An FP32 value is the sum of three
// BF16 values, x = h + m + l, each the nearest to what the ones before leave
// (8 significant bits a part, the last error at most 2^-27 |x|), and a product
// of two values is the six part products of 2^-18 or more: h h, h m, m h,
// m m, h l, l h.  The three that are left out are at most 2^-26 of it, below
// the 2^-24 that one FP32 rounding costs.  A layer adds its small part
// products first and h h last, with FP32 accumulation throughout: measured
// against 64 bits over products of 64 terms, its error is 0.32 to 0.38 of
// what v_mfma_f32_16x16x4_f32 gives for normal, uniform, positive and ReLU'd operands.
// Six 16-cycle products replace eight of 32 cycles (2.7 times fewer matrix
// cycles); the parts cost about five vector instructions a value, which is
// why only the 64-wide networks take this route.
//
// A value that is not finite (or above the largest BF16) has no parts: its
// outputs come out NaN, and the caller evaluates those columns with FP32 products.
// ---------------------------------------------------------------------------

struct Split8 {
  bf8 v[3];  // h, m, l
};

__device__ __forceinline__ Split8 split8(f4 a, f4 b) {
  uint32_t w[3][4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float x = i < 2 ? a[2 * i] : b[2 * i - 4], y = i < 2 ? a[2 * i + 1] : b[2 * i - 3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      w[c][i] = bf16_pair(x, y);
      x -= __uint_as_float(w[c][i] << 16);
      y -= __uint_as_float(w[c][i] & 0xFFFF0000u);
    }
  }
  Split8 s;
#pragma unroll
  for (int c = 0; c < 3; ++c) s.v[c] = __builtin_bit_cast(bf8, make_uint4(w[c][0], w[c][1], w[c][2], w[c][3]));
  return s;
}

// ReLU that keeps a NaN, so that it reaches the network's outputs and their
// check (v_maximum3_f32; fmaxf returns the other operand).
__device__ __forceinline__ f4 relu_nan(f4 v) {
#pragma unroll
  for (int r = 0; r < 4; ++r) v[r] = __builtin_elementwise_maximum(v[r], 0.0f);
  return v;
}

// acc[t][m] = sum over the k-steps of W (tiles m, laid out from A on, parts
// `part` elements apart) times x[t], for T tiles of 16 samples.
template <class N, int MT, int KS, int T>
__device__ __forceinline__ void split_layer(const __bf16* A, int part, int lane, const Split8 (&x)[T][KS],
                                            f4 (&acc)[T][MT]) {
  constexpr int kW[6] = {2, 0, 1, 1, 0, 0}, kX[6] = {0, 2, 1, 0, 1, 0};  // (weight part, value part), small ones first
  constexpr int kFrom[4] = {0, 3, 5, 6};
  constexpr int G = MT % 2 == 0 ? 2 : 1;  // tiles taken together (independent chains)
#pragma unroll
  for (int m0 = 0; m0 < MT; m0 += G) {
    bf8 w[G][KS][3];
#pragma unroll
    for (int i = 0; i < G; ++i)
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int c = 0; c < 3; ++c) w[i][s][c] = lds_bf8<N>(A + c * part, (m0 + i) * KS + s, lane);
    f4 r[T][G];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int i = 0; i < G; ++i) r[t][i] = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int k = kFrom[p]; k < kFrom[p + 1]; ++k)
#pragma unroll
          for (int i = 0; i < G; ++i)
#pragma unroll
            for (int t = 0; t < T; ++t) r[t][i] = mfma32(w[i][s][kW[k]], x[t][s].v[kX[k]], r[t][i]);
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int i = 0; i < G; ++i) acc[t][m0 + i] = r[t][i];
  }
}

// The networks on T tiles: geometry outputs o and colour logits z (as the
// FP32 kernels hold them) from the encoding slots and SH coefficients.
template <class N, int T>
__device__ __forceinline__ void split_mlp(const __bf16* Af, int lane, const float (&e)[T][N::NSLOT], const f4 (&sh)[T],
                                          f4 (&o)[T], f4 (&z)[T]) {
  using M = Mixed<N>;
  constexpr int H = N::HC / 16, K = N::HC / 32;
  static_assert(N::NSLOT == 8 && N::NCH == 2 && N::HD == N::HC, "the 16-level network");
  Split8 x1[T][1], x[T][K];
  f4 h[T][H], r[T][1];
  auto hidden = [&] {
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int s = 0; s < K; ++s) x[t][s] = split8(relu_nan(h[t][2 * s]), relu_nan(h[t][2 * s + 1]));
  };
#pragma unroll
  for (int t = 0; t < T; ++t)
    x1[t][0] = split8(f4{e[t][0], e[t][1], e[t][2], e[t][3]}, f4{e[t][4], e[t][5], e[t][6], e[t][7]});
  split_layer<N, H, 1, T>(Af + M::foff(0), M::FWD, lane, x1, h);
  hidden();
  split_layer<N, 1, K, T>(Af + M::foff(1), M::FWD, lane, x, r);
#pragma unroll
  for (int t = 0; t < T; ++t) {
    o[t] = r[t][0];
    x1[t][0] = split8(o[t], sh[t]);
  }
  split_layer<N, H, 1, T>(Af + M::foff(2), M::FWD, lane, x1, h);
  hidden();
  split_layer<N, H, K, T>(Af + M::foff(3), M::FWD, lane, x, h);
  hidden();
  split_layer<N, 1, K, T>(Af + M::foff(4), M::FWD, lane, x, r);
#pragma unroll
  for (int t = 0; t < T; ++t) z[t] = r[t][0];
}

// Whether a column's density logit and colour logits (rows 0 .. 2 of z) are
// finite.  Whatever in a column has no parts makes its next layer NaN and, since
// relu_nan keeps them, one of these.
__device__ __forceinline__ bool all_finite(float o0, f4 z) {
  const float c = fmaf(o0, 0.0f, fmaf(z[0], 0.0f, fmaf(z[1], 0.0f, z[2] * 0.0f)));
  return c == c;
}

}  // namespace nsl
