// Device helpers shared by the gfx950 kernels of the mapping step.
//
// Sample positions decide integer quantities (occupancy cell, trilinear
// cell, AABB membership), so they are formed in IEEE single precision with
// every operation rounded separately, in a fixed order:
//   a = ((u + 0.5) - cx) / fx,  b = ((v + 0.5) - cy) / fy,
//   s = sqrt((a*a + b*b) + 1),  d_i = ((R_i0*a + R_i1*b) + R_i2) / s,
//   x_i = o_i + t*d_i,  xn_i = clamp((x_i - lo_i) * inv_i, 0, 1).
// Contraction into FMA is switched off in these functions, and division and
// square root are the correctly rounded ones (the library is built with
// -fhip-fp32-correctly-rounded-divide-sqrt), so any IEEE implementation of the
// same sequence lands on the same bits.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace nsl {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kWave = 64;
constexpr int kMaxLevels = 16;
constexpr uint32_t kPrime1 = 2654435761u;
constexpr uint32_t kPrime2 = 805459861u;

struct LevelInfo {
  int levels;
  uint32_t table_mask;          // table entries per hashed level - 1 (power of two)
  uint32_t dense_bits;          // bit l set: level l is dense
  int res[kMaxLevels];          // N_l
  uint32_t offset[kMaxLevels];  // first entry of level l
};

struct Aabb {
  float lo[3], hi[3], inv[3];
};

__device__ __forceinline__ void camera_ray(const float* __restrict__ pose,
                                           const float* __restrict__ intr, int u, int v,
                                           float o[3], float d[3], float& s) {
#pragma clang fp contract(off)
  const float a = (((float)u + 0.5f) - intr[2]) / intr[0];
  const float b = (((float)v + 0.5f) - intr[3]) / intr[1];
  s = __builtin_sqrtf((a * a + b * b) + 1.0f);
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    d[i] = ((pose[4 * i] * a + pose[4 * i + 1] * b) + pose[4 * i + 2]) / s;
    o[i] = pose[4 * i + 3];
  }
}

__device__ __forceinline__ float pos_axis(float o, float d, float t) {
#pragma clang fp contract(off)
  return o + t * d;
}

__device__ __forceinline__ float normalise_axis(float x, float lo, float inv) {
#pragma clang fp contract(off)
  float xn = (x - lo) * inv;
  return fminf(fmaxf(xn, 0.0f), 1.0f);
}

// floor(xn*N) taken on the exact product (TwoProduct: xn*N = ph + pl exactly),
// clamped to N-1; f = xn*N - i0 and g = (i0 + 1) - xn*N, each rounded once
// from the exact product (ph - i0 and (i0 + 1) - ph are exact), so both
// trilinear factors keep full relative precision: 1 - f formed from a
// rounded f loses it when f is near 1.
__device__ __forceinline__ int cell_floor(float xn, int n, float& f, float& g) {
  // no contraction: fused, xn*N - i would be rounded once with the product's
  // error inside it, and adding pl would count that error twice
#pragma clang fp contract(off)
  const float nf = (float)n;
  const float ph = xn * nf;
  const float pl = __builtin_fmaf(xn, nf, -ph);
  float fl = __builtin_floorf(ph);
  if (ph == fl && pl < 0.0f) fl -= 1.0f;
  int i = (int)fl;
  if (i > n - 1) i = n - 1;
  f = (ph - (float)i) + pl;
  g = ((float)(i + 1) - ph) - pl;
  return i;
}

__device__ __forceinline__ uint32_t grid_index(uint32_t x, uint32_t y, uint32_t z, int n,
                                               bool dense, uint32_t mask) {
  if (dense) {
    const uint32_t m = (uint32_t)n + 1u;
    return x + m * (y + m * z);
  }
  return (x ^ (y * kPrime1) ^ (z * kPrime2)) & mask;
}

__device__ __forceinline__ float sigmoidf(float z) { return 1.0f / (1.0f + __expf(-z)); }

// A pixel's depth target along its ray and the precision of its measurement
// (Eq. 4 read with Sigma_D a variance): (D_z s, 1 / (Sigma_z s^2)) when D_z
// and Sigma_z are finite and Sigma_z > 0, else (0, 0): an unusable
// measurement carries no depth loss.
__device__ __forceinline__ float2 depth_target(float Dz, float Vz, float s) {
  const bool ok = isfinite(Dz) && isfinite(Vz) && Vz > 0.0f;
  return ok ? make_float2(Dz * s, 1.0f / (Vz * s * s)) : make_float2(0.0f, 0.0f);
}

// One ray's terms of the mapping loss (Eq. 3, 4, 7) and the seeds of its
// adjoint: l_rgb = |I* - I|^2, l_d = pi (d* - D)^2, dL/dI* = k_rgb (I* - I),
// dL/dd* = k_d pi (d* - D), with the caller's factors k (2/R times the loss
// scale, times lambda_D for the depth term, in the step).
struct RayLoss {
  float l_rgb, l_d, gC[3], gD;
};
__device__ __forceinline__ RayLoss ray_loss(const float C[3], float D, float4 target, float pi, float k_rgb,
                                            float k_d) {
  RayLoss o;
  const float e0 = C[0] - target.x, e1 = C[1] - target.y, e2 = C[2] - target.z, ed = D - target.w;
  o.l_rgb = e0 * e0 + e1 * e1 + e2 * e2;
  o.l_d = pi * ed * ed;
  o.gC[0] = k_rgb * e0;
  o.gC[1] = k_rgb * e1;
  o.gC[2] = k_rgb * e2;
  o.gD = k_d * pi * ed;
  return o;
}

// Wave-wide helpers (wave64).
__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

// DPP row shift towards lower lanes: lane i of each 16-lane row receives the
// value of lane i+N of the same row (0 when i+N leaves the row).
template <int N>
__device__ __forceinline__ int row_from_above(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x100 + N, 0xF, 0xF, true);
}
template <int N>
__device__ __forceinline__ float row_from_above(float v) {
  return __int_as_float(row_from_above<N>(__float_as_int(v)));
}
// Lane i receives lane i-N of its row (0 when i-N leaves the row).
template <int N>
__device__ __forceinline__ int row_from_below(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x110 + N, 0xF, 0xF, true);
}

// Cross-lane moves of a whole wave without LDS (every lane is active).
// rotated<N>: lane i of each row gets lane i - N of it, modulo 16.
template <int N>
__device__ __forceinline__ float row_rotated(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + N, 0xF, 0xF, true));
}
// Lane i gets lane i - 1, lane 0 zero.
__device__ __forceinline__ float wave_up_1(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xF, 0xF, true));
}
typedef unsigned u2 __attribute__((ext_vector_type(2)));
// Rows (0, 0, 2, 2) and (1, 1, 3, 3) of v; halves (0, 0) of a and of b.
__device__ __forceinline__ u2 even_odd_rows(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return u2{r[0], r[1]};
}
__device__ __forceinline__ u2 swap_halves(uint32_t a, uint32_t b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  return u2{r[0], r[1]};
}
// Lane i gets lane i - 16 (the first row any value).
__device__ __forceinline__ float wave_up_16(float v) {
  const u2 r = even_odd_rows(v);                  // (0, 0, 2, 2), (1, 1, 3, 3)
  const uint32_t h = swap_halves(r[0], r[1])[0];  // (0, 0, 1, 1)
  return __uint_as_float((lane_id() & 48) == 32 ? h : r[0]);
}

// Sum over each half of the wave, in every lane: pairs of lanes 16 apart, then
// 8, 4, 2 and 1 (from 8 on a rotation brings the lane that many further, as the
// values repeat).
__device__ __forceinline__ float half_sum(float v) {
  const u2 r = even_odd_rows(v);
  v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  v += row_rotated<8>(v);
  v += row_rotated<4>(v);
  v += row_rotated<2>(v);
  return v + row_rotated<1>(v);
}
// Sum over the wave: pairs of lanes 32 apart, then the halves.
__device__ __forceinline__ float wave_sum(float v) {
  const u2 h = swap_halves(__float_as_uint(v), __float_as_uint(v));
  return half_sum(__uint_as_float(h[0]) + __uint_as_float(h[1]));
}

// Inclusive scan across each half of the wave: to each lane the value 1, 2, 4, 8
// and 16 lanes below in turn.
__device__ __forceinline__ float half_incl_scan(float v) {
  const int l = lane_id() & 31;
  float up = wave_up_1(v);
  v += l < 1 ? 0.0f : up;
  up = wave_up_1(wave_up_1(v));
  v += l < 2 ? 0.0f : up;
  up = wave_up_1(wave_up_1(wave_up_1(wave_up_1(v))));
  v += l < 4 ? 0.0f : up;
  const float rot = row_rotated<8>(v), below = wave_up_16(rot);
  v += (l & 8) ? rot : l < 16 ? 0.0f : below;
  up = wave_up_16(v);
  return v + (l < 16 ? 0.0f : up);
}

// Inclusive scan across the wave: to each lane the value 1, 2, 4, 8, 16 and 32
// lanes below in turn.
__device__ __forceinline__ float wave_incl_scan(float v) {
  const int l = lane_id();
  v += wave_up_1(v);
  v += wave_up_1(wave_up_1(v));
  v += wave_up_1(wave_up_1(wave_up_1(wave_up_1(v))));
  const float rot = row_rotated<8>(v), below = wave_up_16(rot);
  v += (l & 8) ? rot : l < 16 ? 0.0f : below;
  const float up = wave_up_16(v);
  v += l < 16 ? 0.0f : up;
  const float half = __uint_as_float(swap_halves(__float_as_uint(v), __float_as_uint(v))[0]);
  return v + (l < 32 ? 0.0f : half);
}

// Inclusive prefix sum over the wave: within each row by DPP shifts, then the
// totals of the rows before.  Every lane is active.
__device__ __forceinline__ uint32_t wave_incl_scan_u32(uint32_t v) {
  v += (uint32_t)row_from_below<1>((int)v);
  v += (uint32_t)row_from_below<2>((int)v);
  v += (uint32_t)row_from_below<4>((int)v);
  v += (uint32_t)row_from_below<8>((int)v);
  const uint32_t t0 = (uint32_t)__builtin_amdgcn_readlane((int)v, 15);
  const uint32_t t1 = t0 + (uint32_t)__builtin_amdgcn_readlane((int)v, 31);
  const uint32_t t2 = t1 + (uint32_t)__builtin_amdgcn_readlane((int)v, 47);
  const int row = lane_id() >> 4;
  return v + (row == 0 ? 0u : row == 1 ? t0 : row == 2 ? t1 : t2);
}

// Whether this lane starts a run of row_cell_runs below (a valid lane whose
// lower row neighbour is invalid, outside the row or in another cell).
__device__ __forceinline__ bool row_run_head(const uint32_t cell[3], bool valid) {
  const int r = threadIdx.x & 15;
  const int vb = row_from_below<1>((int)valid);  // every DPP read with all lanes active
  uint32_t cb[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) cb[i] = (uint32_t)row_from_below<1>((int)cell[i]);
  bool same_below = valid & (r != 0) & (vb != 0);
#pragma unroll
  for (int i = 0; i < 3; ++i) same_below &= cb[i] == cell[i];
  return valid & !same_below;
}

// Runs of consecutive valid lanes of each 16-lane row whose samples lie in
// the same grid cell (equal cell coordinates).  Such lanes share all eight
// corner entries, so one run structure serves every value: a segmented
// suffix sum gives the first lane of each run the sums of v[0..K) over the
// run.  Returns whether this lane starts a run.  When no lane of the wave
// shares its cell with the lane below, the scan is skipped (every lane is
// its own run and keeps its values).
template <int K>
__device__ __forceinline__ bool row_cell_runs(const uint32_t cell[3], bool valid, float (&v)[K]) {
  const int r = threadIdx.x & 15;
  // every neighbour read first, with all lanes active: a DPP read under a
  // partial exec mask (a short-circuit && would make it one) sees inactive
  // lanes as zero
  const int vb = row_from_below<1>((int)valid), va = row_from_above<1>((int)valid);
  uint32_t cb[3], ca[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    cb[i] = (uint32_t)row_from_below<1>((int)cell[i]);
    ca[i] = (uint32_t)row_from_above<1>((int)cell[i]);
  }
  bool same_below = valid & (r != 0) & (vb != 0);
  bool same_above = valid & (r != 15) & (va != 0);
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    same_below &= cb[i] == cell[i];
    same_above &= ca[i] == cell[i];
  }
  if (__ballot(same_below) == 0ull) return true;
  int tail = same_above ? 0 : 1;  // the run continues above this lane
#define NSL_RUN_STEP(N)                                               \
  {                                                                   \
    const int nt = row_from_above<N>(tail);                           \
    float nv[K];                                                      \
    _Pragma("unroll") for (int k = 0; k < K; ++k) nv[k] = row_from_above<N>(v[k]); \
    if (!tail) {                                                      \
      _Pragma("unroll") for (int k = 0; k < K; ++k) v[k] += nv[k];    \
      tail = nt;                                                      \
    }                                                                 \
  }
  // once every lane's sum reaches the end of its run (no lane still has a
  // continuation), the remaining steps would add nothing: runs of one or two
  // samples, the usual case at the middle levels, stop after the first step
  NSL_RUN_STEP(1)
  if (__ballot(!tail) == 0ull) return !same_below;
  NSL_RUN_STEP(2)
  if (__ballot(!tail) == 0ull) return !same_below;
  NSL_RUN_STEP(4)
  if (__ballot(!tail) == 0ull) return !same_below;
  NSL_RUN_STEP(8)
#undef NSL_RUN_STEP
  return !same_below;
}

// The 64-bit word of a (g0, g1) float pair after adding (a, b): the step of
// a compare-and-swap accumulation of both features at once.
__device__ __forceinline__ unsigned long long add_pair_bits(unsigned long long v, float a, float b) {
  const float x = __uint_as_float((unsigned)(v & 0xFFFFFFFFull)) + a;
  const float y = __uint_as_float((unsigned)(v >> 32)) + b;
  return (unsigned long long)__float_as_uint(x) | ((unsigned long long)__float_as_uint(y) << 32);
}

// Copies BYTES (a multiple of 16) from memory to LDS with the workgroup's
// THREADS threads, eight 16-byte loads of a thread in flight at a time.  (The
// compiler leaves a loop of one load and its wait as it is, a memory latency a
// pass: at 49999 samples of the 64-wide network the forward, ten passes, then
// took 17.6 us instead of 15.9 and the backward, nineteen, 66.3 instead of 62.9.)
template <int THREADS, int BYTES>
__device__ __forceinline__ void copy_to_lds(void* dst, const void* __restrict__ src) {
  static_assert(BYTES % 16 == 0, "whole 16-byte pieces");
  constexpr int n = BYTES / 16, full = n / THREADS, kBatch = 8;
  const f4* s = static_cast<const f4*>(src) + threadIdx.x;
  f4* d = static_cast<f4*>(dst) + threadIdx.x;
#pragma unroll
  for (int p = 0; p < full; p += kBatch) {
    f4 v[kBatch];
#pragma unroll
    for (int k = 0; k < kBatch; ++k)
      if (p + k < full) v[k] = s[(p + k) * THREADS];
#pragma unroll
    for (int k = 0; k < kBatch; ++k)
      if (p + k < full) d[(p + k) * THREADS] = v[k];
  }
  if (full * THREADS + (int)threadIdx.x < n) d[full * THREADS] = s[full * THREADS];
}

__device__ __forceinline__ f4 mfma4(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

}  // namespace nsl
