// Rays, samples and the batch cut of the mapping step on gfx950.
//
// The first pass sets up every candidate ray and counts its samples (one
// wave a ray with the occupancy sampler, one thread a ray with the uniform one;
// march_common.h), a scan turns counts into offsets and applies
// the batch cut, the second pass writes the samples.  Up to kEmitScanMax
// candidates the second pass does the scan itself (each workgroup the prefix
// before its candidates, one more workgroup the statistics), else a
// single-block scan runs between the two.
#include "march_common.h"

namespace nsl {

namespace {

using namespace march_detail;

__global__ __launch_bounds__(256) void rays_count_kernel(KeyframeStore kf, MarchParams mp,
                                                         const uint32_t* __restrict__ ids, int n,
                                                         RayBuffers rb) {
  rays_count_block(kf, mp, ids, n, rb, (int)blockIdx.x);
}

constexpr int kScanThreads = 1024, kScanRays = 8;
// Offsets stop here: candidates times samples a ray may reach 2^32 (2^20 of 4096),
// and an offset that wrapped would be below max_samples again, with its samples
// over those of the kept candidates.  A segment's counts (8192 of at most 4096)
// and a ray's samples still fit above it.
constexpr uint32_t kMaxOffset = 0xFFFFFFFFu - (1u << 26);
static_assert((int64_t)kScanRays * kScanThreads * 4096 < (1 << 26), "a segment fits");

// Single-block exclusive scan of the counts, batch cut and statistics, over
// segments of kScanRays * kScanThreads rays: each thread loads kScanRays
// consecutive ones (counts and precisions, 16-byte loads, the next segment's
// before this one is scanned), a wave scan (DPP) and the totals of the waves
// before give its exclusive offset, and the segment's total carries over to the
// next.  What bounds it is the latency of a segment: with four rays a thread,
// fetched when their segment begins, 32768 candidates took 15.5 us instead of 11.6.
__global__ __launch_bounds__(kScanThreads) void scan_cut_kernel(RayBuffers rb, int n, int max_samples) {
  __shared__ uint32_t wtot[kScanThreads / kWave];
  __shared__ uint32_t red[4][kScanThreads / kWave];
  constexpr int Q = kScanRays / 4;
  const int tid = threadIdx.x, wave = tid / kWave;
  uint32_t carry = 0, nr = 0, nk = 0, nm = 0, smax = 0;
  // a caller's arrays may not be
  const bool aligned = (((uintptr_t)rb.offsets | (uintptr_t)rb.counts) & 15u) == 0;
  struct Rays {
    uint32_t count[kScanRays];
    float prec[kScanRays];
  };
  auto fetch = [&](int64_t i0, Rays& r) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int64_t i = i0 + 4 * q;
      uint4 c = make_uint4(0u, 0u, 0u, 0u);
      float4 p = make_float4(1.0f, 1.0f, 1.0f, 1.0f);
      if (aligned && i + 4 <= n) {
        c = *reinterpret_cast<const uint4*>(rb.counts + i);
        p = *reinterpret_cast<const float4*>(rb.prec + i);
      } else {
        if (i < n) c.x = rb.counts[i], p.x = rb.prec[i];
        if (i + 1 < n) c.y = rb.counts[i + 1], p.y = rb.prec[i + 1];
        if (i + 2 < n) c.z = rb.counts[i + 2], p.z = rb.prec[i + 2];
        if (i + 3 < n) c.w = rb.counts[i + 3], p.w = rb.prec[i + 3];
      }
      const uint32_t c4[4] = {c.x, c.y, c.z, c.w};
      const float p4[4] = {p.x, p.y, p.z, p.w};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        r.count[4 * q + k] = c4[k];
        r.prec[4 * q + k] = p4[k];
      }
    }
  };
  constexpr int kSegment = kScanRays * kScanThreads;
  Rays next;
  fetch((int64_t)kScanRays * tid, next);
  for (int64_t seg = 0; seg < n; seg += kSegment) {
    const int64_t i0 = seg + (int64_t)kScanRays * tid;
    const Rays r = next;
    fetch(i0 + kSegment, next);
    uint32_t sum = 0;
#pragma unroll
    for (int k = 0; k < kScanRays; ++k) sum += r.count[k];
    const uint32_t incl = wave_incl_scan_u32(sum);
    if (lane_id() == kWave - 1) wtot[wave] = incl;
    __syncthreads();
    uint32_t run = carry + incl - sum, total = 0;  // exclusive
#pragma unroll
    for (int w = 0; w < kScanThreads / kWave; ++w) {
      run += w < wave ? wtot[w] : 0u;
      total += wtot[w];
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      uint32_t off[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int j = 4 * q + k;
        off[k] = min(run, kMaxOffset);
        run += r.count[j];
        if (i0 + j < n && run <= (uint32_t)max_samples) {
          ++nk;
          smax = run;  // kept candidates are a prefix
          if (r.count[j] > 0) {
            ++nr;
            if (r.prec[j] == 0.0f) ++nm;
          }
        }
      }
      const int64_t i = i0 + 4 * q;
      if (aligned && i + 4 <= n) {
        *reinterpret_cast<uint4*>(rb.offsets + i) = make_uint4(off[0], off[1], off[2], off[3]);
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (i + k < n) rb.offsets[i + k] = off[k];
      }
    }
    carry = min(carry + total, kMaxOffset);
    __syncthreads();
  }
  if (tid == 0) rb.offsets[n] = carry;
  // reductions (wave totals by the scan's last lane)
  nr = wave_incl_scan_u32(nr);
  nk = wave_incl_scan_u32(nk);
  nm = wave_incl_scan_u32(nm);
  for (int o = 32; o > 0; o >>= 1) smax = max(smax, (uint32_t)__shfl_xor((int)smax, o, kWave));
  if (lane_id() == kWave - 1) {
    red[0][wave] = nr;
    red[1][wave] = nk;
    red[2][wave] = nm;
    red[3][wave] = smax;
  }
  __syncthreads();
  if (tid == 0) {
    uint32_t R = 0, K = 0, M = 0, S = 0;
#pragma unroll
    for (int w = 0; w < kScanThreads / kWave; ++w) {
      R += red[0][w];
      K += red[1][w];
      M += red[2][w];
      S = max(S, red[3][w]);
    }
    rb.stats[0] = R;
    rb.stats[1] = S;
    rb.stats[2] = K;
    rb.stats[3] = M;
    if (rb.loss) rb.loss[0] = rb.loss[1] = rb.loss[2] = 0.0f;
  }
}

// The statistics of the batch cut alone (R, S, kept, masked, as
// scan_cut_kernel leaves them), by one workgroup of 256 threads: each thread
// takes a contiguous run of candidates, a scan of the run totals gives its
// offset, and a second pass over its run counts what the cut keeps.  It is the
// emission's longest workgroup: with every pass's loads its own and sums through
// LDS permutes the launch took 9.7 us instead of 8.5 at 4096 candidates of the
// paper-scale map, 4.2 instead of 3.6 at 1024 of the tiny field.
constexpr int kStatsThreads = 256;
__device__ __forceinline__ void cut_stats_block(const RayBuffers& rb, int n, int max_samples) {
  __shared__ uint32_t wtot[kStatsThreads / kWave];
  __shared__ uint32_t red[4][kStatsThreads / kWave];
  const int tid = threadIdx.x, wave = tid / kWave, lane = lane_id();
  const int per = (n + kStatsThreads - 1) / kStatsThreads;
  const int i0 = min(n, tid * per), i1 = min(n, i0 + per);
  // sixteen candidates of a thread in flight at a time; the first sixteen, all
  // of them up to 4096 candidates, are read once and kept for the second pass
  constexpr int kHeld = 16;
  struct Held {
    uint32_t count[kHeld];
    float prec[kHeld];
  };
  auto fetch = [&](int c, Held& h) {
#pragma unroll
    for (int k = 0; k < kHeld; ++k) {
      h.count[k] = c + k < i1 ? rb.counts[c + k] : 0u;
      h.prec[k] = c + k < i1 ? rb.prec[c + k] : 1.0f;
    }
  };
  Held first;
  fetch(i0, first);
  uint32_t sum = 0;
#pragma unroll
  for (int k = 0; k < kHeld; ++k) sum += first.count[k];
  for (int c = i0 + kHeld; c < i1; c += kHeld) {
    uint32_t v[kHeld];
#pragma unroll
    for (int k = 0; k < kHeld; ++k) v[k] = c + k < i1 ? rb.counts[c + k] : 0u;
#pragma unroll
    for (int k = 0; k < kHeld; ++k) sum += v[k];
  }
  const uint32_t incl = wave_incl_scan_u32(sum);
  if (lane == kWave - 1) wtot[wave] = incl;
  __syncthreads();
  uint32_t run = incl - sum;
  for (int w = 0; w < wave; ++w) run += wtot[w];
  uint32_t nr = 0, nk = 0, nm = 0, smax = 0;
  auto count = [&](int c, const Held& h) {
#pragma unroll
    for (int k = 0; k < kHeld; ++k) {
      if (c + k >= i1) continue;
      run += h.count[k];
      if (run <= (uint32_t)max_samples) {  // kept candidates are a prefix
        ++nk;
        smax = run;
        if (h.count[k] > 0) {
          ++nr;
          if (h.prec[k] == 0.0f) ++nm;
        }
      }
    }
  };
  count(i0, first);
  for (int c = i0 + kHeld; c < i1; c += kHeld) {
    Held h;
    fetch(c, h);
    count(c, h);
  }
  nr = wave_incl_scan_u32(nr);
  nk = wave_incl_scan_u32(nk);
  nm = wave_incl_scan_u32(nm);
  for (int o = 32; o > 0; o >>= 1) smax = max(smax, (uint32_t)__shfl_xor((int)smax, o, kWave));
  if (lane == kWave - 1) {
    red[0][wave] = nr;
    red[1][wave] = nk;
    red[2][wave] = nm;
    red[3][wave] = smax;
  }
  __syncthreads();
  if (tid == 0) {
    uint32_t R = 0, K = 0, M = 0, S = 0;
    for (int w = 0; w < kStatsThreads / kWave; ++w) {
      R += red[0][w];
      K += red[1][w];
      M += red[2][w];
      S = max(S, red[3][w]);
    }
    rb.stats[0] = R;
    rb.stats[1] = S;
    rb.stats[2] = K;
    rb.stats[3] = M;
    if (rb.loss) rb.loss[0] = rb.loss[1] = rb.loss[2] = 0.0f;
  }
}

// The samples of each kept candidate (one wave a candidate).  kScan: the
// launch also does what scan_cut_kernel would (for at most kEmitScanMax
// candidates): each workgroup sums the counts before its first candidate
// (sixteen loads in flight per thread) and writes its candidates' offsets,
// and one more workgroup, the first (so that it starts first), sets the
// statistics.
constexpr int kEmitScanMax = 16384;
template <bool kScan>
__global__ __launch_bounds__(256) void emit_kernel(KeyframeStore kf, MarchParams mp, int n,
                                                   RayBuffers rb, float* __restrict__ t_out,
                                                   uint32_t* __restrict__ ray_out) {
  const int w = (int)threadIdx.x / kWave, lane = lane_id();
  const int blk = kScan ? (int)blockIdx.x - 1 : (int)blockIdx.x;
  const int r = blk * kWavesPerBlock + w;
  uint32_t cnt, base;
  // the ray as the counting pass stored it (the same values make_ray gives),
  // fetched before the sums
  float4 ro = make_float4(0.0f, 0.0f, 0.0f, 0.0f), rd = ro;
  if (r >= 0 && r < n && mp.sampler != 0) {
    ro = rb.rays[2 * r];
    rd = rb.rays[2 * r + 1];
  }
  if (kScan) {
    if (blk < 0) {
      cut_stats_block(rb, n, mp.max_samples);
      return;
    }
    __shared__ uint32_t part[kWavesPerBlock], own[kWavesPerBlock];
    const int r0 = blk * kWavesPerBlock;
    const uint32_t mine = r < n ? rb.counts[r] : 0u;
    uint32_t sum = 0;
    for (int i0 = 0; i0 < r0; i0 += 256 * 16) {
      uint32_t v[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const int i = i0 + 256 * k + (int)threadIdx.x;
        v[k] = i < r0 ? rb.counts[i] : 0u;
      }
#pragma unroll
      for (int k = 0; k < 16; ++k) sum += v[k];
    }
    sum = wave_incl_scan_u32(sum);
    if (lane == kWave - 1) {
      part[w] = sum;
      own[w] = mine;
    }
    __syncthreads();
    base = 0;
#pragma unroll
    for (int k = 0; k < kWavesPerBlock; ++k) base += part[k] + (k < w ? own[k] : 0u);
    cnt = own[w];
    if (r < n && lane == 0) {
      rb.offsets[r] = base;
      if (r == n - 1) rb.offsets[n] = base + cnt;
    }
    if (r >= n) return;
  } else {
    if (r >= n) return;
    cnt = rb.counts[r];
    base = rb.offsets[r];
  }
  if (cnt == 0 || base + cnt > (uint32_t)mp.max_samples) return;
  if (mp.sampler == 0) {
    for (int i = lane; i < (int)cnt; i += kWave) {
      t_out[base + i] = uniform_t(mp, i);
      ray_out[base + i] = (uint32_t)r;
    }
    return;
  }
  Ray ray;
  ray.o[0] = ro.x; ray.o[1] = ro.y; ray.o[2] = ro.z; ray.s = ro.w;
  ray.d[0] = rd.x; ray.d[1] = rd.y; ray.d[2] = rd.z;
  int k0, k1;
  if (!lattice_range(ray, mp, k0, k1)) return;
  uint32_t done = 0;
  for (int kb = k0; kb <= k1 && done < cnt; kb += kWave) {
    float t = 0.0f;
    const int kk = kb + lane;
    const bool keep = kk <= k1 && keep_point(ray, kk, mp, kf.occ, kf.grid_res, t);
    const uint64_t mask = __ballot(keep);
    const uint32_t before = (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
    if (keep && done + before < cnt) {
      t_out[base + done + before] = t;
      ray_out[base + done + before] = (uint32_t)r;
    }
    done += (uint32_t)__popcll(mask);
  }
}

}  // namespace

size_t march_block_count(int n) {
  return (size_t)(n + march_detail::kWavesPerBlock - 1) / march_detail::kWavesPerBlock;
}

size_t count_block_count(const MarchParams& mp, int n) {
  return mp.sampler == 0 ? ((size_t)n + 255) / 256 : march_block_count(n);
}

// The emit does the scan itself for 1 <= n <= kEmitScanMax candidates.
static bool emit_scans(int n) { return n >= 1 && n <= kEmitScanMax; }

hipError_t march_rays(const KeyframeStore& kf, const MarchParams& mp, const uint32_t* ids, int n,
                      const RayBuffers& rb, hipStream_t st) {
  if (n > 0)
    hipLaunchKernelGGL(rays_count_kernel, dim3(count_block_count(mp, n)), dim3(256), 0, st, kf, mp, ids, n, rb);
  return march_scan(mp, n, rb, st);
}

hipError_t march_scan(const MarchParams& mp, int n, const RayBuffers& rb, hipStream_t st) {
  if (!emit_scans(n)) hipLaunchKernelGGL(scan_cut_kernel, dim3(1), dim3(kScanThreads), 0, st, rb, n, mp.max_samples);
  return hipGetLastError();
}

hipError_t march_emit(const KeyframeStore& kf, const MarchParams& mp, const uint32_t* /*ids*/, int n,
                      const RayBuffers& rb, float* t_out, uint32_t* ray_out, hipStream_t st) {
  // the rays come from rb, stored by the counting pass from ids
  if (emit_scans(n))
    hipLaunchKernelGGL(emit_kernel<true>, dim3(march_block_count(n) + 1), dim3(256), 0, st, kf, mp, n, rb, t_out,
                       ray_out);
  else if (n > 0)
    hipLaunchKernelGGL(emit_kernel<false>, dim3(march_block_count(n)), dim3(256), 0, st, kf, mp, n, rb, t_out,
                       ray_out);
  return hipGetLastError();
}

}  // namespace nsl
