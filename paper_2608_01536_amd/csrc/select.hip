// Active-column selection kernels for gfx950 and their C ABI entry point,
// celty_select (Sections 1, 2.1 and 3.1: magnitude threshold, then stream
// compaction with wavefront ballots and prefix sums).  The SpMSpV kernels do
// the same selection inside their own prologue; this entry point gives the
// ascending list of active columns on its own.

#include <hip/hip_runtime.h>

#include <climits>
#include <cmath>
#include <cstdint>

#include "celty.h"
#include "common.h"

namespace {

// Global selection, workgroups of 1024 lanes.
//
// select_kernel (x 4-byte aligned): each workgroup lists the active columns of
// its own range, after counting those before it: one launch with no state kept
// between workgroups, at the price of reading x up to the range again (57 KB
// at the widest activation of the LLM shapes, 16 bytes per lane and load, from
// cache).  One workgroup alone takes 0.33 us per 2048 columns, almost all of
// it the listing, and counting takes 0.08, so up to kSelBlocks workgroups
// share the columns: us per call in a graph of 60, one workgroup -> now,
// K = 28672 6.56 -> 3.38, 11008 3.86 -> 2.69, 4096 2.67 -> 2.44.
//   * A range is taken in chunks of STEPS * 2048 columns; in a chunk, lane tid
//     of step j holds the two columns 2 * (j * 1024 + tid) + {0, 1}, read with
//     one 32-bit buffer load (columns past K read as zero: the buffer's size is
//     x's, rounded up to whole words).  All of a chunk's loads are issued
//     before any is used and the lane keeps its activity bits in one register.
//   * The wavefront totals of every (step, wavefront) pair go to LDS; after
//     the chunk's one barrier every wavefront scans all pairs itself (in
//     column order), so the offsets of its own pairs need no second barrier;
//     within a pair, the ballots of the lanes' first and second columns give
//     each active column its position.
//
// select_kernel_any (x only 2-byte aligned, or K <= 1024): steps of 1024
// columns, one column per lane, ranks from a ballot, two barriers per step.
constexpr int kSelBlocks = 64;
constexpr int kSelSteps = 16;

__device__ __forceinline__ bool active(uint32_t half_bits, float tau) {
  return fabsf(half_bits_to_float(half_bits)) > tau;
}

// STEPS: steps of a chunk (1 where every range is one step, else kSelSteps).
// cols: columns of a workgroup's range, a multiple of 2048.
template <int STEPS>
__global__ __launch_bounds__(1024) void select_kernel(const unsigned short* __restrict__ x, int K, float tau,
                                                      int32_t* __restrict__ idx, int32_t* __restrict__ count,
                                                      int cols) {
  constexpr int NW = 1024 / kWave;                                     // 16 wavefronts
  constexpr int PPL = STEPS * NW > kWave ? STEPS * NW / kWave : 1;     // pairs per lane in the scan
  static_assert(NW % PPL == 0 && (STEPS * NW <= kWave || PPL * kWave == STEPS * NW) && 2 * STEPS <= 32, "pair layout");
  __shared__ uint32_t cnt[STEPS * NW];      // pair (j, w) at j * NW + w: column order
  __shared__ uint32_t before[NW];           // active columns before the range, by wavefront
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
  const uint32_t k_lo = blockIdx.x * static_cast<uint32_t>(cols);      // < K
  const uint32_t k_hi = min(static_cast<uint32_t>(K), k_lo + static_cast<uint32_t>(cols));
  const __amdgpu_buffer_rsrc_t xs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<unsigned short*>(x), static_cast<short>(0), static_cast<int>((static_cast<uint32_t>(K) * 2u + 3u) & ~3u),
      0x00020000);
  uint32_t base = 0;
  for (uint32_t it = k_lo; it < k_hi; it += STEPS * 2048) {
    const int steps = static_cast<int>(min(static_cast<uint32_t>(STEPS), (k_hi - it + 2047u) / 2048u));   // uniform
    uint32_t w[STEPS];
#pragma unroll
    for (int j = 0; j < STEPS; ++j)
      w[j] = __builtin_amdgcn_raw_buffer_load_b32(xs, static_cast<int>((it + 2u * (j * 1024 + tid)) * 2u), 0, 0);
    if (it == k_lo) {
      // the columns before the range: 8 per lane and load, four loads in flight
      uint32_t n = 0;   // wavefront-uniform
      for (uint32_t i = 0; i < k_lo; i += 4 * 8192) {
        uint32_t q[4][4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const auto v = __builtin_amdgcn_raw_buffer_load_b128(xs, static_cast<int>((i + u * 8192u + 8u * tid) * 2u), 0, 0);
          q[u][0] = v[0], q[u][1] = v[1], q[u][2] = v[2], q[u][3] = v[3];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (i + u * 8192u < k_lo) {   // uniform
            const bool in = i + u * 8192u + 8u * tid < k_lo;   // all 8 or none: k_lo is a multiple of 2048
#pragma unroll
            for (int c = 0; c < 4; ++c)
              n += static_cast<uint32_t>(__popcll(__ballot(in && active(q[u][c] & 0xFFFFu, tau))) +
                                         __popcll(__ballot(in && active(q[u][c] >> 16, tau))));
          }
        }
      }
      if (lane == 0) before[wv] = n;
    }
    uint32_t bits = 0;   // bits 2j, 2j+1: the lane's two columns of step j
#pragma unroll
    for (int j = 0; j < STEPS; ++j) {
      if (j < steps) {
        const uint32_t k = it + 2u * (j * 1024 + tid);
        const bool a0 = k < static_cast<uint32_t>(K) && active(w[j] & 0xFFFFu, tau);
        const bool a1 = k + 1 < static_cast<uint32_t>(K) && active(w[j] >> 16, tau);
        bits |= ((a0 ? 1u : 0u) | (a1 ? 2u : 0u)) << (2 * j);
        const uint32_t tot = static_cast<uint32_t>(__popcll(__ballot(a0)) + __popcll(__ballot(a1)));
        if (lane == 0) cnt[j * NW + wv] = tot;
      }
    }
    __syncthreads();
    if (it == k_lo)
      base = static_cast<uint32_t>(__builtin_amdgcn_readlane(
          wave_inclusive_scan(lane < NW ? static_cast<int>(before[lane]) : 0), kWave - 1));
    // every wavefront: lane l sums pairs PPL*l .. PPL*l + PPL-1 (those of
    // steps past the chunk's count as zero) and one wavefront scan orders them
    uint32_t c[PPL], lsum = 0;
#pragma unroll
    for (int i = 0; i < PPL; ++i) {
      const int pidx = PPL * lane + i;
      c[i] = pidx < steps * NW ? cnt[pidx] : 0u;
      lsum += c[i];
    }
    const uint32_t incl = static_cast<uint32_t>(wave_inclusive_scan(static_cast<int>(lsum)));
    const uint32_t total = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(incl), kWave - 1));
    // this wavefront's pair (j, wv) is slot wv % PPL of lane (j * NW + wv) / PPL
    const int slot = wv % PPL;
    uint32_t pre = incl - lsum;
#pragma unroll
    for (int i = 0; i < PPL; ++i) pre += i < slot ? c[i] : 0u;
    for (int j = 0; j < steps; ++j) {
      const int src = __builtin_amdgcn_readfirstlane((j * NW + wv) / PPL);
      const uint32_t o = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(pre), src));
      const bool a0 = (bits >> (2 * j)) & 1u, a1 = (bits >> (2 * j + 1)) & 1u;
      // columns of the lanes below come first: both of theirs, then this lane's
      const uint32_t e = base + o + lanes_below(__ballot(a0)) + lanes_below(__ballot(a1));
      const int k = static_cast<int>(it + 2u * (j * 1024 + tid));
      if (a0) idx[e] = k;
      if (a1) idx[e + (a0 ? 1u : 0u)] = k + 1;
    }
    base += total;
    if (it + STEPS * 2048 < k_hi) __syncthreads();   // cnt[] is rewritten by the next chunk
  }
  if (tid == 0 && blockIdx.x == gridDim.x - 1) *count = static_cast<int32_t>(base);
}

__global__ __launch_bounds__(1024) void select_kernel_any(const unsigned short* __restrict__ x, int K, float tau,
                                                          int32_t* __restrict__ idx, int32_t* __restrict__ count) {
  constexpr int NW = 1024 / kWave;
  __shared__ uint32_t wsum[NW];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
  uint32_t base = 0;
  for (int it = 0; it < K; it += 1024) {
    const int k = it + tid;
    const bool act = k < K && fabsf(half_bits_to_float(x[k])) > tau;
    const uint64_t m = __ballot(act);
    const uint32_t rank = lanes_below(m);
    if (lane == 0) wsum[wv] = static_cast<uint32_t>(__popcll(m));
    __syncthreads();
    uint32_t off = base, tot = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const uint32_t cw = wsum[w];
      if (w < wv) off += cw;
      tot += cw;
    }
    if (act) idx[off + rank] = k;
    base += tot;
    __syncthreads();
  }
  if (tid == 0) *count = static_cast<int32_t>(base);
}

}  // namespace

extern "C" celty_status celty_select(const void* x, int32_t K, float tau, int32_t* idx, int32_t* count,
                                     void* stream) {
  if (!x || !idx || !count || K < 1 || std::isnan(tau)) return CELTY_EINVAL;
  if (K > (INT32_MAX - 3) / 2) return CELTY_EINVAL;   // x's byte size is a 32-bit buffer size
  if (misaligned(x, 2) || misaligned(idx, 4) || misaligned(count, 4)) return CELTY_EINVAL;
  // word loads need x 4-byte aligned (the buffer ends at x's last word); up to
  // 1024 columns one step of the plain kernel is quicker
  if (K > 1024 && !misaligned(x, 4)) {
    // one step of 2048 columns per workgroup, more where kSelBlocks do not hold K
    const int steps = (K + 2047) / 2048, per = (steps + kSelBlocks - 1) / kSelBlocks;
    const dim3 grid(static_cast<unsigned>((steps + per - 1) / per));
    hipLaunchKernelGGL(per == 1 ? select_kernel<1> : select_kernel<kSelSteps>, grid, dim3(1024), 0,
                       static_cast<hipStream_t>(stream), static_cast<const unsigned short*>(x), K, tau, idx, count,
                       per * 2048);
  } else {
    hipLaunchKernelGGL(select_kernel_any, dim3(1), dim3(1024), 0, static_cast<hipStream_t>(stream),
                       static_cast<const unsigned short*>(x), K, tau, idx, count);
  }
  return hipGetLastError() == hipSuccess ? CELTY_OK : CELTY_EHIP;
}

