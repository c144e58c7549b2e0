// Phase-transition detection (Algorithm 1, Section III-B.2) over many power traces at once.
//
// Algorithm 1 keeps the last N = W / delta GPU power readings (5 s at 0.2 s: N = 25) and
// reports a CPU -> GPU phase transition as soon as none of them is below P_th (60 W); its
// split of the window into 1 s intervals does not change which readings are tested.  The
// report for a trace is therefore the first position t >= N - 1 whose run of consecutive
// readings that are not below P_th, ending at t, is at least N long.
//
// One wavefront per trace, 64 readings per step (one per lane), four steps loaded together.
// The comparison of a step gives its "not below" mask as a scalar; four empty masks (the
// CPU-bound phase, most of what is read) skip the block.  Otherwise the run ending at each lane is
// the distance to the last failing reading at or before it (or the carried run plus the lane's
// position when there is none), a second ballot finds the first lane whose run reaches N, and
// the run carried on is read from lane 63.  Reading stops at the report's block.
//
// Bound by memory: 65,536 traces x 3000 readings (433 MB up to the reports) take 92 us = 4.7 TB/s
// of needed readings, the rate of a large copy on this card; with the run search in every
// step, eight steps together and four traces per wavefront of a persistent grid 126 us.  (Persistent
// wavefronts: 103 us; a block prefetched 95, eight steps 94: more reads past the report.)
#include "common.h"

namespace openk {

constexpr int kPhaseAhead = 4;

__global__ __launch_bounds__(256) void k_phase_detect(const float *__restrict__ P, int64_t T, int64_t L, int64_t ld,
                                                      float th, int N, int64_t *__restrict__ first) {
  constexpr int BL = 64 * kPhaseAhead;  // readings of a block
  const int lane = threadIdx.x & 63;
  // the wave's index as a scalar, so that the block's buffer resource stays in scalar registers
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t nw = (int64_t)gridDim.x * (blockDim.x >> 6);
  for (int64_t tr = (int64_t)blockIdx.x * (blockDim.x >> 6) + wv; tr < T; tr += nw) {
    const float *row = P + tr * ld;
    int64_t run = 0;  // readings not below the threshold ending just before the current step
    int64_t found = -1;
    // a block through a buffer resource: readings past the trace read nothing, and no branch
    // surrounds the loads
    auto load = [&](float (&v)[kPhaseAhead], int64_t base) {
      const int64_t rem = L - base;
      const __amdgpu_buffer_rsrc_t rs = make_rsrc(row + base, (uint64_t)(rem < BL ? rem : BL) * 4);
#pragma unroll
      for (int u = 0; u < kPhaseAhead; ++u) v[u] = bload_f32(rs, (64 * u + lane) * 4);
    };
    float v[kPhaseAhead];
    for (int64_t base = 0; base < L && found < 0; base += BL) {
      load(v, base);
      // "not below" masks of the steps; bit l is reading base + 64 u + l
      unsigned long long ok[kPhaseAhead], any = 0ull;
#pragma unroll
      for (int u = 0; u < kPhaseAhead; ++u) ok[u] = __ballot(!(v[u] < th));
      const int64_t rem = L - base;
      if (rem < BL) {
#pragma unroll
        for (int u = 0; u < kPhaseAhead; ++u)
          ok[u] &= rem >= 64 * (u + 1) ? ~0ull : rem <= 64 * u ? 0ull : (1ull << (rem - 64 * u)) - 1ull;
      }
#pragma unroll
      for (int u = 0; u < kPhaseAhead; ++u) any |= ok[u];
      if (!any) {  // every reading below: no run survives the block
        run = 0;
        continue;
      }
#pragma unroll
      for (int u = 0; u < kPhaseAhead; ++u) {
        const int64_t c0 = base + 64 * u;
        if (c0 >= L || found >= 0) break;  // wave-uniform
        const unsigned long long m = ok[u];
        if (!m) {
          run = 0;
          continue;
        }
        const unsigned long long upto = lane == 63 ? ~0ull : ((2ull << lane) - 1ull);
        const unsigned long long z = ~m & upto;  // failing readings at or before this lane
        const int64_t r = z ? (int64_t)(lane - (63 - __clzll((long long)z))) : run + lane + 1;
        const unsigned long long hit = __ballot(r >= N && c0 + lane < L);
        if (hit) {
          found = c0 + __ffsll((long long)hit) - 1;
        } else {
          run = readlane_i64(r, 63);
        }
      }
    }
    if (lane == 0) first[tr] = found;
  }
}

}  // namespace openk

using namespace openk;

extern "C" open_status open_phase_detect(open_ctx *ctx, const float *power, int64_t T, int64_t L, int64_t ld,
                                         float threshold, int32_t n_window, int64_t *first_index) {
  if (!ctx) return OPEN_E_INVALID;
  if (T < 0 || L < 0 || ld < L || n_window < 1 || !(threshold == threshold))
    return fail(ctx, OPEN_E_INVALID, "bad shape, window or threshold");
  if (T == 0) return OPEN_OK;
  if (!first_index || (L > 0 && !power)) return fail(ctx, OPEN_E_INVALID, "null pointer");
  OPEN_HIP_TRY(ctx, hipSetDevice(ctx->device));
  // a wavefront per trace up to 2^24 of them (the wavefronts of more take several)
  const int64_t waves = T < (int64_t(1) << 24) ? T : int64_t(1) << 24;
  const unsigned blocks = (unsigned)((waves + 3) / 4);
  OPEN_LAUNCH(ctx, "phase_detect", k_phase_detect, dim3(blocks), dim3(256), 0, power, T, L, ld, threshold, n_window,
              first_index);
  return OPEN_OK;
}
