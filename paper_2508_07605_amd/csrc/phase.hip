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
// Where readings stay around the threshold the search binds: its positions are 32 bits wide, the same
// traces all read to the end take 148 us, with 64-bit positions 172 (as scalar code, 60 operations a
// step on the one scalar unit of a SIMD, 236).  Short traces are bound by what a trace costs beside its
// readings, so up to kPhaseShort of them a wavefront takes several (100,000 x 600: 35 us, 41 with a
// wavefront each; 65,536 x 1500: 66 and 65.7), and up to 64 or 128 readings one or two steps are all
// there is (300,000 x 40: 25 to 28 us, 41 to 52 with four).
#include "common.h"

namespace openk {

constexpr int64_t kPhaseShort = 768;  // readings up to which a wavefront takes several traces

// AH: steps loaded together
template <int AH>
__global__ __launch_bounds__(256) void k_phase_detect(const float *__restrict__ P, int64_t T, int64_t L, int64_t ld,
                                                      float th, int N, int64_t *__restrict__ first) {
  constexpr int BL = 64 * AH;  // readings of a block
  const int lane = threadIdx.x & 63;
  // bits 0 .. lane of a mask's halves
  const uint32_t lo = lane >= 31 ? ~0u : (2u << lane) - 1u;
  const uint32_t hi = lane < 32 ? 0u : lane == 63 ? ~0u : (2u << (lane - 32)) - 1u;
  // the wave's index as a scalar, so that the block's buffer resource stays in scalar registers
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t nw = (int64_t)gridDim.x * (blockDim.x >> 6);
  for (int64_t tr = (int64_t)blockIdx.x * (blockDim.x >> 6) + wv; tr < T; tr += nw) {
    const float *row = P + tr * ld;
    uint32_t run = 0;  // readings not below the threshold ending just before the current step, < N
    int64_t found = -1;
    // a block through a buffer resource: readings past the trace read nothing, and no branch
    // surrounds the loads
    auto load = [&](float (&v)[AH], int64_t base) {
      const int64_t rem = L - base;
      const __amdgpu_buffer_rsrc_t rs = make_rsrc(row + base, (uint64_t)(rem < BL ? rem : BL) * 4);
#pragma unroll
      for (int u = 0; u < AH; ++u) v[u] = bload_f32(rs, (64 * u + lane) * 4);
    };
    float v[AH];
    for (int64_t base = 0; base < L && found < 0; base += BL) {
      load(v, base);
      // "not below" masks of the steps; bit l is reading base + 64 u + l
      unsigned long long ok[AH], any = 0ull;
#pragma unroll
      for (int u = 0; u < AH; ++u) ok[u] = __ballot(!(v[u] < th));
      const int64_t rem = L - base;
      if (rem < BL) {
#pragma unroll
        for (int u = 0; u < AH; ++u)
          ok[u] &= rem >= 64 * (u + 1) ? ~0ull : rem <= 64 * u ? 0ull : (1ull << (rem - 64 * u)) - 1ull;
      }
#pragma unroll
      for (int u = 0; u < AH; ++u) any |= ok[u];
      if (!any) {  // every reading below: no run survives the block
        run = 0;
        continue;
      }
#pragma unroll
      for (int u = 0; u < AH; ++u) {
        const int64_t c0 = base + 64 * u;
        if (c0 >= L || found >= 0) break;  // wave-uniform
        const unsigned long long m = ok[u];
        if (!m) {
          run = 0;
          continue;
        }
        // the last failing reading at or before this lane; past the trace every reading fails
        const uint32_t zlo = ~(uint32_t)m & lo, zhi = ~(uint32_t)(m >> 32) & hi;
        const int last = zhi ? 63 - __builtin_clz(zhi) : 31 - __builtin_clz(zlo);
        const uint32_t r = zhi | zlo ? (uint32_t)(lane - last) : run + lane + 1;
        const unsigned long long hit = __ballot(r >= (uint32_t)N);
        if (hit) {
          found = c0 + __ffsll((long long)hit) - 1;
        } else {
          run = (uint32_t)__builtin_amdgcn_readlane((int)r, 63);
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
  // A wavefront per trace (up to 2^24 of them), or, of short ones, 64 wavefronts per CU that take
  // several; steps that no trace reaches are left out.
  const int64_t cap = L <= kPhaseShort ? (int64_t)ctx->num_cu * 64 : int64_t(1) << 24;
  const int64_t waves = T < cap ? T : cap;
  OPEN_LAUNCH(ctx, "phase_detect", (L <= 64 ? k_phase_detect<1> : L <= 128 ? k_phase_detect<2> : k_phase_detect<4>),
              dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, power, T, L, ld, threshold, n_window, first_index);
  return OPEN_OK;
}
