// Fold-in of a small batch in one launch: bucketing and solves together.
//
// A batch of few rows per compute unit (small_batch) would spend its time on launches (two of the
// bucketing and one per class group).  Here every block takes kSmallRows consecutive rows,
// orders them in LDS by size class, and its wavefronts solve the groups, with the same
// solve_group as the per-class kernels.
//
// Rows are kept in sections, one per (lanes per system, form): within a section the rows are
// ordered costliest class first and cut into groups of 64 / P whatever their classes; a group
// is solved at the dimension of its first (largest) row.  The padding unknowns of the smaller
// ones are exactly zero, so a row's result does not depend on its neighbours.
//
// Bound by latency: the rows' pointers, their entries and the staged factors are three dependent
// reads, then one or two groups per wavefront.  4099 rows of 4..24 entries at rank 32: 15 us,
// against five launches of 51 us (40 us a pass where passes follow each other); 16 rows at
// rank 8: 6 us against 16.
#pragma once
#include "rowsolve.h"

namespace openk {

// A section: P lanes per system, dual or primal form, its dimensions in descending order
template <int P_, bool DUAL_, int... D_>
struct SmallSection {
  static constexpr int P = P_, SYS = 64 / P_;
  static constexpr bool DUAL = DUAL_;
  static constexpr int wave_floats() {
    int m = 0;
    ((m = wave_lds_floats(P_, D_) > m ? wave_lds_floats(P_, D_) : m), ...);
    return m;
  }
  static constexpr int largest() {
    int m = 0;
    ((m = D_ > m ? D_ : m), ...);
    return m;
  }
  static constexpr int smallest() {
    int m = 1 << 30;
    ((m = D_ < m ? D_ : m), ...);
    return m;
  }
  // the section's solve at dimension d (wave-uniform)
  template <int K, int SRC, int OCC>
  static __device__ __forceinline__ void solve(int d, const FRows<K, SRC> &Fr, int n, const RowRef &r,
                                               const int32_t *__restrict__ idx, const float *__restrict__ val,
                                               float lambda, int weighted, float *__restrict__ X,
                                               int32_t *__restrict__ status, float *__restrict__ wl) {
    ((d == D_ ? solve_group<P_, D_, K, DUAL_, SRC, (OCC == 1 || D_ <= 12), false>(Fr, n, r, idx, val, lambda,
                                                                                  weighted, X, status, wl)
              : (void)0),
     ...);
  }
};

template <typename... S>
__host__ __device__ constexpr int small_wave_floats() {
  int m = 0;
  ((m = S::wave_floats() > m ? S::wave_floats() : m), ...);
  return m;
}

template <int K, int SRC, int W, int OCC, typename... S>
__global__ __attribute__((amdgpu_flat_work_group_size(64 * W, 64 * W), amdgpu_waves_per_eu(OCC))) void k_foldin_small(
    const float *__restrict__ F, int n, const int64_t *__restrict__ ptr, const int32_t *__restrict__ idx,
    const float *__restrict__ val, const uint8_t *__restrict__ mask, float lambda, int weighted,
    float *__restrict__ X, int32_t *__restrict__ status, int64_t m) {
  constexpr int NS = sizeof...(S);
  constexpr int WL = small_wave_floats<S...>();
  constexpr int FL = SRC == kRowsLds ? factor_lds_bytes<K>() / 4 : 4;
  static_assert(64 * W >= 4 * kSmallRows, "four threads per row");
  __shared__ __attribute__((aligned(16))) float lds_all[W * WL + FL];
  __shared__ int64_t beg_s[kSmallRows];
  __shared__ int cnt_s[kSmallRows];
  // (256 section + 255 - dimension) 128 + row of the block (primal rows: 255 - a quarter of their
  // entries): distinct, ascending in solving order, costliest first
  __shared__ __attribute__((aligned(16))) int key_s[kSmallRows];
  __shared__ uint8_t order_s[kSmallRows];  // the rows in that order, section after section
  __shared__ int nrow_s[NS];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  FRows<K, SRC> Fr;
  if constexpr (SRC == kRowsLds) {
    Fr.lds = stage_factors<K, W>(F, n, lds_all + W * WL);  // completes at the wait below
  } else {
    Fr.global(F, n);
  }
  // ---- the block's rows: section and dimension of each
  constexpr int none = 1 << 30;
  static_assert(kSmallRows == 128, "row bits of a key");
  if (tid < NS) nrow_s[tid] = 0;
  const int64_t row0 = (int64_t)blockIdx.x * kSmallRows;
  int key = none;
  if (tid < kSmallRows) {
    const int64_t row = row0 + tid;
    if (row < m && (!mask || mask[row])) {
      const int64_t b = ptr[row], c = ptr[row + 1] - b;
      constexpr int dmax = K < 32 ? K : 32;
      const int d = c > dmax ? K : c <= 4 ? 4 : (int)((c + 3) >> 2) * 4;
      int s = 0;
      const int cost = c <= dmax ? d : c < 4 * 255 ? (int)c / 4 : 255;
      ((S::DUAL == (c <= dmax) && d >= S::smallest() && d <= S::largest() ? (void)(key = (256 * s + 255 - cost) * kSmallRows + tid)
                                                                          : (void)0,
        ++s),
       ...);
      beg_s[tid] = b;
      cnt_s[tid] = (int)c;
    }
    key_s[tid] = key;
  }
  __syncthreads();
  // rank of every row: four threads compare it with a quarter of the rows each
  if (tid < 4 * kSmallRows) {
    const int mine = key_s[tid >> 2];
    int pos = 0;
#pragma unroll
    for (int j = 0; j < kSmallRows / 16; ++j) {
      const int4 k4 = *reinterpret_cast<const int4 *>(key_s + (kSmallRows / 4) * (tid & 3) + 4 * j);
      pos += (k4.x < mine) + (k4.y < mine) + (k4.z < mine) + (k4.w < mine);
    }
    pos += quad_xor1_i(pos);
    pos += quad_xor2_i(pos);
    if ((tid & 3) == 0 && mine != none) order_s[pos] = (uint8_t)(tid >> 2);
  }
  if (tid < kSmallRows) {
#pragma unroll
    for (int q = 0; q < NS; ++q) {
      const int rows = __popcll(__ballot(key / (256 * kSmallRows) == q));
      if (lane == 0) atomicAdd(&nrow_s[q], rows);
    }
  }
  if constexpr (SRC == kRowsLds) __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  // ---- groups, section by section, dealt to the wavefronts in order
  float *wl = lds_all + w * WL;
  int g = w, s = 0, first = 0;  // first: the section's place in the order
  (
      [&] {
        const int rows = nrow_s[s], groups = (rows + S::SYS - 1) / S::SYS;
        for (; g < groups; g += W) {
          const int d = S::DUAL ? 255 - (key_s[order_s[first + g * S::SYS]] / kSmallRows & 255) : K;
          const int i = g * S::SYS + lane / S::P;
          RowRef r{-1, 0, 0};
          if (i < rows) {
            const int t = order_s[first + i];
            r = RowRef{(int32_t)(row0 + t), cnt_s[t], beg_s[t]};
          }
          S::template solve<K, SRC, OCC>(__builtin_amdgcn_readfirstlane(d), Fr, n, r, idx, val, lambda, weighted, X,
                                          status, wl);
        }
        g -= groups;
        first += rows;
        ++s;
      }(),
      ...);
}

template <int K, int W, int OCC, typename... S>
open_status launch_small(open_ctx *ctx, const char *name, const float *F, int n, const int64_t *ptr,
                         const int32_t *idx, const float *val, const uint8_t *mask, float lambda, int weighted,
                         float *X, int32_t *status, int64_t m) {
  const dim3 grid((unsigned)((m + kSmallRows - 1) / kSmallRows));
  if (n <= kFactorLdsRows) {
    OPEN_LAUNCH(ctx, name, (k_foldin_small<K, kRowsLds, W, OCC, S...>), grid, dim3(64 * W), 0, F, n, ptr, idx, val, mask,
                lambda, weighted, X, status, m);
  } else {
    OPEN_LAUNCH(ctx, name, (k_foldin_small<K, kRowsBuffer, W, OCC, S...>), grid, dim3(64 * W), 0, F, n, ptr, idx, val, mask,
                lambda, weighted, X, status, m);
  }
  return OPEN_OK;
}

}  // namespace openk
