// Fused prediction + energy-efficient cap selection (Algorithm 2, Section III-B.3).
//
// p_is = u_i . v_s is formed tile by tile on FP32 MFMA (v_mfma_f32_32x32x2_f32): a wavefront
// owns 32 rows, keeps their factor rows in registers (A operand) and streams the setting
// factors through LDS in blocks of 32 settings (B operand, stored transposed with a padded
// stride so the 32 lanes of a half-wave read distinct banks).  The epilogue applies the
// paper's rule to every element without materialising p:
//   p_base = p_ib                          (the same MFMA value the scan sees for s = b)
//   valid  = p > 0  and  1 - p / p_base <= gamma      (float32, correctly rounded division; as
//            the equivalent p >= t with t found once per row, the test being monotone in p)
//   E      = (c_s + g_s) / p: the least E is the greatest key p * iw_s, iw_s = 1 / (c_s + g_s)
//            (float32, one division per setting instead of one per element); the lowest s on
//            ties; the saving (E_base - E) / E_base with E = (c_s + g_s) / p of the pick
// Each lane scans its own settings in ascending order; the 32 lanes of a half-wave are then
// combined by (E, s) in a butterfly.  The full prediction P is written only when asked.
//
// Bound by the FP32 matrix products, 32 of 66 cycles a block of 32 x 32 at rank 64, to which the
// vector ALU's share adds (the two do not overlap): so the scan is five vector operations per
// element (the prediction of the pick is formed again at the end instead of carried), loads and
// stores of V need no address arithmetic, and 1 / (c_s + g_s) is formed once per block of threads.
// Without the row pointers of P and the baselines four wavefronts fit per SIMD.  1,000,003 x 1920
// at rank 64: 2957 -> 2100 us, the products alone 1640; 1,000,000 x 120 at rank 32: 438 -> 186.
#include <math.h>

#include "common.h"

namespace openk {

typedef float f16v __attribute__((ext_vector_type(16)));

// V block s0 (32 settings x K) as K/8 floats per thread of a 256-thread block: load from global
// through a buffer resource over the settings that are left (past the last one: zeros), then
// store transposed into LDS at stride LD
template <int K>
__device__ __forceinline__ void load_block(float (&t)[K / 8], const float *__restrict__ V, int n, int s0) {
  const int left = min(n - s0, 32);
  const __amdgpu_buffer_rsrc_t rv = make_rsrc(V + (int64_t)s0 * K, (uint64_t)left * K * 4);
#pragma unroll
  for (int i = 0; i < K / 8; ++i) t[i] = bload_f32(rv, (int)(threadIdx.x + 256 * i) * 4);
}
template <int K>
__device__ __forceinline__ void store_block(float *Vt, const float (&t)[K / 8]) {
  constexpr int LD = 33;
  float *d = Vt + (threadIdx.x % K) * LD + threadIdx.x / K;
#pragma unroll
  for (int i = 0; i < K / 8; ++i) d[i * (256 / K)] = t[i];
}
// 1 / (c + g) of setting s by the block's first 32 threads, NaN past the last one
__device__ __forceinline__ void store_weight(float *iw, const float *__restrict__ cap_c,
                                             const float *__restrict__ cap_g, int n, int s) {
  if (threadIdx.x < 32) iw[threadIdx.x] = s < n ? 1.0f / (cap_c[s] + cap_g[s]) : __builtin_nanf("");
}

template <int K>
__device__ __forceinline__ f16v tile(const float (&a)[K / 2], const float *Vt, int r, int h) {
  constexpr int H = K / 2, LD = 33;
  f16v acc = {};
#pragma unroll
  for (int s = 0; s < H; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[s], Vt[(h * H + s) * LD + r], acc, 0, 0, 0);
  return acc;
}

// The rule's validity test 1 - p / p_base <= gamma (float32, correctly rounded division and
// subtraction) is monotone in p for p_base > 0: fl(p / p_base) does not decrease as p grows and
// fl(1 - x) does not increase as x grows.  So it holds exactly for p >= t, t the least float for
// which it holds, found once per row.  The real threshold (1 - gamma) p_base is one or two units in
// the last place off at small gamma, so five neighbours are tried at once; as gamma nears 1 the
// rounding of 1 - x spans many units (400 at 0.999, 3 % of t at 0.999999), and the distance doubles
// until t is enclosed and is then halved.  (The bits of positive floats are ordered as the floats
// are; negative numbers and NaN fail.)
__device__ __forceinline__ bool loss_ok(int p, float pb, float gamma) {
  return (1.0f - __builtin_bit_cast(float, p) / pb) <= gamma;
}
__device__ __forceinline__ float least_valid(float pb, float gamma) {
  if (gamma >= 1.0f) return __builtin_bit_cast(float, 1);  // every p > 0 passes
  if (!(pb < __builtin_inff())) return __builtin_nanf("");  // 1 - 0 and 1 - inf / inf: none passes
  const int top = __builtin_bit_cast(int, pb);  // passes: 1 - 1 <= gamma
  const int t = __builtin_bit_cast(int, (1.0f - gamma) * pb);
  int lo = t, hi = t;  // lo fails, hi passes
  bool ok[5];
#pragma unroll
  for (int i = 0; i < 5; ++i) ok[i] = loss_ok(t - 2 + i, pb, gamma);
  if (!ok[0] && ok[4]) return __builtin_bit_cast(float, t + 2 - ok[1] - ok[2] - ok[3]);
  if (ok[2]) {
    for (int d = 1;; d *= 2) {
      lo = hi - d > 0 ? hi - d : 0;  // 0 fails
      if (lo == 0 || !loss_ok(lo, pb, gamma)) break;
      hi = lo;
    }
  } else {
    for (int d = 1;; d *= 2) {
      hi = top - lo > d ? lo + d : top;
      if (hi == top || loss_ok(hi, pb, gamma)) break;
      lo = hi;
    }
  }
  while (hi - lo > 1) {
    const int mid = lo + (hi - lo) / 2;
    if (loss_ok(mid, pb, gamma))
      hi = mid;
    else
      lo = mid;
  }
  return __builtin_bit_cast(float, hi);
}

// lane moves within a row of 16 lanes: neighbours, pairs, and the mirrors, which once lanes hold
// equal values in fours and eights reach the same partners as 4 and 8 lanes apart
template <int CTRL, class T>
__device__ __forceinline__ T dpp_get(T x) {
  const int i = __builtin_bit_cast(int, x);
  return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(i, i, CTRL, 0xf, 0xf, true));
}
// greatest key, then lowest setting, of two lanes
__device__ __forceinline__ void take_better(float &k, int &s, float k2, int s2) {
  const bool take = s2 >= 0 && (s < 0 || k2 > k || (k2 == k && s2 < s));
  k = take ? k2 : k;
  s = take ? s2 : s;
}
// x[v] by a lane's own v
__device__ __forceinline__ float pick16(f16v x, int v) {
  float y = x[0];
#pragma unroll
  for (int i = 1; i < 16; ++i) {
    const float xi = x[i];
    y = v == i ? xi : y;
  }
  return y;
}

template <int K, bool WP>
__global__ __launch_bounds__(256, WP ? 3 : 4) void k_predict_select(const float *__restrict__ U, int64_t m,
                                                        const float *__restrict__ V, int n,
                                                        const float *__restrict__ cap_c,
                                                        const float *__restrict__ cap_g, int base, float gamma,
                                                        float *__restrict__ P, int32_t *__restrict__ best_idx,
                                                        float *__restrict__ best_saving,
                                                        int32_t *__restrict__ status) {
  constexpr int H = K / 2, LD = 33;
  __shared__ float Vt[2][K * LD], iwt[2][32];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int r = lane & 31, h = lane >> 5;
  const int64_t row0 = ((int64_t)blockIdx.x * 4 + w) * 32;
  const int64_t grow = row0 + r;
  // A operand: lane (r, h) holds u_r[h*H .. h*H + H)
  float a[H];
#pragma unroll
  for (int s = 0; s < H; s += 4) {
    const f4 x = grow < m ? *reinterpret_cast<const f4 *>(U + grow * K + h * H + s) : f4{0.f, 0.f, 0.f, 0.f};
    a[s] = x[0];
    a[s + 1] = x[1];
    a[s + 2] = x[2];
    a[s + 3] = x[3];
  }
  // the lane's 16 accumulators are rows 8*(v/4) + 4*h + v%4; row r is register vr of half hr
  const int hr = (r >> 2) & 1, vr = (r >> 3) * 4 + (r & 3);
  // baseline prediction from the same MFMA tile the scan uses
  const int sb0 = (base / 32) * 32, jb = base - sb0;
  float tb[K / 8];
  load_block<K>(tb, V, n, sb0);
  store_block<K>(Vt[1], tb);
  load_block<K>(tb, V, n, 0);  // the scan's first block
  store_weight(iwt[0], cap_c, cap_g, n, r);
  __syncthreads();
  // per row: valid(p) <=> p >= thr (thr > 0, so p > 0 follows; NaN when p_base <= 0: never).
  // Each lane finds its row r's, then the lanes of a half read those of its 16 rows.
  float thr[16];
  {
    const f16v acc = tile<K>(a, Vt[1], r, h);
    f16v pb;
#pragma unroll
    for (int v = 0; v < 16; ++v) pb[v] = __shfl(acc[v], jb + 32 * h, 64);
    const float own = pick16(pb, vr), other = __shfl_xor(own, 32, 64);
    const float pbr = h == hr ? own : other;
    const float t = pbr > 0.f ? least_valid(pbr, gamma) : __builtin_nanf("");
#pragma unroll
    for (int v = 0; v < 16; ++v) thr[v] = __shfl(t, 8 * (v / 4) + 4 * h + (v % 4), 64);
  }
  float bK[16];  // the best key and its setting
  int bS[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    bK[v] = -__builtin_inff();
    bS[v] = -1;
  }
  store_block<K>(Vt[0], tb);
  if (32 < n) load_block<K>(tb, V, n, 32);
  __syncthreads();
  // Double-buffered stream of V blocks: block i is read from Vt[i & 1] while block i + 1 goes
  // into the other buffer and block i + 2 loads into registers; one barrier per block.
  for (int s0 = 0, i = 0; s0 < n; s0 += 32, ++i) {
    const f16v acc = tile<K>(a, Vt[i & 1], r, h);
    if (s0 + 32 < n) {
      store_block<K>(Vt[(i + 1) & 1], tb);
      store_weight(iwt[(i + 1) & 1], cap_c, cap_g, n, s0 + 32 + r);
    }
    if (s0 + 64 < n) load_block<K>(tb, V, n, s0 + 64);
    const int sc = s0 + r;
    const float iw = iwt[i & 1][r];  // past the last setting the key is NaN and never taken
    if (WP && sc < n) {
      float *prow = P + (row0 + 4 * h) * n + sc;
      const int64_t left = m - row0 - 4 * h;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int rv = 8 * (v / 4) + (v % 4);
        if (rv < left) prow[(int64_t)rv * n] = acc[v];
      }
    }
    // branch-free: greatest key p * iw among valid settings, the lane's settings in ascending
    // order, the first on ties
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const float p = acc[v];
      const float key = p * iw;
      const bool better = p >= thr[v] && key > bK[v];
      bK[v] = better ? key : bK[v];
      bS[v] = better ? sc : bS[v];
    }
    __syncthreads();
  }
  // combine the 32 column lanes of each half-wave
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    take_better(bK[v], bS[v], dpp_get<0xB1>(bK[v]), dpp_get<0xB1>(bS[v]));
    take_better(bK[v], bS[v], dpp_get<0x4E>(bK[v]), dpp_get<0x4E>(bS[v]));
    take_better(bK[v], bS[v], dpp_get<0x141>(bK[v]), dpp_get<0x141>(bS[v]));
    take_better(bK[v], bS[v], dpp_get<0x140>(bK[v]), dpp_get<0x140>(bS[v]));
    take_better(bK[v], bS[v], __shfl_xor(bK[v], 16, 64), __shfl_xor(bS[v], 16, 64));
  }
  // Row r's pick goes to both lanes r, and its prediction is formed once more, on the diagonal of
  // a tile whose column r is row r's pick: the same products in the same order give the scan's
  // bits, at the price of one block, where carrying it along would be 16 selects in every block.
  f16v picks;
#pragma unroll
  for (int v = 0; v < 16; ++v) picks[v] = __builtin_bit_cast(float, bS[v]);
  const int own = __builtin_bit_cast(int, pick16(picks, vr)), other = __shfl_xor(own, 32, 64);
  const int pick = h == hr ? own : other;
  const bool okb = pick >= 0;  // never where p_base <= 0
  const int sb = okb ? pick : base;
  float p = 0.f;
  if (best_saving) {
    f16v acc = {};
    const float *vs = V + (int64_t)sb * K + h * H;
#pragma unroll
    for (int s = 0; s < H; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[s], vs[s], acc, 0, 0, 0);
    p = pick16(acc, vr);
  }
  if (h == hr && grow < m) {
    best_idx[grow] = sb;
    if (best_saving) {
      const float ebase = cap_c[base] + cap_g[base];
      const float E = (cap_c[sb] + cap_g[sb]) / p;
      best_saving[grow] = okb ? (ebase - E) / ebase : 0.f;
    }
    if (status) status[grow] = okb ? OPEN_ROW_OK : OPEN_ROW_NONPOS_BASE;
  }
}

}  // namespace openk

using namespace openk;

extern "C" open_status open_predict(open_ctx *ctx, const float *U, int64_t m, const float *V, int32_t n, int32_t k,
                                    float *P, const float *cap_cpu, const float *cap_gpu, int32_t base, float gamma,
                                    int32_t *best_idx, float *best_saving, int32_t *row_status) {
  if (!ctx) return OPEN_E_INVALID;
  if (!(k == 8 || k == 16 || k == 32 || k == 64)) return fail(ctx, OPEN_E_UNSUPPORTED, "rank must be 8, 16, 32 or 64");
  if (m < 0 || n <= 0 || base < 0 || base >= n) return fail(ctx, OPEN_E_INVALID, "bad shape or baseline index");
  if (!(gamma >= 0.0f) || !isfinite(gamma)) return fail(ctx, OPEN_E_INVALID, "gamma must be finite and >= 0");
  if (m > 0 && (!U || !V || !cap_cpu || !cap_gpu || !best_idx))
    return fail(ctx, OPEN_E_INVALID, "pointers must not be NULL");
  if (m == 0) return OPEN_OK;
  OPEN_HIP_TRY(ctx, hipSetDevice(ctx->device));
  const dim3 grid((unsigned)((m + 127) / 128)), block(256);
  switch (k) {
    case 8:
      OPEN_LAUNCH(ctx, "predict_select_k8", (P ? k_predict_select<8, true> : k_predict_select<8, false>), grid, block,
                  0, U, m, V, n, cap_cpu, cap_gpu, base, gamma, P, best_idx, best_saving, row_status);
      break;
    case 16:
      OPEN_LAUNCH(ctx, "predict_select_k16", (P ? k_predict_select<16, true> : k_predict_select<16, false>), grid,
                  block, 0, U, m, V, n, cap_cpu, cap_gpu, base, gamma, P, best_idx, best_saving, row_status);
      break;
    case 32:
      OPEN_LAUNCH(ctx, "predict_select_k32", (P ? k_predict_select<32, true> : k_predict_select<32, false>), grid,
                  block, 0, U, m, V, n, cap_cpu, cap_gpu, base, gamma, P, best_idx, best_saving, row_status);
      break;
    default:
      OPEN_LAUNCH(ctx, "predict_select_k64", (P ? k_predict_select<64, true> : k_predict_select<64, false>), grid,
                  block, 0, U, m, V, n, cap_cpu, cap_gpu, base, gamma, P, best_idx, best_saving, row_status);
      break;
  }
  return OPEN_OK;
}
