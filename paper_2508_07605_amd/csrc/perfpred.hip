// Offline performance predictor (Section III-A.2, "Performance Prediction Model"), batched over
// profiled runs: each run's seven features (CPU cap, GPU cap, memory throughput, IPS, SM clock,
// DRAM active, FP active) map to the run's normalized performance,
//
//   z = (x - mu) * rs,  h1 = ReLU(W1 z + b1),  h2 = ReLU(W2 h1 + b2),  y = w3 . h2 + b3,
//
// with two hidden layers of 64 units.  W1 (64 x 7) and W2 (64 x 64) are used in bfloat16
// (round to nearest even); everything else is float32.  A run with a non-finite feature gets
// y = NaN.
//
// One wavefront per tile of 32 runs, on BF16 MFMA v_mfma_f32_32x32x16_bf16 with the runs along
// the 32 output columns and the hidden units along the rows.  The activations are not rounded
// to bfloat16: each is split into a bfloat16 part and a bfloat16 remainder (a = hi + lo up to
// 2^-18 |a|) and both are multiplied, so the only rounding beyond float32 is the weights'.
//   layer 1: k = 8 g + t pairs weight column t with the feature parts of half g (g = 0 the
//            bfloat16 parts, g = 1 the remainders); the bias b1 rides in slot t = 7 against
//            a constant feature of 1, again as a bfloat16 part and its remainder.
//   layer 2: the hidden index of slot (g, t) in step s = 2 bk + p is chosen as the row that
//            the layer-1 result already holds in that lane, 32 bk + 8 (2p + t/4) + 4 g + t%4,
//            so h1 feeds the next MFMA without moving between lanes; W2 is permuted to match.
//   layer 3: a per-lane dot product over the 32 held units, then the two halves are added.
//
// Bound by the vector operations, 278 a tile, which issue 78 % of the cycles, beside 18 matrix products a
// tile (258 GFLOP for 14,000,003 runs), whose units are busy 38 %: the two overlap in part.  (Moving
// a quarter of the vector operations to products, or two to five wavefronts per SIMD, leaves the
// time as it is within 3 %.)  The features, 28 bytes a run, are read in whole lines and turned
// through LDS; with the seven strided reads a tile that this replaces, and b2 and w3 read from LDS
// in every tile, 14,000,003 runs took 322 us against 297, and 500,000 16.2 against 13.7.
#include "common.h"

namespace openk {

typedef __bf16 pbf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 pbf16x8 __attribute__((ext_vector_type(8)));

constexpr int kPF = 7;   // features
constexpr int kPH = 64;  // hidden units per layer

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  const pbf16x2 v = {(__bf16)a, (__bf16)b};
  return __builtin_bit_cast(uint32_t, v);
}
// a = hi + lo (bfloat16 parts, packed in pairs)
__device__ __forceinline__ void split_pair(float a, float b, uint32_t &hi, uint32_t &lo) {
  hi = pack_bf16(a, b);
  const float ha = __builtin_bit_cast(float, hi << 16), hb = __builtin_bit_cast(float, hi & 0xffff0000u);
  lo = pack_bf16(a - ha, b - hb);
}
// max(x, 0) on the bit pattern: negative floats are negative integers (one integer max, no
// NaN canonicalisation)
__device__ __forceinline__ float relu(float x) {
  const int i = __builtin_bit_cast(int, x);
  return __builtin_bit_cast(float, i > 0 ? i : 0);
}
__device__ __forceinline__ f16 mfma_bf16(uint4 a, uint4 b, f16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(pbf16x8, a), __builtin_bit_cast(pbf16x8, b), c,
                                                 0, 0, 0);
}

__global__ __launch_bounds__(256, 3) void k_perf_predict(int64_t n, const float *__restrict__ X,
                                                      const float *__restrict__ mu, const float *__restrict__ rs,
                                                      const float *__restrict__ W1, const float *__restrict__ b1,
                                                      const float *__restrict__ W2, const float *__restrict__ b2,
                                                      const float *__restrict__ w3, const float *__restrict__ b3,
                                                      float *__restrict__ y) {
  const int lane = threadIdx.x & 63, i32 = lane & 31, g = lane >> 5;
  // the 32 x 32 results hold rows 8 (v/4) + 4 g + v%4 of the tile in register v of the lane
  // layer-1 weights, A operand of row block bk: W1[32 bk + i32][t] for t < 7; slot t = 7 holds
  // the bias, its bfloat16 part in half 0 and the remainder in half 1 (times a feature of 1)
  uint4 a1[2];
#pragma unroll
  for (int bk = 0; bk < 2; ++bk) {
    const float *w = W1 + (32 * bk + i32) * kPF;
    uint32_t bh, bl;
    split_pair(b1[32 * bk + i32], 0.f, bh, bl);
    a1[bk] = uint4{pack_bf16(w[0], w[1]), pack_bf16(w[2], w[3]), pack_bf16(w[4], w[5]),
                   pack_bf16(w[6], __builtin_bit_cast(float, (g == 0 ? bh : bl) << 16))};
  }
  // layer-2 weights, A operand of output block ob and step s = 2 bk + p: slot t of half g is
  // input unit 32 bk + 8 (2p + t/4) + 4 g + t%4.  Each lane's operands depend on the lane
  // only, so the block keeps one copy in LDS: la2[ob][s][lane].
  __shared__ uint4 la2[2][4][kWave];
  for (int q = threadIdx.x; q < 2 * 4 * kWave; q += blockDim.x) {
    const int ob = q / (4 * kWave), s = (q / kWave) % 4, l = q % kWave, li = l & 31, lg = l >> 5;
    const float *w = W2 + (32 * ob + li) * kPH + 32 * (s >> 1) + 4 * lg;
    const int p = s & 1;
    uint32_t qq[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int t0 = 2 * u, t1 = 2 * u + 1;
      qq[u] = pack_bf16(w[8 * (2 * p + t0 / 4) + t0 % 4], w[8 * (2 * p + t1 / 4) + t1 % 4]);
    }
    la2[ob][s][l] = uint4{qq[0], qq[1], qq[2], qq[3]};
  }
  __syncthreads();
  float muf[kPF], rsf[kPF];
#pragma unroll
  for (int f = 0; f < kPF; ++f) {
    muf[f] = mu[f];
    rsf[f] = rs[f];
  }
  const float bias3 = b3[0];
  f16 rb2[2], rw3[2];  // b2 and w3 at the lane's rows
#pragma unroll
  for (int ob = 0; ob < 2; ++ob)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int r = 32 * ob + 8 * (v / 4) + 4 * g + v % 4;
      rb2[ob][v] = b2[r];
      rw3[ob][v] = w3[r];
    }

  const int64_t ntiles = (n + 31) >> 5;
  const int64_t nw = (int64_t)gridDim.x * (blockDim.x >> 6);
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t tile0 = (int64_t)blockIdx.x * (blockDim.x >> 6) + wv;
  // a tile's features, in the order of memory, through a buffer resource over its runs (past the
  // last one: zeros), the next tile's loaded while the current one is computed
  float xn[4];
  __shared__ float xs_all[4][256];  // per wavefront: the tile's 32 x 7 features
  float *xs = xs_all[wv];
  auto load = [&](int64_t tile) {
    const int64_t left = n - (tile << 5);
    const int runs = left >= 32 ? 32 : left > 0 ? (int)left : 0;
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(X + (runs > 0 ? (tile << 5) * kPF : 0), (uint64_t)runs * kPF * 4);
#pragma unroll
    for (int f = 0; f < 4; ++f) xn[f] = bload_f32(rx, (lane + 64 * f) * 4);
  };
  load(tile0);
  for (int64_t tile = tile0; tile < ntiles; tile += nw) {
#pragma unroll
    for (int f = 0; f < 4; ++f) xs[lane + 64 * f] = xn[f];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    float z[8];
    float zero = 0.f;  // stays zero for finite features, NaN otherwise
#pragma unroll
    for (int f = 0; f < kPF; ++f) {
      const float xf = xs[i32 * kPF + f];
      zero = __builtin_fmaf(xf, 0.f, zero);
      z[f] = (xf - muf[f]) * rsf[f];
    }
    z[7] = 1.f;  // multiplies the layer-1 bias parts
    load(tile + nw);
    uint32_t hi[4], lo[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) split_pair(z[2 * u], z[2 * u + 1], hi[u], lo[u]);
    lo[3] = (lo[3] & 0xffffu) | 0x3f800000u;  // slot 7 is 1 in both halves
    const uint4 bx = g == 0 ? uint4{hi[0], hi[1], hi[2], hi[3]} : uint4{lo[0], lo[1], lo[2], lo[3]};
    // layer 1, rectified and split: hh/hl[4 s + u] are slots 2 u, 2 u + 1 of step s
    uint32_t hh[16], hl[16];
#pragma unroll
    for (int bk = 0; bk < 2; ++bk) {
      const f16 d1 = mfma_bf16(a1[bk], bx, f16{});
#pragma unroll
      for (int u = 0; u < 8; ++u)
        split_pair(relu(d1[2 * u]), relu(d1[2 * u + 1]), hh[8 * bk + u], hl[8 * bk + u]);
    }
    // layers 2 and 3, one half of the 64 units at a time (fewer registers live).  The weights in LDS
    // are read through an offset the compiler cannot see through, so that it reads them here in
    // every tile instead of holding them in 32 registers.
    int opq = 0;
    asm volatile("" : "+v"(opq));
    float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ob = 0; ob < 2; ++ob) {
      f16 d2 = rb2[ob];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const uint4 w = la2[ob][s][lane + opq];
        d2 = mfma_bf16(w, uint4{hh[4 * s], hh[4 * s + 1], hh[4 * s + 2], hh[4 * s + 3]}, d2);
        d2 = mfma_bf16(w, uint4{hl[4 * s], hl[4 * s + 1], hl[4 * s + 2], hl[4 * s + 3]}, d2);
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) part[v & 3] = __builtin_fmaf(rw3[ob][v], relu(d2[v]), part[v & 3]);
    }
    float acc = (part[0] + part[1]) + (part[2] + part[3]);
    acc += __shfl_xor(acc, 32, kWave);
    const int64_t e = (tile << 5) + i32;
    if (g == 0 && e < n) y[e] = zero == 0.f ? acc + bias3 : __builtin_nanf("");
  }
}

}  // namespace openk

using namespace openk;

extern "C" open_status open_perf_predict(open_ctx *ctx, const float *X, int64_t n_runs, const float *mu,
                                         const float *rs, const float *W1, const float *b1, const float *W2,
                                         const float *b2, const float *w3, const float *b3, float *y) {
  if (!ctx) return OPEN_E_INVALID;
  if (n_runs < 0) return fail(ctx, OPEN_E_INVALID, "negative run count");
  if (n_runs == 0) return OPEN_OK;
  if (!X || !mu || !rs || !W1 || !b1 || !W2 || !b2 || !w3 || !b3 || !y)
    return fail(ctx, OPEN_E_INVALID, "null pointer");
  OPEN_HIP_TRY(ctx, hipSetDevice(ctx->device));
  const int64_t tiles = (n_runs + 31) / 32;
  // three wavefronts per SIMD stay resident: with four times as many, 300,000 runs took 14.8 us
  // instead of 10.7 (the weights are laid out again by every block) and 14M as long as now
  const int64_t cap = (int64_t)ctx->num_cu * 12;  // waves
  const int64_t waves = tiles < cap ? tiles : cap;
  OPEN_LAUNCH(ctx, "perf_predict", k_perf_predict, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, n_runs, X, mu,
              rs, W1, b1, W2, b2, w3, b3, y);
  return OPEN_OK;
}
