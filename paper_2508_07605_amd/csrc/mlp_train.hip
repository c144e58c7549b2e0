// Forward and backward pass of the surrogate network over a training batch, one launch.
//
// A block takes R rows of the batch (32, or 16 where 32 would leave compute units idle)
// through the whole network; activations and their gradients stay in LDS and registers:
//   first layer   sparse, lane l owns hidden units 4l .. 4l + 3 (the steps of the inference)
//   layers 2, 3   v_mfma_f32_32x32x16_bf16, one wavefront per 32 output columns, weight operands
//                 from the packed copies (L2-resident)
//   loss          output gradient 2 (u - target) / (B k), squared errors summed in float64
//   backward      dz2 = (dout W3) GELU'(z2), dz1 = (dz2 W2) GELU'(z1) on the transposed copies
// and leaves what the weight gradients contract over the batch (wgrad.h): the dense input rows,
// h1, h2 and the three output gradients as bfloat16 operands (the rounding their products take),
// the output gradients in float32 too for the bias gradients.  FWD: only the output.
//
// Bound by the first layer's gather (1 KB of weights per observed entry) and by latency: the
// dense layers of 4096 rows are 1.9 GFLOP forward and backward.  The products keep float32
// accumulation and one order of k, so the values do not depend on R.
//
// At batch 4096, 480 settings, rank 32: 18 us, and 18 us for the weight gradients and Adam
// (wgrad.hip); a step takes 44 us against 220 us as nineteen launches (products through float32
// activations in memory, partial weight gradients, separate reductions, optimizer and packing).
#include <math.h>

#include "mlp_train.h"
#include "mlp_net.h"

namespace openk {

constexpr int kTrWaves = 8, kTrThreads = 64 * kTrWaves;
constexpr int kTrHP = 256 + 8;  // LDS pitch of an activation row (bfloat16)
constexpr int kTrZP = 256 + 4;  // LDS pitch of a z1 row (float32)

template <int R, int CB3, bool FWD>
__global__ __launch_bounds__(kTrThreads) void k_mlp_fwd_bwd(MlpBatch p) {
  constexpr int RW = R / kTrWaves;  // rows of a wavefront in the first layer
  constexpr int KP = 32 * CB3;      // output columns, padded
  __shared__ __attribute__((aligned(16))) uint16_t Ha[R * kTrHP];  // h1, then dz2
  __shared__ __attribute__((aligned(16))) uint16_t Hb[R * kTrHP];  // h2
  __shared__ __attribute__((aligned(16))) uint16_t Ds[R * (KP + 8)];
  __shared__ float Zs[FWD ? 1 : R * kTrZP];
  __shared__ int64_t row_s[R];  // CSR row of each batch row, -1 past the batch
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, i32 = lane & 31, g = lane >> 5;
  const int64_t b0 = (int64_t)blockIdx.x * R;
  const int n = p.n, k = p.k;
  const int XU = pad_units(2 * n);
  uint4 *X0 = reinterpret_cast<uint4 *>(p.X) + b0 / 8 * XU;  // the block's dense input rows
  if constexpr (!FWD) {
    for (int e = threadIdx.x; e < R / 8 * XU; e += kTrThreads) X0[e] = uint4{0u, 0u, 0u, 0u};
  }
  // ---- the wavefront's rows: lanes 0 .. RW - 1 look them up
  int64_t ri = -1, beg_l = 0;
  int cnt_l = 0;
  if (lane < RW) {
    const int64_t b = b0 + RW * w + lane;
    if (b < p.B) {
      ri = p.rows ? p.rows[(p.use_cursor ? p.st->cursor * p.B : 0) + b] : b;
      beg_l = p.ptr[ri];
      cnt_l = (int)(p.ptr[ri + 1] - beg_l);
    }
    row_s[RW * w + lane] = ri;
  }
  // ---- first layer
  const __amdgpu_buffer_rsrc_t rs1 = make_rsrc(p.W1P, (uint64_t)n * 1024);
  const f4 b1v = *reinterpret_cast<const f4 *>(p.b1 + 4 * lane);
  int64_t beg[RW];
  int cnt[RW], ec[RW];
  float ev[RW];
#pragma unroll
  for (int r = 0; r < RW; ++r) {  // the first 64 entries of every row, one per lane
    beg[r] = readlane_i64(beg_l, r);
    cnt[r] = __builtin_amdgcn_readlane(cnt_l, r);
    const bool in = lane < cnt[r];
    const int j = in ? p.col[beg[r] + lane] : -1;
    ev[r] = in ? p.val[beg[r] + lane] : 0.f;
    ec[r] = j >= 0 && j < n ? j : -1;
  }
#pragma unroll
  for (int r = 0; r < RW; ++r) {
    const int lr = RW * w + r;
    f4 z = b1v;
    int cj = ec[r];
    float cv = ev[r];
    for (int t0 = 0; t0 < cnt[r]; t0 += 64) {
      if (t0) {  // rows of more than 64 entries
        const bool in = t0 + lane < cnt[r];
        const int j = in ? p.col[beg[r] + t0 + lane] : -1;
        cv = in ? p.val[beg[r] + t0 + lane] : 0.f;
        cj = j >= 0 && j < n ? j : -1;
      }
      const uint32_t pr = value_pair(cv, cj >= 0);
      const int len = cnt[r] - t0 < 64 ? cnt[r] - t0 : 64;
      for (int e0 = 0; e0 < len; e0 += 8) {  // entries past the row have column -1: exact zeros
        uint4 wv[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) wv[e] = w1_pairs(rs1, __builtin_amdgcn_readlane(cj, e0 + e), lane);
#pragma unroll
        for (int e = 0; e < 8; ++e)
          layer1_step(z, wv[e], (uint32_t)__builtin_amdgcn_readlane((int)pr, e0 + e));
      }
    }
    const bool real = b0 + lr < p.B;
    if constexpr (!FWD) *reinterpret_cast<f4 *>(Zs + lr * kTrZP + 4 * lane) = z;
    uint2 hv = uint2{bf16pack(gelu(z[0]), gelu(z[1])), bf16pack(gelu(z[2]), gelu(z[3]))};
    if (!real) hv = uint2{0u, 0u};
    *reinterpret_cast<uint2 *>(Ha + lr * kTrHP + 4 * lane) = hv;
  }
  // the second layer's operands of this wavefront's 32 columns load across the barrier
  uint4 bw[16];
#pragma unroll
  for (int ks = 0; ks < 16; ++ks) bw[ks] = p.W2P[(w * 16 + ks) * 64 + lane];
  if constexpr (!FWD) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the zeros of X have landed
  __syncthreads();
  if constexpr (!FWD) {
    // observed entries into the dense input rows; h1 as an operand
    uint16_t *X = p.X + b0 * XU;
#pragma unroll
    for (int r = 0; r < RW; ++r) {
      const int lr = RW * w + r;
      uint16_t *xr = X + (lr >> 3) * XU * 8 + (lr & 7);
      for (int t = lane; t < cnt[r]; t += 64) {
        const int j = t == lane ? ec[r] : p.col[beg[r] + t];
        if (j < 0 || j >= n) continue;
        xr[8 * j] = f2bf(t == lane ? ev[r] : p.val[beg[r] + t]);
        xr[8 * (n + j)] = 0x3f80;
      }
    }
    for (int e = threadIdx.x; e < R / 8 * 256; e += kTrThreads) {
      reinterpret_cast<uint4 *>(p.h1)[b0 / 8 * 256 + e] = gather_pack8(Ha + (e >> 8) * 8 * kTrHP + (e & 255), kTrHP);
    }
  }
  // ---- second layer: column 32 w + i32 of rows 8 (v / 4) + 4 g + v % 4
  const int ar = i32 & (R - 1);  // the A operand's row (rows past R repeat and are not used)
  constexpr int NV = R / 2;      // result registers in use
  const int u2 = 32 * w + i32;
  float z2[NV];
  {
    f16 acc = {};
#pragma unroll
    for (int ks = 0; ks < 16; ++ks)
      acc = mfma_bf16_32(*reinterpret_cast<const uint4 *>(Ha + ar * kTrHP + 16 * ks + 8 * g), bw[ks], acc);
    const float bias = p.b2[u2];
    float h[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const int lr = 8 * (v / 4) + 4 * g + (v % 4);
      z2[v] = acc[v] + bias;
      h[v] = b0 + lr < p.B ? gelu(z2[v]) : 0.f;
      Hb[lr * kTrHP + u2] = f2bf(h[v]);
    }
    if constexpr (!FWD) {
#pragma unroll
      for (int q = 0; q < R / 8; ++q) store_pack4(p.h2, b0 / 8 + q, 256, u2, g, h + 4 * q);
    }
  }
  // ---- output layer and loss on the first CB3 wavefronts (operands load across the barrier)
  const int oc = 32 * w + i32;
  float tg[NV];
  double sq = 0.0;
  if (w < CB3) {
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) bw[ks] = p.W3P[(w * 16 + ks) * 64 + lane];
    if constexpr (!FWD) {
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int64_t i = row_s[8 * (v / 4) + 4 * g + (v % 4)];
        tg[v] = i >= 0 && oc < k ? p.target[i * k + oc] : 0.f;
      }
    }
  }
  __syncthreads();
  if (w < CB3) {
    f16 acc = {};
#pragma unroll
    for (int ks = 0; ks < 16; ++ks)
      acc = mfma_bf16_32(*reinterpret_cast<const uint4 *>(Hb + ar * kTrHP + 16 * ks + 8 * g), bw[ks], acc);
    const float bias = oc < k ? p.b3[oc] : 0.f;
    if constexpr (FWD) {
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int64_t b = b0 + 8 * (v / 4) + 4 * g + (v % 4);
        if (b < p.B && oc < k) p.out[b * k + oc] = acc[v] + bias;
      }
    } else {
      const float scale = 2.0f / (float)(p.B * k);
      float dv[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int lr = 8 * (v / 4) + 4 * g + (v % 4);
        const bool real = b0 + lr < p.B && oc < k;
        const float d = (acc[v] + bias) - tg[v];
        dv[v] = real ? scale * d : 0.f;
        if (real) {
          p.d3[(b0 + lr) * k + oc] = dv[v];
          sq += (double)d * (double)d;
        }
        Ds[lr * (KP + 8) + oc] = f2bf(dv[v]);
      }
#pragma unroll
      for (int q = 0; q < R / 8; ++q) store_pack4(p.d3p, b0 / 8 + q, KP, oc, g, dv + 4 * q);
    }
  }
  if constexpr (!FWD) {
    const int KS3 = (k + 15) / 16;
    uint4 b3w[2 * CB3];
#pragma unroll
    for (int ks = 0; ks < 2 * CB3; ++ks)
      b3w[ks] = ks < KS3 ? p.W3T[(w * KS3 + ks) * 64 + lane] : uint4{0u, 0u, 0u, 0u};
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) bw[ks] = p.W2T[(w * 16 + ks) * 64 + lane];
    if (blockIdx.x == 0 && threadIdx.x == kTrThreads - 1) train_state_begin(p.st);
    __syncthreads();
    // ---- dz2 = (dout W3) GELU'(z2); h1 is no longer needed
    f16 acc = {};
#pragma unroll
    for (int ks = 0; ks < 2 * CB3; ++ks)
      if (ks < KS3)
        acc = mfma_bf16_32(*reinterpret_cast<const uint4 *>(Ds + ar * (KP + 8) + 16 * ks + 8 * g), b3w[ks], acc);
    float dz[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const int lr = 8 * (v / 4) + 4 * g + (v % 4);
      dz[v] = b0 + lr < p.B ? acc[v] * gelu_grad(z2[v]) : 0.f;
      if (b0 + lr < p.B) p.d2[(b0 + lr) * 256 + u2] = dz[v];
      Ha[lr * kTrHP + u2] = f2bf(dz[v]);
    }
#pragma unroll
    for (int q = 0; q < R / 8; ++q) store_pack4(p.d2p, b0 / 8 + q, 256, u2, g, dz + 4 * q);
    __syncthreads();
    // ---- dz1 = (dz2 W2) GELU'(z1)
    acc = f16{};
#pragma unroll
    for (int ks = 0; ks < 16; ++ks)
      acc = mfma_bf16_32(*reinterpret_cast<const uint4 *>(Ha + ar * kTrHP + 16 * ks + 8 * g), bw[ks], acc);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const int lr = 8 * (v / 4) + 4 * g + (v % 4);
      dz[v] = b0 + lr < p.B ? acc[v] * gelu_grad(Zs[lr * kTrZP + u2]) : 0.f;
      if (b0 + lr < p.B) p.d1[(b0 + lr) * 256 + u2] = dz[v];
    }
#pragma unroll
    for (int q = 0; q < R / 8; ++q) store_pack4(p.d1p, b0 / 8 + q, 256, u2, g, dz + 4 * q);
    if (w < CB3) {
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) sq += __shfl_xor(sq, off, 64);
      if (lane == 0) p.lpart[(int64_t)blockIdx.x * CB3 + w] = sq;
    }
  }
}

// rows per block: 16 where blocks of 32 rows would not cover the compute units
int mlp_batch_rows(const open_ctx *ctx, int64_t B) { return B <= 16 * (int64_t)ctx->num_cu ? 16 : 32; }
int mlp_batch_loss_parts(const open_ctx *ctx, int64_t B, int k) {
  return (int)(pad_rows(B) / mlp_batch_rows(ctx, B)) * ((k + 31) / 32);
}

template <int CB3, bool FWD>
static open_status launch_batch(open_ctx *ctx, const MlpBatch &p) {
  const int R = mlp_batch_rows(ctx, p.B);
  const int64_t rows = FWD ? p.B : pad_rows(p.B);
  const dim3 grid((unsigned)((rows + R - 1) / R));
  const char *name = FWD ? "mlp_forward" : "mlp_fwd_bwd";
  if (R == 16) {
    OPEN_LAUNCH(ctx, name, (k_mlp_fwd_bwd<16, CB3, FWD>), grid, dim3(kTrThreads), 0, p);
  } else {
    OPEN_LAUNCH(ctx, name, (k_mlp_fwd_bwd<32, CB3, FWD>), grid, dim3(kTrThreads), 0, p);
  }
  return OPEN_OK;
}

open_status mlp_batch_launch(open_ctx *ctx, const MlpBatch &p, bool forward_only) {
  if (p.k > 32) return forward_only ? launch_batch<2, true>(ctx, p) : launch_batch<2, false>(ctx, p);
  return forward_only ? launch_batch<1, true>(ctx, p) : launch_batch<1, false>(ctx, p);
}

}  // namespace openk
