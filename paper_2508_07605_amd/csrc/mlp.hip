// Fold-in surrogate network: training and inference.
//
//   x  = [r * mask ; mask]                      (length 2n, never materialised)
//   z1 = W1 x + b1 = b1 + sum_{j in O} (r_j W1[:, j] + W1[:, n + j])    sparse first layer
//   h1 = GELU(z1);  z2 = W2 h1 + b2;  h2 = GELU(z2);  u = W3 h2 + b3
//   GELU(z) = z/2 (1 + erf(z / sqrt 2))
//
// Weights live as float32 masters (updated by Adam) and as bfloat16 copies (round to
// nearest even) for the products.  The sparse first layer accumulates value x weight in
// float32 from a transposed bfloat16 copy of W1 (one contiguous hidden vector per input
// feature).  The dense products run on BF16 MFMA (v_mfma_f32_32x32x16_bf16) with float32
// accumulation.  The batched forward and the training step are in mlp_train.hip and
// wgrad.hip; here are the fused inference, the weight copies, the seeded shuffle and the handle.
#include <limits.h>
#include <math.h>
#include <string.h>

#include <new>

#include "common.h"
#include "dense.h"
#include "mlp_net.h"
#include "mlp_train.h"

namespace openk {

// ---------------------------------------------------------------- bfloat16 weight copies
// First-layer weights as one 32-bit pair per (setting j, hidden unit h): low half
// bf16(W1[h][j]) (the weight of the value r_j), high half bf16(W1[h][n + j]) (the weight of the
// mask bit).  A lane's four units of one setting are one 16-byte load.
__global__ void k_pack_w1p(const float *__restrict__ W1, int H, int n, uint32_t *__restrict__ W1P) {
  const int64_t total = (int64_t)H * n, twon = 2 * (int64_t)n;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t j = e / H, h = e % H;
    W1P[e] = bf16pack(W1[h * twon + j], W1[h * twon + n + j]);
  }
}

// W (N x Kd, row-major; with T its transpose) as MFMA operands in the order of mfma_slot, zero
// past its edges: rows padded to 32, k to 16.
template <bool T>
__global__ void k_pack_mfma(const float *__restrict__ W, int N, int Kd, uint16_t *__restrict__ P) {
  const int KS = (Kd + 15) / 16, total = (N + 31) / 32 * 32 * KS * 16;
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < total; e += gridDim.x * blockDim.x) {
    const int o = e / (16 * KS), i = e % (16 * KS);
    const float x = o < N && i < Kd ? (T ? W[(int64_t)i * N + o] : W[(int64_t)o * Kd + i]) : 0.f;
    P[mfma_slot(o, i, KS)] = f2bf(x);
  }
}

// ---------------------------------------------------------------- step state, shuffle, fallback
__global__ void k_train_state_reset(TrainState *st) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *st = TrainState{0, 0, 0.f, 0.f, 0};
}

// ---- seeded shuffle of the training rows, on the device
// SplitMix64 output function (Steele, Lea and Flood, OOPSLA 2014): a 64-bit mixing bijection.
__host__ __device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z += 0x9e3779b97f4a7c15ull;
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  return z ^ (z >> 31);
}

// perm[i] for i < m: a four-round balanced Feistel network on 2h-bit integers (4^h >= m,
// round keys key_r = mix64(mix64(seed) + 4 epoch + r), round function mix64(R ^ key_r) masked to
// h bits) is a bijection of [0, 4^h); walking its cycle from i until the value falls below m
// restricts it to a bijection of [0, m) (every cycle through i returns to i, so the walk ends).
// Thread 0 also rewinds the batch cursor of the epoch.
__global__ __launch_bounds__(256) void k_shuffle(int64_t m, int h, uint64_t seed, int64_t epoch,
                                                 int64_t *__restrict__ perm, TrainState *__restrict__ st) {
  const uint64_t base = mix64(seed) + 4ull * (uint64_t)epoch;
  uint64_t key[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) key[r] = mix64(base + (uint64_t)r);
  const uint64_t mask = (1ull << h) - 1ull;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < m; i += (int64_t)gridDim.x * 256) {
    uint64_t x = (uint64_t)i;
    do {
      uint64_t L = x >> h, R = x & mask;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const uint64_t nl = R;
        R = L ^ (mix64(R ^ key[r]) & mask);
        L = nl;
      }
      x = (L << h) | R;
    } while (x >= (uint64_t)m);
    perm[i] = (int64_t)x;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) st->cursor = 0;
}

__global__ void k_count_u8(int64_t m, const uint8_t *__restrict__ f, int64_t *__restrict__ out) {
  __shared__ int64_t red[256];
  int64_t c = 0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < m; i += (int64_t)gridDim.x * 256) c += f[i];
  red[threadIdx.x] = c;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < (unsigned)s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[blockIdx.x] = red[0];
}

// ---------------------------------------------------------------- fused inference
// Surrogate fold-in of a tile of kIR rows per block iteration (persistent grid), the network
// and the fallback test in one kernel:
//   first layer  each wavefront owns 16 consecutive rows, lane l hidden units 4l..4l+3.  The
//                row pointers of the 16 rows come in one load, their entries (contiguous in
//                the CSR) are staged in LDS up to kCap at a time, and the entries are taken as
//                one stream across the rows: the weight pairs of the next eight entries load
//                while the current eight are added, and a row is closed (GELU, bfloat16 into
//                the LDS tile) when the stream passes its end.
//   second layer BF16 MFMA, this wavefront's 64 output columns, its W2 operands streamed from
//                the packed copy (L2-resident) four steps ahead -> GELU -> LDS
//   third layer  MFMA -> u to global and LDS
//   residual     observed-entry RMS residual against the setting factors (four lanes per row;
//                the entries from the staging area when they fit) -> fallback flag.
// Every arithmetic step matches the batched forward (same products, same order, same
// roundings).
constexpr int kIR = 64;       // rows per tile
constexpr int kHP = 256 + 8;  // LDS pitch of an activation row (bf16)
constexpr int kCap = 176;     // entries staged per wavefront (three blocks per CU up to rank 32)
static_assert(kCap % 8 == 0, "a staged chunk is padded to a multiple of eight entries");

template <int K>
__global__ __launch_bounds__(256, 3) void k_mlp_infer(int64_t m, const int64_t *__restrict__ ptr,
                                                      const int32_t *__restrict__ col, const float *__restrict__ val,
                                                      int n, const uint32_t *__restrict__ W1P,
                                                      const float *__restrict__ b1, const uint4 *__restrict__ W2P,
                                                      const float *__restrict__ b2, const uint4 *__restrict__ W3P,
                                                      const float *__restrict__ b3, const float *__restrict__ F,
                                                      float tau, float *__restrict__ U, float *__restrict__ rho,
                                                      uint8_t *__restrict__ flag) {
  constexpr int CB3 = (K + 31) / 32;  // 32-column blocks of the output layer
  constexpr int PF = 4;               // W2 steps loaded ahead
  __shared__ __attribute__((aligned(16))) uint16_t Hs[kIR * kHP];
  __shared__ float Us[kIR * K];
  // per wavefront: {column or -1, value pair, value bits, 0} of its rows' entries
  __shared__ uint4 Stg[4][kCap];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int i32 = lane & 31;
  const float b2c[2] = {b2[64 * w + i32], b2[64 * w + 32 + i32]};
  const f4 b1v = *reinterpret_cast<const f4 *>(b1 + 4 * lane);
  const uint2 hb1 = uint2{bf16pack(gelu(b1v[0]), gelu(b1v[1])), bf16pack(gelu(b1v[2]), gelu(b1v[3]))};
  const uint4 *w2w = W2P + (int64_t)(2 * w) * 16 * 64 + lane;  // step (cb, ks) at w2w[(cb*16 + ks)*64]
  const __amdgpu_buffer_rsrc_t rs1 = make_rsrc(W1P, (uint64_t)n * 1024);
  uint4 *stg = Stg[w];
  const int64_t ntiles = (m + kIR - 1) / kIR;
  // The next tile's row pointers and the first staged chunk of its entries are loaded while
  // the current tile is in its later phases.  Lane q <= 16 holds P_q, the first entry of row
  // 16 w + q of the tile (rows past m are empty); lane l holds entries l + 64 i of the chunk.
  constexpr int PK = (kCap + 63) / 64;
  auto load_ptrs = [&](int64_t tile) -> int64_t {
    const int64_t prow = tile * kIR + 16 * w + (lane < 16 ? lane : 16);
    return tile < ntiles ? ptr[prow < m ? prow : m] : 0;
  };
  int pcol[PK];
  float pval[PK];
  auto load_chunk0 = [&](int64_t pvn) {
    const int64_t e0 = readlane_i64(pvn, 0);
    const int64_t nn = readlane_i64(pvn, 16) - e0;
#pragma unroll
    for (int i = 0; i < PK; ++i) {
      const int t = lane + 64 * i;
      pcol[i] = t < nn && t < kCap ? col[e0 + t] : -1;
      pval[i] = t < nn && t < kCap ? val[e0 + t] : 0.f;
    }
  };
  int64_t pv_next = load_ptrs(blockIdx.x);
  load_chunk0(pv_next);
  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int64_t r0 = tile * kIR;
    // ---- first layer (sparse), GELU, bfloat16 into LDS
    const int64_t pv = pv_next;
    const int64_t E0 = readlane_i64(pv, 0);
    const int nent = (int)(readlane_i64(pv, 16) - E0);  // the wavefront's entries, < 2^31
    int cur = 0;                                      // row of the wavefront being accumulated
    int nxt = (int)(readlane_i64(pv, 1) - E0);        // first entry (relative) after it
    f4 z = b1v;
    auto advance = [&]() {
      ++cur;
      nxt = cur < 16 ? (int)(readlane_i64(pv, cur + 1) - E0) : INT_MAX;
    };
    // closes row cur (GELU, bfloat16 into the tile), then stores every following empty row
    // ending at or before entry u: rows without entries are GELU(b1)
    auto close_rows = [&](int u) {
      *reinterpret_cast<uint2 *>(Hs + (16 * w + cur) * kHP + 4 * lane) =
          uint2{bf16pack(gelu(z[0]), gelu(z[1])), bf16pack(gelu(z[2]), gelu(z[3]))};
      z = b1v;
      advance();
      while (u >= nxt) {
        *reinterpret_cast<uint2 *>(Hs + (16 * w + cur) * kHP + 4 * lane) = hb1;
        advance();
      }
    };
    for (int cs = 0; cs < nent; cs += kCap) {
      const int clen = nent - cs < kCap ? nent - cs : kCap;
      const int cpad = (clen + 7) & ~7;  // the chunk padded with entries that add nothing
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();  // the previous chunk's reads of the staging area are done
      if (cs == 0) {
#pragma unroll
        for (int i = 0; i < PK; ++i) {
          const int t = lane + 64 * i;
          if (t < cpad) {
            const int j = pcol[i];
            const float r = pval[i];
            const bool ok = t < clen && j >= 0 && j < n;
            stg[t] = t < clen ? uint4{(uint32_t)(ok ? j : -1), value_pair(r, ok), __builtin_bit_cast(uint32_t, r), 0u}
                              : uint4{0xffffffffu, 0u, 0u, 0u};
          }
        }
      } else {
        for (int t = lane; t < cpad; t += 64) {
          uint4 e = uint4{0xffffffffu, 0u, 0u, 0u};
          if (t < clen) {
            const int j = col[E0 + cs + t];
            const float r = val[E0 + cs + t];
            const bool ok = j >= 0 && j < n;
            e = uint4{(uint32_t)(ok ? j : -1), value_pair(r, ok), __builtin_bit_cast(uint32_t, r), 0u};
          }
          stg[t] = e;
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      // two register sets of eight entries' weight pairs: one loads while the other is added
      uint4 wa[8], wb[8];
      uint32_t qa[8], qb[8];
      // the loads are issued in entry order (scheduling barriers), so that each entry waits
      // only for its own weights and not for the younger loads of the other set
      auto fetch = [&](uint4 (&wv)[8], uint32_t (&q)[8], int u0) {
        uint4 st[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) st[e] = stg[u0 + e];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          q[e] = st[e].y;
          wv[e] = w1_pairs(rs1, (int)st[e].x, lane);
          __builtin_amdgcn_sched_barrier(0);
        }
      };
      // a padding entry adds exact zeros; a row it closes has ended at or before it
      auto consume = [&](const uint4 (&wv)[8], const uint32_t (&q)[8], int u0) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          // rows end at one entry in ~14: the close is laid out of line, so that the common
          // path falls through instead of taking a branch per entry
          if (__builtin_expect(cs + u0 + e >= nxt, 0)) close_rows(cs + u0 + e);
          layer1_step(z, wv[e], q[e]);
        }
      };
      // Every fetch is unconditional (past the chunk it reloads entries 0..7, which are not
      // taken): a conditional one would make the waits count as if the other set had not been
      // issued, and each entry would wait for the younger loads too.
      fetch(wa, qa, 0);
      for (int u0 = 0; u0 < cpad; u0 += 16) {
        fetch(wb, qb, u0 + 8 < cpad ? u0 + 8 : 0);
        consume(wa, qa, u0);
        if (u0 + 8 >= cpad) break;
        fetch(wa, qa, u0 + 16 < cpad ? u0 + 16 : 0);
        consume(wb, qb, u0 + 8);
      }
    }
    if (cur < 16) close_rows(INT_MAX - 1);
    pv_next = load_ptrs(tile + gridDim.x);
    // the lane index through an opaque copy: the per-lane addresses of the later phases are
    // formed here in each tile instead of being hoisted out of the tile loop (and spilled)
    int lane_o = lane;
    asm volatile("" : "+v"(lane_o));
    const int i32o = lane_o & 31, go = (lane_o >> 5) & 1;
    __syncthreads();
    // ---- second layer: this wavefront's 64 output columns for all kIR rows
    f16 acc[2][2] = {};
    {
      // an offset the compiler cannot see through, so that the W2 loads stay in the tile loop
      // instead of being hoisted into 128 live registers
      int opq = 0;
      asm volatile("" : "+v"(opq));
      const uint4 *w2t = w2w + opq;
      uint4 ring[PF][2];
#pragma unroll
      for (int ks = 0; ks < PF; ++ks)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) ring[ks][cb] = w2t[(cb * 16 + ks) * 64];
#pragma unroll
      for (int ks = 0; ks < 16; ++ks) {
        const uint4 bw0 = ring[ks % PF][0], bw1 = ring[ks % PF][1];
        if (ks + PF < 16) {
          ring[ks % PF][0] = w2t[(ks + PF) * 64];
          ring[ks % PF][1] = w2t[(16 + ks + PF) * 64];
        }
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) {
          const uint4 a = *reinterpret_cast<const uint4 *>(Hs + (32 * rb + i32o) * kHP + 16 * ks + 8 * go);
          acc[rb][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                              __builtin_bit_cast(bf16x8, bw0), acc[rb][0], 0, 0, 0);
          acc[rb][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                              __builtin_bit_cast(bf16x8, bw1), acc[rb][1], 0, 0, 0);
        }
      }
    }
    load_chunk0(pv_next);
    __syncthreads();  // every wavefront has read the first layer's tile
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int rr = 32 * rb + 8 * (v / 4) + 4 * go + (v % 4);
          Hs[rr * kHP + 64 * w + 32 * cb + i32o] = f2bf(gelu(acc[rb][cb][v] + b2c[cb]));
        }
    __syncthreads();
    // ---- third layer: tiles (row block, 32 outputs) on the first 2 CB3 wavefronts
    if (w < 2 * CB3) {
      const int rb = w & 1, cb = w >> 1;
      const int oc = 32 * cb + i32o;  // output column supplied / received by this lane
      f16 acc3 = {};
      int opq = 0;
      asm volatile("" : "+v"(opq));  // keeps the operand loads in the tile loop
      const uint4 *w3t = W3P + cb * 16 * 64 + lane + opq;
      uint4 bw[16];
#pragma unroll
      for (int ks = 0; ks < 16; ++ks) bw[ks] = w3t[ks * 64];
#pragma unroll
      for (int ks = 0; ks < 16; ++ks) {
        const uint4 a = *reinterpret_cast<const uint4 *>(Hs + (32 * rb + i32o) * kHP + 16 * ks + 8 * go);
        acc3 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, bw[ks]),
                                                      acc3, 0, 0, 0);
      }
      if (oc < K) {
        const float bias = b3[oc];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int rr = 32 * rb + 8 * (v / 4) + 4 * go + (v % 4);
          const float x = acc3[v] + bias;
          Us[rr * K + oc] = x;
          if (r0 + rr < m) U[(r0 + rr) * K + oc] = x;
        }
      }
    }
    __syncthreads();
    // ---- observed-entry RMS residual: four lanes per row, K/4 dimensions each
    {
      constexpr int KQ = K / 4;
      constexpr int RQ = K <= 32 ? 8 : 4;  // entries per row in flight
      const int lr = 16 * w + (lane_o >> 2), pq = lane_o & 3;
      const int64_t row = r0 + lr;
      // the row's entries [P_q, P_q+1) from the lanes that loaded them (empty past m)
      const int q = lane_o >> 2;
      const int64_t t0 = (int64_t)(((uint64_t)(uint32_t)__shfl((int)((uint64_t)pv >> 32), q, 64) << 32) |
                                   (uint32_t)__shfl((int)(uint32_t)pv, q, 64));
      const int64_t t1 = (int64_t)(((uint64_t)(uint32_t)__shfl((int)((uint64_t)pv >> 32), q + 1, 64) << 32) |
                                   (uint32_t)__shfl((int)(uint32_t)pv, q + 1, 64));
      const int cnt = (int)(t1 - t0);
      int cmax = cnt;
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) {
        const int o = __shfl_xor(cmax, off, 64);
        cmax = o > cmax ? o : cmax;
      }
      float ssq = 0.f;
      const bool staged = nent <= kCap;  // wave-uniform: this row's entries are in stg
      const int sofs = (int)(t0 - E0);
      for (int t0b = 0; t0b < cmax; t0b += RQ) {
        // RQ entries in flight: indices and values, then the factor rows, then the dots
        int jv[RQ];
        float rv[RQ];
        const float *fv[RQ];
#pragma unroll
        for (int e = 0; e < RQ; ++e) {
          const int t = t0b + e;
          const bool in = t < cnt;
          if (staged) {
            const uint4 st = stg[in ? sofs + t : 0];
            jv[e] = in ? (int)st.x : -1;
            rv[e] = in ? __builtin_bit_cast(float, st.z) : 0.f;
          } else {
            jv[e] = in ? col[t0 + t] : -1;
            rv[e] = in ? val[t0 + t] : 0.f;
          }
          const bool okj = jv[e] >= 0 && jv[e] < n;
          fv[e] = F + (int64_t)(okj ? jv[e] : 0) * K + pq * KQ;
        }
        float fx[RQ][KQ];
#pragma unroll
        for (int e = 0; e < RQ; ++e)
#pragma unroll
          for (int a = 0; a < KQ; ++a) fx[e][a] = fv[e][a];
#pragma unroll
        for (int e = 0; e < RQ; ++e) {
          float d = 0.f;
#pragma unroll
          for (int a = 0; a < KQ; ++a) d = __builtin_fmaf(Us[lr * K + pq * KQ + a], fx[e][a], d);
          d += __shfl_xor(d, 1, 64);
          d += __shfl_xor(d, 2, 64);
          const float er = rv[e] - d;
          if (jv[e] >= 0 && jv[e] < n) ssq = __builtin_fmaf(er, er, ssq);
        }
      }
      if (pq == 0 && row < m) {
        const float rh = cnt > 0 ? sqrtf(ssq / (float)cnt) : 0.f;
        rho[row] = rh;
        flag[row] = (cnt > 0) && !(rh <= tau);
      }
    }
    __syncthreads();  // the tile buffers are reused
  }
}

}  // namespace openk

// ---------------------------------------------------------------- handle
struct open_mlp {
  open_ctx *ctx = nullptr;
  int n = 0, k = 0, H = 0;
  int64_t np = 0;
  int64_t off_b1 = 0, off_w2 = 0, off_b2 = 0, off_w3 = 0, off_b3 = 0;
  float *w = nullptr, *g = nullptr, *am = nullptr, *av = nullptr;  // masters, gradient, Adam moments
  uint32_t *w1p = nullptr;                                         // W1 weight pairs, bfloat16 (n x H)
  uint4 *w2p = nullptr, *w3p = nullptr;                            // W2, W3 as MFMA operands
  uint4 *w2t = nullptr, *w3t = nullptr;                            // and their transposes (training)
  openk::TrainState *tstate = nullptr;                             // device optimizer state
  // a training batch of up to cap rows: packed operands of the weight gradients, output
  // gradients, partial losses
  int64_t cap = 0;
  uint16_t *x = nullptr, *h1 = nullptr, *h2 = nullptr, *d1p = nullptr, *d2p = nullptr, *d3p = nullptr;
  float *d1 = nullptr, *d2 = nullptr, *d3 = nullptr;
  double *lpart = nullptr, *loss = nullptr;
  // inference scratch
  int64_t icap = 0;
  float *rho = nullptr;
  uint8_t *flag = nullptr;
  int64_t *cnt = nullptr;
};

namespace openk {

constexpr int kMaxBatchRows = 16384;

static void mlp_free_batch(open_mlp *p) {
  for (uint16_t **f : {&p->x, &p->h1, &p->h2, &p->d1p, &p->d2p, &p->d3p}) {
    (void)hipFree(*f);
    *f = nullptr;
  }
  for (float **f : {&p->d1, &p->d2, &p->d3}) {
    (void)hipFree(*f);
    *f = nullptr;
  }
  (void)hipFree(p->lpart);
  p->lpart = nullptr;
  p->cap = 0;
}

static open_status mlp_batch_buffers(open_mlp *p, int64_t B) {
  open_ctx *ctx = p->ctx;
  if (B <= p->cap) return OPEN_OK;
  if (ctx->capturing) return fail(ctx, OPEN_E_UNSUPPORTED, "buffer growth during graph capture");
  OPEN_HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
  mlp_free_batch(p);
  const size_t R = (size_t)pad_rows(B), H = (size_t)p->H;
  const size_t h = sizeof(uint16_t) * R * H, f = sizeof(float) * R * H;
  // partial losses: one per block of at least 16 rows and 32 outputs
  const size_t parts = R / 16 * ((size_t)pad_units(p->k) / 32);
  if (hipMalloc(&p->x, sizeof(uint16_t) * R * (size_t)pad_units(2 * p->n)) || hipMalloc(&p->h1, h) ||
      hipMalloc(&p->h2, h) || hipMalloc(&p->d1p, h) || hipMalloc(&p->d2p, h) ||
      hipMalloc(&p->d3p, sizeof(uint16_t) * R * (size_t)pad_units(p->k)) || hipMalloc(&p->d1, f) ||
      hipMalloc(&p->d2, f) || hipMalloc(&p->d3, sizeof(float) * R * (size_t)p->k) ||
      hipMalloc(&p->lpart, sizeof(double) * parts)) {
    (void)hipGetLastError();
    mlp_free_batch(p);
    return fail(ctx, OPEN_E_NOMEM, "surrogate batch buffers");
  }
  p->cap = B;
  return OPEN_OK;
}

static open_status mlp_repack(open_mlp *p) {
  OPEN_LAUNCH(p->ctx, "mlp_pack_w1p", k_pack_w1p, dim3(1024), dim3(256), 0, p->w, p->H, p->n, p->w1p);
  const int H = p->H, k = p->k;
  OPEN_LAUNCH(p->ctx, "mlp_pack_w2p", k_pack_mfma<false>, dim3(64), dim3(256), 0, p->w + p->off_w2, H, H,
              (uint16_t *)p->w2p);
  OPEN_LAUNCH(p->ctx, "mlp_pack_w2t", k_pack_mfma<true>, dim3(64), dim3(256), 0, p->w + p->off_w2, H, H,
              (uint16_t *)p->w2t);
  OPEN_LAUNCH(p->ctx, "mlp_pack_w3p", k_pack_mfma<false>, dim3(16), dim3(256), 0, p->w + p->off_w3, k, H,
              (uint16_t *)p->w3p);
  OPEN_LAUNCH(p->ctx, "mlp_pack_w3t", k_pack_mfma<true>, dim3(16), dim3(256), 0, p->w + p->off_w3, H, k,
              (uint16_t *)p->w3t);
  return OPEN_OK;
}

static MlpBatch mlp_batch(const open_mlp *p, int64_t B, const int64_t *rows, int use_cursor, const int64_t *ptr,
                          const int32_t *col, const float *val) {
  MlpBatch b = {};
  b.B = B;
  b.rows = rows;
  b.use_cursor = use_cursor;
  b.ptr = ptr;
  b.col = col;
  b.val = val;
  b.n = p->n;
  b.k = p->k;
  b.W1P = p->w1p;
  b.b1 = p->w + p->off_b1;
  b.b2 = p->w + p->off_b2;
  b.b3 = p->w + p->off_b3;
  b.W2P = p->w2p;
  b.W3P = p->w3p;
  b.W2T = p->w2t;
  b.W3T = p->w3t;
  b.st = p->tstate;
  return b;
}

// Loss and gradients of a batch, in two launches: forward and backward, then the weight
// gradients, with the Adam update (lr > 0) or into p->g (lr = 0).
static open_status mlp_step(open_mlp *p, int64_t B, const int64_t *rows, int use_cursor, const int64_t *ptr,
                            const int32_t *col, const float *val, const float *target, float lr, float *loss_out,
                            float *loss_steps) {
  open_ctx *ctx = p->ctx;
  const int H = p->H, k = p->k, n = p->n;
  MlpBatch b = mlp_batch(p, B, rows, use_cursor, ptr, col, val);
  b.target = target;
  b.X = p->x;
  b.h1 = p->h1;
  b.h2 = p->h2;
  b.d1p = p->d1p;
  b.d2p = p->d2p;
  b.d3p = p->d3p;
  b.d1 = p->d1;
  b.d2 = p->d2;
  b.d3 = p->d3;
  b.lpart = p->lpart;
  open_status st;
  if ((st = mlp_batch_launch(ctx, b, false))) return st;
  WgradStep g = {};
  g.l[0] = {p->d1p, p->x, p->d1, H, 2 * n, 0, nullptr, nullptr, (uint16_t *)p->w1p};
  g.l[1] = {p->d2p, p->h1, p->d2, H, H, p->off_w2, (uint16_t *)p->w2p, (uint16_t *)p->w2t, nullptr};
  g.l[2] = {p->d3p, p->h2, p->d3, k, H, p->off_w3, (uint16_t *)p->w3p, (uint16_t *)p->w3t, nullptr};
  g.B = B;
  g.w = p->w;
  g.g = p->g;
  g.m = p->am;
  g.v = p->av;
  g.lr = lr;
  g.st = p->tstate;
  g.lpart = p->lpart;
  g.nlpart = mlp_batch_loss_parts(ctx, B, k);
  g.ltotal = B * k;
  g.loss_d = p->loss;
  g.loss_f = loss_out;
  g.loss_steps = loss_steps;
  return wgrad_step(ctx, "mlp_wgrad_adam", g, lr > 0.f);
}

// ---------------------------------------------------------------- shared with the NCF training
// (declared in dense.h)
open_status dense_train_state_reset(open_ctx *ctx, TrainState *st) {
  OPEN_LAUNCH(ctx, "train_state_reset", k_train_state_reset, dim3(1), dim3(64), 0, st);
  return OPEN_OK;
}

open_status dense_shuffle(open_ctx *ctx, int64_t m, uint64_t seed, int64_t epoch, int64_t *perm, TrainState *st) {
  int h = 1;
  while (h < 31 && (int64_t(1) << (2 * h)) < m) ++h;
  const int64_t blocks = (m + 255) / 256 < 4096 ? (m + 255) / 256 : 4096;
  OPEN_LAUNCH(ctx, "shuffle", k_shuffle, dim3((unsigned)blocks), dim3(256), 0, m, h, seed, epoch, perm, st);
  return OPEN_OK;
}

// Seeded initial weights: every weight and bias of a layer with fan-in f uniform on
// [-1/sqrt(f), 1/sqrt(f)), element e of the flat parameter vector drawn as
// (mix64(seed ^ mix64(e)) >> 40) * 2^-24 in [0, 1).
static void seeded_init(open_mlp *p, uint64_t seed, float *w) {
  struct Seg {
    int64_t off, len;
    int fan_in;
  };
  const int64_t H = p->H, n2 = 2 * (int64_t)p->n, k = p->k;
  const Seg seg[] = {{0, H * n2, (int)n2},          {p->off_b1, H, (int)n2}, {p->off_w2, H * H, (int)H},
                     {p->off_b2, H, (int)H},       {p->off_w3, k * H, (int)H}, {p->off_b3, k, (int)H}};
  for (const Seg &sg : seg) {
    const double a = 1.0 / sqrt((double)sg.fan_in);
    for (int64_t i = 0; i < sg.len; ++i) {
      const uint64_t e = (uint64_t)(sg.off + i);
      const double u = (double)(mix64(seed ^ mix64(e)) >> 40) * (1.0 / 16777216.0);
      w[sg.off + i] = (float)(a * (2.0 * u - 1.0));
    }
  }
}

}  // namespace openk

using namespace openk;

extern "C" {

int64_t open_mlp_num_params(int32_t n, int32_t k, int32_t hidden) {
  return (int64_t)hidden * 2 * n + hidden + (int64_t)hidden * hidden + hidden + (int64_t)k * hidden + k;
}

open_status open_mlp_create(open_ctx *ctx, open_mlp **out, int32_t n, int32_t k, int32_t hidden,
                            const float *init_host, uint64_t seed) {
  if (!ctx) return OPEN_E_INVALID;
  if (!out) return fail(ctx, OPEN_E_INVALID, "null output handle");
  *out = nullptr;
  if (hidden != 256) return fail(ctx, OPEN_E_UNSUPPORTED, "hidden width must be 256");
  if (!(k == 8 || k == 16 || k == 32 || k == 64)) return fail(ctx, OPEN_E_UNSUPPORTED, "rank must be 8, 16, 32 or 64");
  if (n <= 0 || n > 4096) return fail(ctx, OPEN_E_INVALID, "n must be in [1, 4096]");
  OPEN_HIP_TRY(ctx, hipSetDevice(ctx->device));
  open_mlp *p = new (std::nothrow) open_mlp();
  if (!p) return fail(ctx, OPEN_E_NOMEM, "handle");
  p->ctx = ctx;
  p->n = n;
  p->k = k;
  p->H = hidden;
  p->np = open_mlp_num_params(n, k, hidden);
  p->off_b1 = (int64_t)hidden * 2 * n;
  p->off_w2 = p->off_b1 + hidden;
  p->off_b2 = p->off_w2 + (int64_t)hidden * hidden;
  p->off_w3 = p->off_b2 + hidden;
  p->off_b3 = p->off_w3 + (int64_t)k * hidden;
  const size_t bytes = sizeof(float) * (size_t)p->np;
  if (hipMalloc(&p->w, bytes) || hipMalloc(&p->g, bytes) || hipMalloc(&p->am, bytes) || hipMalloc(&p->av, bytes) ||
      hipMalloc(&p->w1p, sizeof(uint32_t) * (size_t)hidden * n) || hipMalloc(&p->w2p, sizeof(uint4) * 8192) ||
      hipMalloc(&p->w3p, sizeof(uint4) * 2048) ||
      hipMalloc(&p->w2t, sizeof(uint4) * 8192) || hipMalloc(&p->w3t, sizeof(uint4) * 2048) ||
      hipMalloc(&p->loss, sizeof(double) * 8) ||
      hipMalloc(&p->tstate, sizeof(TrainState))) {
    (void)hipGetLastError();
    open_mlp_destroy(p);
    return fail(ctx, OPEN_E_NOMEM, "surrogate parameters");
  }
  open_status st;
  if (init_host) {
    st = open_mlp_set_weights(p, init_host);
  } else {
    float *w0 = new (std::nothrow) float[(size_t)p->np];
    if (!w0) {
      open_mlp_destroy(p);
      return fail(ctx, OPEN_E_NOMEM, "initial weights");
    }
    seeded_init(p, seed, w0);
    st = open_mlp_set_weights(p, w0);
    delete[] w0;
  }
  if (st) {
    open_mlp_destroy(p);
    return st;
  }
  *out = p;
  return OPEN_OK;
}

open_status open_mlp_destroy(open_mlp *p) {
  if (!p) return OPEN_E_INVALID;
  if (p->ctx) (void)hipStreamSynchronize(p->ctx->stream);
  mlp_free_batch(p);
  (void)hipFree(p->w);
  (void)hipFree(p->g);
  (void)hipFree(p->am);
  (void)hipFree(p->av);
  (void)hipFree(p->w1p);
  (void)hipFree(p->w2p);
  (void)hipFree(p->w3p);
  (void)hipFree(p->w2t);
  (void)hipFree(p->w3t);
  (void)hipFree(p->tstate);
  (void)hipFree(p->loss);
  (void)hipFree(p->rho);
  (void)hipFree(p->flag);
  (void)hipFree(p->cnt);
  delete p;
  return OPEN_OK;
}

open_status open_mlp_get_weights(open_mlp *p, float *host_out) {
  if (!p || !host_out) return OPEN_E_INVALID;
  open_ctx *ctx = p->ctx;
  OPEN_HIP_TRY(ctx, hipMemcpyAsync(host_out, p->w, sizeof(float) * p->np, hipMemcpyDeviceToHost, ctx->stream));
  OPEN_HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
  return OPEN_OK;
}

open_status open_mlp_set_weights(open_mlp *p, const float *host_in) {
  if (!p || !host_in) return OPEN_E_INVALID;
  open_ctx *ctx = p->ctx;
  OPEN_HIP_TRY(ctx, hipMemcpyAsync(p->w, host_in, sizeof(float) * p->np, hipMemcpyHostToDevice, ctx->stream));
  OPEN_LAUNCH(ctx, "fill", k_fill_i32, dim3(256), dim3(256), 0, (int *)p->am, p->np, 0);
  OPEN_LAUNCH(ctx, "fill", k_fill_i32, dim3(256), dim3(256), 0, (int *)p->av, p->np, 0);
  OPEN_LAUNCH(ctx, "mlp_train_state_reset", k_train_state_reset, dim3(1), dim3(64), 0, p->tstate);
  open_status st = mlp_repack(p);
  if (st) return st;
  OPEN_HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
  return OPEN_OK;
}

open_status open_mlp_forward(open_mlp *p, int64_t m, const int64_t *row_ptr, const int32_t *col, const float *val,
                             float *U_hat) {
  if (!p) return OPEN_E_INVALID;
  open_ctx *ctx = p->ctx;
  if (m < 0 || m >= INT32_MAX || (m > 0 && (!row_ptr || !col || !val || !U_hat)))
    return fail(ctx, OPEN_E_INVALID, "bad shape or pointer");
  OPEN_HIP_TRY(ctx, hipSetDevice(ctx->device));
  if (m == 0) return OPEN_OK;
  // a launch takes 2^26 rows at most: 512 threads for every 32 rows, fewer than 2^32 in a grid
  constexpr int64_t kLaunchRows = int64_t(1) << 26;
  open_status st = OPEN_OK;
  for (int64_t r0 = 0; r0 < m && !st; r0 += kLaunchRows) {
    MlpBatch b = mlp_batch(p, m - r0 < kLaunchRows ? m - r0 : kLaunchRows, nullptr, 0, row_ptr + r0, col, val);
    b.out = U_hat + r0 * p->k;
    st = mlp_batch_launch(ctx, b, true);
  }
  return st;
}

open_status open_mlp_loss_grad(open_mlp *p, int64_t m, const int64_t *row_ptr, const int32_t *col,
                               const float *val, const float *target, double *loss, float *grads_host) {
  if (!p) return OPEN_E_INVALID;
  open_ctx *ctx = p->ctx;
  if (m <= 0 || m > kMaxBatchRows || !row_ptr || !col || !val || !target || !loss || !grads_host)
    return fail(ctx, OPEN_E_INVALID, "bad shape or pointer (batch of 1..16384 rows)");
  OPEN_HIP_TRY(ctx, hipSetDevice(ctx->device));
  open_status st;
  if ((st = mlp_batch_buffers(p, m))) return st;
  if ((st = mlp_step(p, m, nullptr, 0, row_ptr, col, val, target, 0.f, nullptr, nullptr))) return st;
  OPEN_HIP_TRY(ctx, hipMemcpyAsync(grads_host, p->g, sizeof(float) * p->np, hipMemcpyDeviceToHost, ctx->stream));
  double *h;
  if ((st = pinned_get(ctx, 64, (void **)&h))) return st;
  OPEN_HIP_TRY(ctx, hipMemcpyAsync(h, p->loss, sizeof(double), hipMemcpyDeviceToHost, ctx->stream));
  OPEN_HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
  *loss = h[0];
  return OPEN_OK;
}

open_status open_mlp_train_step(open_mlp *p, int64_t m, const int64_t *row_ptr, const int32_t *col,
                                const float *val, const float *target, const int64_t *rows, int32_t batch, float lr,
                                float *loss_out) {
  if (!p) return OPEN_E_INVALID;
  open_ctx *ctx = p->ctx;
  if (m <= 0 || m >= INT32_MAX || batch <= 0 || batch > kMaxBatchRows || (!rows && batch > m) || !row_ptr || !col ||
      !val || !target)
    return fail(ctx, OPEN_E_INVALID, "bad shape or pointer (batch of 1..16384 rows)");
  if (!(lr > 0.0f) || !isfinite(lr)) return fail(ctx, OPEN_E_INVALID, "learning rate must be finite and > 0");
  OPEN_HIP_TRY(ctx, hipSetDevice(ctx->device));
  open_status st;
  if ((st = mlp_batch_buffers(p, batch))) return st;
  return mlp_step(p, batch, rows, 0, row_ptr, col, val, target, lr, loss_out, nullptr);
}

open_status open_mlp_train(open_mlp *p, int64_t m, const int64_t *row_ptr, const int32_t *col, const float *val,
                           const float *target, int32_t batch, float lr, int32_t epochs, uint64_t seed,
                           float *loss_hist) {
  if (!p) return OPEN_E_INVALID;
  open_ctx *ctx = p->ctx;
  if (m <= 0 || m >= INT32_MAX || !row_ptr || !col || !val || !target)
    return fail(ctx, OPEN_E_INVALID, "bad shape or pointer");
  if (batch <= 0 || batch > kMaxBatchRows || batch > m)
    return fail(ctx, OPEN_E_INVALID, "batch must be in [1, min(16384, m)]");
  if (epochs < 0) return fail(ctx, OPEN_E_INVALID, "epochs must be >= 0");
  if (!(lr > 0.0f) || !isfinite(lr)) return fail(ctx, OPEN_E_INVALID, "learning rate must be finite and > 0");
  if (epochs == 0) return OPEN_OK;
  OPEN_HIP_TRY(ctx, hipSetDevice(ctx->device));
  const int64_t spe = m / batch;  // full batches per epoch; the remainder is left to later shuffles
  const int64_t total = spe * epochs;
  int h = 1;
  while (h < 31 && (int64_t(1) << (2 * h)) < m) ++h;
  open_status st;
  if ((st = mlp_batch_buffers(p, batch))) return st;
  int64_t *perm = nullptr;
  float *losses = nullptr;
  int64_t *t0h = nullptr;
  if (hipMalloc(&perm, sizeof(int64_t) * (size_t)m) || hipMalloc(&losses, sizeof(float) * (size_t)total)) {
    (void)hipGetLastError();
    (void)hipFree(perm);
    (void)hipFree(losses);
    return fail(ctx, OPEN_E_NOMEM, "training buffers");
  }
  // the per-step losses are indexed by the Adam step count, which may not start at zero
  if ((st = pinned_get(ctx, 64, (void **)&t0h))) {
    (void)hipFree(perm);
    (void)hipFree(losses);
    return st;
  }
  if (hipMemcpyAsync(t0h, p->tstate, sizeof(int64_t), hipMemcpyDeviceToHost, ctx->stream) != hipSuccess ||
      hipStreamSynchronize(ctx->stream) != hipSuccess) {
    (void)hipFree(perm);
    (void)hipFree(losses);
    return fail(ctx, OPEN_E_DEVICE, "reading the step counter");
  }
  const int64_t t0 = t0h[0];
  float *loss_rec = losses - t0;  // loss of Adam step t lands in losses[t - t0]
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  auto one_step = [&]() -> open_status {
    return mlp_step(p, batch, perm, 1, row_ptr, col, val, target, lr, nullptr, loss_rec);
  };
  const int64_t sblocks = (m + 255) / 256 < 4096 ? (m + 255) / 256 : 4096;
  for (int32_t e = 0; e < epochs && st == OPEN_OK; ++e) {
    OPEN_LAUNCH(ctx, "mlp_shuffle", k_shuffle, dim3((unsigned)sblocks), dim3(256), 0, m, h, seed, (int64_t)e, perm,
                p->tstate);
    for (int64_t b = 0; b < spe && st == OPEN_OK; ++b) {
      if (!exec) {
        // the first step runs eagerly (it sizes every workspace), the next one is recorded
        if ((st = one_step())) break;
        if (b + 1 < spe || e + 1 < epochs) {
          if ((st = graph_capture(ctx, one_step, &graph))) break;
          if (hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0) != hipSuccess) {
            (void)hipGetLastError();
            st = fail(ctx, OPEN_E_DEVICE, "graph instantiation failed");
          }
        }
        continue;
      }
      if (hipGraphLaunch(exec, ctx->stream) != hipSuccess) st = fail(ctx, OPEN_E_DEVICE, "graph launch failed");
    }
  }
  if (exec) (void)hipGraphExecDestroy(exec);
  if (graph) (void)hipGraphDestroy(graph);
  if (st == OPEN_OK && loss_hist) {
    float *hl = new (std::nothrow) float[(size_t)total];
    if (!hl) {
      st = fail(ctx, OPEN_E_NOMEM, "loss history");
    } else {
      if (hipMemcpyAsync(hl, losses, sizeof(float) * (size_t)total, hipMemcpyDeviceToHost, ctx->stream) != hipSuccess ||
          hipStreamSynchronize(ctx->stream) != hipSuccess) {
        st = fail(ctx, OPEN_E_DEVICE, "reading the losses");
      } else {
        for (int32_t e = 0; e < epochs; ++e) {
          double sum = 0.0;
          for (int64_t b = 0; b < spe; ++b) sum += hl[e * spe + b];
          loss_hist[e] = (float)(sum / (double)spe);
        }
      }
      delete[] hl;
    }
  }
  (void)hipStreamSynchronize(ctx->stream);
  (void)hipFree(perm);
  (void)hipFree(losses);
  return st;
}

open_status open_mlp_foldin(open_mlp *p, const float *F, int64_t m, const int64_t *row_ptr, const int32_t *col,
                            const float *val, float tau, float lambda, int32_t weighted, float *U_out,
                            uint8_t *used_fallback, float *rho, int64_t *n_fallback) {
  if (!p) return OPEN_E_INVALID;
  open_ctx *ctx = p->ctx;
  if (m < 0 || m >= INT32_MAX || !F || (m > 0 && (!row_ptr || !col || !val || !U_out)))
    return fail(ctx, OPEN_E_INVALID, "bad shape or pointer");
  if (!(tau >= 0.0f)) return fail(ctx, OPEN_E_INVALID, "tau must be >= 0");
  if (!(lambda >= 0.0f) || !isfinite(lambda)) return fail(ctx, OPEN_E_INVALID, "lambda must be finite and >= 0");
  if (m == 0) {
    if (n_fallback) *n_fallback = 0;
    return OPEN_OK;
  }
  OPEN_HIP_TRY(ctx, hipSetDevice(ctx->device));
  open_status st;
  if (m > p->icap) {
    OPEN_HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
    (void)hipFree(p->rho);
    (void)hipFree(p->flag);
    (void)hipFree(p->cnt);
    p->rho = nullptr;
    p->flag = nullptr;
    p->cnt = nullptr;
    if (hipMalloc(&p->rho, sizeof(float) * m) || hipMalloc(&p->flag, m) || hipMalloc(&p->cnt, sizeof(int64_t) * 512)) {
      (void)hipGetLastError();
      p->icap = 0;
      return fail(ctx, OPEN_E_NOMEM, "surrogate fold-in buffers");
    }
    p->icap = m;
  }
  float *r = rho ? rho : p->rho;
  uint8_t *f = used_fallback ? used_fallback : p->flag;
  // network, residual and fallback flag in one persistent kernel
  const int64_t tiles = (m + kIR - 1) / kIR;
  // resident blocks per CU: three (LDS about 50 KB each) up to rank 32, two at rank 64
  const int64_t per_cu = p->k == 64 ? 2 : 3;
  const unsigned grid = (unsigned)(tiles < (int64_t)ctx->num_cu * per_cu ? tiles : (int64_t)ctx->num_cu * per_cu);
  const float *W = p->w;
  switch (p->k) {
    case 8:
      OPEN_LAUNCH(ctx, "mlp_infer", k_mlp_infer<8>, dim3(grid), dim3(256), 0, m, row_ptr, col, val, p->n, p->w1p,
                  W + p->off_b1, p->w2p, W + p->off_b2, p->w3p, W + p->off_b3, F, tau, U_out, r, f);
      break;
    case 16:
      OPEN_LAUNCH(ctx, "mlp_infer", k_mlp_infer<16>, dim3(grid), dim3(256), 0, m, row_ptr, col, val, p->n, p->w1p,
                  W + p->off_b1, p->w2p, W + p->off_b2, p->w3p, W + p->off_b3, F, tau, U_out, r, f);
      break;
    case 32:
      OPEN_LAUNCH(ctx, "mlp_infer", k_mlp_infer<32>, dim3(grid), dim3(256), 0, m, row_ptr, col, val, p->n, p->w1p,
                  W + p->off_b1, p->w2p, W + p->off_b2, p->w3p, W + p->off_b3, F, tau, U_out, r, f);
      break;
    default:
      OPEN_LAUNCH(ctx, "mlp_infer", k_mlp_infer<64>, dim3(grid), dim3(256), 0, m, row_ptr, col, val, p->n, p->w1p,
                  W + p->off_b1, p->w2p, W + p->off_b2, p->w3p, W + p->off_b3, F, tau, U_out, r, f);
      break;
  }
  // re-solve the flagged rows with the ridge fold-in (only they are bucketed)
  RowRef *list;
  int64_t *cls;
  if (small_batch(ctx, p->n, p->k, m)) {
    if ((st = small_batch_launch(ctx, F, p->n, p->k, row_ptr, col, val, f, lambda, weighted, U_out, nullptr, m)))
      return st;
  } else if ((st = bucket_rows(ctx, m, row_ptr, p->n, p->k, &list, &cls, INT64_MAX, f)) ||
             (st = rowsolve_launch(ctx, F, p->n, p->k, row_ptr, col, val, lambda, weighted, list, cls, U_out, nullptr,
                                   m))) {
    return st;
  }
  if (n_fallback) {
    OPEN_LAUNCH(ctx, "mlp_count_fallback", k_count_u8, dim3(256), dim3(256), 0, m, f, p->cnt);
    int64_t *h;
    if ((st = pinned_get(ctx, sizeof(int64_t) * 256, (void **)&h))) return st;
    OPEN_HIP_TRY(ctx, hipMemcpyAsync(h, p->cnt, sizeof(int64_t) * 256, hipMemcpyDeviceToHost, ctx->stream));
    OPEN_HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
    int64_t s = 0;
    for (int i = 0; i < 256; ++i) s += h[i];
    *n_fallback = s;
  }
  return OPEN_OK;
}

}  // extern "C"
