// Neural collaborative filtering fold-in (Section III-B.1 model, Section III-B.2 online
// imputation): each new application's embedding e is learned with the setting embeddings and
// the network frozen, by `steps` steps of gradient descent from e = 0 on
//   L(e) = (1/q) sum_j (y(e, s_j) - r_j)^2 + mu |e|^2,
//   y(e, s) = w3 . SELU(W2 SELU(W1 [e; s] + b1) + b2) + b3,   d = 32, 64 hidden units.
//
// The setting half of the first layer is the same for every application and every step, so
// a table C[j] = W1[:, d:] s_j + b1 (n x 64) is built once per call; a step then needs only
// a = W1[:, :d] e, and a setting's first pre-activation is a + C[j].
#include <math.h>

#include <new>

#include "common.h"
#include "mlp_net.h"
#include "wgrad.h"

namespace openk {

constexpr int kNcfD = 32, kNcfH = 64;
constexpr int kNcfMaxSteps = 100000;  // bounds a launch's run time
constexpr int kNcfTwoPairs = 24;     // applications per CU above which a wavefront takes two pairs

// both sides computed and selected: as branches, the 64 evaluations of a tile run one after the other
__device__ __forceinline__ void selu_and_grad(float z, float &h, float &dh) {
  const float ez = __expf(z);
  const float hn = kSeluL * kSeluA * (ez - 1.f), dn = kSeluL * kSeluA * ez;
  const float hp = kSeluL * z;
  const bool pos = z > 0.f;
  h = pos ? hp : hn;
  dh = pos ? kSeluL : dn;
}

// C[j][l] = b1[l] + sum_k W1[l][d + k] S[j][k]
__global__ void k_ncf_table(const float *__restrict__ S, int n, const float *__restrict__ W1,
                            const float *__restrict__ b1, float *__restrict__ C) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)n * kNcfH) return;
  const int j = (int)(t / kNcfH), l = (int)(t % kNcfH);
  float acc = b1[l];
  for (int k = 0; k < kNcfD; ++k) acc = __builtin_fmaf(W1[l * 2 * kNcfD + kNcfD + k], S[(int64_t)j * kNcfD + k], acc);
  C[t] = acc;
}

// Observation tiles on FP32 MFMA (v_mfma_f32_32x32x2f32), 32 columns to a tile; the MFMA keeps
// columns apart, so each column simply carries its own application's embedding.  Every 32 x 32
// result holds, in register v of lane (j, g), row 8 (v/4) + 4 g + v%4 of its block; hidden unit
// U(b, v, g) = 32 b + that row, embedding index K(v, g) = that row.  Each product's contraction
// index is ordered so that its B operand is a register the lane already holds:
//   a   = W1e e         (64 x 32):  step s, half g <-> embedding K(s, g)   (e kept as e[K(v, g)])
//   Z2  = W2 H1         (64 x 64):  step t, half g <-> hidden U(t/16, t%16, g)
//   dH1 = W2^T dZ2      (64 x 64):  step t, half g <-> layer-2 unit U(t/16, t%16, g)
//   DE  = W1e^T dZ1     (32 x 64):  step t, half g <-> hidden U(t/16, t%16, g)
// so activations never move between lanes.  The A operands depend on the lane only and sit in
// LDS once per block, slot-major so that consecutive lanes read consecutive 16-byte words.
// DE's columns (observations) are summed across each application's 16 lanes of a half.
//
// Columns.  A wavefront takes NP pairs of applications of about the same length.  A pair's tile
// holds 16 observations of each of its two (lane j = l % 32 is column j, g = l / 32 the half).
// With NP = 2 a last part of at most 8 observations per application shares one tile among all
// four: in each half of 16 columns, columns 0..7 belong to the first pair's application and
// 8..15 to the second's.  a is computed once, in that shared layout, and a pair's tile takes it
// from column 0 or 8 of each half as it adds it to the table row.
// Bound by the matrix cores and the vector ALU, which share their time on FP32 products: a
// 32 x 32 x 2 product next to 16 independent FMAs takes 109 cycles, 66 and 45 alone.  Per step
// and four applications that is 160 products a tile and 32 for a: 192 up to 8 observations, 352
// up to 16, 512 up to 24, where two wavefronts of one pair each need 384, 384 and 704; SELU is
// evaluated once per unit, its derivative kept in the register of its argument.  65,536
// applications of 4..24 observations, 30 steps: 10.2 -> 7.3 ms, 68 % of the time in products.
constexpr int kNcfTA = 0, kNcfTF = 8, kNcfTB = 24, kNcfTE = 40, kNcfTW3 = 48, kNcfTB2 = 56, kNcfTSlots = 64;

__device__ __forceinline__ f16 mfma32(float a, float b, f16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ int ncf_row(int v, int g) { return 8 * (v >> 2) + 4 * g + (v & 3); }

// lane moves within a row of 16 lanes
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E;                // quad_perm
constexpr int kDppHalfMirror = 0x141, kDppMirror = 0x140;
constexpr int kDppRor8 = 0x128, kDppBcast = 0x150;             // + column
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float x) {
  const int i = __builtin_bit_cast(int, x);
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(i, i, CTRL, 0xf, 0xf, true));
}
// the sum over 8 and over 16 lanes, pairing lanes 1, 2, 4 and 8 apart (the mirrors meet the same
// partial sums as those, since lanes already summed hold equal values)
__device__ __forceinline__ float sum8(float x) {
  x += dpp_mov<kDppXor1>(x);
  x += dpp_mov<kDppXor2>(x);
  x += dpp_mov<kDppHalfMirror>(x);
  return x;
}
__device__ __forceinline__ float sum16(float x) {
  x = sum8(x);
  x += dpp_mov<kDppMirror>(x);
  return x;
}

// `hi` from 8 lanes on, in the banks of four lanes of BANKS, `lo` in the others
template <int BANKS>
__device__ __forceinline__ float ror8_into(float lo, float hi) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, lo),
                                                               __builtin_bit_cast(int, hi), kDppRor8, 0xf, BANKS,
                                                               false));
}

template <int NP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_ncf_foldin(
    int64_t m, const RowRef *__restrict__ list, const int32_t *__restrict__ col, const float *__restrict__ val, int n,
    const float *__restrict__ C, const float *__restrict__ W1, const float *__restrict__ W2,
    const float *__restrict__ b2, const float *__restrict__ w3, const float *__restrict__ b3, int steps, float eta,
    float mu, float *__restrict__ E, float *__restrict__ Lout, int32_t *__restrict__ status) {
  // tab[slot][lane]: per-lane operands, four floats per slot
  __shared__ f4 tab[kNcfTSlots][kWave];
  {
    const int l = threadIdx.x & 63, j = l & 31, g = l >> 5;
    auto put = [&](int slot, int q, float x) { reinterpret_cast<float *>(&tab[slot + q / 4][l])[q & 3] = x; };
    for (int q = threadIdx.x >> 6; q < 32; q += 4) {
      const int b = q >> 4, u = 32 * b + ncf_row(q & 15, g);
      // a = W1e e: A[b][s] = W1e[32 b + j][K(s, g)]
      put(kNcfTA, q, W1[(32 * b + j) * 2 * kNcfD + ncf_row(q & 15, g)]);
      // Z2 = W2 H1: A[ob][t] = W2[32 ob + j][U(t)], and dH1 = W2^T dZ2: A[b][t] = W2[U(t)][32 b + j]
#pragma unroll
      for (int ob = 0; ob < 2; ++ob) {
        put(kNcfTF, 32 * ob + q, W2[(32 * ob + j) * kNcfH + u]);
        put(kNcfTB, 32 * ob + q, W2[u * kNcfH + 32 * ob + j]);
      }
      // DE = W1e^T dZ1: A[t] = W1e[U(t)][j]
      put(kNcfTE, q, W1[u * 2 * kNcfD + j]);
      // w3 and b2 at this lane's rows
      put(kNcfTW3, q, w3[u]);
      put(kNcfTB2, q, b2[u]);
    }
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, jl = lane & 31, g = lane >> 5;
  const float bias3 = b3[0];
  // The table reads go through an offset the compiler cannot see through, renewed every tile,
  // so that it reads the operands from LDS where they are used instead of holding all 256 in
  // registers.
  int toff = 0;
  auto T = [&](int slot, int q) {
    return reinterpret_cast<const float *>(&tab[0][0])[((slot + q / 4) * kWave + lane + toff) * 4 + (q & 3)];
  };

  // columns 0..15 of a tile belong to the first application of a pair, 16..31 to the second;
  // `second`: a column of the second pair in the shared layout
  const int half = jl >> 4, jc = jl & 15;
  const bool second = NP == 2 && jc >= 8;
  const uint64_t appmask = 0x0000ffff0000ffffull << (16 * half);
  const int64_t ngroups = (m + 2 * NP - 1) / (2 * NP);
  const int64_t nw = (int64_t)gridDim.x * (blockDim.x >> 6);
  // the last of the list, where the applications with the most tiles are, first
  for (int64_t gr = ngroups - 1 - ((int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)); gr >= 0; gr -= nw) {
    // the application of this lane's columns in each pair's tiles: its entries, cnt = 0 of them
    // where it is refused
    int64_t beg[NP];
    int cnt[NP], st[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const int64_t li = 2 * NP * gr + 2 * p + half;  // an entry of the size-ordered list
      const RowRef rec = li < m ? list[li] : RowRef{0, 0, 0};
      beg[p] = rec.beg;
      st[p] = rec.cnt <= 0 ? 1 : 0;
      bool bad_idx = false, bad_val = false;
      for (int t = jc + 16 * g; st[p] == 0 && t < rec.cnt; t += 32) {
        const int j = col[beg[p] + t];
        bad_idx = bad_idx || j < 0 || j >= n;
        bad_val = bad_val || !__builtin_isfinite(val[beg[p] + t]);
      }
      if (st[p] == 0 && (__ballot(bad_idx) & appmask)) st[p] = 5;
      else if (st[p] == 0 && (__ballot(bad_val) & appmask)) st[p] = 3;
      cnt[p] = st[p] == 0 ? rec.cnt : 0;
    }
    int qm = max(cnt[0], cnt[NP - 1]);
    qm = __builtin_amdgcn_readfirstlane(max(qm, __shfl_xor(qm, 16, kWave)));
    // tiles of 16 observations per application in each pair, then the shared one
    const int shared = NP == 2 && (qm & 15) >= 1 && (qm & 15) <= 8 ? 1 : 0;
    const int full = (qm >> 4) + ((qm & 15) && !shared ? 1 : 0);
    const int ntiles = NP * full + shared;
    const int cnt_own = second ? cnt[NP - 1] : cnt[0];
    const bool live_own = cnt_own > 0;
    float e[16];  // e[v] = embedding K(v, g) of this column's application in the shared layout
#pragma unroll
    for (int v = 0; v < 16; ++v) e[v] = 0.f;
    float lossv = 0.f;
    for (int it = 0; ntiles > 0 && it <= steps; ++it) {
      // a at this lane's hidden units
      asm volatile("" : "+v"(toff));
      f16 a[2] = {};
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int s2 = 0; s2 < 16; ++s2) a[b] = mfma32(T(kNcfTA, 16 * b + s2), e[s2], a[b]);
      // sums of the tiles under way, and those set aside: the first pair's, then, under the shared
      // tile, both pairs' columns 8..15 (the second's in lanes 0..7)
      f16 de = {}, aside = {};
      float sq = 0.f, sq_aside = 0.f;
      for (int x = 0; x < ntiles; ++x) {
        asm volatile("" : "+v"(toff));
        const int part = x < full ? 0 : x < NP * full ? 1 : 2;  // first pair, second pair, shared
        int64_t t0;
        int t, q;
        if (NP == 2 && part == 2) {
          t0 = second ? beg[NP - 1] : beg[0];
          t = 16 * full + (jc & 7);
          q = cnt_own;
          if (full > 0) {  // the shared columns go on from the pairs' sums
#pragma unroll
            for (int v = 0; v < 16; ++v) {
              const float d1 = de[v];
              de[v] = ror8_into<0xc>(aside[v], d1);
              aside[v] = ror8_into<0x3>(aside[v], d1);
            }
            const float s1 = sq;
            sq = ror8_into<0xc>(sq_aside, s1);
            sq_aside = ror8_into<0x3>(sq_aside, s1);
          }
        } else {
          if (NP == 2 && x == full) {
            aside = de;
            sq_aside = sq;
            de = f16{};
            sq = 0.f;
          }
          t0 = part ? beg[NP - 1] : beg[0];
          t = 16 * (x - part * full) + jc;
          q = part ? cnt[NP - 1] : cnt[0];
        }
        const bool valid = t < q;
        const float *crow = C + (int64_t)(valid ? col[t0 + t] : 0) * kNcfH;
        const float r = valid ? val[t0 + t] : 0.f;
        // forward: Z2 = b2 + W2 SELU(a + c)
        f16 z2[2];
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int v = 0; v < 16; ++v) z2[b][v] = T(kNcfTB2, 16 * b + v);
        float cz[32];
#pragma unroll
        for (int q2 = 0; q2 < 32; ++q2) cz[q2] = crow[32 * (q2 >> 4) + ncf_row(q2 & 15, g)];
        if (NP == 1 || part == 2) {
#pragma unroll
          for (int q2 = 0; q2 < 32; ++q2) cz[q2] += a[q2 >> 4][q2 & 15];
        } else if (part == 0) {
#pragma unroll
          for (int q2 = 0; q2 < 32; ++q2) cz[q2] += dpp_mov<kDppBcast>(a[q2 >> 4][q2 & 15]);
        } else {
#pragma unroll
          for (int q2 = 0; q2 < 32; ++q2) cz[q2] += dpp_mov<kDppBcast + 8>(a[q2 >> 4][q2 & 15]);
        }
#pragma unroll
        for (int q2 = 0; q2 < 32; ++q2) {
          float h1;
          selu_and_grad(cz[q2], h1, cz[q2]);  // cz now holds SELU'(z1)
#pragma unroll
          for (int ob = 0; ob < 2; ++ob) z2[ob] = mfma32(T(kNcfTF, 32 * ob + q2), h1, z2[ob]);
        }
        // the derivatives are computed here and not where they are used: that would keep the 64
        // comparisons instead
#pragma unroll
        for (int q2 = 0; q2 < 32; ++q2) asm volatile("" : "+v"(cz[q2]));
        // output and residual of this column's observation (each half holds half of the sum)
        float yp = 0.f;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            float h2, d2;
            selu_and_grad(z2[b][v], h2, d2);
            z2[b][v] = d2;  // z2 now holds SELU'(z2)
            yp = __builtin_fmaf(T(kNcfTW3, 16 * b + v), h2, yp);
          }
#pragma unroll
        for (int q2 = 0; q2 < 32; ++q2) {
          float d2 = z2[q2 >> 4][q2 & 15];
          asm volatile("" : "+v"(d2));
          z2[q2 >> 4][q2 & 15] = d2;
        }
        const float y = yp + __shfl_xor(yp, 32, kWave) + bias3;
        const float res = valid ? y - r : 0.f;
        sq = __builtin_fmaf(res, res, sq);
        if (it == steps) continue;  // the last pass only evaluates the loss
        // backward: dH1 = W2^T dZ2, dZ2 = (2 res / q) w3 SELU'(z2)
        const float dy = 2.f * res * (q > 0 ? 1.f / (float)q : 0.f);
        f16 dh1[2] = {};
#pragma unroll
        for (int q2 = 0; q2 < 32; ++q2) {
          const float dz2 = dy * T(kNcfTW3, q2) * z2[q2 >> 4][q2 & 15];
#pragma unroll
          for (int b = 0; b < 2; ++b) dh1[b] = mfma32(T(kNcfTB, 32 * b + q2), dz2, dh1[b]);
        }
        // DE += W1e^T (dH1 * SELU'(a + c))
#pragma unroll
        for (int q2 = 0; q2 < 32; ++q2) de = mfma32(T(kNcfTE, q2), dh1[q2 >> 4][q2 & 15] * cz[q2], de);
      }
      // the squared residuals and DE summed over each application's 16 columns: the pairs' own
      // columns, the first 8 of them as the shared tile left them
      const bool alone = shared && full == 0;  // the shared tile is all there is
      auto first_of = [&](float d, float as) { return shared && !second ? d : as; };
      auto second_of = [&](float d, float as) { return shared ? dpp_mov<kDppRor8>(second ? d : as) : d; };
      if (it == steps) {
        float ee = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) ee = __builtin_fmaf(e[v], e[v], ee);
        // squared residuals: one per column in each half; embedding: each half holds 16 indices
        float sqt;
        if (NP == 1) {
          sqt = sum16(g == 0 ? sq : 0.f);
        } else if (alone) {
          sqt = sum8(g == 0 ? sq : 0.f);
        } else {
          const float s0 = sum16(g == 0 ? first_of(sq, sq_aside) : 0.f);
          const float s1 = sum16(g == 0 ? second_of(sq, sq_aside) : 0.f);
          sqt = second ? s1 : s0;
        }
        const float iq = live_own ? 1.f / (float)cnt_own : 0.f;
        lossv = sqt * iq + mu * (ee + __shfl_xor(ee, 32, kWave));
        break;
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        float s;
        if (NP == 1) {
          s = sum16(de[v]);
        } else if (alone) {
          s = sum8(de[v]);
        } else {
          const float s0 = sum16(first_of(de[v], aside[v])), s1 = sum16(second_of(de[v], aside[v]));
          s = second ? s1 : s0;
        }
        if (live_own) e[v] -= eta * (s + 2.f * mu * e[v]);
      }
    }
    const int64_t li = 2 * NP * gr + 2 * (second ? 1 : 0) + half;
    if (li < m && (jc & (NP == 2 ? 7 : 15)) == 0) {
      const int64_t i = list[li].row;
#pragma unroll
      for (int v = 0; v < 16; ++v) E[i * kNcfD + ncf_row(v, g)] = e[v];
      if (g == 0) {
        if (Lout) Lout[i] = live_own ? lossv : 0.f;
        if (status) status[i] = second ? st[NP - 1] : st[0];
      }
    }
  }
}

// ---------------------------------------------------------------- offline training
// The model is trained on the dense offline matrix R (applications x settings, every entry
// observed) in batches of whole applications: batch row b = g n + j pairs application
// apps[g] with setting j.  A step is two launches: k_ncf_fwd_bwd takes R rows per block (one
// wavefront per 32 of the 64 hidden units) through the forward and backward pass on
// v_mfma_f32_32x32x16_bf16 with the activations in LDS and registers, and wgrad_step contracts
// the weight gradients over the batch, sums the embedding gradients in order and applies Adam.
// Bound by launch and load latency: 3840 rows are 0.2 GFLOP.  At 8 x 480: 12 us, and 18 us for
// the second launch; a step takes 37 us against 250 us as sixteen launches, of which the
// embedding sums took 129 (one thread per sum, each read waited for).
struct NcfBatch {
  int64_t B;                 // batch rows, G n
  int G, n;
  const int64_t *apps;       // the batch's applications, from apps + st->cursor * G with use_cursor
  int use_cursor;
  const float *E, *S, *W1, *b1, *W2, *b2, *w3, *b3, *R;
  uint16_t *X, *h1, *h2, *d1p, *d2p, *dyp;  // packed operands, 64 (dyp: 32) wide
  float *d1, *d2, *dy, *dX;                 // output gradients and the input gradient
  double *lpart;             // one per block
  int64_t *apps_out, *mark;  // the batch's applications and their step tag, for wgrad_step
  TrainState *st;
};

// this lane's B operands of a 64 x 64 weight matrix, output tile w, four steps of k; T: of its
// transpose
template <bool T>
__device__ __forceinline__ void load_operand(uint4 (&bw)[4], const float *__restrict__ W, int w, int i32, int g) {
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int o = 32 * w + i32, i = 16 * ks + 8 * g + e;
      x[e] = T ? W[i * 64 + o] : W[o * 64 + i];
    }
    bw[ks] = uint4{bf16pack(x[0], x[1]), bf16pack(x[2], x[3]), bf16pack(x[4], x[5]), bf16pack(x[6], x[7])};
  }
}

template <int R>
__global__ __launch_bounds__(128) void k_ncf_fwd_bwd(NcfBatch p) {
  constexpr int P = 64 + 8, NV = R / 2;  // LDS pitch (bfloat16), result registers in use
  __shared__ __attribute__((aligned(16))) uint16_t Xs[R * P];   // the inputs, then dz2
  __shared__ __attribute__((aligned(16))) uint16_t Hs[R * P];   // h1, then dz1
  __shared__ __attribute__((aligned(16))) uint16_t H2[R * P];
  __shared__ float dys[R];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, i32 = lane & 31, g = lane >> 5;
  const int64_t b0 = (int64_t)blockIdx.x * R;
  const int64_t *apps = p.apps + (p.use_cursor ? p.st->cursor * p.G : 0);
  const int u = 32 * w + i32, ar = i32 & (R - 1);
  uint4 bw[4], bw2[4];
  load_operand<false>(bw, p.W1, w, i32, g);
  load_operand<false>(bw2, p.W2, w, i32, g);
  // ---- the inputs [e ; s], eight values per thread and round
#pragma unroll
  for (int t = tid; t < R * 8; t += 128) {
    const int lr = t >> 3, c = (t & 7) * 8;
    const int64_t b = b0 + lr;
    uint4 v = uint4{0u, 0u, 0u, 0u};
    if (b < p.B) {
      const int64_t a = b / p.n, j = b - a * p.n;
      // the parameter vector's arrays start at any multiple of four bytes
      const float *src = c < kNcfD ? p.E + apps[a] * kNcfD + c : p.S + j * kNcfD + (c - kNcfD);
      v = uint4{bf16pack(src[0], src[1]), bf16pack(src[2], src[3]), bf16pack(src[4], src[5]),
                bf16pack(src[6], src[7])};
    }
    *reinterpret_cast<uint4 *>(Xs + lr * P + c) = v;
  }
  __syncthreads();
  for (int e = tid; e < R / 8 * 64; e += 128)
    reinterpret_cast<uint4 *>(p.X)[b0 / 8 * 64 + e] = gather_pack8(Xs + (e >> 6) * 8 * P + (e & 63), P);
  // ---- forward: z1, z2 of hidden unit u for rows 8 (v / 4) + 4 g + v % 4
  float s1[NV], s2[NV], hv[NV];  // SELU' of both layers
  f16 acc = {};
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
    acc = mfma_bf16_32(*reinterpret_cast<const uint4 *>(Xs + ar * P + 16 * ks + 8 * g), bw[ks], acc);
  float bias = p.b1[u];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int lr = 8 * (v / 4) + 4 * g + (v % 4);
    const float z = acc[v] + bias;
    s1[v] = selu_grad(z);
    hv[v] = b0 + lr < p.B ? selu(z) : 0.f;
    Hs[lr * P + u] = f2bf(hv[v]);
  }
#pragma unroll
  for (int q = 0; q < R / 8; ++q) store_pack4(p.h1, b0 / 8 + q, 64, u, g, hv + 4 * q);
  __syncthreads();
  acc = f16{};
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
    acc = mfma_bf16_32(*reinterpret_cast<const uint4 *>(Hs + ar * P + 16 * ks + 8 * g), bw2[ks], acc);
  bias = p.b2[u];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int lr = 8 * (v / 4) + 4 * g + (v % 4);
    const float z = acc[v] + bias;
    s2[v] = selu_grad(z);
    hv[v] = b0 + lr < p.B ? selu(z) : 0.f;
    H2[lr * P + u] = f2bf(hv[v]);
  }
#pragma unroll
  for (int q = 0; q < R / 8; ++q) store_pack4(p.h2, b0 / 8 + q, 64, u, g, hv + 4 * q);
  load_operand<true>(bw2, p.W2, w, i32, g);  // for the backward pass
  load_operand<true>(bw, p.W1, w, i32, g);
  __syncthreads();
  // ---- output and loss: w3 as column 0 of the product, on the first wavefront
  if (w == 0) {
    acc = f16{};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const float *s = p.w3 + 16 * ks + 8 * g;
      uint4 b = uint4{0u, 0u, 0u, 0u};
      if (i32 == 0)
        b = uint4{bf16pack(s[0], s[1]), bf16pack(s[2], s[3]), bf16pack(s[4], s[5]), bf16pack(s[6], s[7])};
      acc = mfma_bf16_32(*reinterpret_cast<const uint4 *>(H2 + ar * P + 16 * ks + 8 * g), b, acc);
    }
    const float scale = 2.0f / (float)p.B;
    double sq = 0.0;
    float dv[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const int lr = 8 * (v / 4) + 4 * g + (v % 4);
      const int64_t b = b0 + lr;
      dv[v] = 0.f;
      if (i32 == 0) {
        if (b < p.B) {
          const int64_t a = b / p.n;
          const float d = (acc[v] + p.b3[0]) - p.R[apps[a] * p.n + (b - a * p.n)];
          dv[v] = scale * d;
          p.dy[b] = dv[v];
          sq += (double)d * (double)d;
        }
        dys[lr] = dv[v];
      }
    }
#pragma unroll
    for (int q = 0; q < R / 8; ++q) store_pack4(p.dyp, b0 / 8 + q, 32, i32, g, dv + 4 * q);
    sq += __shfl_xor(sq, 32, 64);
    if (lane == 0) p.lpart[blockIdx.x] = sq;
  }
  __syncthreads();
  // ---- backward: dz2 = (dy w3) SELU'(z2), the factors rounded as in a product
  const float w3u = bf2f(f2bf(p.w3[u]));
  float dz[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int lr = 8 * (v / 4) + 4 * g + (v % 4);
    dz[v] = (bf2f(f2bf(dys[lr])) * w3u) * s2[v];
    if (b0 + lr < p.B) p.d2[(b0 + lr) * 64 + u] = dz[v];
    Xs[lr * P + u] = f2bf(dz[v]);
  }
#pragma unroll
  for (int q = 0; q < R / 8; ++q) store_pack4(p.d2p, b0 / 8 + q, 64, u, g, dz + 4 * q);
  __syncthreads();
  // dz1 = (dz2 W2) SELU'(z1)
  acc = f16{};
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
    acc = mfma_bf16_32(*reinterpret_cast<const uint4 *>(Xs + ar * P + 16 * ks + 8 * g), bw2[ks], acc);
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int lr = 8 * (v / 4) + 4 * g + (v % 4);
    dz[v] = acc[v] * s1[v];
    if (b0 + lr < p.B) p.d1[(b0 + lr) * 64 + u] = dz[v];
    Hs[lr * P + u] = f2bf(dz[v]);
  }
#pragma unroll
  for (int q = 0; q < R / 8; ++q) store_pack4(p.d1p, b0 / 8 + q, 64, u, g, dz + 4 * q);
  __syncthreads();
  // dX = dz1 W1
  acc = f16{};
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
    acc = mfma_bf16_32(*reinterpret_cast<const uint4 *>(Hs + ar * P + 16 * ks + 8 * g), bw[ks], acc);
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int lr = 8 * (v / 4) + 4 * g + (v % 4);
    if (b0 + lr < p.B) p.dX[(b0 + lr) * 64 + u] = acc[v];
  }
  if (blockIdx.x == 0) {
    for (int a = tid; a < p.G; a += 128) {
      p.apps_out[a] = apps[a];
      p.mark[apps[a]] = p.st->t + 1;
    }
    __syncthreads();
    if (tid == 0) train_state_begin(p.st);
  }
}

// Parameter packing of the trained model (float32): E (m_off x d), S (n x d), W1 (H x 2d),
// b1 (H), W2 (H x H), b2 (H), w3 (H), b3 (1).
struct NcfLayout {
  int64_t E, S, W1, b1, W2, b2, w3, b3, total;
  NcfLayout(int64_t m_off, int64_t n) {
    E = 0;
    S = E + m_off * kNcfD;
    W1 = S + n * kNcfD;
    b1 = W1 + (int64_t)kNcfH * 2 * kNcfD;
    W2 = b1 + kNcfH;
    b2 = W2 + (int64_t)kNcfH * kNcfH;
    w3 = b2 + kNcfH;
    b3 = w3 + kNcfH;
    total = b3 + 1;
  }
};

// Whether the bias gradients' sums have a launch of their own (wgrad.hip): in large batches they are the
// second launch's longest chain, unless a few applications' sums over very many settings are.  A
// step of the training, us, in one launch / apart: 512 applications x 480 settings 1410 / 1060, 34 x
// 480 117 / 88, 5 x 1920 72 / 59, 18 x 480 70 / 58, 3 x 4096 84 / 79, but 2 x 4096 73 / 78, 1 x 10,000
// 126 / 131, and of few rows 24 x 120 33.7 / 33.2, 16 x 120 28.7 / 31.8, 4 x 120 25 / 29.
static bool bias_apart(int G, int n) { return G >= 4 && (int64_t)G * n > 8192; }

// Device buffers of one training call.
struct NcfTrainBufs {
  uint16_t *X = nullptr, *h1 = nullptr, *h2 = nullptr, *d1p = nullptr, *d2p = nullptr, *dyp = nullptr;
  float *d1 = nullptr, *d2 = nullptr, *dy = nullptr, *dX = nullptr, *g = nullptr, *am = nullptr, *av = nullptr;
  double *lpart = nullptr, *loss = nullptr;
  int64_t *apps = nullptr, *mark = nullptr;
  TrainState *st = nullptr;
  float *bias = nullptr;  // bias_apart
  void release() {
    for (uint16_t *q : {X, h1, h2, d1p, d2p, dyp}) (void)hipFree(q);
    for (float *q : {d1, d2, dy, dX, g, am, av, bias}) (void)hipFree(q);
    for (int64_t *q : {apps, mark}) (void)hipFree(q);
    (void)hipFree(lpart);
    (void)hipFree(loss);
    (void)hipFree(st);
  }
  // G n batch rows, np parameters; training: Adam moments, otherwise the gradient
  bool alloc(int64_t m_off, int G, int n, int64_t np, bool train) {
    const size_t Bp = (size_t)pad_rows((int64_t)G * n), h = sizeof(uint16_t) * Bp * kNcfH;
    const size_t f = sizeof(float) * Bp * kNcfH, pb = sizeof(float) * (size_t)np;
    const bool ok = !hipMalloc(&X, h) && !hipMalloc(&h1, h) && !hipMalloc(&h2, h) && !hipMalloc(&d1p, h) &&
                    !hipMalloc(&d2p, h) && !hipMalloc(&dyp, h / 2) && !hipMalloc(&d1, f) && !hipMalloc(&d2, f) &&
                    !hipMalloc(&dy, sizeof(float) * Bp) && !hipMalloc(&dX, f) &&
                    (train ? !hipMalloc(&am, pb) && !hipMalloc(&av, pb) : !hipMalloc(&g, pb)) &&
                    !hipMalloc(&lpart, sizeof(double) * (Bp / 16)) && !hipMalloc(&loss, sizeof(double) * 8) &&
                    !hipMalloc(&apps, sizeof(int64_t) * (size_t)G) &&
                    !hipMalloc(&mark, sizeof(int64_t) * (size_t)m_off) && !hipMalloc(&st, sizeof(TrainState)) &&
                    (!bias_apart(G, n) ||
                     !hipMalloc(&bias, sizeof(float) * kWgBiasPart * (2 * kNcfH / 32 + 1)));
    if (!ok) (void)hipGetLastError();
    return ok;
  }
};

// no application is in a batch yet; the step state starts over
static open_status ncf_train_begin(open_ctx *ctx, NcfTrainBufs &b, int64_t m_off) {
  OPEN_LAUNCH(ctx, "fill", k_fill_i32, dim3(64), dim3(256), 0, (int *)b.mark, 2 * m_off, 0);
  return dense_train_state_reset(ctx, b.st);
}

// Loss and gradient of one batch of G applications (apps on the device, from the cursor's batch
// with use_cursor): the Adam step with lr > 0, the gradient in b.g otherwise; the loss to b.loss
// and, when given, to loss_steps[t].
static open_status ncf_step(open_ctx *ctx, const NcfLayout &L, int64_t m_off, int n, const float *R, float *P,
                            const int64_t *apps, int use_cursor, int G, NcfTrainBufs &b, float lr,
                            float *loss_steps) {
  const int64_t B = (int64_t)G * n;
  NcfBatch k = {};
  k.B = B;
  k.G = G;
  k.n = n;
  k.apps = apps;
  k.use_cursor = use_cursor;
  k.E = P + L.E;
  k.S = P + L.S;
  k.W1 = P + L.W1;
  k.b1 = P + L.b1;
  k.W2 = P + L.W2;
  k.b2 = P + L.b2;
  k.w3 = P + L.w3;
  k.b3 = P + L.b3;
  k.R = R;
  k.X = b.X;
  k.h1 = b.h1;
  k.h2 = b.h2;
  k.d1p = b.d1p;
  k.d2p = b.d2p;
  k.dyp = b.dyp;
  k.d1 = b.d1;
  k.d2 = b.d2;
  k.dy = b.dy;
  k.dX = b.dX;
  k.lpart = b.lpart;
  k.apps_out = b.apps;
  k.mark = b.mark;
  k.st = b.st;
  // rows per block: 16 where blocks of 32 would not cover the compute units
  const int rows = B <= 16 * (int64_t)ctx->num_cu ? 16 : 32;
  const unsigned blocks = (unsigned)(pad_rows(B) / rows);
  if (rows == 16) {
    OPEN_LAUNCH(ctx, "ncf_fwd_bwd", k_ncf_fwd_bwd<16>, dim3(blocks), dim3(128), 0, k);
  } else {
    OPEN_LAUNCH(ctx, "ncf_fwd_bwd", k_ncf_fwd_bwd<32>, dim3(blocks), dim3(128), 0, k);
  }
  WgradStep w = {};
  w.l[0] = {b.d1p, b.X, b.d1, kNcfH, 2 * kNcfD, L.W1};
  w.l[1] = {b.d2p, b.h1, b.d2, kNcfH, kNcfH, L.W2};
  w.l[2] = {b.dyp, b.h2, b.dy, 1, kNcfH, L.w3};
  w.emb.G = G;
  w.emb.n = n;
  w.emb.m = m_off;
  w.emb.dX = b.dX;
  w.emb.apps = b.apps;
  w.emb.mark = b.mark;
  w.emb.e = L.E;
  w.emb.s = L.S;
  w.B = B;
  w.w = P;
  w.g = b.g;
  w.m = b.am;
  w.v = b.av;
  w.lr = lr;
  w.st = b.st;
  w.lpart = b.lpart;
  w.nlpart = (int)blocks;
  w.ltotal = B;
  w.loss_d = b.loss;
  w.loss_steps = loss_steps;
  w.bias = b.bias;
  return wgrad_step(ctx, "ncf_wgrad_adam", w, lr > 0.f);
}

constexpr int64_t kNcfMaxBatch = int64_t(1) << 20;  // batch entries (applications x settings)

static open_status ncf_train_check(open_ctx *ctx, int64_t m_off, int32_t n, int32_t d, const float *R,
                                   const float *params, int64_t G) {
  if (d != kNcfD) return fail(ctx, OPEN_E_UNSUPPORTED, "embedding width must be 32");
  if (m_off < 1 || n < 1 || m_off > INT32_MAX) return fail(ctx, OPEN_E_INVALID, "bad matrix shape");
  if (!R || !params) return fail(ctx, OPEN_E_INVALID, "null pointer");
  if (G < 1 || G > m_off || G * n > kNcfMaxBatch)
    return fail(ctx, OPEN_E_INVALID, "applications per batch must be in [1, m_off] with at most 2^20 entries");
  return OPEN_OK;
}

}  // namespace openk

using namespace openk;

extern "C" int64_t open_ncf_num_params(int64_t m_off, int32_t n) { return NcfLayout(m_off, n).total; }

extern "C" open_status open_ncf_loss_grad(open_ctx *ctx, int64_t m_off, int32_t n, int32_t d, const float *R,
                                          const float *params, const int64_t *apps, int32_t G, double *loss,
                                          float *grads_host) {
  if (!ctx) return OPEN_E_INVALID;
  open_status st = ncf_train_check(ctx, m_off, n, d, R, params, G);
  if (st) return st;
  if (!apps || !loss || !grads_host) return fail(ctx, OPEN_E_INVALID, "null pointer");
  OPEN_HIP_TRY(ctx, hipSetDevice(ctx->device));
  const NcfLayout L(m_off, n);
  NcfTrainBufs b;
  if (!b.alloc(m_off, G, n, L.total, false)) {
    b.release();
    return fail(ctx, OPEN_E_NOMEM, "NCF training buffers");
  }
  st = ncf_train_begin(ctx, b, m_off);
  if (!st) st = ncf_step(ctx, L, m_off, n, R, const_cast<float *>(params), apps, 0, G, b, 0.f, nullptr);
  double *h = nullptr;
  if (!st) st = pinned_get(ctx, 64, (void **)&h);
  if (!st && (hipMemcpyAsync(grads_host, b.g, sizeof(float) * L.total, hipMemcpyDeviceToHost, ctx->stream) ||
              hipMemcpyAsync(h, b.loss, sizeof(double), hipMemcpyDeviceToHost, ctx->stream) ||
              hipStreamSynchronize(ctx->stream)))
    st = fail(ctx, OPEN_E_DEVICE, "reading the gradient");
  if (!st) *loss = h[0];
  (void)hipStreamSynchronize(ctx->stream);
  b.release();
  return st;
}

extern "C" open_status open_ncf_train(open_ctx *ctx, int64_t m_off, int32_t n, int32_t d, const float *R,
                                      float *params, int32_t apps_per_batch, float lr, int32_t epochs, uint64_t seed,
                                      float *loss_hist) {
  if (!ctx) return OPEN_E_INVALID;
  open_status st = ncf_train_check(ctx, m_off, n, d, R, params, apps_per_batch);
  if (st) return st;
  if (epochs < 0 || !(lr > 0.f) || !isfinite(lr)) return fail(ctx, OPEN_E_INVALID, "bad epochs or learning rate");
  if (epochs == 0) return OPEN_OK;
  OPEN_HIP_TRY(ctx, hipSetDevice(ctx->device));
  const NcfLayout L(m_off, n);
  const int G = apps_per_batch;
  const int64_t spe = m_off / G, total = spe * epochs;
  NcfTrainBufs b;
  int64_t *perm = nullptr;
  float *losses = nullptr;
  if (!b.alloc(m_off, G, n, L.total, true) || hipMalloc(&perm, sizeof(int64_t) * m_off) ||
      hipMalloc(&losses, sizeof(float) * total)) {
    (void)hipGetLastError();
    b.release();
    (void)hipFree(perm);
    (void)hipFree(losses);
    return fail(ctx, OPEN_E_NOMEM, "NCF training buffers");
  }
  OPEN_LAUNCH(ctx, "fill", k_fill_i32, dim3(256), dim3(256), 0, (int *)b.am, L.total, 0);
  OPEN_LAUNCH(ctx, "fill", k_fill_i32, dim3(256), dim3(256), 0, (int *)b.av, L.total, 0);
  st = ncf_train_begin(ctx, b, m_off);
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  auto one_step = [&]() -> open_status {
    return ncf_step(ctx, L, m_off, n, R, params, perm, 1, G, b, lr, losses);
  };
  for (int32_t e = 0; e < epochs && st == OPEN_OK; ++e) {
    if ((st = dense_shuffle(ctx, m_off, seed, e, perm, b.st))) break;
    for (int64_t s = 0; s < spe && st == OPEN_OK; ++s) {
      if (!exec) {
        if ((st = one_step())) break;  // the first step runs eagerly, the next one is recorded
        if (s + 1 < spe || e + 1 < epochs) {
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
          for (int64_t s = 0; s < spe; ++s) sum += hl[e * spe + s];
          loss_hist[e] = (float)(sum / (double)spe);
        }
      }
      delete[] hl;
    }
  }
  (void)hipStreamSynchronize(ctx->stream);
  b.release();
  (void)hipFree(perm);
  (void)hipFree(losses);
  return st;
}

extern "C" open_status open_ncf_foldin(open_ctx *ctx, const float *S, int32_t n, int32_t d, const float *W1,
                                       const float *b1, const float *W2, const float *b2, const float *w3,
                                       const float *b3, int64_t m, const int64_t *row_ptr, const int32_t *col,
                                       const float *val, int32_t steps, float eta, float mu, float *E_out,
                                       float *loss_out, int32_t *row_status) {
  if (!ctx) return OPEN_E_INVALID;
  if (d != kNcfD) return fail(ctx, OPEN_E_UNSUPPORTED, "embedding width must be 32");
  if (n < 1 || m < 0 || steps < 0 || steps > kNcfMaxSteps || !(eta == eta) || !(mu == mu))
    return fail(ctx, OPEN_E_INVALID, "bad sizes, steps, eta or mu");
  if (m == 0) return OPEN_OK;
  if (m > INT32_MAX) return fail(ctx, OPEN_E_UNSUPPORTED, "more than 2^31 - 1 rows");
  if (!S || !W1 || !b1 || !W2 || !b2 || !w3 || !b3 || !row_ptr || !col || !val || !E_out)
    return fail(ctx, OPEN_E_INVALID, "null pointer");
  OPEN_HIP_TRY(ctx, hipSetDevice(ctx->device));
  void *tab = nullptr;
  open_status st;
  if ((st = ws_get(ctx, open_ctx::WS_NCF, sizeof(float) * (size_t)n * kNcfH, &tab))) return st;
  const int64_t tt = (int64_t)n * kNcfH;
  OPEN_LAUNCH(ctx, "ncf_table", k_ncf_table, dim3((unsigned)((tt + 255) / 256)), dim3(256), 0, S, n, W1, b1,
              (float *)tab);
  // applications in order of observed count, so that the two of a wavefront need about as
  // many observation tiles
  RowRef *list = nullptr;
  int64_t *cls = nullptr;
  if ((st = bucket_rows(ctx, m, row_ptr, n, kNcfD, &list, &cls, kSplitMin))) return st;
  // two pairs per wavefront once the pairs alone give every SIMD its two wavefronts and more: at
  // 8192 applications of 4..24 observations, 30 steps, 1062 us against 1343, at 6000 1053 against
  // 1081, at 4096 (one wavefront per SIMD, longer) 755 against 648.  Where the last tiles are more than
  // half full only the work on a is shared, and whole rounds of wavefronts decide: with 9..16
  // observations, 10 steps, 317 against 322 us at 6145 applications, 476 against 404 at 10,000 (two
  // rounds of half as many), 612 against 630 at 16,384, 1192 against 1236 at 32,768; with 1..8 180
  // against 320 at 6145.
  const int64_t cap = (int64_t)ctx->num_cu * 64;  // waves, all blocks handed out as they end
  const bool two = m > (int64_t)ctx->num_cu * kNcfTwoPairs;
  const int64_t groups = two ? (m + 3) / 4 : (m + 1) / 2;
  const int64_t waves = groups < cap ? groups : cap;
  OPEN_LAUNCH(ctx, "ncf_foldin", (two ? k_ncf_foldin<2> : k_ncf_foldin<1>), dim3((unsigned)((waves + 3) / 4)),
              dim3(256), 0, m, (const RowRef *)list, col, val, n, (const float *)tab, W1, W2, b2, w3, b3, steps, eta,
              mu, E_out, loss_out, row_status);
  return OPEN_OK;
}
