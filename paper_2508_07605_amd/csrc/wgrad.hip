// Weight gradients, bias gradients and the Adam update of a training step in one launch.
//
// A layer's weight gradient is a contraction over the batch, G[m][n] = sum_b A[b][m] X[b][n].
// The batch is cut into S slices of kc rows; a wavefront sums a slice of a 32 x 32 tile of G on
// v_mfma_f32_32x32x16_bf16 (operands straight from the packed arrays, 16 bytes per lane), and
// the block that owns the tile adds the slices in slice order through LDS, so the result does
// not depend on scheduling.  The thread that ends up with an element updates it: no gradient,
// no partial sum and no separate optimizer pass goes through memory.
//
// Bound by the latency of the operand reads (the other launch of the step wrote them from all
// XCDs, so the first touch misses the L2): every wavefront keeps 12 to 16 loads of 1 KB in
// flight, and the block shapes below keep the launch within one block per CU at batch 4096.
// The blocks of one XCD (dealt round-robin) take the same few input tiles.
//
// At batch 4096 and 960-256-256-32: 18 us (bias sums alone 12, first layer alone 15, an empty
// launch 4); with 16 slices a round, 64 registers and two blocks per CU 23 us.
#include "wgrad.h"
#include "mlp_net.h"

namespace openk {

constexpr int kWgWaves = 16;
constexpr int kWgThreads = 64 * kWgWaves;

// batch slices of an M x N layer: about 1024 / (64 x 64 tiles) of them, at most 256, each a
// multiple of 32 rows
static int wgrad_slices(int64_t B, int M, int N, int *kc) {
  const int64_t tiles = (int64_t)((M + 63) / 64) * ((N + 63) / 64);
  int64_t S = (1024 + tiles - 1) / tiles;
  if (S > 256) S = 256;
  int64_t c = (B + S - 1) / S;
  c = (c + 31) / 32 * 32;
  *kc = (int)c;
  return (int)((B + c - 1) / c);
}

__device__ __forceinline__ float adam_update(const WgradStep &p, int64_t i, float gi, float c1, float c2) {
  const float mi = 0.9f * p.m[i] + 0.1f * gi;
  const float vi = 0.999f * p.v[i] + 0.001f * gi * gi;
  p.m[i] = mi;
  p.v[i] = vi;
  const float wi = p.w[i] - p.lr * (mi / c1) / (sqrtf(vi / c2) + 1e-8f);
  p.w[i] = wi;
  return wi;
}

// Shape of a layer's blocks, by its slice count: NT tiles side by side share the output
// gradients; a block keeps VR of a tile's 16 result registers (16 / VR blocks repeat the
// products), so that 128 KB of LDS hold SL slices and few slices are left to a second round.
//   S <= 16  NT 2, VR 16, 16 slices a round (wide layers: the reads of A are shared)
//   S <= 64  NT 1, VR 16, 32 slices
//   else     NT 1, VR 4, 128 slices (narrow layers: few tiles, many short slices)
constexpr int kWgLdsFloats = 32768;
template <int NT, int VR>
constexpr int wg_slots() { return kWgLdsFloats / (NT * VR * 64); }

// Block q of a layer.
template <bool ADAM, int NT, int VR>
__device__ __forceinline__ void weight_tiles(const WgradStep &p, const WgradLayer &l, int q, float *buf) {
  constexpr int SL = wg_slots<NT, VR>(), U = NT == 2 ? 2 : 4;  // slices a round; 32-row units in flight
  constexpr int PARTS = 16 / VR;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int i32 = lane & 31, g = lane >> 5;
  const int ntm = (l.M + 31) / 32, ntn = (l.N + 31) / 32, Au = 32 * ntm, Xu = 32 * ntn;
  const int mb = (ntm + l.nt - 1) / l.nt * PARTS, ng = (ntn + NT - 1) / NT;
  const int n0 = ((q & 7) + 8 * ((q >> 3) / mb)) * NT, mq = (q >> 3) % mb;
  const int m0 = mq / PARTS * l.nt, v0 = mq % PARTS * VR;
  if (n0 >= ng * NT) return;  // uniform
  const bool two = NT == 2 && n0 + 1 < ntn;
  const int64_t Bp = pad_rows(p.B);
  const int ups = l.kc / 32;                  // units of a slice
  float tot[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) tot[t] = 0.f;
  const int per = l.nt > 1 ? l.S : SL;        // slices summed per round
  for (int r0 = 0; r0 < l.S; r0 += per) {
    // the wavefront's slices of the round: s0, s0 + 16, ...
    const int sub = l.nt > 1 ? w / l.S : 0, s0 = l.nt > 1 ? w % l.S : r0 + w;
    const int send = r0 + per < l.S ? r0 + per : l.S;
    const int ns = sub < l.nt && m0 + sub < ntm && s0 < send ? (l.nt > 1 ? 1 : (send - s0 + 15) / 16) : 0;
    const int units = ns * ups;
    if (r0) __syncthreads();  // the previous round's sums are read
    f16 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = f16{};
    for (int u0 = 0; u0 < units; u0 += U) {
      uint4 a[U][2], x[U][NT][2];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t b = (int64_t)(s0 + 16 * ((u0 + u) / ups)) * l.kc + 32 * ((u0 + u) % ups);
        const bool in = u0 + u < units && b < Bp;  // past the last slice's rows: zeros
        const uint4 *pa = reinterpret_cast<const uint4 *>(l.A) + (b / 8 + g) * Au + 32 * (m0 + sub) + i32;
        const uint4 *px = reinterpret_cast<const uint4 *>(l.X) + (b / 8 + g) * Xu + 32 * n0 + i32;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          a[u][e] = in ? pa[2 * e * Au] : uint4{0u, 0u, 0u, 0u};
#pragma unroll
          for (int t = 0; t < NT; ++t)
            x[u][t][e] = in && (t == 0 || two) ? px[2 * e * Xu + 32 * t] : uint4{0u, 0u, 0u, 0u};
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (u0 + u < units) {
#pragma unroll
          for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[t] = mfma_bf16_32(a[u][e], x[u][t][e], acc[t]);
          if ((u0 + u + 1) % ups == 0) {  // the slice is done: its slot
            float *dst = buf + (w + 16 * ((u0 + u) / ups)) * (NT * VR * 64) + lane;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
#pragma unroll
              for (int v = 0; v < 16; ++v)
                if (PARTS == 1 || v / VR * VR == v0) dst[(t * VR + v % VR) * 64] = acc[t][v];
              acc[t] = f16{};
            }
          }
        }
      }
    }
    __syncthreads();
    // thread (w, lane), w < VR: register v0 + w of lane `lane`, of every tile side by side
    if (w < VR) {
      const int left = l.S - r0 < per ? l.S - r0 : per;
#pragma unroll 4
      for (int i = 0; i < left; ++i) {
#pragma unroll
        for (int t = 0; t < NT; ++t) tot[t] += buf[((i * NT + t) * VR + w) * 64 + lane];
      }
    }
  }
  if (w >= VR) return;
  const float c1 = p.st->c1, c2 = p.st->c2;
  const int vr = v0 + w, mr = 8 * (vr / 4) + 4 * g + (vr % 4);
  for (int s = 0; s < l.nt; ++s) {
    if (s) {  // the block's further tiles (one round: their slices are still in LDS)
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        tot[t] = 0.f;
        for (int i = 0; i < l.S; ++i) tot[t] += buf[(((s * l.S + i) * NT + t) * VR + w) * 64 + lane];
      }
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int m = 32 * (m0 + s) + mr, n = 32 * (n0 + t) + i32;
      if (m >= l.M || n >= l.N) continue;
      const int64_t i = l.w + (int64_t)m * l.N + n;
      if constexpr (!ADAM) {
        p.g[i] = tot[t];
      } else {
        const uint16_t h = f2bf(adam_update(p, i, tot[t], c1, c2));
        if (l.P) l.P[mfma_slot(m, n, (l.N + 15) / 16)] = h;
        if (l.PT) l.PT[mfma_slot(n, m, (l.M + 15) / 16)] = h;
        if (l.pairs) {
          const int half = l.N / 2, mask = n >= half;
          l.pairs[2 * ((int64_t)(n - half * mask) * l.M + m) + mask] = h;
        }
      }
    }
  }
}

// blocks of a layer (kept in step with weight_tiles) and their shape
static void wgrad_shape(WgradLayer &l) {
  const int ntm = (l.M + 31) / 32, ntn = (l.N + 31) / 32;
  const int NT = l.S <= 16 ? 2 : 1, parts = l.S > 64 ? 4 : 1;
  // few slices: a block takes several tiles, so that its wavefronts have work
  l.nt = l.S <= kWgWaves / 2 ? kWgWaves / l.S : 1;
  if (l.nt > ntm) l.nt = ntm;
  l.blocks = 8 * (((ntn + NT - 1) / NT + 7) / 8) * ((ntm + l.nt - 1) / l.nt) * parts;
}

// Bias gradients of kWgBias outputs: per slice four sums over the rows 32 c + 8 kg + e (kg =
// 0..3), added in order, then the slices in order.  A thread's (slice, c) groups of eight rows
// load four at a time: the chain of dependent reads is what this part is bound by.  A block goes
// through all slices of its outputs; with many rows that chain is the launch's longest, and the
// slices' sums come from k_wgrad_bias, eight slices to a block.
constexpr int kWgBias = 32;
constexpr int kWgBiasSlices = kWgThreads / (4 * kWgBias);  // slices in parallel
// the thread's slices s0, s0 + kWgBiasSlices, ... (ns of them): their sums to dst[slice][kg][output]
__device__ __forceinline__ void bias_slices(const WgradStep &p, const WgradLayer &l, int q, int s0, int ns, float *dst) {
  constexpr int G = 4;  // groups in flight
  const int u = threadIdx.x % kWgBias, kg = threadIdx.x / kWgBias % 4, m = kWgBias * q + u;
  const int gps = l.kc / 32;  // groups of a slice
  const int groups = m < l.M ? ns * gps : 0;
  float x = 0.f;
  for (int g0 = 0; g0 < groups; g0 += G) {
    float d[G][8];
#pragma unroll
    for (int c = 0; c < G; ++c) {
      const int64_t b = (int64_t)(s0 + kWgBiasSlices * ((g0 + c) / gps)) * l.kc + 32 * ((g0 + c) % gps) + 8 * kg;
#pragma unroll
      for (int e = 0; e < 8; ++e) d[c][e] = g0 + c < groups && b + e < p.B ? l.Af[(b + e) * l.M + m] : 0.f;
    }
#pragma unroll
    for (int c = 0; c < G; ++c) {
      if (g0 + c < groups) {
#pragma unroll
        for (int e = 0; e < 8; ++e) x += d[c][e];
        if ((g0 + c + 1) % gps == 0) {
          dst[((s0 + kWgBiasSlices * ((g0 + c) / gps)) * 4 + kg) * kWgBias + u] = x;
          x = 0.f;
        }
      }
    }
  }
}
template <bool ADAM>
__device__ __forceinline__ void bias_sums(const WgradStep &p, const WgradLayer &l, int q, const float *part, float *buf) {
  static_assert(kWgBiasPart <= kWgLdsFloats, "every slice has a slot");
  if (part) {
    for (int i = threadIdx.x; i < l.S * 4 * kWgBias; i += kWgThreads) buf[i] = part[i];
  } else {
    const int sl = threadIdx.x / (4 * kWgBias);
    bias_slices(p, l, q, sl, sl < l.S ? (l.S - sl + kWgBiasSlices - 1) / kWgBiasSlices : 0, buf);
  }
  __syncthreads();
  const int u = threadIdx.x, m = kWgBias * q + u;
  if (u < kWgBias && m < l.M) {
    float tot = 0.f;
#pragma unroll 4
    for (int i = 0; i < l.S; ++i) {
      const float *r = buf + i * 4 * kWgBias + u;
      tot += ((r[0] + r[kWgBias]) + r[2 * kWgBias]) + r[3 * kWgBias];
    }
    const int64_t i = l.w + (int64_t)l.M * l.N + m;
    if constexpr (ADAM)
      adam_update(p, i, tot, p.st->c1, p.st->c2);
    else
      p.g[i] = tot;
  }
}
// the slices' bias sums of all layers: block (x, y) takes slices 8 x .. 8 x + 7 of the y-th 32 outputs
__global__ __launch_bounds__(kWgThreads) void k_wgrad_bias(WgradStep p) {
  int q = blockIdx.y;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const int nb = (p.l[i].M + kWgBias - 1) / kWgBias;
    if (q < nb) {
      const int s = kWgBiasSlices * blockIdx.x + (int)threadIdx.x / (4 * kWgBias);
      return bias_slices(p, p.l[i], q, s, s < p.l[i].S ? 1 : 0, p.bias + (int64_t)blockIdx.y * kWgBiasPart);
    }
    q -= nb;
  }
}

// ---- embeddings
constexpr int kEmbD = 32;

// gE of application g of the batch: the rows of dX through LDS, summed in setting order by
// one thread per dimension
template <bool ADAM>
__device__ __forceinline__ void app_embedding(const WgradStep &p, int g, float *buf) {
  const WgradEmb &e = p.emb;
  constexpr int RS = kWgLdsFloats / kEmbD;  // settings a round
  float x = 0.f;
  for (int j0 = 0; j0 < e.n; j0 += RS) {
    const int left = e.n - j0 < RS ? e.n - j0 : RS;
    if (j0) __syncthreads();
    const float *src = e.dX + ((int64_t)g * e.n + j0) * 2 * kEmbD;
    for (int t = threadIdx.x; t < left * (kEmbD / 4); t += kWgThreads)
      reinterpret_cast<f4 *>(buf)[t] =
          *reinterpret_cast<const f4 *>(src + (t / (kEmbD / 4)) * 2 * kEmbD + 4 * (t % (kEmbD / 4)));
    __syncthreads();
    if (threadIdx.x < kEmbD) {
#pragma unroll 16
      for (int j = 0; j < left; ++j) x += buf[j * kEmbD + threadIdx.x];
    }
  }
  if (threadIdx.x < kEmbD) {
    const int64_t i = e.e + e.apps[g] * kEmbD + threadIdx.x;
    if constexpr (ADAM)
      adam_update(p, i, x, p.st->c1, p.st->c2);
    else
      p.g[i] = x;
  }
}

// gS of 1024 elements (setting, dimension): applications in order
template <bool ADAM>
__device__ __forceinline__ void setting_embeddings(const WgradStep &p, int q) {
  const WgradEmb &e = p.emb;
  const int64_t t = (int64_t)q * kWgThreads + threadIdx.x;
  if (t >= (int64_t)e.n * kEmbD) return;
  const float *src = e.dX + t / kEmbD * 2 * kEmbD + kEmbD + t % kEmbD;
  float x = 0.f;
#pragma unroll 8
  for (int g = 0; g < e.G; ++g) x += src[(int64_t)g * e.n * 2 * kEmbD];
  if constexpr (ADAM)
    adam_update(p, e.s + t, x, p.st->c1, p.st->c2);
  else
    p.g[e.s + t] = x;
}

// blocks of other_embeddings, 1024 elements each: capped, since a grid holds fewer than 2^32 threads
constexpr int64_t kWgMaxOther = int64_t(1) << 20;
__host__ __device__ inline int other_blocks(int64_t m) {
  const int64_t b = (m * kEmbD + kWgThreads - 1) / kWgThreads;
  return (int)(b < kWgMaxOther ? b : kWgMaxOther);
}
// Elements of E, 1024 at a time: the applications outside the batch have zero gradient (Adam still
// moves them by their moments)
template <bool ADAM>
__device__ __forceinline__ void other_embeddings(const WgradStep &p, int q) {
  const WgradEmb &e = p.emb;
  for (int64_t t = (int64_t)q * kWgThreads + threadIdx.x; t < e.m * kEmbD; t += kWgMaxOther * kWgThreads) {
    if (e.mark[t / kEmbD] == p.st->tag) continue;
    if constexpr (ADAM)
      adam_update(p, e.e + t, 0.f, p.st->c1, p.st->c2);
    else
      p.g[e.e + t] = 0.f;
  }
}

// the batch loss, and the step state's counters (read by no other block of this launch)
template <bool ADAM>
__device__ __forceinline__ void loss_and_state(const WgradStep &p, double *red) {
  double a = 0.0;
  for (int i = threadIdx.x; i < p.nlpart; i += kWgThreads) a += p.lpart[i];
  red[threadIdx.x] = a;
  __syncthreads();
  for (int s = kWgThreads / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double loss = red[0] / (double)p.ltotal;
    if (p.loss_d) p.loss_d[0] = loss;
    if (p.loss_f) p.loss_f[0] = (float)loss;
    if (p.loss_steps) p.loss_steps[p.st->t] = (float)loss;
    if constexpr (ADAM) {
      p.st->t += 1;
      p.st->cursor += 1;
    }
  }
}

template <bool ADAM>
__global__ __launch_bounds__(kWgThreads) void k_wgrad_step(WgradStep p) {
  __shared__ __attribute__((aligned(16))) float buf[kWgLdsFloats];
  // the longest chains first: the embedding and bias sums, the loss
  int q = blockIdx.x;
  if (p.emb.G > 0) {
    const int ns = (int)(((int64_t)p.emb.n * kEmbD + kWgThreads - 1) / kWgThreads);
    const int no = other_blocks(p.emb.m);
    if (q < p.emb.G) return app_embedding<ADAM>(p, q, buf);
    q -= p.emb.G;
    if (q < ns) return setting_embeddings<ADAM>(p, q);
    q -= ns;
    if (q < no) return other_embeddings<ADAM>(p, q);
    q -= no;
  }
  const float *part = p.bias;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const int nb = (p.l[i].M + kWgBias - 1) / kWgBias;
    if (q < nb) return bias_sums<ADAM>(p, p.l[i], q, part ? part + (int64_t)q * kWgBiasPart : nullptr, buf);
    q -= nb;
    if (part) part += (int64_t)nb * kWgBiasPart;
  }
  if (q == 0) return loss_and_state<ADAM>(p, reinterpret_cast<double *>(buf));
  --q;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    if (q < p.l[i].blocks) {
      if (p.l[i].S <= 16) return weight_tiles<ADAM, 2, 16>(p, p.l[i], q, buf);
      if (p.l[i].S <= 64) return weight_tiles<ADAM, 1, 16>(p, p.l[i], q, buf);
      return weight_tiles<ADAM, 1, 4>(p, p.l[i], q, buf);
    }
    q -= p.l[i].blocks;
  }
}

open_status wgrad_step(open_ctx *ctx, const char *name, WgradStep p, bool adam) {
  unsigned blocks = 1;
  if (p.emb.G > 0)
    blocks += (unsigned)(p.emb.G + ((int64_t)p.emb.n * kEmbD + kWgThreads - 1) / kWgThreads + other_blocks(p.emb.m));
  int outputs = 0, slices = 0;  // 32 outputs each, of all layers; most slices of a layer
  for (WgradLayer &l : p.l) {
    l.S = wgrad_slices(p.B, l.M, l.N, &l.kc);
    wgrad_shape(l);
    blocks += (unsigned)(l.blocks + (l.M + kWgBias - 1) / kWgBias);
    outputs += (l.M + kWgBias - 1) / kWgBias;
    slices = l.S > slices ? l.S : slices;
  }
  if (p.bias) {
    const dim3 grid((unsigned)((slices + kWgBiasSlices - 1) / kWgBiasSlices), (unsigned)outputs);
    OPEN_LAUNCH(ctx, "wgrad_bias", k_wgrad_bias, grid, dim3(kWgThreads), 0, p);
  }
  if (adam) {
    OPEN_LAUNCH(ctx, name, k_wgrad_step<true>, dim3(blocks), dim3(kWgThreads), 0, p);
  } else {
    OPEN_LAUNCH(ctx, name, k_wgrad_step<false>, dim3(blocks), dim3(kWgThreads), 0, p);
  }
  return OPEN_OK;
}

}  // namespace openk
