// Split-K ridge solve of long rows (weighted-lambda ALS, the completion step of Section III-B):
//   x_i = (sum_{j in O_i} f_j f_j^T + lambda w_i I)^-1  sum_{j in O_i} r_ij f_j
// for the rows with at least kSplitMin observations (size class kSplitClass of the
// bucketing).  These are the columns of the ALS column half-sweep (solved on the column
// view, F = U): a few hundred of them hold most of the observed entries, so one system per
// lane group would leave the chip idle; instead
//   1. k_split_prefix  cuts every long row into equal parts and numbers them;
//   2. k_split_gram    one wavefront per part forms the partial Gram matrix on FP32 MFMA
//                      (the observation index is the contraction index, so one register of
//                      u values is both operands) and the partial right-hand side;
//   3. k_split_solve   one wavefront per row sums its partials in part order (the result
//                      does not depend on scheduling), adds the ridge and solves by LDL^T.
#include "common.h"

namespace openk {

constexpr int kSplitStage = 256;   // entries staged per wavefront, twice
constexpr int kSplitFlush = 1024;  // entries summed in one accumulator
constexpr int kXcds = 8;           // accelerator complex dies of the MI355X, each with its own L2
constexpr int64_t kMaxRangeRows = 4096;  // rows of a matrix whose parts follow the XCDs' factor ranges
constexpr float kSplitSum = 4.0f;  // entries that cost as much as adding a part
constexpr int kPrefixThreads = 1024;
constexpr int kGramWaves = 4;      // wavefronts of a block

// MFMA geometry per rank.  v_mfma_f32_16x16x4f32 takes four observations; a lane holds the
// dimensions KB i + b, b = 0 .. KB - 1, of one of them (i = lane % 16), a contiguous load of KB
// floats, and block (b, c <= b) of the Gram matrix pairs the dimensions b and c modulo KB.
// Only the lower blocks are formed: 3 of 4 at rank 32, 10 of 16 at rank 64.
template <int K>
struct SplitGeo {
  static constexpr int KB = K <= 16 ? 1 : K / 16;
  static constexpr int NB = KB * (KB + 1) / 2;
  static constexpr int GRAM = NB * 256;               // partial Gram floats (MFMA register order)
  static constexpr int PST = GRAM + 16 * KB;          // and the partial right-hand side
  static constexpr int STEPS = K == 64 ? 4 : 8;       // MFMA steps whose factor rows load together
  static constexpr int BLOCKS = K == 64 ? 2 : 4;      // blocks per CU (registers)
};

static int split_part_floats(int k) {
  switch (k) {
    case 8: return SplitGeo<8>::PST;
    case 16: return SplitGeo<16>::PST;
    case 32: return SplitGeo<32>::PST;
    default: return SplitGeo<64>::PST;
  }
}

// Parts.  Where the factor matrix does not fit an XCD's L2 (`ranges`), a row has 8 s parts and XCD x
// takes parts x s .. x s + s - 1: the entries are sorted by index, so it gathers from one
// eighth of the factors.  Otherwise a row has one part per kSplitFlush entries.  `len`: part
// length aimed at (ranges only), so that the parts of an XCD fill its wavefronts evenly.  Few rows
// would then have hundreds of parts each, which one wavefront has to add up: a part costs that about
// as much as kSplitSum entries cost the products, so sqrt(kSplitSum cnt) is the least of both (one row
// of 100,000 entries, us, with 696 parts / now: rank 8 102 / 69, 32 166 / 92, 64 319 / 178).
__device__ __forceinline__ int split_parts(int cnt, bool ranges, int64_t len) {
  if (!ranges) return (cnt + kSplitFlush - 1) / kSplitFlush;
  const int64_t own = (int64_t)__builtin_sqrtf(kSplitSum * (float)cnt);
  len = len > own ? len : own;
  const int64_t s = (cnt + 8 * len - 1) / (8 * len);
  return (int)(8 * (s < 1 ? 1 : s));
}

// start[i] = first part of long row i (list position cls[2 kSplitClass] + i), start[count] = total
// parts, start[count + 1] = most parts of a row
__global__ __launch_bounds__(kPrefixThreads) void k_split_prefix(const RowRef *__restrict__ list,
                                                                 const int64_t *__restrict__ cls, int ranges,
                                                                 int waves_per_xcd, int64_t *__restrict__ start) {
  __shared__ int64_t part[kPrefixThreads];
  const int64_t s0 = cls[2 * kSplitClass], cnt = cls[2 * kSplitClass + 1];
  const int64_t per = (cnt + kPrefixThreads - 1) / kPrefixThreads;
  const int64_t b0 = threadIdx.x * per, b1 = b0 + per < cnt ? b0 + per : cnt;
  auto block_scan = [&](int64_t s) {  // inclusive; part[last] = total
    part[threadIdx.x] = s;
    __syncthreads();
    for (int off = 1; off < kPrefixThreads; off <<= 1) {
      const int64_t x = threadIdx.x >= (unsigned)off ? part[threadIdx.x - off] : 0;
      __syncthreads();
      part[threadIdx.x] += x;
      __syncthreads();
    }
  };
  int64_t len = 1;
  if (ranges) {
    int64_t t = 0;
    for (int64_t i = b0; i < b1; ++i) t += list[s0 + i].cnt;
    block_scan(t);
    len = part[kPrefixThreads - 1] / (8 * (int64_t)waves_per_xcd);
    len = len < kSplitMin / 8 ? kSplitMin / 8 : len;
    // a little longer: rows of equal length then take a whole number of rounds
    len += len / 8;
    __syncthreads();
  }
  int64_t s = 0, m1 = 0;
  for (int64_t i = b0; i < b1; ++i) {
    const int64_t c = split_parts(list[s0 + i].cnt, ranges, len);
    s += c;
    m1 = c > m1 ? c : m1;
  }
  block_scan(s);
  int64_t run = threadIdx.x ? part[threadIdx.x - 1] : 0;
  for (int64_t i = b0; i < b1; ++i) {
    start[i] = run;
    run += split_parts(list[s0 + i].cnt, ranges, len);
  }
  if (threadIdx.x == kPrefixThreads - 1) start[cnt] = part[kPrefixThreads - 1];
  __syncthreads();
  part[threadIdx.x] = m1;
  __syncthreads();
  for (int off = kPrefixThreads / 2; off > 0; off >>= 1) {
    if (threadIdx.x < (unsigned)off && part[threadIdx.x + off] > part[threadIdx.x])
      part[threadIdx.x] = part[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) start[cnt + 1] = part[0];
}

// Partial Gram and right-hand side of every part.  A wavefront takes parts in turn (persistent
// grid); workgroups are dealt to the 8 XCDs round-robin.
//
// Bound by the matrix units (24 cycles per observation and SIMD at rank 32, 80 at rank 64) and the
// gathers from L2.  Parts of equal length keep the wavefronts busy to the end; the accumulators of
// both sums are emptied every kSplitFlush entries, so that a longer part loses no accuracy.  12.7M entries at
// rank 32 (480 columns): 240 us, at rank 64 23.5M entries 1.2 ms; with 32 x 32 x 2 products (all of
// the upper triangle too), chunks of 1024 entries (3.05 per wavefront: four rounds for some) and
// a partial Gram written per chunk 380 us and 1.9 ms.  Asking for two blocks per CU keeps the
// accumulators out of the accumulation registers: at rank 64 each product otherwise came with two
// register moves, which take issue time that the products need (622 -> 568 us a launch).
template <int K, bool FAR>
__global__ __launch_bounds__(64 * kGramWaves, 2) void k_split_gram(const float *__restrict__ Uf,
                                                               const int32_t *__restrict__ ri,
                                                               const float *__restrict__ cv,
                                                               const RowRef *__restrict__ list,
                                                               const int64_t *__restrict__ cls, int ranges,
                                                               const int64_t *__restrict__ start, int nF,
                                                               float *__restrict__ part, int32_t *__restrict__ pflag) {
  using G = SplitGeo<K>;
  constexpr int KB = G::KB, NB = G::NB, ST = G::STEPS;
  typedef float fkb __attribute__((ext_vector_type(KB == 1 ? 2 : KB)));  // (KB = 1: one float used)
  __shared__ int jl_all[kGramWaves][2][kSplitStage];
  __shared__ float rl_all[kGramWaves][2][kSplitStage];
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int64_t s0 = cls[2 * kSplitClass], cnt = cls[2 * kSplitClass + 1];
  if (cnt == 0) return;
  const __amdgpu_buffer_rsrc_t urs = make_rsrc(Uf, (uint64_t)nF * K * sizeof(float));
  const int i16 = lane & 15, o = lane >> 4;  // dimension group and observation slot of this lane
  const bool dim_ok = K >= 16 || i16 < K;
  // virtual index v = c * cnt + row, part c of the wavefront's range of every row in turn
  const bool xr = ranges && gridDim.x % kXcds == 0;
  const int xcd = (int)(blockIdx.x % kXcds);
  const int64_t most = start[cnt + 1];
  const int64_t nw = (xr ? gridDim.x / kXcds : gridDim.x) * (int64_t)kGramWaves;
  const int64_t wv = (xr ? blockIdx.x / kXcds : blockIdx.x) * (int64_t)kGramWaves + w;
  const int64_t total = (xr ? most / kXcds : most) * cnt;
  for (int64_t v = wv; v < total; v += nw) {
    const int64_t row = v % cnt, c = v / cnt;
    const int64_t p0 = start[row], np = start[row + 1] - p0;
    if (c >= (xr ? np / kXcds : np)) continue;  // this row has fewer parts (wave-uniform)
    const int64_t p = xr ? xcd * (np / kXcds) + c : c;
    const RowRef rr = list[s0 + row];
    const int e0 = (int)(rr.cnt * p / np), e1 = (int)(rr.cnt * (p + 1) / np);
    const int len = e1 - e0;
    const int32_t *ip = ri + rr.beg + e0;
    const float *vp = cv + rr.beg + e0;
    f4 acc[NB], sum[NB];
    float b[KB], bsum[KB];
#pragma unroll
    for (int q = 0; q < NB; ++q) acc[q] = sum[q] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < KB; ++q) b[q] = bsum[q] = 0.f;
    int flags = 0;  // 1: non-finite value, 2: index outside [0, nF)
    // indices and values of a stage: loaded a stage ahead, then kept in LDS; rejected or absent
    // entries get the index -1, which reads zeros through the buffer resource
    int jn[kSplitStage / 64];
    float rn[kSplitStage / 64];
    auto fetch = [&](int t0) {
#pragma unroll
      for (int e = 0; e < kSplitStage / 64; ++e) {
        const int t = t0 + 64 * e + lane;
        jn[e] = t < len ? ip[t] : -1;
        rn[e] = t < len ? vp[t] : 0.f;
      }
    };
    auto stage = [&](int t0) {
      int *jl = jl_all[w][(t0 / kSplitStage) & 1];
      float *rl = rl_all[w][(t0 / kSplitStage) & 1];
      __builtin_amdgcn_wave_barrier();  // the reads of two stages ago are done
#pragma unroll
      for (int e = 0; e < kSplitStage / 64; ++e) {
        const bool in = t0 + 64 * e + lane < len;
        const bool ok = jn[e] >= 0 && jn[e] < nF;
        if (in && !ok) flags |= 2;
        if (in && !__builtin_isfinite(rn[e])) flags |= 1;
        jl[64 * e + lane] = ok ? jn[e] : -1;
        rl[64 * e + lane] = rn[e];
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    // factor rows of ST steps (4 ST entries), loaded one batch ahead of the matrix units
    fkb un[ST];
    float vn[ST];
    auto gather = [&](int t0) {
      const int *jl = jl_all[w][(t0 / kSplitStage) & 1] + t0 % kSplitStage;
      const float *rl = rl_all[w][(t0 / kSplitStage) & 1] + t0 % kSplitStage;
#pragma unroll
      for (int u = 0; u < ST; ++u) {
        const int j = jl[4 * u + o];
        vn[u] = rl[4 * u + o];
        const uint32_t off = dim_ok ? ((uint32_t)j * K + KB * i16) * 4u : 0xfffffff0u;
        if constexpr (FAR && KB == 1)
          un[u][0] = far_load<1>(Uf, dim_ok ? j : -1, K, dim_ok ? i16 : 0)[0];
        else if constexpr (FAR)
          un[u] = far_load<KB>(Uf, j, K, KB * i16);
        else if constexpr (KB == 1)
          un[u][0] = bload_f32(urs, (int)off);
        else if constexpr (KB == 2)
          un[u] = __builtin_bit_cast(fkb, __builtin_amdgcn_raw_buffer_load_b64(urs, (int)off, 0, 0));
        else
          un[u] = __builtin_bit_cast(fkb, __builtin_amdgcn_raw_buffer_load_b128(urs, (int)off, 0, 0));
      }
    };
    fetch(0);
    stage(0);
    fetch(kSplitStage);
    gather(0);
    for (int t0 = 0; t0 < len; t0 += 4 * ST) {
      fkb u[ST];
      float val[ST];
#pragma unroll
      for (int e = 0; e < ST; ++e) {
        u[e] = un[e];
        val[e] = vn[e];
      }
      const int t1 = t0 + 4 * ST;
      if (t1 % kSplitStage == 0 && t1 < len) {  // wave-uniform
        stage(t1);
        fetch(t1 + kSplitStage);
      }
      if (t1 < len) gather(t1);
#pragma unroll
      for (int e = 0; e < ST; ++e) {
        int q = 0;
#pragma unroll
        for (int b1 = 0; b1 < KB; ++b1)
#pragma unroll
          for (int b2 = 0; b2 <= b1; ++b2, ++q)
            acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(u[e][b1], u[e][b2], acc[q], 0, 0, 0);
#pragma unroll
        for (int b1 = 0; b1 < KB; ++b1) b[b1] = __builtin_fmaf(val[e], u[e][b1], b[b1]);
      }
      if (t1 % kSplitFlush == 0) {
#pragma unroll
        for (int q = 0; q < NB; ++q) {
          sum[q] += acc[q];
          acc[q] = f4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int q = 0; q < KB; ++q) {
          bsum[q] += b[q];
          b[q] = 0.f;
        }
      }
    }
    float *dst = part + (p0 + p) * G::PST;
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      sum[q] += acc[q];
#pragma unroll
      for (int e = 0; e < 4; ++e) dst[(4 * q + e) * 64 + lane] = sum[q][e];
    }
    // the right-hand side over the four observation slots, in dimension order
#pragma unroll
    for (int q = 0; q < KB; ++q) {
      b[q] += bsum[q];
      b[q] += __shfl_xor(b[q], 16, 64);
      b[q] += __shfl_xor(b[q], 32, 64);
      if (lane < 16) dst[G::GRAM + KB * lane + q] = b[q];
    }
    const unsigned long long f1 = __ballot(flags & 1), f2 = __ballot(flags & 2);
    if (lane == 0) pflag[p0 + p] = (f1 ? 1 : 0) | (f2 ? 2 : 0);
  }
}

// One wavefront per long row: sum its partials, add the ridge, LDL^T with lane c holding column
// c of the symmetric matrix in registers (lanes past K repeat), the pivot row passed through
// LDS, forward substitution fused in; back substitution by lane reads.  Bound by the chain of K
// pivots: 7 us for 480 rows at rank 32, 80 us for 5000 rows at rank 64 (27 and 400 us with the
// matrix in LDS, a barrier between every step and three times the partial sums).  Where a row has
// many parts, by their sum: several parts' loads go out together (one row of 696 parts at rank 32,
// whole pass, 267 -> 166 us).
template <int K>
__global__ __launch_bounds__(64) void k_split_solve(const RowRef *__restrict__ list, const int64_t *__restrict__ cls,
                                                    const int64_t *__restrict__ start,
                                                    const float *__restrict__ part,
                                                    const int32_t *__restrict__ pflag, float lambda, int weighted,
                                                    float *__restrict__ X, int32_t *__restrict__ status) {
  using G = SplitGeo<K>;
  constexpr int KB = G::KB, NB = G::NB, LD = K + 1;
  __shared__ __attribute__((aligned(16))) float prow[64];
  __shared__ float mat[K * LD];
  const int64_t s0 = cls[2 * kSplitClass], cnt = cls[2 * kSplitClass + 1];
  const int64_t i = blockIdx.x;
  if (i >= cnt) return;
  const RowRef rr = list[s0 + i];
  const int lane = threadIdx.x, i16 = lane & 15, o = lane >> 4;
  const int64_t g0 = start[i], g1 = start[i + 1];
  f4 gs[NB];
  float b = 0.f;
#pragma unroll
  for (int q = 0; q < NB; ++q) gs[q] = f4{0.f, 0.f, 0.f, 0.f};
  int flags = 0;
  // U parts' loads together; added in part order
  auto add = [&](int64_t g, auto Un) {
    constexpr int U = decltype(Un)::value;
    f4 x[U][NB];
    float y[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float *src = part + (g + u) * G::PST;
#pragma unroll
      for (int q = 0; q < NB; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) x[u][q][e] = src[(4 * q + e) * 64 + lane];
      y[u] = src[G::GRAM + lane % K];
      flags |= pflag[g + u];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int q = 0; q < NB; ++q) gs[q] += x[u][q];
      b += y[u];
    }
  };
  constexpr int U = K == 64 ? 2 : K == 32 ? 4 : 8;
  int64_t g = g0;
  for (; g + U <= g1; g += U) add(g, std::integral_constant<int, U>{});
  for (; g < g1; ++g) add(g, std::integral_constant<int, 1>{});
  // lane (i16, o) holds, of block (b1, b2), column KB i16 + b2 and rows KB (4 o + e) + b1
  {
    int q = 0;
#pragma unroll
    for (int b1 = 0; b1 < KB; ++b1)
#pragma unroll
      for (int b2 = 0; b2 <= b1; ++b2, ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int r = KB * (4 * o + e) + b1, c = KB * i16 + b2;
          if (r < K && c < K) {
            mat[r * LD + c] = gs[q][e];
            mat[c * LD + r] = gs[q][e];
          }
        }
  }
  __syncthreads();
  const int me = lane % K;
  const float reg = lambda * (weighted ? (float)rr.cnt : 1.0f);
  float a[K];
#pragma unroll
  for (int r = 0; r < K; ++r) a[r] = mat[r * LD + me] + (r == me ? reg : 0.f);
  int bad = 0;
  float dd = 1.f;  // d of the lane's column
  sfor<0, K>([&](auto Pp) {
    constexpr int p = decltype(Pp)::value;
    prow[lane] = a[p];  // row p of the trailing matrix: also column p below the pivot
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    float gc[K];
    sfor<p / 4, K / 4>([&](auto Q) {
      constexpr int q = decltype(Q)::value;
      const f4 x = *reinterpret_cast<const f4 *>(prow + 4 * q);
      gc[4 * q] = x[0];
      gc[4 * q + 1] = x[1];
      gc[4 * q + 2] = x[2];
      gc[4 * q + 3] = x[3];
    });
    const float dp = gc[p];
    bad |= !(dp > 0.f && __builtin_isfinite(dp));
    const float lc = me > p ? a[p] / dp : 0.f;
    sfor<p + 1, K>([&](auto R) {
      constexpr int r = decltype(R)::value;
      a[r] = __builtin_fmaf(-gc[r], lc, a[r]);
    });
    b = __builtin_fmaf(-lc, readlane_f32(b, p), b);
    dd = me == p ? dp : dd;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();  // the buffer is rewritten at the next pivot
  });
  // x_r = (y_r - sum_{p > r} d_r L[p][r] x_p) / d_r, and a[p] of lane r is d_r L[p][r]
  const float rd = 1.0f / dd;
  sfor_down<0, K>([&](auto Pp) {
    constexpr int p = decltype(Pp)::value;
    const float xp = readlane_f32(b * rd, p);
    b = me < p ? __builtin_fmaf(-a[p], xp, b) : b;
  });
  const bool good = !bad && flags == 0;
  if (lane < K) X[(int64_t)rr.row * K + lane] = good ? b * rd : 0.f;
  if (status && lane == 0)
    status[rr.row] = (flags & 2) ? OPEN_ROW_BADINDEX
                     : (flags & 1) ? OPEN_ROW_NONFINITE
                     : bad        ? OPEN_ROW_NONPOS_PIVOT
                                  : OPEN_ROW_OK;
}

template <int K>
static open_status split_launch_k(open_ctx *ctx, const float *F, int nF, const int32_t *ri, const float *cv,
                                  const RowRef *list, const int64_t *cls, int64_t *start, float *part,
                                  int32_t *pflag, float lambda, int weighted, float *X, int32_t *status,
                                  int64_t max_rows, int ranges, unsigned blocks) {
  OPEN_LAUNCH(ctx, "split_prefix", k_split_prefix, dim3(1), dim3(kPrefixThreads), 0, list, cls, ranges,
              (int)(blocks * kGramWaves / kXcds), start);
  OPEN_LAUNCH(ctx, "split_gram", (far_factors(nF, K) ? k_split_gram<K, true> : k_split_gram<K, false>), dim3(blocks),
              dim3(64 * kGramWaves), 0, F, ri, cv, list, cls, ranges,
              (const int64_t *)start, nF, part, pflag);
  OPEN_LAUNCH(ctx, "split_solve", k_split_solve<K>, dim3((unsigned)max_rows), dim3(64), 0, list, cls,
              (const int64_t *)start, (const float *)part, (const int32_t *)pflag, lambda, weighted, X, status);
  return OPEN_OK;
}

open_status splitk_launch(open_ctx *ctx, const float *F, int nF, int k, const int32_t *idx, const float *val,
                          float lambda, int weighted, const RowRef *list, const int64_t *cls, float *X,
                          int32_t *status, int64_t m, int64_t nnz) {
  // at most nnz / kSplitMin long rows
  int64_t max_rows = nnz / kSplitMin + 1;
  if (max_rows > m) max_rows = m;
  if (max_rows < 1) return OPEN_OK;
  if (max_rows > INT32_MAX) return fail(ctx, OPEN_E_UNSUPPORTED, "too many long rows");
  // Ranges of the factors per XCD pay once these no longer fit an L2 (4 MB) beside the entries, and
  // where the rows are few and long (the column half-sweep): every row then has at least
  // eight parts, whose partial sums cost memory and time.
  const int ranges = (int64_t)nF * k * (int64_t)sizeof(float) > (int64_t(2) << 20) && m <= kMaxRangeRows;
  const unsigned blocks = (unsigned)(ctx->num_cu * (k == 64 ? SplitGeo<64>::BLOCKS : SplitGeo<32>::BLOCKS));
  // parts: at least total / (8 waves of an XCD) entries long up to a row's eight, or kSplitFlush
  // entries but for a row's last
  const int64_t max_parts = ranges ? (int64_t)blocks * kGramWaves + 8 * max_rows + 8 : nnz / kSplitFlush + max_rows + 1;
  void *cs = nullptr, *pt = nullptr, *cf = nullptr;
  open_status st;
  // start: one entry per long row, the total, and the most parts of a row
  if ((st = ws_get(ctx, open_ctx::WS_SPLIT_START, sizeof(int64_t) * (size_t)(max_rows + 2), &cs))) return st;
  if ((st = ws_get(ctx, open_ctx::WS_SPLIT_PART, sizeof(float) * (size_t)max_parts * split_part_floats(k), &pt)))
    return st;
  if ((st = ws_get(ctx, open_ctx::WS_SPLIT_FLAG, sizeof(int32_t) * (size_t)max_parts, &cf))) return st;
  int64_t *c = (int64_t *)cs;
  float *p = (float *)pt;
  int32_t *f = (int32_t *)cf;
  switch (k) {
    case 8: return split_launch_k<8>(ctx, F, nF, idx, val, list, cls, c, p, f, lambda, weighted, X, status, max_rows,
                                   ranges, blocks);
    case 16: return split_launch_k<16>(ctx, F, nF, idx, val, list, cls, c, p, f, lambda, weighted, X, status, max_rows,
                                   ranges, blocks);
    case 32: return split_launch_k<32>(ctx, F, nF, idx, val, list, cls, c, p, f, lambda, weighted, X, status, max_rows,
                                   ranges, blocks);
    case 64: return split_launch_k<64>(ctx, F, nF, idx, val, list, cls, c, p, f, lambda, weighted, X, status, max_rows,
                                   ranges, blocks);
    default: return fail(ctx, OPEN_E_UNSUPPORTED, "rank must be 8, 16, 32 or 64");
  }
}

}  // namespace openk
