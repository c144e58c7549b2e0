// ALS-WR fit support: column view of the CSR (exact stable counting sort), the objective
// reduced in float64 in a fixed order, the observed-entry residual, and the sweep driver.
#include <math.h>
#include <string.h>

#include "common.h"

namespace openk {

// Column view on the device: an exact stable counting sort of the entries by column.
//
// Rows are cut into chunks of kCscRows; a block owns a chunk and keeps, per column, one bit per
// row of the chunk that has an entry there.  The rank of an entry among the chunk's entries of
// its column is then a bit count, so all entries of a chunk are placed at once, ordered by
// column and, within a column, by row.
//   count   entries per (chunk, column), chunk-major
//   scan    per column: exclusive over the chunks of a segment, in place; then over the segments
//           and the columns (one block), which also gives col_ptr
//   place   position = segment base + chunk offset + rank
// The place kernel puts a chunk's entries in order in LDS first, so that neighbouring lanes store
// neighbouring entries of a column (17 in a run at 480 columns, 2.6 at 1920); consecutive chunks,
// which write next to each other, are dealt to one XCD's L2.  Bound by the latency of its steps,
// one or two blocks of 16 wavefronts per CU.  12.7M entries, 200,003 x 480: count 28, scan 15, place
// 94 us (118 with one block per CU); stored entry by entry as ranked 358 us, and with chunks of 256 rows per wavefront that
// walked its rows one by one 109, 15 and 860.  19.5M entries, 500,009 x 1920: place 272 us, stored
// as ranked 577.  Every window ranks all of the chunk's entries again, so a chunk of more than
// kCscMaxWins windows stores them as ranked, once: whole view of full rows, windows against as
// ranked, 50,000 x 1920 (24 windows) 9.2 and 4.9 ms, 3000 x 4096 (94) 32 and 2.0, 100,000 x 960
// (12) 4.7 and 4.4, 50,000 rows of 900 in 1920 (11) 2.33 and 2.46, 100,000 x 480 (6) 1.5 and 2.0.
// Chunks of few entries need no large window: where there are more chunks than CUs and the window of
// two blocks that share a CU holds the mean chunk, that window is taken, and the exceptional chunk,
// which then has the CU's wavefronts to wait for, is stored as ranked past kCscPairWins windows.  Whole
// view, one block per CU with the scan's walk by one thread per column against now: 2M rows of 0 to 2
// in 2 columns 283 and 175 us, 10M 1261 and 712, 2M of 0 to 4 in 120 320 and 223; 1M rows of 2 in 480
// but for 128 full ones 409 and 311, with 12 windows allowed 486.
constexpr int kCscRows = 128;          // rows of a chunk: two 64-bit masks per column
constexpr int kCscThreads = 512;
constexpr int kCscPlaceThreads = 1024;
constexpr int kCscWin = 10240;         // entries put in order in LDS at a time (fewer for many columns)
constexpr int kCscMaxWins = 12;        // more of them in a chunk: its entries are stored as ranked
constexpr int kCscPairLds = 79 * 1024; // LDS of a place block when two share a CU
constexpr int kCscPairWins = 4;        // and its most windows
constexpr int kCscSeg = 64;            // chunks of a scan segment
// chunks of a launch: a grid holds fewer than 2^32 threads, which 2^31 rows would pass
constexpr int kCscLaunchChunks = 1 << 21;
static_assert(kCscLaunchChunks % kCscSeg == 0, "a launch holds whole segments");
constexpr int kMaxCols = 4096;

// the chunk of a block among the launch's `count` from chunk0 on: blocks are dealt to the 8 XCDs
// round-robin, so XCD x walks the x-th eighth of them
__device__ __forceinline__ int csc_chunk(int chunk0, int count) {
  const int per = (count + 7) / 8;
  const int c = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  return (int)(blockIdx.x >> 3) < per && c < count ? chunk0 + c : -1;
}

// the chunk's row pointers relative to its first entry, and the column masks
struct CscChunk {
  int64_t r0, e0;
  int rows, len;
};
template <int TH>
__device__ __forceinline__ CscChunk csc_begin(int64_t m, int n, const int64_t *__restrict__ ptr, int chunk,
                                              int *rp, unsigned long long *mask) {
  CscChunk c;
  c.r0 = (int64_t)chunk * kCscRows;
  c.rows = (int)(m - c.r0 < kCscRows ? m - c.r0 : kCscRows);
  c.e0 = ptr[c.r0];
  for (int i = threadIdx.x; i <= kCscRows; i += TH)
    rp[i] = (int)(ptr[c.r0 + (i < c.rows ? i : c.rows)] - c.e0);
  for (int j = threadIdx.x; j < 2 * n; j += TH) mask[j] = 0ull;
  __syncthreads();
  c.len = rp[kCscRows];
  return c;
}
// row (of the chunk) of its entry t: the last one that starts at or before t
__device__ __forceinline__ int csc_row(const int *rp, int t) {
  int r = 0;
#pragma unroll
  for (int s = kCscRows / 2; s > 0; s >>= 1) r += rp[r + s] <= t ? s : 0;
  return r;
}
template <int TH>
__device__ __forceinline__ void csc_masks(const CscChunk &c, int n, const int32_t *__restrict__ col, const int *rp,
                                          unsigned long long *mask) {
  for (int t = threadIdx.x; t < c.len; t += TH) {
    const int j = col[c.e0 + t];
    if (j < 0 || j >= n) continue;  // rejected by the index check
    const int r = csc_row(rp, t);
    atomicOr(&mask[2 * j + (r >> 6)], 1ull << (r & 63));
  }
  __syncthreads();
}

__global__ __launch_bounds__(kCscThreads) void k_csc_count(int64_t m, int n, const int64_t *__restrict__ ptr,
                                                           const int32_t *__restrict__ col, int chunk0, int count,
                                                           int32_t *__restrict__ hist) {
  extern __shared__ unsigned long long mask_s[];  // [n][2]
  __shared__ int rp[kCscRows + 1];
  const int chunk = csc_chunk(chunk0, count);
  if (chunk < 0) return;
  const CscChunk c = csc_begin<kCscThreads>(m, n, ptr, chunk, rp, mask_s);
  csc_masks<kCscThreads>(c, n, col, rp, mask_s);
  for (int j = threadIdx.x; j < n; j += kCscThreads)
    hist[(int64_t)chunk * n + j] = __popcll(mask_s[2 * j]) + __popcll(mask_s[2 * j + 1]);
}

// hist[c][j] -> entries of column j in the chunks of c's segment before c; seg[s][j] = its total
__global__ __launch_bounds__(256) void k_csc_segments(int n, int nchunk, int seg0, int32_t *__restrict__ hist,
                                                      int64_t *__restrict__ seg) {
  const int j = blockIdx.x * 256 + threadIdx.x, sg = seg0 + (int)blockIdx.y, c0 = sg * kCscSeg;
  if (j >= n) return;
  int run = 0;
  for (int b = 0; b < kCscSeg; b += 16) {
    int v[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) v[e] = c0 + b + e < nchunk ? hist[(int64_t)(c0 + b + e) * n + j] : 0;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      if (c0 + b + e < nchunk) hist[(int64_t)(c0 + b + e) * n + j] = run;
      run += v[e];
    }
  }
  seg[(int64_t)sg * n + j] = run;
}

// seg[s][j] -> position of segment s's first entry of column j; col_ptr.  One block.  Thread t owns
// columns t, t + 1024, ...; SPLIT (at most 512 columns, and more segments than a thread loads at once):
// 1024 / n threads share a column, each with a stretch of its segments, as a single thread's walk over
// them is a serial chain: at 10M rows x 2 columns 1221 segments, 8 loads at a time and twice.
template <bool SPLIT>
__global__ __launch_bounds__(1024) void k_csc_bases(int n, int nseg, int64_t *__restrict__ seg,
                                                    int64_t *__restrict__ col_ptr) {
  __shared__ int64_t scan[1024];
  const int P = SPLIT ? 1024 / n : 1, per = (nseg + P - 1) / P;
  int64_t before = 0;  // entries of the columns before this round's
  for (int j0 = 0; j0 < n; j0 += 1024) {
    const int j = j0 + (int)threadIdx.x / P;
    const int s0 = SPLIT ? (int)threadIdx.x % P * per : 0, s1 = SPLIT && s0 + per < nseg ? s0 + per : nseg;
    int64_t tot = 0;
    if (j < n)
      for (int s = s0; s < s1; s += 8) {
        int64_t v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = s + e < s1 ? seg[(int64_t)(s + e) * n + j] : 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) tot += v[e];
      }
    scan[threadIdx.x] = tot;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
      const int64_t v = threadIdx.x >= (unsigned)off ? scan[threadIdx.x - off] : 0;
      __syncthreads();
      scan[threadIdx.x] += v;
      __syncthreads();
    }
    int64_t run = before + scan[threadIdx.x] - tot;
    before += scan[1023];
    if (j < n) {
      if (s0 == 0) col_ptr[j] = run;
      for (int s = s0; s < s1; s += 8) {
        int64_t v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = s + e < s1 ? seg[(int64_t)(s + e) * n + j] : 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          if (s + e < s1) seg[(int64_t)(s + e) * n + j] = run;
          run += v[e];
        }
      }
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) col_ptr[n] = before;
}

// The chunk's entries are first put in order in LDS, `win` of them at a time, and then written out
// in that order: neighbouring lanes write neighbouring entries of a column.  (Too many for that:
// stored as ranked.)
__global__ __launch_bounds__(kCscPlaceThreads) void k_csc_place(int64_t m, int n, const int64_t *__restrict__ ptr,
                                                                const int32_t *__restrict__ col,
                                                                const float *__restrict__ val, int chunk0, int count,
                                                                int win, int max_wins,
                                                                const int32_t *__restrict__ hist,
                                                                const int64_t *__restrict__ seg,
                                                                int32_t *__restrict__ row_idx,
                                                                float *__restrict__ cval) {
  constexpr int TH = kCscPlaceThreads;
  // [n][2] masks, [n] global minus chunk position of a column's first entry, [win] entries
  // (column and row of the chunk, value), [n] chunk position
  extern __shared__ unsigned long long mask_s[];
  __shared__ int rp[kCscRows + 1], wsum[TH / 64];
  int64_t *shift = reinterpret_cast<int64_t *>(mask_s + 2 * n);
  uint2 *ent = reinterpret_cast<uint2 *>(shift + n);
  int *first = reinterpret_cast<int *>(ent + win);
  const int chunk = csc_chunk(chunk0, count);
  if (chunk < 0) return;
  const CscChunk c = csc_begin<TH>(m, n, ptr, chunk, rp, mask_s);
  csc_masks<TH>(c, n, col, rp, mask_s);
  // exclusive scan of the columns' counts: thread t owns columns per t .. per t + per - 1
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, per = (n + TH - 1) / TH;
  auto entries = [&](int j) { return __popcll(mask_s[2 * j]) + __popcll(mask_s[2 * j + 1]); };
  int own = 0;
  for (int j = per * threadIdx.x; j < per * ((int)threadIdx.x + 1) && j < n; ++j) own += entries(j);
  int run = own;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int x = __shfl_up(run, off, 64);
    run += lane >= off ? x : 0;
  }
  if (lane == 63) wsum[w] = run;
  __syncthreads();
  int total = 0;
  run -= own;
#pragma unroll
  for (int i = 0; i < TH / 64; ++i) {
    run += i < w ? wsum[i] : 0;
    total += wsum[i];
  }
  for (int j = per * threadIdx.x; j < per * ((int)threadIdx.x + 1) && j < n; ++j) {
    first[j] = run;
    shift[j] = seg[(int64_t)(chunk / kCscSeg) * n + j] + hist[(int64_t)chunk * n + j] - run;
    run += entries(j);
  }
  // rank of the entry of row r among the chunk's entries of column j
  auto rank_of = [&](int j, int r) {
    const unsigned long long lo = mask_s[2 * j], hi = mask_s[2 * j + 1];
    const unsigned long long below = (1ull << (r & 63)) - 1ull;
    return r < 64 ? __popcll(lo & below) : __popcll(lo) + __popcll(hi & below);
  };
  if (total > max_wins * win) {
    __syncthreads();
#pragma unroll 4
    for (int t = threadIdx.x; t < c.len; t += TH) {
      const int j = col[c.e0 + t];
      if (j < 0 || j >= n) continue;
      const int r = csc_row(rp, t);
      const int64_t p = shift[j] + first[j] + rank_of(j, r);
      row_idx[p] = (int32_t)(c.r0 + r);
      cval[p] = val[c.e0 + t];
    }
    return;
  }
  for (int w0 = 0; w0 < total; w0 += win) {
    __syncthreads();
    for (int t = threadIdx.x; t < c.len; t += TH) {
      const int j = col[c.e0 + t];
      if (j < 0 || j >= n) continue;
      const int r = csc_row(rp, t);
      const int q = first[j] + rank_of(j, r) - w0;
      if (q >= 0 && q < win) ent[q] = uint2{(uint32_t)(j * kCscRows + r), __builtin_bit_cast(uint32_t, val[c.e0 + t])};
    }
    __syncthreads();
    const int nw = total - w0 < win ? total - w0 : win;
    for (int q = threadIdx.x; q < nw; q += TH) {
      const uint2 e = ent[q];
      const int64_t p = shift[e.x / kCscRows] + w0 + q;
      const uint32_t v = e.y;
      row_idx[p] = (int32_t)(c.r0 + (int)(e.x % kCscRows));
      cval[p] = __builtin_bit_cast(float, v);
    }
  }
}

// flag[0] |= 1 if some column index lies outside [0, n)
__global__ void k_check_cols(int64_t nnz, const int32_t *__restrict__ col, int n, int *__restrict__ flag) {
  int bad = 0;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < nnz; t += (int64_t)gridDim.x * blockDim.x)
    bad |= (col[t] < 0) | (col[t] >= n);
  if (__any(bad) && (threadIdx.x & 63) == 0) atomicOr(flag, 1);
}

// Synchronous check that every column index is in range (OPEN_E_INVALID otherwise).
static open_status check_cols(open_ctx *ctx, int64_t nnz, const int32_t *col, int n) {
  if (nnz <= 0) return OPEN_OK;
  void *flag;
  int *h;
  open_status st;
  if ((st = ws_get(ctx, open_ctx::WS_FLAG, 256, &flag))) return st;
  if ((st = pinned_get(ctx, 64, (void **)&h))) return st;
  OPEN_LAUNCH(ctx, "fill", k_fill_i32, dim3(1), dim3(64), 0, (int *)flag, 1, 0);
  int64_t blocks = (nnz + 255) / 256;
  if (blocks > ctx->num_cu * 8) blocks = ctx->num_cu * 8;
  OPEN_LAUNCH(ctx, "check_cols", k_check_cols, dim3((unsigned)blocks), dim3(256), 0, nnz, col, n, (int *)flag);
  OPEN_HIP_TRY(ctx, hipMemcpyAsync(h, flag, sizeof(int), hipMemcpyDeviceToHost, ctx->stream));
  OPEN_HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
  if (h[0]) return fail(ctx, OPEN_E_INVALID, "a column index lies outside [0, n)");
  return OPEN_OK;
}

open_status csr_to_csc_dev(open_ctx *ctx, int64_t m, int n, int64_t nnz, const int64_t *row_ptr, const int32_t *col,
                           const float *val, int64_t *col_ptr, int32_t *row_idx, float *cval) {
  const int nchunk = (int)((m + kCscRows - 1) / kCscRows);
  const int nseg = (nchunk + kCscSeg - 1) / kCscSeg;
  void *hist, *seg;
  open_status st;
  if ((st = ws_get(ctx, open_ctx::WS_HIST, sizeof(int32_t) * (size_t)n * (size_t)(nchunk > 0 ? nchunk : 1), &hist)))
    return st;
  if ((st = ws_get(ctx, open_ctx::WS_SPLIT, sizeof(int64_t) * (size_t)n * (size_t)(nseg > 0 ? nseg : 1), &seg)))
    return st;
  const size_t lds = sizeof(unsigned long long) * 2 * (size_t)n;
  const size_t cols = (2 * sizeof(unsigned long long) + sizeof(int64_t) + sizeof(int)) * (size_t)n;
  const size_t room = (size_t)(156 * 1024 - cols) / sizeof(uint2);  // n <= kMaxCols: at least 5632
  int win = room < (size_t)kCscWin ? (int)room : kCscWin, max_wins = kCscMaxWins;
  const int64_t pair = cols < (size_t)kCscPairLds ? (int64_t)((kCscPairLds - cols) / sizeof(uint2)) : 0;
  if (nchunk > ctx->num_cu && pair * nchunk >= nnz) {
    win = pair < win ? (int)pair : win;
    max_wins = kCscPairWins;
  }
  auto launch_chunks = [&](int c0) { return nchunk - c0 < kCscLaunchChunks ? nchunk - c0 : kCscLaunchChunks; };
  auto launch_blocks = [](int count) { return dim3(8 * (unsigned)((count + 7) / 8)); };
  for (int c0 = 0; c0 < nchunk; c0 += launch_chunks(c0)) {
    const int count = launch_chunks(c0), segs = (count + kCscSeg - 1) / kCscSeg;
    OPEN_LAUNCH(ctx, "csc_count", k_csc_count, launch_blocks(count), dim3(kCscThreads), lds, m, n, row_ptr, col, c0,
                count, (int32_t *)hist);
    OPEN_LAUNCH(ctx, "csc_segments", k_csc_segments, dim3((unsigned)((n + 255) / 256), (unsigned)segs), dim3(256), 0, n,
                nchunk, c0 / kCscSeg, (int32_t *)hist, (int64_t *)seg);
  }
  OPEN_LAUNCH(ctx, "csc_bases", (n <= 512 && nseg > 8 ? k_csc_bases<true> : k_csc_bases<false>), dim3(1), dim3(1024), 0, n, nseg, (int64_t *)seg, col_ptr);
  for (int c0 = 0; c0 < nchunk; c0 += launch_chunks(c0)) {
    const int count = launch_chunks(c0);
    OPEN_LAUNCH(ctx, "csc_place", k_csc_place, launch_blocks(count), dim3(kCscPlaceThreads),
                cols + sizeof(uint2) * (size_t)win, m, n, row_ptr, col, val, c0, count, win, max_wins,
                (const int32_t *)hist, (const int64_t *)seg, row_idx, cval);
  }
  return OPEN_OK;
}

// ---------------------------------------------------------------- objective and residual
constexpr int kRedBlocks = 1024;

// One wavefront per row (grid-stride).  Per row the squared errors and |u_i|^2 are formed
// in float32 and added to a per-lane float64 accumulator; lanes and waves are combined in
// a fixed order, then a second kernel adds the block partials in order.
template <int K>
__global__ __launch_bounds__(256) void k_objective_rows(int64_t m, int n, const int64_t *__restrict__ ptr,
                                                        const int32_t *__restrict__ col,
                                                        const float *__restrict__ val, const float *__restrict__ U,
                                                        const float *__restrict__ V, float lambda, int weighted,
                                                        double *__restrict__ part) {
  __shared__ double red[256];
  const int lane = threadIdx.x & 63;
  double acc = 0.0;
  const int64_t nw = (int64_t)gridDim.x * 4;
  for (int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); i < m; i += nw) {
    const float *u = U + i * K;
    const int64_t b = ptr[i], e = ptr[i + 1];
    for (int64_t t = b + lane; t < e; t += 64) {
      const int j = col[t];
      if (j < 0 || j >= n) continue;
      const float *v = V + (int64_t)j * K;
      float p = 0.f;
#pragma unroll
      for (int a = 0; a < K; ++a) p = __builtin_fmaf(u[a], v[a], p);
      const float d = val[t] - p;
      acc += (double)(d * d);
    }
    if (lane < K) {
      const float w = weighted ? (float)(e - b) : 1.0f;
      acc += (double)lambda * (double)w * (double)(u[lane] * u[lane]);
    }
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < (unsigned)s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// lambda * sum_j w^j |v_j|^2 with w^j from the column pointer (or 1); one block, fixed order
template <int K>
__global__ __launch_bounds__(256) void k_objective_cols(int n, const int64_t *__restrict__ col_ptr,
                                                        const float *__restrict__ V, float lambda, int weighted,
                                                        const double *__restrict__ part, int nparts,
                                                        double *__restrict__ out) {
  __shared__ double red[256];
  double acc = 0.0;
  for (int j = threadIdx.x; j < n; j += 256) {
    float s = 0.f;
#pragma unroll
    for (int a = 0; a < K; ++a) s = __builtin_fmaf(V[(int64_t)j * K + a], V[(int64_t)j * K + a], s);
    const double w = weighted ? (double)(col_ptr[j + 1] - col_ptr[j]) : 1.0;
    acc += (double)lambda * w * (double)s;
  }
  for (int b = threadIdx.x; b < nparts; b += 256) acc += part[b];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < (unsigned)s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = red[0];
}

template <int K>
__global__ __launch_bounds__(256) void k_residual(int64_t m, int n, const int64_t *__restrict__ ptr,
                                                  const int32_t *__restrict__ col, const float *__restrict__ val,
                                                  const float *__restrict__ U, const float *__restrict__ V,
                                                  float *__restrict__ rho) {
  const int lane = threadIdx.x & 63;
  const int64_t nw = (int64_t)gridDim.x * 4;
  for (int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); i < m; i += nw) {
    const float *u = U + i * K;
    const int64_t b = ptr[i], e = ptr[i + 1];
    float acc = 0.f;
    for (int64_t t = b + lane; t < e; t += 64) {
      const int j = col[t];
      if (j < 0 || j >= n) continue;
      const float *v = V + (int64_t)j * K;
      float p = 0.f;
#pragma unroll
      for (int a = 0; a < K; ++a) p = __builtin_fmaf(u[a], v[a], p);
      const float d = val[t] - p;
      acc = __builtin_fmaf(d, d, acc);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (lane == 0) rho[i] = e > b ? sqrtf(acc / (float)(e - b)) : 0.f;
  }
}

template <int K>
static open_status objective_impl(open_ctx *ctx, int64_t m, int n, const int64_t *row_ptr, const int32_t *col,
                                  const float *val, const float *U, const float *V, float lambda, int weighted,
                                  const int64_t *col_ptr, double *out_dev) {
  void *part;
  open_status st;
  if ((st = ws_get(ctx, open_ctx::WS_MISC, sizeof(double) * (kRedBlocks + 8), &part))) return st;
  OPEN_LAUNCH(ctx, "objective_rows", k_objective_rows<K>, dim3(kRedBlocks), dim3(256), 0, m, n, row_ptr, col, val, U, V,
              lambda, weighted, (double *)part);
  OPEN_LAUNCH(ctx, "objective_cols", k_objective_cols<K>, dim3(1), dim3(256), 0, n, col_ptr, V, lambda, weighted,
              (const double *)part, kRedBlocks, out_dev);
  return OPEN_OK;
}

static open_status objective_dispatch(open_ctx *ctx, int k, int64_t m, int n, const int64_t *row_ptr,
                                      const int32_t *col, const float *val, const float *U, const float *V,
                                      float lambda, int weighted, const int64_t *col_ptr, double *out_dev) {
  switch (k) {
    case 8: return objective_impl<8>(ctx, m, n, row_ptr, col, val, U, V, lambda, weighted, col_ptr, out_dev);
    case 16: return objective_impl<16>(ctx, m, n, row_ptr, col, val, U, V, lambda, weighted, col_ptr, out_dev);
    case 32: return objective_impl<32>(ctx, m, n, row_ptr, col, val, U, V, lambda, weighted, col_ptr, out_dev);
    default: return objective_impl<64>(ctx, m, n, row_ptr, col, val, U, V, lambda, weighted, col_ptr, out_dev);
  }
}

}  // namespace openk

using namespace openk;

extern "C" {

open_status open_csr_to_csc(open_ctx *ctx, int64_t m, int32_t n, const int64_t *row_ptr, const int32_t *col,
                            const float *val, int64_t *col_ptr, int32_t *row_idx, float *cval) {
  if (!ctx) return OPEN_E_INVALID;
  if (m < 0 || m >= INT32_MAX) return fail(ctx, OPEN_E_INVALID, "row count must be in [0, 2^31 - 1)");
  if (n <= 0 || n > kMaxCols) return fail(ctx, OPEN_E_INVALID, "column count must be in [1, 4096]");
  if (!row_ptr || !col_ptr || (m > 0 && (!col || !val || !row_idx || !cval)))
    return fail(ctx, OPEN_E_INVALID, "pointers must not be NULL");
  OPEN_HIP_TRY(ctx, hipSetDevice(ctx->device));
  int64_t nnz = 0;
  if (m > 0) {
    OPEN_HIP_TRY(ctx, hipMemcpyAsync(&nnz, row_ptr + m, sizeof(int64_t), hipMemcpyDeviceToHost, ctx->stream));
    OPEN_HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
  }
  open_status st = check_cols(ctx, nnz, col, n);
  if (st) return st;
  return csr_to_csc_dev(ctx, m, n, nnz, row_ptr, col, val, col_ptr, row_idx, cval);
}

open_status open_objective(open_ctx *ctx, int64_t m, int32_t n, int32_t k, const int64_t *row_ptr,
                           const int32_t *col, const float *val, const float *U, const float *V, float lambda,
                           int32_t weighted, double *out) {
  if (!ctx) return OPEN_E_INVALID;
  if (!(k == 8 || k == 16 || k == 32 || k == 64)) return fail(ctx, OPEN_E_UNSUPPORTED, "rank must be 8, 16, 32 or 64");
  if (m < 0 || m >= INT32_MAX || n <= 0 || n > kMaxCols || !out || !U || !V || !row_ptr)
    return fail(ctx, OPEN_E_INVALID, "bad shape or pointer");
  OPEN_HIP_TRY(ctx, hipSetDevice(ctx->device));
  // the column weights w^j are the column counts: they come from the column-view pass
  void *cp, *ri, *cv;
  open_status st;
  int64_t nnz;
  OPEN_HIP_TRY(ctx, hipMemcpyAsync(&nnz, row_ptr + m, sizeof(int64_t), hipMemcpyDeviceToHost, ctx->stream));
  OPEN_HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
  if ((st = check_cols(ctx, nnz, col, n))) return st;
  if ((st = ws_get(ctx, open_ctx::WS_CSC_PTR, sizeof(int64_t) * (n + 1), &cp))) return st;
  if ((st = ws_get(ctx, open_ctx::WS_CSC_IDX, sizeof(int32_t) * (size_t)(nnz > 0 ? nnz : 1), &ri))) return st;
  if ((st = ws_get(ctx, open_ctx::WS_CSC_VAL, sizeof(float) * (size_t)(nnz > 0 ? nnz : 1), &cv))) return st;
  if ((st = csr_to_csc_dev(ctx, m, n, nnz, row_ptr, col, val, (int64_t *)cp, (int32_t *)ri, (float *)cv))) return st;
  double *h;
  if ((st = pinned_get(ctx, 64, (void **)&h))) return st;
  void *d;
  if ((st = ws_get(ctx, open_ctx::WS_OBJ, 256, &d))) return st;
  if ((st = objective_dispatch(ctx, k, m, n, row_ptr, col, val, U, V, lambda, weighted, (const int64_t *)cp,
                               (double *)d)))
    return st;
  OPEN_HIP_TRY(ctx, hipMemcpyAsync(h, d, sizeof(double), hipMemcpyDeviceToHost, ctx->stream));
  OPEN_HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
  *out = h[0];
  return OPEN_OK;
}

open_status open_residual(open_ctx *ctx, int64_t m, int32_t n, int32_t k, const int64_t *row_ptr,
                          const int32_t *col, const float *val, const float *U, const float *V, float *rho) {
  if (!ctx) return OPEN_E_INVALID;
  if (!(k == 8 || k == 16 || k == 32 || k == 64)) return fail(ctx, OPEN_E_UNSUPPORTED, "rank must be 8, 16, 32 or 64");
  if (m < 0 || m >= INT32_MAX || n <= 0 || (m > 0 && (!rho || !U || !V || !row_ptr)))
    return fail(ctx, OPEN_E_INVALID, "bad shape or pointer");
  if (m == 0) return OPEN_OK;
  OPEN_HIP_TRY(ctx, hipSetDevice(ctx->device));
  int64_t blocks = (m + 3) / 4;
  if (blocks > ctx->num_cu * 8) blocks = ctx->num_cu * 8;
  const dim3 g((unsigned)blocks), b(256);
  switch (k) {
    case 8: OPEN_LAUNCH(ctx, "residual", k_residual<8>, g, b, 0, m, n, row_ptr, col, val, U, V, rho); break;
    case 16: OPEN_LAUNCH(ctx, "residual", k_residual<16>, g, b, 0, m, n, row_ptr, col, val, U, V, rho); break;
    case 32: OPEN_LAUNCH(ctx, "residual", k_residual<32>, g, b, 0, m, n, row_ptr, col, val, U, V, rho); break;
    default: OPEN_LAUNCH(ctx, "residual", k_residual<64>, g, b, 0, m, n, row_ptr, col, val, U, V, rho); break;
  }
  return OPEN_OK;
}

// ALS-WR sweeps.  The column view and both bucketings are built once per call.
open_status open_fit(open_ctx *ctx, int64_t m, int32_t n, int32_t k, const int64_t *row_ptr, const int32_t *col,
                     const float *val, float lambda, int32_t weighted, int32_t sweeps, float *U, float *V,
                     double *obj_hist) {
  if (!ctx) return OPEN_E_INVALID;
  if (!(k == 8 || k == 16 || k == 32 || k == 64)) return fail(ctx, OPEN_E_UNSUPPORTED, "rank must be 8, 16, 32 or 64");
  if (m <= 0 || m >= INT32_MAX || n <= 0 || n > kMaxCols || sweeps < 0 || !row_ptr || !col || !val || !U || !V)
    return fail(ctx, OPEN_E_INVALID, "bad shape or pointer");
  if (!(lambda >= 0.0f) || !isfinite(lambda)) return fail(ctx, OPEN_E_INVALID, "lambda must be finite and >= 0");
  OPEN_HIP_TRY(ctx, hipSetDevice(ctx->device));
  int64_t nnz;
  OPEN_HIP_TRY(ctx, hipMemcpyAsync(&nnz, row_ptr + m, sizeof(int64_t), hipMemcpyDeviceToHost, ctx->stream));
  OPEN_HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
  // caller-independent buffers of this call: the column view and the two bucketings
  int64_t *cp = nullptr;
  int32_t *ri = nullptr;
  RowRef *list_r = nullptr, *list_c = nullptr;
  float *cv = nullptr;
  int64_t *cls_r = nullptr, *cls_c = nullptr;
  double *obj_d = nullptr;
  open_status st = OPEN_OK;
  auto cleanup = [&]() {
    (void)hipStreamSynchronize(ctx->stream);
    (void)hipFree(cp);
    (void)hipFree(ri);
    (void)hipFree(cv);
    (void)hipFree(list_r);
    (void)hipFree(list_c);
    (void)hipFree(cls_r);
    (void)hipFree(cls_c);
    (void)hipFree(obj_d);
  };
  if (hipMalloc(&cp, sizeof(int64_t) * (n + 1)) != hipSuccess ||
      hipMalloc(&ri, sizeof(int32_t) * (size_t)(nnz > 0 ? nnz : 1)) != hipSuccess ||
      hipMalloc(&cv, sizeof(float) * (size_t)(nnz > 0 ? nnz : 1)) != hipSuccess ||
      hipMalloc(&list_r, sizeof(RowRef) * (size_t)m) != hipSuccess ||
      hipMalloc(&list_c, sizeof(RowRef) * (size_t)n) != hipSuccess ||
      hipMalloc(&cls_r, sizeof(int64_t) * 2 * kNumClasses) != hipSuccess ||
      hipMalloc(&cls_c, sizeof(int64_t) * 2 * kNumClasses) != hipSuccess ||
      hipMalloc(&obj_d, sizeof(double) * 2 * (sweeps > 0 ? sweeps : 1)) != hipSuccess) {
    (void)hipGetLastError();
    cleanup();
    return fail(ctx, OPEN_E_NOMEM, "fit buffers");
  }
  do {
    if ((st = check_cols(ctx, nnz, col, n))) break;
    if ((st = csr_to_csc_dev(ctx, m, n, nnz, row_ptr, col, val, cp, ri, cv))) break;
    RowRef *l;
    int64_t *c;
    if ((st = bucket_rows(ctx, m, row_ptr, n, k, &l, &c, kSplitMin))) break;
    if (hipMemcpyAsync(list_r, l, sizeof(RowRef) * m, hipMemcpyDeviceToDevice, ctx->stream) != hipSuccess ||
        hipMemcpyAsync(cls_r, c, sizeof(int64_t) * 2 * kNumClasses, hipMemcpyDeviceToDevice, ctx->stream) !=
            hipSuccess) {
      st = fail(ctx, OPEN_E_DEVICE, "copy");
      break;
    }
    if ((st = bucket_rows(ctx, n, cp, (int)m, k, &l, &c, kSplitMin))) break;
    if (hipMemcpyAsync(list_c, l, sizeof(RowRef) * n, hipMemcpyDeviceToDevice, ctx->stream) != hipSuccess ||
        hipMemcpyAsync(cls_c, c, sizeof(int64_t) * 2 * kNumClasses, hipMemcpyDeviceToDevice, ctx->stream) !=
            hipSuccess) {
      st = fail(ctx, OPEN_E_DEVICE, "copy");
      break;
    }
    auto sweep = [&]() -> open_status {
      open_status e;
      if ((e = rowsolve_launch(ctx, V, n, k, row_ptr, col, val, lambda, weighted, list_r, cls_r, U, nullptr, m)))
        return e;
      if ((e = splitk_launch(ctx, V, n, k, col, val, lambda, weighted, list_r, cls_r, U, nullptr, m, nnz))) return e;
      if ((e = rowsolve_launch(ctx, U, (int)m, k, cp, ri, cv, lambda, weighted, list_c, cls_c, V, nullptr, n)))
        return e;
      return splitk_launch(ctx, U, (int)m, k, ri, cv, lambda, weighted, list_c, cls_c, V, nullptr, n, nnz);
    };
    if (!obj_hist && sweeps >= 2 && !ctx->prof_on) {
      // the first sweep runs eagerly (and sizes the workspaces); the others replay it as one graph
      if ((st = sweep())) break;
      hipGraph_t g = nullptr;
      if ((st = graph_capture(ctx, sweep, &g))) break;
      hipGraphExec_t ex = nullptr;
      if (hipGraphInstantiate(&ex, g, nullptr, nullptr, 0) != hipSuccess) {
        (void)hipGetLastError();
        (void)hipGraphDestroy(g);
        st = fail(ctx, OPEN_E_DEVICE, "graph instantiation failed");
        break;
      }
      for (int s = 1; s < sweeps && !st; ++s)
        if (hipGraphLaunch(ex, ctx->stream) != hipSuccess) st = fail(ctx, OPEN_E_DEVICE, "graph launch failed");
      (void)hipStreamSynchronize(ctx->stream);  // the graph is released below
      (void)hipGraphExecDestroy(ex);
      (void)hipGraphDestroy(g);
      break;
    }
    for (int s = 0; s < sweeps && !st; ++s) {
      if ((st = rowsolve_launch(ctx, V, n, k, row_ptr, col, val, lambda, weighted, list_r, cls_r, U, nullptr, m)))
        break;
      if ((st = splitk_launch(ctx, V, n, k, col, val, lambda, weighted, list_r, cls_r, U, nullptr, m, nnz))) break;
      if (obj_hist &&
          (st = objective_dispatch(ctx, k, m, n, row_ptr, col, val, U, V, lambda, weighted, cp, obj_d + 2 * s)))
        break;
      if ((st = rowsolve_launch(ctx, U, (int)m, k, cp, ri, cv, lambda, weighted, list_c, cls_c, V, nullptr, n)))
        break;
      if ((st = splitk_launch(ctx, U, (int)m, k, ri, cv, lambda, weighted, list_c, cls_c, V, nullptr, n, nnz))) break;
      if (obj_hist &&
          (st = objective_dispatch(ctx, k, m, n, row_ptr, col, val, U, V, lambda, weighted, cp, obj_d + 2 * s + 1)))
        break;
    }
    if (!st && obj_hist && sweeps > 0) {
      if (hipMemcpyAsync(obj_hist, obj_d, sizeof(double) * 2 * sweeps, hipMemcpyDeviceToHost, ctx->stream) ||
          hipStreamSynchronize(ctx->stream))
        st = fail(ctx, OPEN_E_DEVICE, "objective copy");
    }
  } while (0);
  cleanup();
  return st;
}

// Warm-started refit on the union of the offline rows and newly arrived rows: the new rows are
// folded in against the current V, then `sweeps` ALS sweeps run on the union from there.
open_status open_refit(open_ctx *ctx, int64_t m_old, int64_t m_new, int32_t n, int32_t k, const int64_t *row_ptr,
                       const int32_t *col, const float *val, float lambda, int32_t weighted, int32_t sweeps, float *U,
                       float *V, double *obj_hist) {
  if (!ctx) return OPEN_E_INVALID;
  if (m_old < 0 || m_new < 0 || m_old + m_new <= 0 || !U || !V || !row_ptr)
    return fail(ctx, OPEN_E_INVALID, "bad shape or pointer");
  open_status st;
  if (m_new > 0 &&
      (st = open_foldin(ctx, V, n, k, m_new, row_ptr + m_old, col, val, lambda, weighted, U + m_old * (int64_t)k,
                        nullptr)))
    return st;
  return open_fit(ctx, m_old + m_new, n, k, row_ptr, col, val, lambda, weighted, sweeps, U, V, obj_hist);
}

}  // extern "C"
