// Rank-64 ridge solves of rows with more than 32 observed entries (the primal form of the
// fold-in and of the ALS row half-sweep, Section III-B.2, with the ALS-WR weighting of the
// paper's CF reference):
//     (sum_{j in O_i} f_j f_j^T + lambda w_i I_64) u_i = sum_{j in O_i} r_ij f_j.
// The 64 x 64 system of a row does not fit the register layouts of the other size classes.  In large
// batches a wavefront takes four rows:
//   Gram   row by row on v_mfma_f32_16x16x4f32, four observations a step.  Lane (i, o), i = lane % 16,
//          o = lane / 16, loads the dimensions 4 i .. 4 i + 3 of observation o (16 bytes); block b
//          of 16 dimensions is {4 i + b}, and the ten blocks of the lower triangle are formed
//          transposed: register e of lane (i, o) is row 16 b + i, column 16 c + 4 o + e.  Indices
//          and values are staged in LDS 256 at a time, the next ones (of the next row too) loading
//          meanwhile.  All four rows stay in registers, 160 of them.
//   Layout the four lanes i, 16 + i, 32 + i, 48 + i exchange their pieces of the four systems
//          (lane-row swaps, no LDS): then lane row q holds system q, lane i its rows 16 b + i.
//   Solve  right-looking LDL^T without pivoting (SPD) of the four systems at once, 16 lanes each,
//          with the forward substitution fused in: pivot entries move by DPP row broadcast.  The
//          back substitution is a sum per lane and a reduction over the 16 lanes per unknown.
//   Output lane i writes the dimensions 4 i .. 4 i + 3 of its system (16 bytes).
// Bound by the matrix units (80 cycles per observation and SIMD) and the solve's VALU (8000 per row);
// two wavefronts per SIMD overlap part of it.  78,000 rows of 33 to 1023 entries (11.9M): 0.83 ms,
// of which the products need 0.39; 0.93 with the units dealt to the wavefronts in turn; with one row
// per wavefront (32 x 32 x 2 products, one column per lane, every pivot row through LDS: 22,000
// cycles a solve) 1.2 ms, 1.33 before the rows were taken longest first.
//
// Few rows leave a wavefront no four of them, and four in turn are then what the call waits for.  A
// row on its own takes all 64 lanes: the Gram matrix goes through LDS, lane l holds row l of it, the
// multipliers of a pivot go through LDS too (the next pivot's by a lane read, ahead of the others),
// and the back substitution is the one above on 16 lanes.  Both forms take the same products in the
// same order, so a row's bits do not depend on the form.  A pass over m rows, us, each on its own /
// two and more per wavefront (2048 wavefronts on the card):
//   m     of 40 entries  of 100     of 480
//   16      42             43         59 / 132
//   2048    48 / 72        54 / 92    84 / 209
//   4096    68 / 57        79 / 68   139 / 136
// so a row is on its own up to one row a wavefront, and up to two where half of the rows have
// kP64Long entries or more (2049 rows of 480: 111 / 135).  Otherwise units of up to four rows, with
// three or two where these fill the last round better: 6100 rows of 480 175 us with three, 211 with
// four; but past one round of four only where half of the rows have kP64VeryLong entries (12,000 rows
// of 480 320 / 394, of 200 190 / 171).
#include "rowsolve.h"

namespace openk {

constexpr int kP64Waves = 8;    // wavefronts per block
constexpr int kP64Rows = 4;     // rows of a unit, at most
constexpr int kP64Stage = 256;  // entries staged per wavefront, twice
constexpr int kP64Steps = 4;    // MFMA steps (four observations each) whose rows load together
constexpr int kP64Pitch = 68;   // LDS pitch of a row's matrix: 16-byte words of 16 rows cover the banks
constexpr int kP64Long = 128, kP64VeryLong = 384;  // entries, for the rows of a unit

// value of lane SRC of the lane's row of 16 (DPP row broadcast)
template <int SRC>
__device__ __forceinline__ float row16_bcast(float x) {
  return __builtin_bit_cast(float,
                            __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x150 + SRC, 0xf, 0xf, true));
}
// sum over the lane's row of 16
__device__ __forceinline__ float row16_sum(float x) {
  x += quad_xor1(x);
  x += quad_xor2(x);
  x += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x141, 0xf, 0xf, true));  // half mirror
  x += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x140, 0xf, 0xf, true));  // mirror
  return x;
}
// x[q], q = 0..3, of lane row o -> x[o] of lane row q (a 4 x 4 transposition over the lane rows)
__device__ __forceinline__ void swap_lane_rows(float &x0, float &x1, float &x2, float &x3) {
  auto half = [](float &a, float &b) {  // upper half of a <-> lower half of b
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b),
                                                    false, false);
    const unsigned ra = r[0], rb = r[1];  // (a bit cast of the vector element itself reads element 0)
    a = __builtin_bit_cast(float, ra);
    b = __builtin_bit_cast(float, rb);
  };
  auto quarter = [](float &a, float &b) {  // odd rows of a <-> even rows of b
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b),
                                                    false, false);
    const unsigned ra = r[0], rb = r[1];  // (a bit cast of the vector element itself reads element 0)
    a = __builtin_bit_cast(float, ra);
    b = __builtin_bit_cast(float, rb);
  };
  half(x0, x2);
  half(x1, x3);
  quarter(x0, x1);
  quarter(x2, x3);
}

// What both forms share: a wavefront's staging and the Gram matrix of a row.
template <bool FAR>
struct P64Gram {
  const float *__restrict__ F;
  const int32_t *__restrict__ idx;
  const float *__restrict__ val;
  int (*jl_buf)[kP64Stage];
  float (*rl_buf)[kP64Stage];
  __amdgpu_buffer_rsrc_t rs;
  int n, lane, i16, o;
  int stg = 0;  // staging buffer in use
  int jn[kP64Stage / 64];
  float rn[kP64Stage / 64];

  __device__ __forceinline__ void fetch(int64_t beg, int len, int t0) {
#pragma unroll
    for (int e = 0; e < kP64Stage / 64; ++e) {
      const int t = t0 + 64 * e + lane;
      jn[e] = t < len ? idx[beg + t] : -1;
      rn[e] = t < len ? val[beg + t] : 0.f;
    }
  }
  // The ten lower blocks, with the ridge on the diagonal, and the lane's part of the right-hand
  // side of the `len` entries from `beg` on (fetched before); fl: 1 non-finite value, 2 index
  // outside [0, n).  Meanwhile the first entries of the next row load (next() fetches them).
  template <class Next>
  __device__ __forceinline__ void row(int64_t beg, int len, float reg, f4 (&acc)[10], float (&b)[4], int &fl,
                                      Next &&next) {
#pragma unroll
    for (int e = 0; e < 10; ++e) acc[e] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int e = 0; e < 4; ++e) b[e] = 0.f;
    fl = 0;
    // the staged registers -> LDS, then the following entries (of this row or the next) load
    auto stage = [&](int t0) {
      stg ^= 1;
      int *jl = jl_buf[stg];
      float *rl = rl_buf[stg];
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int e = 0; e < kP64Stage / 64; ++e) {
        const bool in = t0 + 64 * e + lane < len;
        const bool ok = jn[e] >= 0 && jn[e] < n;
        if (in && !ok) fl |= 2;
        if (in && !__builtin_isfinite(rn[e])) fl |= 1;
        jl[64 * e + lane] = ok ? jn[e] : -1;
        rl[64 * e + lane] = rn[e];
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      if (t0 + kP64Stage < len)
        fetch(beg, len, t0 + kP64Stage);
      else
        next();
    };
    f4 un[kP64Steps];
    float vn[kP64Steps];
    auto gather = [&](int t0) {
      const int *jl = jl_buf[stg] + t0 % kP64Stage;
      const float *rl = rl_buf[stg] + t0 % kP64Stage;
#pragma unroll
      for (int e = 0; e < kP64Steps; ++e) {
        const int j = jl[4 * e + o];
        vn[e] = rl[4 * e + o];
        if constexpr (FAR)
          un[e] = far_load<4>(F, j, 64, 4 * i16);
        else
          un[e] = bload_f4(rs, (int)(((uint32_t)j * 64u + 4u * i16) * 4u));  // j = -1 wraps out of range: zeros
      }
    };
    stage(0);
    if (len > 0) gather(0);
    for (int t0 = 0; t0 < len; t0 += 4 * kP64Steps) {
      f4 f[kP64Steps];
      float v[kP64Steps];
#pragma unroll
      for (int e = 0; e < kP64Steps; ++e) {
        f[e] = un[e];
        v[e] = vn[e];
      }
      const int t1 = t0 + 4 * kP64Steps;
      if (t1 < len) {  // wave-uniform
        if (t1 % kP64Stage == 0) stage(t1);
        gather(t1);
      }
#pragma unroll
      for (int e = 0; e < kP64Steps; ++e) {
        int t = 0;
#pragma unroll
        for (int bi = 0; bi < 4; ++bi)
#pragma unroll
          for (int bj = 0; bj <= bi; ++bj, ++t)
            acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(f[e][bj], f[e][bi], acc[t], 0, 0, 0);
#pragma unroll
        for (int bi = 0; bi < 4; ++bi) b[bi] = __builtin_fmaf(v[e], f[e][bi], b[bi]);
      }
    }
    // ridge on the diagonal: lane (i, o), register e of a diagonal block is row i, column 4 o + e
#pragma unroll
    for (int bi = 0; bi < 4; ++bi)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[tri(bi, bi)][e] += i16 == 4 * o + e ? reg : 0.f;
#pragma unroll
    for (int bi = 0; bi < 4; ++bi) {
      b[bi] += __shfl_xor(b[bi], 16, 64);
      b[bi] += __shfl_xor(b[bi], 32, 64);
    }
    const unsigned long long f1 = __ballot(fl & 1), f2 = __ballot(fl & 2);
    fl = (f1 ? 1 : 0) | (f2 ? 2 : 0);
  }
};

// The row's output: block b of lane i (of 16) is dimension 4 i + b.
__device__ __forceinline__ void p64_store(float *__restrict__ X, int32_t *__restrict__ status, int row, int cnt,
                                          int i16, const float (&x)[4], int flags, int bad) {
  const bool good = !bad && flags == 0 && cnt > 0;
  *reinterpret_cast<f4 *>(X + (int64_t)row * 64 + 4 * i16) = good ? f4{x[0], x[1], x[2], x[3]} : f4{0.f, 0.f, 0.f, 0.f};
  if (status && i16 == 0)
    status[row] = cnt == 0      ? OPEN_ROW_EMPTY
                  : (flags & 2) ? OPEN_ROW_BADINDEX
                  : (flags & 1) ? OPEN_ROW_NONFINITE
                  : bad         ? OPEN_ROW_NONPOS_PIVOT
                                : OPEN_ROW_OK;
}

// x_p = z_p - sum_{c > p} L[c][p] x_c over the 16 lanes of a system, lane i with the rows 16 b + i:
// nl(b, p) is its -L[16 b + i][p]
template <class NL>
__device__ __forceinline__ void p64_back(const float (&z)[4], float (&xv)[4], int i16, NL &&nl) {
#pragma unroll
  for (int b = 0; b < 4; ++b) xv[b] = 0.f;
  sfor_down<0, 64>([&](auto Pp) {
    constexpr int p = decltype(Pp)::value, bp = p / 16, pp = p % 16;
    float part = __builtin_fmaf(nl(std::integral_constant<int, bp>{}, Pp), xv[bp], 0.f);
    sfor<bp + 1, 4>([&](auto B) { part = __builtin_fmaf(nl(B, Pp), xv[B], part); });
    part = row16_sum(part);
    const float xp = row16_bcast<pp>(z[bp]) + part;
    xv[bp] = i16 == pp ? xp : xv[bp];
  });
}

template <bool FAR>
__global__ __launch_bounds__(64 * kP64Waves) __attribute__((amdgpu_waves_per_eu(2))) void k_primal64(
    const float *__restrict__ F, int n, const int32_t *__restrict__ idx, const float *__restrict__ val,
    const RowRef *__restrict__ list, const int64_t *__restrict__ cls, int c_lo, int c_hi, float lambda, int weighted,
    float *__restrict__ X, int32_t *__restrict__ status) {
  // per wavefront: the staged indices and values; in their place, the matrix of a row that is solved
  // on its own, and behind it two rows of 64
  __shared__ __attribute__((aligned(16))) float lds_all[kP64Waves][64 * kP64Pitch + 128];
  static_assert(4 * kP64Stage <= 64 * kP64Pitch, "staging lies in the matrix area");
  __shared__ int qnext;
  const int64_t first = cls[2 * c_lo];
  const int64_t count = cls[2 * c_hi] + cls[2 * c_hi + 1] - first;
  if ((int64_t)blockIdx.x >= count) return;  // block has no work (uniform)
  if (threadIdx.x == 0) qnext = 2 * kP64Waves;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int i16 = lane & 15, o = lane >> 4;
  P64Gram<FAR> gram{F, idx, val, reinterpret_cast<int(*)[kP64Stage]>(lds_all[w]),
                    reinterpret_cast<float(*)[kP64Stage]>(lds_all[w] + 2 * kP64Stage)};
  if constexpr (!FAR) gram.rs = make_rsrc(F, (uint64_t)n * 64 * sizeof(float));
  gram.n = n;
  gram.lane = lane;
  gram.i16 = i16;
  gram.o = o;
  __syncthreads();
  const GroupQueue<kP64Waves> queue{&qnext};
  const int64_t waves = (int64_t)gridDim.x * kP64Waves;
  // wave-major and the longest rows first: units that cost alike go to different compute units.  A
  // block's units are handed out to its wavefronts one ahead (a unit's records load meanwhile), the
  // first two rounds in order of the wavefronts: then a second unit, where not all get one, goes to
  // the older wavefront of each SIMD, which has precedence (12,000 rows of 200: 171 us a pass, 215
  // with two of them on one SIMD, 181 with the younger ones).
  const int64_t u0 = (int64_t)blockIdx.x + (int64_t)gridDim.x * w;
  const int64_t u1 = u0 + waves;
  auto ridge = [&](int len) { return lambda * (weighted ? (float)len : 1.0f); };

  const bool apart = count <= waves || (count <= 2 * waves && list[first + count / 2].cnt >= kP64Long);
  if (apart) {  // one row at a time
    float *mat = lds_all[w], *lrow = lds_all[w] + 64 * kP64Pitch;
    auto record = [&](int64_t u) -> RowRef { return u < count ? list[first + count - 1 - u] : RowRef{-1, 0, 0}; };
    RowRef rec = record(u0);
    gram.fetch(rec.beg, rec.cnt, 0);
    for (int64_t u = u0, un; u < count; u = un) {
      un = u == u0 ? u1 : count;  // two at most
      const RowRef nxt = record(un);
      f4 acc[10];
      float b[4];
      int flags;
      gram.row(rec.beg, rec.cnt, ridge(rec.cnt), acc, b, flags, [&] { gram.fetch(nxt.beg, nxt.cnt, 0); });
      // the lower blocks to LDS: lane l takes row l (of the order 16 b + i)
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();  // the staged entries are read
#pragma unroll
      for (int bi = 0; bi < 4; ++bi)
#pragma unroll
        for (int bj = 0; bj <= bi; ++bj)
          *reinterpret_cast<f4 *>(mat + (16 * bi + i16) * kP64Pitch + 16 * bj + 4 * o) = acc[tri(bi, bj)];
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      float a[64];
      sfor<0, 16>([&](auto Q) {
        constexpr int q = decltype(Q)::value;
        const f4 x = *reinterpret_cast<const f4 *>(mat + lane * kP64Pitch + 4 * q);
#pragma unroll
        for (int e = 0; e < 4; ++e) a[4 * q + e] = x[e];
      });
      float rhs = o == 0 ? b[0] : o == 1 ? b[1] : o == 2 ? b[2] : b[3];
      // LDL^T with fused forward substitution, the same products in the same order as below: a[p]
      // becomes -L[.][p] under the pivot and stays d_p in lane p; lanes above it stay as they are (entries
      // past a lane's block are never used).  The next pivot's column is updated first, by a lane read, and its factors go to
      // the other row buffer while the rest of this pivot's arrive.
      int bad = 0, me = lane;
      float l = 0.f, v = 0.f, s;
      auto pivot = [&](auto Pp) {
        constexpr int p = decltype(Pp)::value;
        asm volatile("" : "+v"(me));  // compared afresh: 64 lane masks would not fit the scalar registers
        const float d = readlane_f32(a[p], p);
        const bool below = me > p;
        bad |= !(d > 0.f);
        s = __builtin_amdgcn_rcpf(d);
        v = below ? a[p] : 0.f;
        l = -v * s;
        lrow[64 * (p & 1) + lane] = l;
        const float under = __builtin_fmaf(-v, readlane_f32(rhs, p) * s, rhs);
        rhs = below ? under : rhs;
        a[p] = below ? l : a[p];
      };
      pivot(std::integral_constant<int, 0>{});
      sfor<0, 63>([&](auto Pp) {
        constexpr int p = decltype(Pp)::value;
        const float vp = v;
        a[p + 1] = __builtin_fmaf(readlane_f32(l, p + 1), vp, a[p + 1]);
        f4 x[16];
        sfor<(p + 2) / 4, 16>([&](auto Q) {
          x[decltype(Q)::value] = *reinterpret_cast<const f4 *>(lrow + 64 * (p & 1) + 4 * decltype(Q)::value);
        });
        pivot(std::integral_constant<int, p + 1>{});
        sfor<p + 2, 64>([&](auto J) {
          constexpr int j = decltype(J)::value;
          a[j] = __builtin_fmaf(x[j / 4][j % 4], vp, a[j]);
        });
      });
      // back substitution: 16 lanes with four rows each
      sfor<0, 16>([&](auto Q) {
        constexpr int q = decltype(Q)::value;
        const f4 x = {a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]};
        *reinterpret_cast<f4 *>(mat + lane * kP64Pitch + 4 * q) = x;
      });
      lrow[lane] = rhs;  // y
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      float z[4], xv[4];
#pragma unroll
      for (int bi = 0; bi < 4; ++bi) {
        const int r = 16 * bi + i16;
        z[bi] = lrow[r] * __builtin_amdgcn_rcpf(mat[r * kP64Pitch + r]);
      }
      p64_back(z, xv, i16, [&](auto B, auto Pp) {
        return mat[(16 * decltype(B)::value + i16) * kP64Pitch + decltype(Pp)::value];
      });
      if (o == 0) p64_store(X, status, rec.row, rec.cnt, i16, xv, flags, bad);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();  // the matrix is rewritten by the next row
      rec = nxt;
    }
    return;
  }

  const int64_t full = waves * kP64Rows, rounds = (count + full - 1) / full;
  const bool even = count > 2 * waves && (rounds == 1 || list[first + count / 2].cnt >= kP64VeryLong);
  const int per = even ? (int)((count + waves * rounds - 1) / (waves * rounds)) : kP64Rows;
  const int64_t units = (count + per - 1) / per;
  // the unit's records, row q in lane q (a missing row is an empty one)
  auto records = [&](int64_t u) -> RowRef {
    const int64_t sl = (units - 1 - u) * per + lane;
    return u < units && lane < per && sl < count ? list[first + sl] : RowRef{-1, 0, 0};
  };
  RowRef rec = records(u0);
  if (u0 < units) gram.fetch(readlane_i64(rec.beg, 0), __builtin_amdgcn_readlane(rec.cnt, 0), 0);
  for (int64_t u = u0, un; u < units; u = un) {
    un = u == u0 ? u1 : (int64_t)blockIdx.x + (int64_t)gridDim.x * queue.take();
    const RowRef nxt = records(un);
    float g[kP64Rows][40];  // the four lower block triangles, block (b, c <= b), register e: [4 tri(b, c) + e]
    float rhs[4] = {0.f, 0.f, 0.f, 0.f};
    int flags = 0;          // of the lane row's system
    sfor<0, kP64Rows>([&](auto Q) {
      constexpr int q = decltype(Q)::value;
      const int len = __builtin_amdgcn_readlane(rec.cnt, q);
      f4 acc[10];
      float b[4];
      int fl;
      gram.row(readlane_i64(rec.beg, q), len, ridge(len), acc, b, fl, [&] {
        if constexpr (q + 1 < kP64Rows)
          gram.fetch(readlane_i64(rec.beg, q + 1), __builtin_amdgcn_readlane(rec.cnt, q + 1), 0);
        else
          gram.fetch(readlane_i64(nxt.beg, 0), __builtin_amdgcn_readlane(nxt.cnt, 0), 0);
      });
#pragma unroll
      for (int t = 0; t < 10; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) g[q][4 * t + e] = acc[t][e];
#pragma unroll
      for (int bi = 0; bi < 4; ++bi) rhs[bi] = o == q ? b[bi] : rhs[bi];
      flags = o == q ? fl : flags;
    });
    // lane row q, lane i: st[b][c] = row 16 b + i, column c of system q
    float st[4][64];
    sfor<0, 4>([&](auto B) {
      constexpr int b = decltype(B)::value;
      sfor<0, b + 1>([&](auto C) {
        constexpr int c = decltype(C)::value;
        sfor<0, 4>([&](auto E) {
          constexpr int t = 4 * tri(b, c) + decltype(E)::value;
          swap_lane_rows(g[0][t], g[1][t], g[2][t], g[3][t]);
          sfor<0, 4>([&](auto O) { st[b][16 * c + 4 * decltype(O)::value + decltype(E)::value] = g[O][t]; });
        });
      });
    });
    // ---- LDL^T with fused forward substitution: st[b][p] becomes -L[.][p] below the pivot
    int bad = 0;
    sfor<0, 64>([&](auto Pp) {
      constexpr int p = decltype(Pp)::value, bp = p / 16, pp = p % 16;
      const float d = row16_bcast<pp>(st[bp][p]);
      bad |= !(d > 0.f);
      const float s = __builtin_amdgcn_rcpf(d);
      const float zp = row16_bcast<pp>(rhs[bp]) * s;  // y_p / d_p
      float gc[4];
      sfor<bp, 4>([&](auto B) {
        constexpr int b = decltype(B)::value;
        float v = st[b][p];
        if constexpr (b == bp) v = i16 > pp ? v : 0.f;
        gc[b] = v;
        rhs[b] = __builtin_fmaf(-v, zp, rhs[b]);
        st[b][p] = -v * s;
      });
      rhs[bp] = i16 == pp ? zp : rhs[bp];
      sfor<p + 1, 64>([&](auto J) {
        constexpr int j = decltype(J)::value;
        const float lj = row16_bcast<j % 16>(st[j / 16][p]);  // -L[j][p]
        sfor<j / 16, 4>([&](auto B) {
          constexpr int b = decltype(B)::value;
          st[b][j] = __builtin_fmaf(lj, gc[b], st[b][j]);
        });
      });
    });
    float xv[4];
    p64_back(rhs, xv, i16, [&](auto B, auto Pp) { return st[B][Pp]; });
    // the lane row's record
    const int my_row = __shfl(rec.row, o, 64), my_cnt = __shfl(rec.cnt, o, 64);
    if (my_row >= 0) p64_store(X, status, my_row, my_cnt, i16, xv, flags, bad);
    rec = nxt;
  }
}

// The group of the primal size classes at rank 64 (n_i > 32 below the split-K length): one
// variant, a persistent grid of up to one block per CU.
OPEN_GROUP(g_k64_primal) {
  if (choice != 0) return fail(ctx, OPEN_E_INVALID, "kernel variant out of range");
  int64_t blocks = m < ctx->num_cu ? m : ctx->num_cu;
  if (blocks < 1) blocks = 1;
  OPEN_LAUNCH(ctx, "ridge_k64_primal", (far_factors(n, 64) ? k_primal64<true> : k_primal64<false>),
              dim3((unsigned)blocks), dim3(64 * kP64Waves), 0, F, n, idx, val, list, cls, kPrimalLo, kPrimalHi, lambda,
              weighted, X, status);
  return OPEN_OK;
}

}  // namespace openk
