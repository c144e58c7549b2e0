// Rank-64 ridge solves of rows with more than 32 observed entries (the primal form of the
// fold-in and of the ALS row half-sweep, Section III-B.2, with the ALS-WR weighting of the
// paper's CF reference):
//     (sum_{j in O_i} f_j f_j^T + lambda w_i I_64) u_i = sum_{j in O_i} r_ij f_j.
// The 64 x 64 system of a row does not fit the register layouts of the other size classes.  A
// wavefront takes four rows:
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
#include "rowsolve.h"

namespace openk {

constexpr int kP64Waves = 8;    // wavefronts per block
constexpr int kP64Rows = 4;     // rows of a wavefront
constexpr int kP64Stage = 256;  // entries staged per wavefront, twice
constexpr int kP64Steps = 4;    // MFMA steps (four observations each) whose rows load together

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

template <bool FAR>
__global__ __launch_bounds__(64 * kP64Waves) __attribute__((amdgpu_waves_per_eu(2))) void k_primal64(
    const float *__restrict__ F, int n, const int32_t *__restrict__ idx, const float *__restrict__ val,
    const RowRef *__restrict__ list, const int64_t *__restrict__ cls, int c_lo, int c_hi, float lambda, int weighted,
    float *__restrict__ X, int32_t *__restrict__ status) {
  __shared__ int jl_all[kP64Waves][2][kP64Stage];
  __shared__ float rl_all[kP64Waves][2][kP64Stage];
  __shared__ int qnext;
  if (threadIdx.x == 0) qnext = kP64Waves;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int i16 = lane & 15, o = lane >> 4;
  const int64_t first = cls[2 * c_lo];
  const int64_t count = cls[2 * c_hi] + cls[2 * c_hi + 1] - first;
  const int64_t units = (count + kP64Rows - 1) / kP64Rows;
  const __amdgpu_buffer_rsrc_t rs = make_rsrc(F, (uint64_t)n * 64 * sizeof(float));
  __syncthreads();
  const GroupQueue<kP64Waves> queue{&qnext};
  // wave-major and the longest rows first: units that cost alike go to different compute units; a
  // block's units are handed out to its wavefronts, one ahead (its records load meanwhile)
  const int64_t u0 = (int64_t)blockIdx.x + (int64_t)gridDim.x * w;
  // the unit's records, row q in lane q
  auto records = [&](int64_t u) -> RowRef {
    const int64_t sl = (units - 1 - u) * kP64Rows + lane;
    return u < units && lane < kP64Rows && sl < count ? list[first + sl] : RowRef{-1, 0, 0};
  };
  RowRef rec = records(u0);
  int jn[kP64Stage / 64];
  float rn[kP64Stage / 64];
  auto fetch = [&](int64_t beg, int len, int t0) {
#pragma unroll
    for (int e = 0; e < kP64Stage / 64; ++e) {
      const int t = t0 + 64 * e + lane;
      jn[e] = t < len ? idx[beg + t] : -1;
      rn[e] = t < len ? val[beg + t] : 0.f;
    }
  };
  int stg = 0;  // staging buffer in use
  if (u0 < units) fetch(readlane_i64(rec.beg, 0), __builtin_amdgcn_readlane(rec.cnt, 0), 0);
  for (int64_t u = u0, un; u < units; u = un) {
    un = (int64_t)blockIdx.x + (int64_t)gridDim.x * queue.take();
    const RowRef nxt = records(un);
    float g[kP64Rows][40];  // the four lower block triangles, block (b, c <= b), register e: [4 tri(b, c) + e]
    float rhs[4] = {0.f, 0.f, 0.f, 0.f};
    int flags = 0;          // of the lane row's system: 1 non-finite value, 2 index outside [0, n)
    sfor<0, kP64Rows>([&](auto Q) {
      constexpr int q = decltype(Q)::value;
      const int len = __builtin_amdgcn_readlane(rec.cnt, q);
      const int64_t beg = readlane_i64(rec.beg, q);
      f4 acc[10];
#pragma unroll
      for (int e = 0; e < 10; ++e) acc[e] = f4{0.f, 0.f, 0.f, 0.f};
      float b[4] = {0.f, 0.f, 0.f, 0.f};
      int fl = 0;
      // the staged registers -> LDS, then the following entries (of this row or the next) load
      auto stage = [&](int t0) {
        stg ^= 1;
        int *jl = jl_all[w][stg];
        float *rl = rl_all[w][stg];
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
        else if constexpr (q + 1 < kP64Rows)
          fetch(readlane_i64(rec.beg, q + 1), __builtin_amdgcn_readlane(rec.cnt, q + 1), 0);
        else
          fetch(readlane_i64(nxt.beg, 0), __builtin_amdgcn_readlane(nxt.cnt, 0), 0);
      };
      f4 un[kP64Steps];
      float vn[kP64Steps];
      auto gather = [&](int t0) {
        const int *jl = jl_all[w][stg] + t0 % kP64Stage;
        const float *rl = rl_all[w][stg] + t0 % kP64Stage;
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
      const float reg = lambda * (weighted ? (float)len : 1.0f);
#pragma unroll
      for (int bi = 0; bi < 4; ++bi)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[tri(bi, bi)][e] += i16 == 4 * o + e ? reg : 0.f;
#pragma unroll
      for (int t = 0; t < 10; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) g[q][4 * t + e] = acc[t][e];
#pragma unroll
      for (int bi = 0; bi < 4; ++bi) {
        float s = b[bi];
        s += __shfl_xor(s, 16, 64);
        s += __shfl_xor(s, 32, 64);
        rhs[bi] = o == q ? s : rhs[bi];
      }
      const unsigned long long f1 = __ballot(fl & 1), f2 = __ballot(fl & 2);
      const int all = (f1 ? 1 : 0) | (f2 ? 2 : 0);
      flags = o == q ? all : flags;
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
    // ---- back substitution: x_p = z_p - sum_{c > p} L[c][p] x_c
    float xv[4] = {0.f, 0.f, 0.f, 0.f};
    sfor_down<0, 64>([&](auto Pp) {
      constexpr int p = decltype(Pp)::value, bp = p / 16, pp = p % 16;
      float part = __builtin_fmaf(st[bp][p], xv[bp], 0.f);
      sfor<bp + 1, 4>([&](auto B) { part = __builtin_fmaf(st[B][p], xv[B], part); });
      part = row16_sum(part);
      const float xp = row16_bcast<pp>(rhs[bp]) + part;
      xv[bp] = i16 == pp ? xp : xv[bp];
    });
    // the lane row's record
    const int my_row = __shfl(rec.row, o, 64), my_cnt = __shfl(rec.cnt, o, 64);
    if (my_row >= 0) {
      const bool good = !bad && flags == 0 && my_cnt > 0;
      // block b of lane i is dimension 4 i + b
      *reinterpret_cast<f4 *>(X + (int64_t)my_row * 64 + 4 * i16) =
          good ? f4{xv[0], xv[1], xv[2], xv[3]} : f4{0.f, 0.f, 0.f, 0.f};
      if (status && i16 == 0)
        status[my_row] = my_cnt == 0   ? OPEN_ROW_EMPTY
                         : (flags & 2) ? OPEN_ROW_BADINDEX
                         : (flags & 1) ? OPEN_ROW_NONFINITE
                         : bad         ? OPEN_ROW_NONPOS_PIVOT
                                       : OPEN_ROW_OK;
    }
    rec = nxt;
  }
}

// The group of the primal size classes at rank 64 (n_i > 32 below the split-K length): one
// variant, a persistent grid of up to one block per CU.
OPEN_GROUP(g_k64_primal) {
  if (choice != 0) return fail(ctx, OPEN_E_INVALID, "kernel variant out of range");
  int64_t blocks = (m + kP64Waves * kP64Rows - 1) / (kP64Waves * kP64Rows);
  const int64_t cap = ctx->num_cu;
  if (blocks > cap) blocks = cap;
  if (blocks < 1) blocks = 1;
  OPEN_LAUNCH(ctx, "ridge_k64_primal", (far_factors(n, 64) ? k_primal64<true> : k_primal64<false>), dim3((unsigned)blocks), dim3(64 * kP64Waves), 0, F, n, idx, val,
              list, cls, kPrimalLo, kPrimalHi, lambda, weighted, X, status);
  return OPEN_OK;
}

}  // namespace openk
