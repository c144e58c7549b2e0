// Device pieces of the surrogate network shared by its inference and its training: bfloat16
// packing, the activations, the sparse first layer's steps and the MFMA operand order.
#pragma once
#include "common.h"

namespace openk {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

typedef float f2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
// float32 -> bfloat16, round to nearest even (NaN stays NaN): the gfx950 conversion
// instruction v_cvt_pk_bf16_f32, two values at a time; bf16pack(a, b) has a in the low half
__device__ __forceinline__ uint32_t bf16pack(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2v{a, b}, bf16x2v));
}
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ __forceinline__ float bf2f(uint16_t b) { return __builtin_bit_cast(float, (uint32_t)b << 16); }

// GELU(z) = z Phi(z) (the erf form), with Phi(z) evaluated as the logistic function of an odd
// polynomial, Phi(z) ~ 1 / (1 + exp(-(a z + b z^3 + c z^5))), whose three coefficients were
// fitted to minimise the largest error of GELU over the real line (a = 1.5950157,
// b = 0.07401132, c = -7.030379e-4; the polynomial is taken at z clamped to [-10, 10], where
// it is increasing; GELU is taken as 0 below -10).  Largest absolute error of GELU: 2.5e-5,
// below the bfloat16 rounding of the activations that follows.  One exponential, one
// reciprocal and eight other instructions.
// The constants below are -log2(e) times the coefficients (the exponential is exp2).
constexpr float kGeluC0 = -2.301121234893799f, kGeluC1 = -0.10677576065063477f, kGeluC2 = 0.0010142693063244224f;
__device__ __forceinline__ float gelu_t(float z) {
  const float zc = __builtin_amdgcn_fmed3f(z, -10.0f, 10.0f);
  const float z2 = zc * zc;
  return zc * __builtin_fmaf(z2, __builtin_fmaf(z2, kGeluC2, kGeluC1), kGeluC0);
}
__device__ __forceinline__ float gelu(float z) {
  const float v = z * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(gelu_t(z)));
  return z < -10.0f ? 0.0f : v;  // below -10 the clamped polynomial would leave z 9e-13
}
// SELU (Klambauer et al. 2017) and its derivative (the right-hand value at 0 is not taken: z > 0)
constexpr float kSeluA = 1.6732632423543772f, kSeluL = 1.0507009873554805f;
__device__ __forceinline__ float selu(float z) { return z > 0.f ? kSeluL * z : kSeluL * kSeluA * (__expf(z) - 1.f); }
__device__ __forceinline__ float selu_grad(float z) { return z > 0.f ? kSeluL : kSeluL * kSeluA * __expf(z); }
// derivative of the GELU above: s + z s'(z), s = 1 / (1 + e), e = 2^t(z),
// s' = -s^2 e ln2 t'(z), t' = C0 + 3 C1 z^2 + 5 C2 z^4 (0 where z is clamped)
__device__ __forceinline__ float gelu_grad(float z) {
  const float e = __builtin_amdgcn_exp2f(gelu_t(z));
  const float sg = __builtin_amdgcn_rcpf(1.0f + e);
  const float z2 = z * z;
  const float tp = __builtin_fabsf(z) < 10.0f
                       ? __builtin_fmaf(z2, __builtin_fmaf(z2, 5.0f * kGeluC2, 3.0f * kGeluC1), kGeluC0)
                       : 0.0f;
  return sg - z * sg * sg * e * 0.69314718055994531f * tp;
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// Place (in bfloat16 values) of element (o, i) of an N x Kd operand packed in the B (or A)
// order of v_mfma_f32_32x32x16_bf16: tiles of 32 rows o, KS steps of 16 along i; lane
// 32 g + o % 32 of step ks holds i = 16 ks + 8 g .. + 8 as one 16-byte word.
__host__ __device__ __forceinline__ int64_t mfma_slot(int64_t o, int64_t i, int64_t KS) {
  return (((o >> 5) * KS + (i >> 4)) * 64 + ((i >> 3) & 1) * 32 + (o & 31)) * 8 + (i & 7);
}

__device__ __forceinline__ f16 mfma_bf16_32(uint4 a, uint4 b, f16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                 0);
}

// four consecutive batch rows (4 hf .. 4 hf + 3 of group b8) of one unit, rounded, into an operand
// of the weight gradients ([batch / 8][units][8], wgrad.h)
__device__ __forceinline__ void store_pack4(uint16_t *P, int64_t b8, int units, int unit, int hf, const float *x) {
  const uint2 v = uint2{bf16pack(x[0], x[1]), bf16pack(x[2], x[3])};
  *reinterpret_cast<uint2 *>(P + ((b8 * units + unit) * 8 + 4 * hf)) = v;
}
// eight consecutive batch rows (row r at x + r * pitch) of one unit as an operand's 16-byte word
__device__ __forceinline__ uint4 gather_pack8(const uint16_t *x, int pitch) {
  uint32_t q[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) q[c] = (uint32_t)x[2 * c * pitch] | ((uint32_t)x[(2 * c + 1) * pitch] << 16);
  return uint4{q[0], q[1], q[2], q[3]};
}

// The value r of an observed entry as the pair (bf16(r), 1) that multiplies a weight pair
// (value weight, mask weight): one dot product adds a r + c.  The value is rounded to bfloat16
// like the weights (relative error at most 2^-9).  An entry whose column is outside [0, n)
// takes the pair (0, 0): it adds nothing.
__device__ __forceinline__ uint32_t value_pair(float r, bool valid) {
  return valid ? (uint32_t)f2bf(r) | (0x3f80u << 16) : 0u;
}

// The lane's weight pairs of setting j (four units, 16 bytes) from the packed first layer
// through a buffer resource over n settings: j outside [0, n) reads zeros.
__device__ __forceinline__ uint4 w1_pairs(__amdgpu_buffer_rsrc_t rs, int j, int lane) {
  const uint32_t off = ((uint32_t)j << 10) + 16u * (uint32_t)lane;  // j = -1 wraps out of range
  return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, 0));
}

// z += a r + c for the lane's four units (w: their weight pairs), one bfloat16 dot product
// per unit with float32 accumulation.  Every first-layer evaluation (training and inference)
// takes exactly these steps in the row's entry order.
__device__ __forceinline__ void layer1_step(f4 &z, uint4 w, uint32_t p) {
  const bf16x2 y = __builtin_bit_cast(bf16x2, p);
  const uint32_t wq[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
  for (int q = 0; q < 4; ++q) z[q] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, wq[q]), y, z[q], false);
}

}  // namespace openk
