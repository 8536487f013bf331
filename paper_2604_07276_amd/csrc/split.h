// FP32 matrix-core operands as two f16 terms.
//
// gfx950 multiplies f16 sixteen times as fast as FP32 (v_mfma_f32_16x16x32_f16
// takes 16 cycles for 16x16x32, v_mfma_f32_16x16x4_f32 32 for 16x16x4).  An
// FP32 value scaled by a power of two, so that the largest of its row lies in
// [2^14, 2^15), is written as x = hi + lo, hi = f16(x), lo = f16(x - hi): 22 to
// 24 significant bits down to 2^-17 of the row's largest value and an absolute
// 2^-39 of that value below.  Both terms share one dword (hi in the low half),
// so a packed array has the size and the indexing of the FP32 one, and one
// 16-byte read of four packed values is a whole f16 operand: eight slots,
// (hi, lo) of four depths.  Against it the other operand is fed twice, with
// its lo terms and then its hi terms duplicated into both slots of each depth,
// which sums all four products hi hi + hi lo + lo hi + lo lo of 16 depths in
// two MFMAs (32 cycles) where FP32 takes four (128 cycles).
//
// The products of f16 terms are exact and the matrix core rounds once or so
// per MFMA instead of once per depth.  Scales are powers of two and so exact;
// f16 subnormals are not flushed by these instructions.  Forces on small systems
// are off by 5e-7 to 2.7e-6 of their root mean square, where the whole model in
// FP32 on the CPU is off by 1.1e-6 to 6.4e-6; without the lo terms it would be
// 2.5e-4 and more (tests/test_gpu_split_scales.py bounds it at 2e-5).
//
// The bound on small values is one against the row's largest, so rows must not
// hold values of very different scales that matter alike.  Each row of W^T and
// of the pair tensors has a scale of its own, and the channels of W_Q and W_K,
// and of W_V and W_O, are balanced when weights are loaded.  An infinite value
// makes its row's products NaN; in FP32 they would be infinite or NaN, and NaN
// after the next sum over features of both signs.
//
// Only products of the input-gradient adjoint take these operands.  The
// forward up to the attention logits keeps FP32 MFMAs in their order: its
// rounding, whichever it is, is amplified at rare centres (about 1e4-fold), so
// that another rounding moves the forces by 1e-5 of their size, where the
// adjoint, which is linear in what it propagates, moves them by 4e-7.
#ifndef DPA1_SPLIT_H
#define DPA1_SPLIT_H

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dpa1 {
namespace split {

typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t packx4 __attribute__((ext_vector_type(4)));
typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));

// Power-of-two scale that takes a largest magnitude m to [2^14, 2^15), and its
// inverse.  m below 2^-100 (zero rows) takes that of 2^-100.
struct Scale {
  float up, down;
};
__host__ __device__ __forceinline__ Scale scale_of(float m) {
  uint32_t b;
  __builtin_memcpy(&b, &m, 4);
  b = (b >> 23) & 255u;
  b = b < 27u ? 27u : (b > 254u ? 254u : b);
  const uint32_t u = (268u - b) << 23, d = (b - 14u) << 23;
  Scale s;
  __builtin_memcpy(&s.up, &u, 4);
  __builtin_memcpy(&s.down, &d, 4);
  return s;
}

// The inverse of scale_of's up.
__device__ __forceinline__ float down_of(float up) {
  return __builtin_bit_cast(float, (254u << 23) - __builtin_bit_cast(uint32_t, up));
}

// Four scaled values, each as hi | lo << 16.
__device__ __forceinline__ packx4 pack(const floatx4 &x) {
  packx4 o;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const floatx2 a = {x[2 * i], x[2 * i + 1]};
    const halfx2 h = __builtin_convertvector(a, halfx2);
    const floatx2 rest = {a[0] - (float)h[0], a[1] - (float)h[1]};
    const halfx2 l = __builtin_convertvector(rest, halfx2);
    const uint32_t hu = __builtin_bit_cast(uint32_t, h), lu = __builtin_bit_cast(uint32_t, l);
    o[2 * i] = __builtin_amdgcn_perm(lu, hu, 0x05040100u);
    o[2 * i + 1] = __builtin_amdgcn_perm(lu, hu, 0x07060302u);
  }
  return o;
}

// The hi (lo) terms of four packed values in both slots of each depth.
__device__ __forceinline__ halfx8 dup_hi(const packx4 &p) {
  packx4 o;
#pragma unroll
  for (int i = 0; i < 4; ++i) o[i] = __builtin_amdgcn_perm(p[i], p[i], 0x01000100u);
  return __builtin_bit_cast(halfx8, o);
}
__device__ __forceinline__ halfx8 dup_lo(const packx4 &p) {
  packx4 o;
#pragma unroll
  for (int i = 0; i < 4; ++i) o[i] = __builtin_amdgcn_perm(p[i], p[i], 0x03020302u);
  return __builtin_bit_cast(halfx8, o);
}

__device__ __forceinline__ floatx4 mfma(const packx4 &a, const halfx8 &b, const floatx4 &c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(halfx8, a), b, c, 0, 0, 0);
}

__device__ __forceinline__ float max_abs(float m, const floatx4 &x) {
  return fmaxf(fmaxf(fmaxf(m, fabsf(x[0])), fmaxf(fabsf(x[1]), fabsf(x[2]))), fabsf(x[3]));
}
// Largest over the four lanes that hold one row (lanes that share lane % 16).
__device__ __forceinline__ float row_max(float m) {
  m = fmaxf(m, __shfl_xor(m, 16));
  return fmaxf(m, __shfl_xor(m, 32));
}

}  // namespace split
}  // namespace dpa1

#endif  // DPA1_SPLIT_H
