// Arithmetic shared by the Q4_0 GEMM kernels: the same dequantized halves and
// the same SwiGLU in every tile form, so results do not depend on which one a
// shape takes.
#pragma once
#include <hip/hip_runtime.h>

namespace mzk {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// four values of a caller's output, which may start at any element
typedef f32x4 f32x4_out __attribute__((aligned(4)));
typedef f16x4 f16x4_out __attribute__((aligned(2)));
typedef __attribute__((address_space(3))) void lds_void;

__device__ __forceinline__ float silu(float g) { return g / (1.0f + __expf(-g)); }

// silu(g) * u as the GEMM epilogues store it: one rounding, of the product to
// f16 (v_fma_mixlo_f16).  The empty asm keeps it a single half: packed into a
// vector, the product would be rounded to fp32 first.
__device__ __forceinline__ _Float16 swiglu_f16(float g, float u) {
  _Float16 h = (_Float16)(silu(g) * u);
  asm volatile("" : "+v"(h));
  return h;
}

// (x & mask) | magic in one instruction (the mask from a scalar register, the
// magic from a vector register: one scalar operand per VOP3 on this chip)
__device__ __forceinline__ uint32_t and_or(uint32_t x, uint32_t mask, uint32_t magic) {
  uint32_t r;
  asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "s"(mask), "v"(magic));
  return r;
}

// Code pair m (bits 4m and 16 + 4m) of a pre-ordered dword -> d * (q - 8) of
// both, as packed halves.  The integer-to-half step is the published
// exponent-bias conversion of 4-bit integers (Kim et al., arXiv:2211.10017):
// OR-ing a code into the mantissa of a half whose ulp is 1 (or 1/16 for the
// codes of odd pairs) and subtracting the bias gives it exactly.
__device__ __forceinline__ uint32_t dequant_pair(uint32_t w, int m, f16x2 d2) {
  const uint32_t mag_lo = 0x64006400u;   // 1024: code bits 0-3 add q
  const uint32_t mag_hi = 0x54005400u;   // 64: code bits 4-7 add q (ulp 1/16)
  const f16x2 off_lo = {(_Float16)1032.0f, (_Float16)1032.0f};
  const f16x2 off_hi = {(_Float16)72.0f, (_Float16)72.0f};
  const uint32_t v = m < 2 ? w : w >> 8;
  const f16x2 c = __builtin_bit_cast(f16x2, and_or(v, m & 1 ? 0x00F000F0u : 0x000F000Fu, m & 1 ? mag_hi : mag_lo));
  return __builtin_bit_cast(uint32_t, (c - (m & 1 ? off_hi : off_lo)) * d2);
}

// The 8 codes of one dword -> 4 f16x2 of d * (q - 8), pair m in component m.
__device__ __forceinline__ uint4 dequant_dword(uint32_t w, f16x2 d2) {
  return uint4{dequant_pair(w, 0, d2), dequant_pair(w, 1, d2), dequant_pair(w, 2, d2), dequant_pair(w, 3, d2)};
}

}  // namespace mzk
