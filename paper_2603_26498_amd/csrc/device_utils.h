// Small device helpers for gfx950 kernels (wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>
#include "tcmv_internal.h"

namespace tcmv {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

// round-to-nearest-even fp32 -> bf16 (hardware conversion on gfx950)
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  __bf16 b = (__bf16)f;
  return __builtin_bit_cast(uint16_t, b);
}
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  f32x2 v = {lo, hi};
  bf16x2 r = __builtin_convertvector(v, bf16x2);
  return __builtin_bit_cast(uint32_t, r);
}

// GELU, erf form: x/2 * (1 + erf(x / sqrt 2))
__device__ __forceinline__ float gelu_erf(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }

// GELU for bf16 outputs: gelu(x) = max(x, 0) - |x| * Phi(-|x|), with the lower tail of the normal distribution
// evaluated as 2^G(|x|), G a polynomial of degree 5 fitted to log2 Phi(-a) on [0, 5.5] (|error| <= 3.6e-4, so the
// tail is accurate in RELATIVE terms: 2.5e-4).  G goes on falling beyond 5.5, so nothing holds its argument there: the
// product stays within 1.1e-7 of zero (2e-8 * |x| where it was held) and reaches zero.  Absolute error of the product
// <= 3.5e-5; after rounding to bf16 the result is within one bf16 unit in the last place of the rounded exact value (or
// within 2^-22 of it where that is larger), for every finite x; NaN for infinities.  5 fused multiply-adds, one exp2 and two
// other vector instructions, each about 1 % of a large product's write-out.
__device__ __forceinline__ float gelu_bf16(float x) {
  const float a = fabsf(x);
  float t = fmaf(-0.00023325323f, a, 0.004869808f);
  t = fmaf(t, a, -0.044599235f);
  t = fmaf(t, a, -0.46968046f);
  t = fmaf(t, a, -1.1462616f);
  t = fmaf(t, a, -1.0003588f);
  const float tail = __builtin_amdgcn_exp2f(t);     // Phi(-|x|)
  return fmaf(-fabsf(x), tail, fmaxf(x, 0.0f));
}

// silu(x) = x / (1 + exp(-x)) of four values, with the bits of the division.  The compiler's division (12 instructions with
// its scaling and special cases) is most of a gated product's write-out: the quotient by the hardware's reciprocal (1 ulp)
// instead, put right by its own remainder.  Over all 2^32 arguments that gives the division's bits wherever |x| <= 87.3
// (without the remainder 2.4 % of them are one step off); beyond, the denominator's reciprocal is subnormal or the
// remainder not a number, and such a lane divides.
__device__ __forceinline__ void silu4(const float (&x)[4], float (&y)[4]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float d = 1.0f + __expf(-x[j]), r = __builtin_amdgcn_rcpf(d), q = x[j] * r;
    y[j] = fmaf(-fmaf(d, q, -x[j]), r, q);           // this sign keeps that of a zero
  }
  if (__builtin_expect(fmaxf(fmaxf(fabsf(x[0]), fabsf(x[1])), fmaxf(fabsf(x[2]), fabsf(x[3]))) > 87.0f, 0)) {
#pragma unroll
    for (int j = 0; j < 4; ++j) y[j] = x[j] / (1.0f + __expf(-x[j]));
  }
}

// compile-time loop: f(std::integral_constant<int, 0>) ... f(<N-1>)
template <int I, int N, class F>
__device__ __forceinline__ void static_for_impl(F& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for_impl<I + 1, N>(f);
  }
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) { static_for_impl<0, N>(f); }

// Workgroup `block` of a launch's touching workgroups (a multiple of 8, of nt threads each) reads a word of every line that is
// its own.  Workgroup ids modulo 8 are XCDs: each takes one contiguous eighth of the bytes that are touched.  Those are the rows
// that the product's workgroups on that XCD read where the whole matrix is touched and the output has at most eight tiles of
// rows (the workgroups then walk its columns in such eighths).  Elsewhere, for a matrix that touch_blocks cut short or an
// output of more rows, other XCDs read most of the lines, and what is gained is that they come from the last-level cache.
__device__ __forceinline__ void touch_lines(const Touch& t, unsigned block, unsigned blocks, unsigned nt) {
  const uint32_t part = block & 7, stride = (blocks >> 3) * nt;
  for (int r = 0; r < 4; ++r) {
    const uint32_t lines = t.bytes[r] >> 7;            // a last line that is not whole stays untouched
    const uint32_t lo = (uint32_t)((uint64_t)lines * part >> 3), hi = (uint32_t)((uint64_t)lines * (part + 1) >> 3);
    const char* p = reinterpret_cast<const char*>(t.p[r]);
    for (uint32_t i = lo + (block >> 3) * nt + threadIdx.x; i < hi; i += kTouchLines * stride) {
      uint32_t v[kTouchLines];
#pragma unroll
      for (int j = 0; j < kTouchLines; ++j) v[j] = *reinterpret_cast<const uint32_t*>(p + (size_t)min(i + j * stride, hi - 1) * 128);
#pragma unroll
      for (int j = 0; j < kTouchLines; ++j) asm volatile("" ::"v"(v[j]));
    }
  }
}

// Sum over the 64 lanes, in every lane: the pairs of an exchange with lane ^ 32, ^ 16, ^ 8, ^ 4, ^ 2, ^ 1 (from ^ 4 on the
// lane four further in the row of 16 holds the same value as lane ^ 4), through the vector ALU instead of LDS.
template <int CTRL>
__device__ __forceinline__ float add_dpp(float v) {
  return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float wave_sum(float v) {
  const auto half = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(half[0]) + __uint_as_float(half[1]);
  const auto row = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(row[0]) + __uint_as_float(row[1]);
  v = add_dpp<0x128>(v);                           // row_ror:8
  v = add_dpp<0x124>(v);                           // row_ror:4
  v = add_dpp<0x4E>(v);                            // quad_perm [2,3,0,1]
  return add_dpp<0xB1>(v);                         // quad_perm [1,0,3,2]
}

}  // namespace tcmv
