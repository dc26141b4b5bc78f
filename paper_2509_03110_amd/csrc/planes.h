// Plane values: an fp32 number as NP bfloat16 numbers (see kernels_conv_gemm.hip).
#pragma once
#include <hip/hip_runtime.h>

namespace lsam {

// The pieces of x, as bfloat16 bit patterns.
template <int NP>
__device__ __forceinline__ void split_planes(float x, unsigned short (&o)[NP]) {
  const unsigned ux = __builtin_bit_cast(unsigned, x);
  o[0] = __builtin_bit_cast(unsigned short, static_cast<__bf16>(x));
  if constexpr (NP == 3) {
    // above the largest bfloat16 the rounding would overflow: cut instead (infinity and NaN stay as they are)
    const unsigned mag = ux & 0x7FFFFFFFu;
    if (mag >= 0x7F7F8000u && mag <= 0x7F800000u) o[0] = (unsigned short)(ux >> 16);
    const float r1 = mag < 0x7F800000u ? x - __builtin_bit_cast(float, (unsigned)o[0] << 16) : 0.f;
    o[1] = __builtin_bit_cast(unsigned short, static_cast<__bf16>(r1));
    const float r2 = r1 - __builtin_bit_cast(float, (unsigned)o[1] << 16);
    o[2] = __builtin_bit_cast(unsigned short, static_cast<__bf16>(r2));
  }
}

// The pieces of N values, two to a word, in 6 operations a value instead of the 19 of one at a time: two conversions share an
// instruction.  Numbers that the rounding would make infinite, or that are, come out wrong: the caller looks for them once for
// many values (past_rounding of their largest; NaN needs no care: its pieces are NaN and so is what they are multiplied
// into), and then takes split_words_any.
template <int NP, int N>
__device__ __forceinline__ void split_words(const float (&x)[N], unsigned (&o)[NP][N / 2]) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int w = 0; w < N / 2; ++w) {
    float a = x[2 * w], b = x[2 * w + 1];
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      o[q][w] = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{a, b}, bf16x2));
      a -= __builtin_bit_cast(float, o[q][w] << 16);
      b -= __builtin_bit_cast(float, o[q][w] & 0xFFFF0000u);
    }
  }
}
template <int NP, int N>
__device__ __forceinline__ void split_words_any(const float (&x)[N], unsigned (&o)[NP][N / 2]) {
#pragma unroll
  for (int w = 0; w < N / 2; ++w) {
    unsigned short lo[NP], hi[NP];
    split_planes<NP>(x[2 * w], lo);
    split_planes<NP>(x[2 * w + 1], hi);
#pragma unroll
    for (int q = 0; q < NP; ++q) o[q][w] = (unsigned)lo[q] | (unsigned)hi[q] << 16;
  }
}
__device__ __forceinline__ float largest_of(float most, float x) { return __builtin_fmaxf(most, __builtin_fabsf(x)); }
__device__ __forceinline__ bool past_rounding(float most) {
  return __builtin_expect(most >= __builtin_bit_cast(float, 0x7F7F8000u), 0);
}

// Results with three planes from their two sums, the products of the leading pieces and the other
// five: `leading` becomes both.  An infinite leading sum (or NaN) is the result: the leading piece of a
// finite number is finite, of an infinite one the number itself, so these products overflow, or are
// infinite or NaN, where the products of the numbers are, while the small ones may then be infinite
// with the other sign.  (One look at the largest of sixteen: a compare and a choice for each value cost
// 16-channel layers 1.3 %.)
template <typename F32x16>
__device__ __forceinline__ void join_sums(F32x16& leading, F32x16& small) {
  float most = 0.f;
#pragma unroll
  for (int e = 0; e < 16; ++e) most = __builtin_fmaxf(most, __builtin_fabsf(leading[e]));
  if (__builtin_expect(__builtin_isinf(most), 0)) {
#pragma unroll
    for (int e = 0; e < 16; ++e)
      if (__builtin_isinf(leading[e])) small[e] = 0.f;
  }
#pragma unroll
  for (int e = 0; e < 16; ++e) leading[e] += small[e];
}

}  // namespace lsam
