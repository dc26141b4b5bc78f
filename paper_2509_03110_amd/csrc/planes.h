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

}  // namespace lsam
