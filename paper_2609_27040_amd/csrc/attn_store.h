// Final attention outputs in the caller's element type (device code only).
#pragma once

#include "kernels.h"

namespace ema {

// fp32 -> bf16 with round to nearest, ties to even; NaN stays a quiet NaN.
__device__ __forceinline__ uint16_t f32_to_bf16_rne(float v) {
  const uint32_t u = __builtin_bit_cast(uint32_t, v);
  if ((u & 0x7fffffffu) > 0x7f800000u) return uint16_t((u >> 16) | 0x0040u);
  return uint16_t((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

// out[idx] = v in a.out_dtype (fp16 conversion rounds to nearest even).
__device__ __forceinline__ void store_out(const AttnArgs& a, int64_t idx, float v) {
  if (a.out_dtype == kOutF32) {
    static_cast<float*>(a.out)[idx] = v;
  } else if (a.out_dtype == kOutBF16) {
    static_cast<uint16_t*>(a.out)[idx] = f32_to_bf16_rne(v);
  } else {
    static_cast<_Float16*>(a.out)[idx] = _Float16(v);
  }
}

typedef float out_f32x4 __attribute__((ext_vector_type(4)));

// out[idx .. idx + 4) = v (idx a multiple of 4): one store where the output is
// aligned for it, else one per element.
__device__ __forceinline__ void store_out4(const AttnArgs& a, int64_t idx, out_f32x4 v) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  if (!a.out_vec) {
#pragma unroll 1
    for (int i = 0; i < 4; ++i)
      store_out(a, idx + i, i == 0 ? v[0] : i == 1 ? v[1] : i == 2 ? v[2] : v[3]);
  } else if (a.out_dtype == kOutF32) {
    *reinterpret_cast<out_f32x4*>(static_cast<float*>(a.out) + idx) = v;
  } else {
    uint32_t h[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      h[i] = a.out_dtype == kOutBF16 ? f32_to_bf16_rne(v[i])
                                     : __builtin_bit_cast(uint16_t, _Float16(v[i]));
    *reinterpret_cast<u32x2*>(static_cast<uint16_t*>(a.out) + idx) =
        u32x2{h[0] | (h[1] << 16), h[2] | (h[3] << 16)};
  }
}

}  // namespace ema
