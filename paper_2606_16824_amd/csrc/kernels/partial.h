// Stores of an attention kernel's split-K partials (device code).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../cw_internal.h"

namespace cw {
namespace part {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// Elements elem .. elem + 3 of the unnormalised partial O: fp32, or bf16 (relative
// rounding 2^-9, the range of fp32).
__device__ __forceinline__ void put4(const ExtendParams& p, size_t elem, f32x4 v) {
  if (p.part_f32) {
    *reinterpret_cast<f32x4*>(static_cast<float*>(p.part_o) + elem) = v;
  } else {
    bf16x4 v4;
#pragma unroll
    for (int e = 0; e < 4; ++e) v4[e] = static_cast<__bf16>(v[e]);
    *reinterpret_cast<u32x2*>(static_cast<uint16_t*>(p.part_o) + elem) = __builtin_bit_cast(u32x2, v4);
  }
}

}  // namespace part
}  // namespace cw
