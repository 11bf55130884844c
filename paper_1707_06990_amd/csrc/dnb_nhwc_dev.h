// Device helpers shared by the bf16 / NHWC kernel files: bf16 conversions, the 16-byte operand
// fragment and its matrix instruction.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dnb {
namespace nhwc {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16;

__device__ __forceinline__ float bf2f(u16 v) { return __uint_as_float((unsigned)v << 16); }
// round to nearest even (the hardware conversion of gfx950)
__device__ __forceinline__ u16 f2bf(float f) {
  const __bf16 b = (__bf16)f;
  return __builtin_bit_cast(u16, b);
}

union V8 {          // 8 bf16 = 16 bytes
  uint4 q;
  u16 h[8];
  bf16x8 v;
};

__device__ __forceinline__ f32x4 mfma_bf16(const V8& a, const V8& b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, b.v, c, 0, 0, 0);
}

}  // namespace
}  // namespace nhwc
}  // namespace dnb
