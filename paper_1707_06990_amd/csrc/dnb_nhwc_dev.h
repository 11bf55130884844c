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

// Packed weights are kept in fragment order: [taps][M-tile of 16][K-step of 32][lane][8], lane (j, g)
// holding row j, K indexes 8g..8g+7.  A wave's operand load is then 1 KB of consecutive memory; as rows
// of K32 elements it was sixteen 64-byte pieces at strides that fall on few L2 channels.  With the row
// sums of dnb_stats.h: DenseNet-264-shaped step 16.0 -> 15.1 ms, DenseNet-161-shaped 14.0 -> 13.0 ms.
__device__ __forceinline__ const u16* wfrag(const u16* W, int K32, int mtile, int kstep) {
  return W + ((int64_t)mtile * (K32 >> 5) + kstep) * 512 + (threadIdx.x & 63) * 8;
}
// position e inside one tap's [M16][K32] block -> row, K index
__device__ __forceinline__ void wunfrag(int e, int K32, int& m, int& k) {
  const int mt = e / (16 * K32), r = e - mt * 16 * K32, lane = (r >> 3) & 63;
  m = mt * 16 + (lane & 15);
  k = (r >> 9) * 32 + 8 * (lane >> 4) + (r & 7);
}

__device__ __forceinline__ f32x4 mfma_bf16(const V8& a, const V8& b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, b.v, c, 0, 0, 0);
}

}  // namespace
}  // namespace nhwc
}  // namespace dnb
