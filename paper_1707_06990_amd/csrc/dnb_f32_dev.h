// Device helpers shared by the fp32 convolution kernel files.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dnb_internal.h"

namespace dnb {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// D(16x16) += A(16x4) * B(4x16).  Lane l supplies A[l%16][l/16] and B[l/16][l%16] and holds
// D[4*(l/16)+r][l%16] in register r.
__device__ __forceinline__ f32x4 mfma16(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ float4 ldg4(const float* p) { return *reinterpret_cast<const float4*>(p); }
// 16 bytes of LDS in one instruction.  Through float4, a struct, the compiler takes such an access apart where its
// elements are used one by one and, knowing only 4-byte alignment of the LDS array, makes pairs of floats of it, which
// meet banks that the pitches here avoid for 16 bytes.
__device__ __forceinline__ float4 lds_ld4(const float* p) {
  const f32x4 v = *reinterpret_cast<const f32x4*>(p);
  return make_float4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ void lds_st4(float* p, const float4& v) {
  *reinterpret_cast<f32x4*>(p) = (f32x4){v.x, v.y, v.z, v.w};
}
__device__ __forceinline__ float4 zero4() { return make_float4(0.f, 0.f, 0.f, 0.f); }
__device__ __forceinline__ float elem(const float4& v, int e) {
  return e == 0 ? v.x : (e == 1 ? v.y : (e == 2 ? v.z : v.w));
}

__device__ __forceinline__ const float* wfrag(const float* W, int Kpad, int mtile, int chunk) {
  return W + ((int64_t)mtile * (Kpad >> 4) + chunk) * 256 + (threadIdx.x & 63) * 4;
}
// position e inside one tap's [M16][K16] block -> row, channel
__device__ __forceinline__ void wunfrag(int e, int K16, int& m, int& c) {
  const int mt = e / (16 * K16), r = e - mt * 16 * K16, lane = (r >> 2) & 63;
  m = mt * 16 + (lane & 15);
  c = (r >> 8) * 16 + 4 * (r & 3) + (lane >> 4);
}

// Sums the accumulators of the K-split waves of a workgroup (fixed order 0,1,2,...).  M-tile a
// is owned by wave a % nw: every other wave writes its copy of the tile to LDS, the owner adds
// the copies (its own stays in registers, inserted at its place in the order) and keeps the
// result.  red: [MT*NT][nw-1 slots][64 lanes][4].
template <int MT, int NT>
__device__ __forceinline__ void ksplit_reduce(f32x4 (&acc)[MT][NT], float* red, int wave, int lane, int nw) {
  __syncthreads();  // (wave = index inside the K group, nw = waves per K group, red = the group's buffer)
  if (nw == 1) return;
#pragma unroll
  for (int a = 0; a < MT; ++a) {
    const int owner = a % nw;
    if (wave != owner) {
      const int slot = (wave - owner - 1 + nw) % nw;
#pragma unroll
      for (int t = 0; t < NT; ++t)
        *reinterpret_cast<float4*>(&red[((((a * NT + t) * (nw - 1)) + slot) * 64 + lane) * 4]) =
            make_float4(acc[a][t][0], acc[a][t][1], acc[a][t][2], acc[a][t][3]);
    }
  }
  __syncthreads();
#pragma unroll
  for (int a = 0; a < MT; ++a) {
    const int owner = a % nw;
    if (wave == owner) {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        f32x4 s = (f32x4){0.f, 0.f, 0.f, 0.f};
        for (int w = 0; w < nw; ++w) {
          if (w == owner) {
            s[0] += acc[a][t][0]; s[1] += acc[a][t][1]; s[2] += acc[a][t][2]; s[3] += acc[a][t][3];
          } else {
            const int slot = (w - owner - 1 + nw) % nw;
            const float4 v = *reinterpret_cast<const float4*>(
                &red[((((a * NT + t) * (nw - 1)) + slot) * 64 + lane) * 4]);
            s[0] += v.x; s[1] += v.y; s[2] += v.z; s[3] += v.w;
          }
        }
        acc[a][t] = s;
      }
    }
  }
}

// A pending sum of partials carried out by extra workgroups, of 256 threads, of a weight-gradient launch or, without a
// bottleneck, of BN's reduction: kind 1 is k_sum_partials' job, kind 2 k_sum_wgrad3x3's,
// with the same grouping and order of additions, so the sums have the same bits either way.
struct SumRole {
  int kind, wgs;  // kind 0: none; wgs: workgroups the sum needs
  const float* part;
  float* out;
  int splits, G, per;
  long long count;  // elements of one partial
  int gy, gz, mtw, ctw, cin, cout;
};

__device__ __forceinline__ void sum_role(const SumRole& sr, int wg) {
  extern __shared__ float sh[];  // the launch's dynamic LDS: at least 1 KB in every launch that carries a sum
  const int epb = 256 / sr.G;
  const int le = threadIdx.x % epb, grp = threadIdx.x / epb;
  const long long f = (long long)wg * epb + le;
  float s = 0.f;
  if (f < sr.count) {
    int i = grp * sr.per;
    const int end = min(sr.splits, i + sr.per);
    for (; i + 8 <= end; i += 8) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = sr.part[(long long)(i + u) * sr.count + f];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; i < end; ++i) s += sr.part[(long long)i * sr.count + f];
  }
  sh[threadIdx.x] = s;
  __syncthreads();
  if (grp == 0 && f < sr.count) {
    float t = sh[le];
    for (int g = 1; g < sr.G; ++g) t += sh[g * epb + le];
    if (sr.kind == 1) {
      sr.out[f] = t;
    } else {
      const int NT = sr.mtw * sr.ctw * 9;
      const int rr = (int)(f & 3), lane = (int)((f >> 2) & 63);
      const long long tl = f >> 8;
      const int tile = (int)(tl % NT), blk = (int)(tl / NT);
      const int yb = blk % sr.gy, z = blk / sr.gy;
      const int tap = tile % 9, y = (tile / 9) % sr.ctw, x = tile / (9 * sr.ctw);
      const int m = z * (sr.mtw * 16) + x * 16 + 4 * (lane >> 4) + rr;
      const int c = yb * (sr.ctw * 16) + y * 16 + (lane & 15);
      if (m < sr.cout && c < sr.cin) sr.out[((long long)m * sr.cin + c) * 9 + tap] = t;
    }
  }
}

// Grouping of a sum of `splits` partials (the same rule the stand-alone sum kernels use).
inline void sum_grouping(int kind, int splits, int* G, int* per) {
  int g = 1;
  if (kind == 2) { while (g < 16 && splits / (g * 2) >= 4) g *= 2; }   // at least 4 partials per group
  else           { while (g < 16 && splits / g > 16) g <<= 1; }         // about 16 splits per thread
  *G = g;
  *per = (splits + g - 1) / g;
}

inline SumRole make_sum_role(PendingSum* absorb) {
  SumRole sr{};
  if (absorb && absorb->kind != 0) {
    sr.kind = absorb->kind;
    sr.part = absorb->part; sr.out = absorb->out; sr.splits = absorb->splits; sr.count = absorb->count;
    sr.gy = absorb->gy; sr.gz = absorb->gz; sr.mtw = absorb->mtw; sr.ctw = absorb->ctw;
    sr.cin = absorb->cin; sr.cout = absorb->cout;
    sum_grouping(sr.kind, sr.splits, &sr.G, &sr.per);
    const int epb = 256 / sr.G;
    sr.wgs = (int)((sr.count + epb - 1) / epb);
    absorb->kind = 0;
  }
  return sr;
}

}  // namespace
}  // namespace dnb
