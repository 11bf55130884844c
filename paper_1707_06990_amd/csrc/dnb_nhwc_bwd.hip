// bf16 / NHWC backward chain of a bottleneck layer: the kernels that carry the dependence from layer
// l+1 to layer l.
//
//   k_dgrad3s / k_dgrad3   3x3 data gradient of g_l, ReLU mask of BN2 and its two sums in the epilogue
//   k_bn2_apply            gradient of b_l from those sums (element-wise on P x B)
//   dgrad1_body            1x1 data gradient; BN1+ReLU backward and the concatenation's backward
//                          (accumulate into the slab G) in the epilogue, with BN1's two sums
//
// The last is a role of the weight-gradient launch (dnb_nhwc_wgrad.hip), which only needs db_l too, and takes
// layers in pairs: layer l-1 needs of layer l only its own slice of the slab, so beside layer l's weight
// gradients only those k channels are formed, and beside layer l-1's the channels of both layers below, in one
// pass over the slab.  Three launches a layer, and 5 bytes per element of a layer's concatenated input instead of
// 10.  (One at a time where a block has no room for the second gradient of a b_l that a pair keeps, the same role.)
//
// BN1's backward is  du = s*(dz - dbeta/P - xhat*dgamma/P),  dz = the masked gradient, s = gamma*istd.
// Its first term needs no sum, so it is added into the slab where dz is formed; the other two are
// constants per channel times 1 and xhat, and xhat does not depend on the layer (a channel's
// statistics are those of the produced feature).  They are therefore collected per channel,
//   K0 = sum_l s_l*dbeta_l/P,   K1 = sum_l s_l*dgamma_l/P,
// and taken off once, where a slice of the slab is finally read:  g = G - K0 - K1*xhat.  A layer
// by itself then moves 10 bytes per element of its concatenated input (x 2, G 4 + 4) instead of the 22 of
// separate passes (gradient written 2; reduction 2 + 2; element-wise pass 2 + 2 + 4 + 4; the slab's
// initial copy of dy, another 6 per element of the block's output, goes away too: the first layer
// that touches the slab reads dy in its place).  Against the separate passes, on one stream where
// those ran beside a helper stream: DenseNet-264-shaped step at batch 32, 22.5 -> 20.4 ms;
// DenseNet-161-shaped, 17.4 -> 17.2 ms at batch 32, 10.6 -> 8.0 ms at batch 2.
#include "dnb_internal.h"
#include "dnb_nhwc_dev.h"
#include "dnb_stats.h"

namespace dnb {
namespace nhwc {

namespace {

// ---------------------------------------------------------------- 3x3 data gradient

struct Dgrad3Args {
  const u16* dy;                        // last layer: the slice of dy, row stride g_ld; else null
  const float* G; int64_t g_ld;         // slab at the slice's first channel
  const u16* x; int64_t x_ld;           // features at the slice's first channel
  BwdSums S;                            // BN1 sums of layers above, not yet in K: they cover the slice
  int c;                                // the slice's first channel
  float2* K; int K_set;                 // K0, K1 of what came before (K_set: there was something)
  const float *mean, *istd;             // of the slice's features
  float inv_p;
  u16* gl;                              // out: g_l, [P][k] (not written for the last layer)
  int k;
  const u16* W; int M16, K32;           // packed weights, nine taps of [M16][K32]
  const u16* b; const float2* fold2; const float *mean_b, *istd_b;
  int B;
  u16* dz;                              // out [P][B]: masked gradient of BN2's output
  float2* part2; int T2;                // out [T2][B]: BN2's sums
  int H, Wd, tpi, tiles, gy;
};

// Unsigned division of x < 2^31 by a fixed d <= 2^30: m = ceil(2^s / d) with s = 31 + ceil(log2 d), so that
// m*d - 2^s < d <= 2^(s-31) and the excess x*(m*d - 2^s) stays below 2^s.
struct DivBy {
  unsigned m;
  int s;
  __device__ __forceinline__ unsigned div(unsigned x) const { return (unsigned)(((unsigned long long)x * m) >> s); }
};

// Sum over the T partials of channel ch, the NW waves taking every NW-th; call with all threads,
// ch clamped into range.  sh: NW*64 float2.  Result valid in wave 0.
template <int NW>
__device__ __forceinline__ float2 sum_partials64(const float2* __restrict__ part, int T, int C, int ch, float2* sh) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float2 s = make_float2(0.f, 0.f);
  int t = wave;
  for (; t + 7 * NW < T; t += 8 * NW) {
    float2 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = part[(int64_t)(t + NW * u) * C + ch];
#pragma unroll
    for (int u = 0; u < 8; ++u) { s.x += v[u].x; s.y += v[u].y; }
  }
  for (; t + 3 * NW < T; t += 4 * NW) {
    float2 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = part[(int64_t)(t + NW * u) * C + ch];
#pragma unroll
    for (int u = 0; u < 4; ++u) { s.x += v[u].x; s.y += v[u].y; }
  }
  for (; t < T; t += NW) { const float2 v = part[(int64_t)t * C + ch]; s.x += v.x; s.y += v.y; }
  __syncthreads();
  sh[wave * 64 + lane] = s;
  __syncthreads();
  float2 r = sh[lane];
#pragma unroll
  for (int w = 1; w < NW; ++w) { r.x += sh[w * 64 + lane].x; r.y += sh[w * 64 + lane].y; }
  return r;
}

// The same for channels ch and ch + 1 (ch even, C even), four waves.  sh: 4*64 float4.
__device__ __forceinline__ float4 sum_partials128(const float2* __restrict__ part, int T, int C, int ch, float4* sh) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  int t = wave;
  auto add = [&](const float4& v) { s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w; };
  for (; t + 28 < T; t += 32) {
    float4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const float4*>(part + (int64_t)(t + 4 * u) * C + ch);
#pragma unroll
    for (int u = 0; u < 8; ++u) add(v[u]);
  }
  for (; t < T; t += 4) add(*reinterpret_cast<const float4*>(part + (int64_t)t * C + ch));
  __syncthreads();
  sh[wave * 64 + lane] = s;
  __syncthreads();
  s = sh[lane];
#pragma unroll
  for (int w = 1; w < 4; ++w) add(sh[w * 64 + lane]);
  return s;
}

// Extra workgroups of the 3x3 data gradient: 64 channels of S's BN1, their parameter gradients and, where a
// layer further down will read them, K0 / K1.
template <int NW>
__device__ __forceinline__ void finish_bn1(const Dgrad3Args& A, int wg, float2* sh) {
  const int i = wg * 64 + (threadIdx.x & 63), ic = min(i, A.S.width - 1), ch = A.S.base + ic;
  float2 k = make_float2(0.f, 0.f);
  if (A.K_set) k = A.K[ch];
  for (int q = 0; q < A.S.n; ++q) {
    const float2 s = sum_partials64<NW>(q ? A.S.part[1] : A.S.part[0], A.S.T, A.S.width, ic, sh);
    const float sc = (q ? A.S.fold1[1] : A.S.fold1[0])[ch].x * A.inv_p;
    k = make_float2(__fmaf_rn(sc, s.x, k.x), __fmaf_rn(sc, s.y, k.y));
    if (threadIdx.x < 64 && i < A.S.width) {
      (q ? A.S.dbeta[1] : A.S.dbeta[0])[ch] = s.x;
      (q ? A.S.dgamma[1] : A.S.dgamma[0])[ch] = s.y;
    }
    __syncthreads();
  }
  if (threadIdx.x < 64 && i < A.S.width && ch < A.c) A.K[ch] = k;
}
// K0, K1 of the slice's channel ic, with what S holds; valid in wave 0.  Call with all threads.
template <int NW>
__device__ __forceinline__ float2 slice_k(const Dgrad3Args& A, int ic, float2* sh) {
  float2 k = make_float2(0.f, 0.f);
  if (A.K_set) k = A.K[A.c + ic];
  for (int q = 0; q < A.S.n; ++q) {
    const float2 s = sum_partials64<NW>(q ? A.S.part[1] : A.S.part[0], A.S.T, A.S.width, A.c - A.S.base + ic, sh);
    const float sc = (q ? A.S.fold1[1] : A.S.fold1[0])[A.c + ic].x * A.inv_p;
    k = make_float2(__fmaf_rn(sc, s.x, k.x), __fmaf_rn(sc, s.y, k.y));
    __syncthreads();
  }
  return k;
}

// Output channels (B of them) on M, pixels of one image on N.  A workgroup owns a tile of 64*NT
// consecutive pixels and MT M-tiles; its four waves split the pixels (NT N-tiles each) and every wave
// forms all MT M-tiles, so nothing is added across waves but the two sums at the end.  The slice
// of the slab is corrected, rounded to bf16 and staged once per tile with a halo of a row and a
// pixel on either side; in passes of 64 channels (k above 64).  Workgroups walk over tiles T2 apart.
// BYPASS: the coefficients of a pass's channels are formed before it, else all of them first.
template <int NT, int MT, bool BYPASS>
__global__ __launch_bounds__(256) void k_dgrad3(Dgrad3Args A) {
  extern __shared__ u16 lds[];
  __shared__ float2 sh[256];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, j = lane & 15, g = lane >> 4;
  const int nconv = A.T2 * A.gy;
  if ((int)blockIdx.x >= nconv) { finish_bn1<4>(A, (int)blockIdx.x - nconv, sh); return; }
  constexpr int PITCH = 64 + 8, TP = 64 * NT;
  const int HW = A.H * A.Wd, W = A.Wd, halo = W + 1, seg = TP + 2 * halo;
  const int pw = blockIdx.x / A.gy, m0 = (blockIdx.x % A.gy) * MT * 16;
  float* coef = reinterpret_cast<float*>(lds + seg * PITCH);  // [3][kc]: K0, K1*istd, mean
  const int kc = BYPASS ? 64 : A.k;
  auto form_coef = [&](int c0, int at) {  // of channels c0..c0+63, to positions at..
    const int i = c0 + lane, ic = min(i, A.k - 1);
    const float2 k = slice_k<4>(A, ic, sh);
    if (wave == 0 && i < A.k) {
      coef[at + lane] = k.x;
      coef[kc + at + lane] = k.y * A.istd[ic];
      coef[2 * kc + at + lane] = A.mean[ic];
    }
  };
  if (!BYPASS && !A.dy)
    for (int c0 = 0; c0 < A.k; c0 += 64) form_coef(c0, c0);
  float s0[MT][4], s1[MT][4], fs[MT][4], ft[MT][4], mu[MT][4];
  int mch[MT];
#pragma unroll
  for (int a = 0; a < MT; ++a) {
    mch[a] = m0 + a * 16 + 4 * g;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = min(mch[a] + r, A.B - 1);
      const float2 f = A.fold2[m];
      fs[a][r] = f.x; ft[a][r] = f.y; mu[a][r] = A.mean_b[m];
      s0[a][r] = s1[a][r] = 0.f;
    }
  }

  for (int tile = pw; tile < A.tiles; tile += A.T2) {
    const int img = tile / A.tpi, q0 = (tile - img * A.tpi) * TP;
    const int64_t p0 = (int64_t)img * HW;
    f32x4 acc[MT][NT];
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[a][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    uint2 braw[MT][NT];  // b_l at the outputs' positions, requested before the staging
    bool lok[NT], rok[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int q = q0 + (wave * NT + t) * 16 + j, qc = min(q, HW - 1), wc = q % W;
      lok[t] = wc != 0;
      rok[t] = wc != W - 1;
#pragma unroll
      for (int a = 0; a < MT; ++a)
        braw[a][t] = *reinterpret_cast<const uint2*>(A.b + (p0 + qc) * A.B + min(mch[a], A.B - 4));
    }
    for (int c0 = 0; c0 < A.K32; c0 += 64) {
      const int kw = min(64, A.K32 - c0), vsh = kw == 64 ? 3 : 2, nvec = seg << vsh, cb = BYPASS ? c0 : 0;
      if (BYPASS && !A.dy) form_coef(c0, 0);  // (its barriers: the previous pass has read the last ones)
      __syncthreads();  // coefficients written; the previous pass's fragment reads are done
      for (int base = 0; base < nvec; base += 4 * 256) {
        uint4 ga[4], gb[4], xr[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {  // loads unconditional at clamped addresses
          const int idx = min(base + u * 256 + tid, nvec - 1), s = idx >> vsh;
          const int ch = min(c0 + 8 * (idx & ((1 << vsh) - 1)), A.k - 8);
          const int64_t p = p0 + min(max(q0 - halo + s, 0), HW - 1);
          if (A.dy) {
            ga[u] = *reinterpret_cast<const uint4*>(A.dy + p * A.g_ld + ch);
          } else {
            const float* gp = A.G + p * A.g_ld + ch;
            ga[u] = *reinterpret_cast<const uint4*>(gp);
            gb[u] = *reinterpret_cast<const uint4*>(gp + 4);
            xr[u] = *reinterpret_cast<const uint4*>(A.x + p * A.x_ld + ch);
          }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int idx = base + u * 256 + tid;
          if (idx < nvec) {
            const int s = idx >> vsh, v = idx & ((1 << vsh) - 1), ch = c0 + 8 * v, q = q0 - halo + s;
            V8 o;
            o.q = make_uint4(0u, 0u, 0u, 0u);
            if (q >= 0 && q < HW && ch < A.k) {
              if (A.dy) {
                o.q = ga[u];
              } else {
                V8 xv;
                xv.q = xr[u];
                const float gf[8] = {__uint_as_float(ga[u].x), __uint_as_float(ga[u].y), __uint_as_float(ga[u].z),
                                     __uint_as_float(ga[u].w), __uint_as_float(gb[u].x), __uint_as_float(gb[u].y),
                                     __uint_as_float(gb[u].z), __uint_as_float(gb[u].w)};
#pragma unroll
                for (int e = 0; e < 8; ++e)
                  o.h[e] = f2bf(gf[e] - coef[ch - cb + e] - coef[kc + ch - cb + e] * (bf2f(xv.h[e]) - coef[2 * kc + ch - cb + e]));
                if (m0 == 0 && s >= halo && s < halo + TP)
                  *reinterpret_cast<uint4*>(A.gl + (p0 + q) * A.k + ch) = o.q;
              }
            }
            *reinterpret_cast<uint4*>(&lds[s * PITCH + 8 * v]) = o.q;
          }
        }
      }
      __syncthreads();
#pragma unroll
      for (int t9 = 0; t9 < 9; ++t9) {
        const int di = t9 / 3 - 1, dj = t9 % 3 - 1;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
          if (kk * 32 < kw) {
            V8 wv[MT], bv[NT];
#pragma unroll
            for (int a = 0; a < MT; ++a)
              wv[a].q = *reinterpret_cast<const uint4*>(
                  wfrag(A.W + (int64_t)t9 * A.M16 * A.K32, A.K32, min(m0 + a * 16, A.M16 - 16) >> 4, (c0 >> 5) + kk));
#pragma unroll
            for (int t = 0; t < NT; ++t) {
              bv[t].q = *reinterpret_cast<const uint4*>(
                  &lds[((wave * NT + t) * 16 + j + halo + di * W + dj) * PITCH + kk * 32 + 8 * g]);
              if ((dj < 0 && !lok[t]) || (dj > 0 && !rok[t])) bv[t].q = make_uint4(0u, 0u, 0u, 0u);
            }
#pragma unroll
            for (int a = 0; a < MT; ++a)
#pragma unroll
              for (int t = 0; t < NT; ++t) acc[a][t] = mfma_bf16(wv[a], bv[t], acc[a][t]);
          }
        }
      }
    }
    // ReLU mask of BN2, the two sums over what is stored
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int q = q0 + (wave * NT + t) * 16 + j;
        if (q < HW && mch[a] < A.B) {
          const float bf[4] = {bf2f((u16)braw[a][t].x), bf2f((u16)(braw[a][t].x >> 16)), bf2f((u16)braw[a][t].y),
                               bf2f((u16)(braw[a][t].y >> 16))};
          u16 h[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            h[r] = __fmaf_rn(bf[r], fs[a][r], ft[a][r]) > 0.f ? f2bf(acc[a][t][r]) : (u16)0;
            const float dz = bf2f(h[r]);
            s0[a][r] += dz;
            s1[a][r] = __fmaf_rn(dz, bf[r] - mu[a][r], s1[a][r]);
          }
          *reinterpret_cast<uint2*>(A.dz + (p0 + q) * A.B + mch[a]) =
              make_uint2((unsigned)h[0] | ((unsigned)h[1] << 16), (unsigned)h[2] | ((unsigned)h[3] << 16));
        }
      }
  }
  // sums: over the 16 pixel lanes, then over the waves
  __syncthreads();
  float* red = reinterpret_cast<float*>(lds);  // [4][MT*16][2]
#pragma unroll
  for (int a = 0; a < MT; ++a)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float u = row16_sum(s0[a][r]), v = row16_sum(s1[a][r]);
      if (j == 0) {
        float* p = red + ((wave * MT + a) * 16 + 4 * g + r) * 2;
        p[0] = u; p[1] = v;
      }
    }
  __syncthreads();
  if (tid < MT * 16) {
    const int m = m0 + tid;
    if (m < A.B) {
      float u = 0.f, v = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) { u += red[(w * MT * 16 + tid) * 2]; v += red[(w * MT * 16 + tid) * 2 + 1]; }
      A.part2[(int64_t)pw * A.B + m] = make_float2(u, v * A.istd_b[m]);
    }
  }
}

// The same for growth rates up to 64 (K-steps KS = 1 or 2 of 32 channels), which is every network of the
// paper's family.  A workgroup walks over tiles of 64 pixels of the flat pixel axis of all images (a tap
// outside a pixel's image is a read of a row of zeros); each of its eight waves forms one M-tile of up to
// eight of all 64 pixels, so a tile's slice is staged once for 128 channels, the wave's weights (nine taps)
// stay in its registers, and the sums need no exchange.  The next tile's slice is requested before the
// current tile's products and staged into the other LDS buffer after them; the first tile's is in flight
// while the coefficients' partial sums are added.  U: vectors of 8 channels a thread stages per tile.
// Bounds: few pixels, two memory latencies (partial sums, slice), the staging and 36 or 72 MFMAs a wave; many,
// LDS reads (36 or 72 KB a tile and wave) and the traffic of b and dz.  us a launch at 32 images, against
// k_dgrad3 (which waited for its weights tap by tap, staged the tile for every 16 or 32 output channels and
// rounded each image up to whole tiles): 32 channels to 128, 14x14 8.9 (14.2), 7x7 7.8 (9.4), 28x28 14.5 (23),
// 56x56 35.6 (56); 48 to 192, 14x14 13 (20), 28x28 28 (43), 56x56 79 (108).
template <int KS, int U>
__global__ __launch_bounds__(512) void k_dgrad3s(Dgrad3Args A, int T, DivBy dhw, DivBy dw) {
  extern __shared__ __attribute__((aligned(16))) u16 lds[];
  __shared__ float2 sh[512];
  __shared__ __attribute__((aligned(16))) float coef[3][64];  // K0, K1*istd, mean
  constexpr int VS = KS == 2 ? 3 : 2, PITCH = 32 * KS + 8, RS = 512 >> VS;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), j = lane & 15, g = lane >> 4;
  const int nconv = (A.T2 + 7) / 8 * 8 * A.gy;
  if ((int)blockIdx.x >= nconv) { finish_bn1<8>(A, (int)blockIdx.x - nconv, sh); return; }
  const int slot = blockIdx.x >> 3, grp = slot % A.gy, pw = (slot / A.gy) * 8 + (blockIdx.x & 7);
  if (pw >= A.T2) return;
  const int W = A.Wd, HW = A.H * W, halo = W + 1, seg = 64 + 2 * halo, BUFE = (seg + 1) * PITCH, P = A.tiles;
  const int v = tid & ((1 << VS) - 1), r = tid >> VS, ch = min(8 * v, A.k - 8);
  const bool cok = 8 * v < A.k;

  // staging: three loads a vector (two of them again what the first brings where dy stands in for the slab)
  struct Raw { uint4 a, b, x; };
  const int gsz = A.dy ? 2 : 4, goff = A.dy ? 0 : 16;
  const unsigned grow = (unsigned)A.g_ld * gsz, xrow = (unsigned)(A.dy ? A.g_ld : A.x_ld) * 2;
  Raw raw[U];
  auto request = [&](int tile) {
    const int first = max(tile * 64 - halo, 0);  // scalar bases at the tile's first row, 32-bit offsets from there
    const char* gb = (A.dy ? reinterpret_cast<const char*>(A.dy) : reinterpret_cast<const char*>(A.G)) + (int64_t)first * grow;
    const char* xb = (A.dy ? reinterpret_cast<const char*>(A.dy) : reinterpret_cast<const char*>(A.x)) + (int64_t)first * xrow;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int s = min(r + u * RS, seg - 1);
      const unsigned row = min(max(tile * 64 - halo + s, 0), P - 1) - first;
      const unsigned o = row * grow + ch * gsz;
      raw[u].a = *reinterpret_cast<const uint4*>(gb + o);
      raw[u].b = *reinterpret_cast<const uint4*>(gb + (o + goff));
      raw[u].x = *reinterpret_cast<const uint4*>(xb + (row * xrow + 2 * ch));
    }
  };
  float k0[8], k1[8], mu0[8];
  auto deposit = [&](int tile, int buf) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int s = r + u * RS, p = tile * 64 - halo + s;
      V8 o, xv;
      xv.q = raw[u].x;
      const float gf[8] = {__uint_as_float(raw[u].a.x), __uint_as_float(raw[u].a.y), __uint_as_float(raw[u].a.z),
                           __uint_as_float(raw[u].a.w), __uint_as_float(raw[u].b.x), __uint_as_float(raw[u].b.y),
                           __uint_as_float(raw[u].b.z), __uint_as_float(raw[u].b.w)};
#pragma unroll
      for (int e = 0; e < 8; ++e) o.h[e] = f2bf(gf[e] - k0[e] - k1[e] * (bf2f(xv.h[e]) - mu0[e]));
      if (A.dy) o.q = raw[u].a;
      if (!A.dy && grp == 0 && cok && s >= halo && s < halo + 64 && p < P)
        *reinterpret_cast<uint4*>(A.gl + (int64_t)p * A.k + ch) = o.q;
      if (!cok) o.q = make_uint4(0u, 0u, 0u, 0u);
      if (s < seg) *reinterpret_cast<uint4*>(lds + buf * BUFE + s * PITCH + 8 * v) = o.q;
    }
  };
  request(pw);

  // the groups share the M-tiles evenly (192 channels: six and six, not eight and four: 56x56 block 1010 -> 987 us a step)
  const int mtiles = A.M16 >> 4, per = (mtiles + A.gy - 1) / A.gy, mt = grp * per + wave;
  const int mch = mt * 16 + 4 * g, mc = min(mch, A.B - 4);
  const bool m_ok = wave < per && mt < mtiles;  // uniform
  V8 wv[9][KS];
#pragma unroll
  for (int t9 = 0; t9 < 9; ++t9)
#pragma unroll
    for (int kk = 0; kk < KS; ++kk)
      wv[t9][kk].q = *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(A.W) +
                                                     (((int64_t)t9 * mtiles + min(mt, mtiles - 1)) * KS + kk) * 1024 + (unsigned)lane * 16);
  float fs[4], ft[4], mu[4], s0[4], s1[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float2 f = A.fold2[mc + e];
    fs[e] = f.x; ft[e] = f.y; mu[e] = A.mean_b[mc + e];
    s0[e] = s1[e] = 0.f;
  }
  if (!A.dy) {
    const int ic = min(lane, A.k - 1);
    const float2 k = slice_k<8>(A, ic, sh);
    if (wave == 0) {
      coef[0][lane] = k.x;
      coef[1][lane] = k.y * A.istd[ic];
      coef[2][lane] = A.mean[ic];
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 8; ++e) { k0[e] = coef[0][ch + e]; k1[e] = coef[1][ch + e]; mu0[e] = coef[2][ch + e]; }
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) k0[e] = k1[e] = mu0[e] = 0.f;
  }
  if (tid < PITCH / 4) *reinterpret_cast<uint4*>(lds + (tid / (PITCH / 8)) * BUFE + seg * PITCH + 8 * (tid % (PITCH / 8))) = make_uint4(0u, 0u, 0u, 0u);
  deposit(pw, 0);
  __syncthreads();

  int buf = 0;
  for (int tile = pw; tile < T; tile += A.T2, buf ^= 1) {
    const int next = min(tile + A.T2, T - 1);
    request(next);
    if (m_ok) {
      uint2 braw[4];
      unsigned mask[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int p = tile * 64 + t * 16 + j, pc = min(p, P - 1);
        braw[t] = *reinterpret_cast<const uint2*>(A.b + (int64_t)pc * A.B + mc);
        const int q = pc - (int)dhw.div(pc) * HW, y = (int)dw.div(q), x = q - y * W;
        const unsigned r3 = (x > 0 ? 1u : 0u) | 2u | (x < W - 1 ? 4u : 0u);
        mask[t] = (y > 0 ? r3 : 0u) | (r3 << 3) | (y < A.H - 1 ? r3 << 6 : 0u);
      }
      f32x4 acc[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[t] = (f32x4){0.f, 0.f, 0.f, 0.f};
      const u16* lb = lds + buf * BUFE + 8 * g;
#pragma unroll
      for (int t9 = 0; t9 < 9; ++t9) {
        const int off = (halo + (t9 / 3 - 1) * W + t9 % 3 - 1 + j) * PITCH;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const u16* xp = lb + ((mask[t] >> t9) & 1 ? off + t * 16 * PITCH : seg * PITCH);
#pragma unroll
          for (int kk = 0; kk < KS; ++kk) {
            V8 x;
            x.q = *reinterpret_cast<const uint4*>(xp + kk * 32);
            acc[t] = mfma_bf16(wv[t9][kk], x, acc[t]);
          }
        }
      }
      // ReLU mask of BN2, the two sums over what is stored
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int p = tile * 64 + t * 16 + j;
        if (p < P && mch < A.B) {
          const float bf[4] = {bf2f((u16)braw[t].x), bf2f((u16)(braw[t].x >> 16)), bf2f((u16)braw[t].y), bf2f((u16)(braw[t].y >> 16))};
          u16 h[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            h[e] = __fmaf_rn(bf[e], fs[e], ft[e]) > 0.f ? f2bf(acc[t][e]) : (u16)0;
            const float dz = bf2f(h[e]);
            s0[e] += dz;
            s1[e] = __fmaf_rn(dz, bf[e] - mu[e], s1[e]);
          }
          *reinterpret_cast<uint2*>(A.dz + (int64_t)p * A.B + mch) =
              make_uint2((unsigned)h[0] | ((unsigned)h[1] << 16), (unsigned)h[2] | ((unsigned)h[3] << 16));
        }
      }
    }
    if (tile + A.T2 < T) deposit(next, buf ^ 1);
    __syncthreads();
  }
  if (m_ok) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float a = row16_sum(s0[e]), b = row16_sum(s1[e]);
      if (j == 0 && mch < A.B) A.part2[(int64_t)pw * A.B + mch + e] = make_float2(a, b * A.istd_b[mch + e]);
    }
  }
}

// ---------------------------------------------------------------- BN2 backward, element-wise

// out[c] = sum over T of part[T][C], one workgroup per 64 channels
__global__ __launch_bounds__(256) void k_sum_pairs(const float2* __restrict__ part, int T, int C, float2* __restrict__ out) {
  __shared__ float2 sh[256];
  const int ch = blockIdx.x * 64 + (threadIdx.x & 63);
  const float2 s = sum_partials64<4>(part, T, C, min(ch, C - 1), sh);
  if (threadIdx.x < 64 && ch < C) out[ch] = s;
}

// db = s2*(dz - dbeta/P - xhat*dgamma/P) in place.  Thread = (8-channel vector, pixel row); grid
// (pixel ranges, groups of 8*L channels).  Every workgroup adds the T partials of its channels
// itself (T is small: see launch_dgrad3), the first of a group stores the parameter gradients.
__global__ __launch_bounds__(256) void k_bn2_apply(u16* __restrict__ dz, const u16* __restrict__ b, int64_t P, int B,
                                                   int ppb, int lsh, float inv_p, const float2* __restrict__ fold2,
                                                   const float* __restrict__ mean, const float* __restrict__ istd,
                                                   const float2* __restrict__ part, int T, float* __restrict__ dgamma,
                                                   float* __restrict__ dbeta) {
  __shared__ float4 sh[256];
  __shared__ float4 co[256];  // scale, scale*dbeta/P, scale*dgamma/P*istd, mean
  const int L = 1 << lsh, rows = 256 >> lsh, cvl = threadIdx.x & (L - 1), pr = threadIdx.x >> lsh;
  const int cb = blockIdx.y * L * 8, ch0 = cb + cvl * 8;
  const int64_t p0 = (int64_t)blockIdx.x * ppb, p1 = min(P, p0 + ppb);
  const bool ok = ch0 < B;
  const int chc = ok ? ch0 : 0;
  V8 d0[2], b0[2];  // the first rows' data, in flight while the sums are formed
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int64_t p = min(p0 + pr + u * rows, p1 - 1);
    d0[u].q = *reinterpret_cast<const uint4*>(dz + p * B + chc);
    b0[u].q = *reinterpret_cast<const uint4*>(b + p * B + chc);
  }
  for (int c0 = 0; c0 < L * 8; c0 += 128) {  // two channels a lane (B % 8 == 0)
    const int cl = c0 + 2 * (threadIdx.x & 63), ch = cb + cl;
    const float4 s = sum_partials128(part, T, B, min(ch, B - 2), sh);
    if (threadIdx.x < 64 && cl < L * 8 && ch < B) {
      const float sx[2] = {s.x, s.z}, sy[2] = {s.y, s.w};
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const float sc = fold2[ch + e].x;
        co[cl + e] = make_float4(sc, sc * (sx[e] * inv_p), sc * (sy[e] * inv_p) * istd[ch + e], mean[ch + e]);
        if (blockIdx.x == 0) { dbeta[ch + e] = sx[e]; dgamma[ch + e] = sy[e]; }
      }
    }
  }
  __syncthreads();
  if (!ok) return;
  float4 f[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) f[e] = co[cvl * 8 + e];
  for (int64_t pb = p0 + pr; pb < p1; pb += 2 * rows) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int64_t p = pb + u * rows;
      if (p < p1) {
        V8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e)
          o.h[e] = f2bf(__fmaf_rn(f[e].x, bf2f(d0[u].h[e]), -f[e].y) - f[e].z * (bf2f(b0[u].h[e]) - f[e].w));
        *reinterpret_cast<uint4*>(dz + p * B + ch0) = o.q;
      }
      const int64_t pn = min(p + 2 * rows, p1 - 1);
      if (pb + 2 * rows < p1) {
        d0[u].q = *reinterpret_cast<const uint4*>(dz + pn * B + ch0);
        b0[u].q = *reinterpret_cast<const uint4*>(b + pn * B + ch0);
      }
    }
  }
}

// ---------------------------------------------------------------- 1x1 data gradient + BN1 backward

struct Dgrad1Args {
  const u16* db; int B;                 // gradient of b_l [P][B]
  const u16* W; int C16, B32;           // packed weights [C16][B32]
  const u16* x; int64_t x_ld;           // concatenated features
  const u16* dy; float* G; int64_t g_ld;  // slab; dy replaces its first read (FIRST)
  const float2* fold1; const float *mean, *istd;
  float2* part1; int C;                 // out [T1][C]
  int64_t P;
  int ppw;                              // pixels per wave, a multiple of 32
};

// One layer with more than kDgrad1MaxB outputs (fewer: dgrad1_body of dnb_nhwc_wgrad.hip, which keeps the weights
// in LDS).  Output channels on M, pixels on N.  A workgroup owns 32 channels (two M-tiles) and a range of pixels, of
// which each wave walks a quarter in steps of 32 (two N-tiles); weights and gradients are read in the loop over K.
template <bool FIRST>
__global__ __launch_bounds__(256) void k_dgrad1(Dgrad1Args A) {
  __shared__ float red[4][32][2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, j = lane & 15, g = lane >> 4;
  const int c0 = blockIdx.x * 32;
  const int64_t pw0 = ((int64_t)blockIdx.y * 4 + wave) * A.ppw;
  const int64_t pw1 = min(A.P, pw0 + A.ppw);
  const int ksteps = A.B32 >> 5;
  const u16* wr[2];
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    wr[a] = wfrag(A.W, A.B32, min(c0 + a * 16, A.C16 - 16) >> 4, 0);
  }
  float sc[2][4], sf[2][4], mu[2][4], s0[2][4], s1[2][4];
  int ch[2];
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    ch[a] = min(c0 + a * 16 + 4 * g, A.C - 4);  // C % 8 == 0: a lane's four channels are in or out together
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float2 f = A.fold1[ch[a] + r];
      sc[a][r] = f.x; sf[a][r] = f.y; mu[a][r] = A.mean[ch[a] + r];
      s0[a][r] = s1[a][r] = 0.f;
    }
  }
  const bool cok[2] = {c0 + 4 * g < A.C, c0 + 16 + 4 * g < A.C};

  for (int64_t pb = pw0; pb < pw1; pb += 32) {
    int64_t p[2];
    uint2 xr[2][2], dr[2][2];
    float4 gr[2][2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      p[t] = min(pb + t * 16 + j, pw1 - 1);  // clamped: masked below
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        xr[t][a] = *reinterpret_cast<const uint2*>(A.x + p[t] * A.x_ld + ch[a]);
        if (FIRST) dr[t][a] = *reinterpret_cast<const uint2*>(A.dy + p[t] * A.g_ld + ch[a]);
        else gr[t][a] = *reinterpret_cast<const float4*>(A.G + p[t] * A.g_ld + ch[a]);
      }
    f32x4 acc[2][2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int a = 0; a < 2; ++a) acc[t][a] = (f32x4){0.f, 0.f, 0.f, 0.f};
    for (int s = 0; s < ksteps; ++s) {
      V8 ww[2], dd[2];
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        ww[a].q = *reinterpret_cast<const uint4*>(wr[a] + 512 * s);
        dd[a].q = *reinterpret_cast<const uint4*>(A.db + p[a] * A.B + min(32 * s + 8 * g, A.B - 8));
      }
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int a = 0; a < 2; ++a) acc[t][a] = mfma_bf16(ww[a], dd[t], acc[t][a]);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        if (pb + t * 16 + j < pw1 && cok[a]) {
          const float xf[4] = {bf2f((u16)xr[t][a].x), bf2f((u16)(xr[t][a].x >> 16)), bf2f((u16)xr[t][a].y),
                               bf2f((u16)(xr[t][a].y >> 16))};
          float gv[4];
          if (FIRST) {
            gv[0] = bf2f((u16)dr[t][a].x); gv[1] = bf2f((u16)(dr[t][a].x >> 16));
            gv[2] = bf2f((u16)dr[t][a].y); gv[3] = bf2f((u16)(dr[t][a].y >> 16));
          } else {
            gv[0] = gr[t][a].x; gv[1] = gr[t][a].y; gv[2] = gr[t][a].z; gv[3] = gr[t][a].w;
          }
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float dz = __fmaf_rn(xf[r], sc[a][r], sf[a][r]) > 0.f ? acc[t][a][r] : 0.f;
            gv[r] = __fmaf_rn(sc[a][r], dz, gv[r]);
            s0[a][r] += dz;
            s1[a][r] = __fmaf_rn(dz, xf[r] - mu[a][r], s1[a][r]);
          }
          *reinterpret_cast<float4*>(A.G + p[t] * A.g_ld + ch[a]) = make_float4(gv[0], gv[1], gv[2], gv[3]);
        }
      }
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float u = row16_sum(s0[a][r]), v = row16_sum(s1[a][r]);
      if (j == 0) { red[wave][a * 16 + 4 * g + r][0] = u; red[wave][a * 16 + 4 * g + r][1] = v; }
    }
  __syncthreads();
  if (tid < 32 && c0 + tid < A.C) {
    float u = 0.f, v = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q) { u += red[q][tid][0]; v += red[q][tid][1]; }
    A.part1[(int64_t)blockIdx.y * A.C + c0 + tid] = make_float2(u, v * A.istd[c0 + tid]);
  }
}

// ---------------------------------------------------------------- gradient of the block input

// dx0 = bf16(G - K0 - K1*xhat) on the block input's channels, with the last BN1 sums (which cover exactly these
// channels) finished on the way.  grid (groups of 256 channels, pixel ranges).
__global__ __launch_bounds__(256) void k_dx0(const float* __restrict__ G, int64_t g_ld, const u16* __restrict__ x,
                                             int64_t x_ld, u16* __restrict__ dx0, int64_t P, int C, int ppb, float inv_p,
                                             const float2* __restrict__ K, BwdSums S, const float* __restrict__ mean,
                                             const float* __restrict__ istd) {
  __shared__ float co[3][256];
  const int cb = blockIdx.x * 256;
  {
    const int ch = cb + threadIdx.x, cc = min(ch, C - 1);
    float2 k = K ? K[cc] : make_float2(0.f, 0.f);
    for (int q = 0; q < S.n; ++q) {
      const float2* part = q ? S.part[1] : S.part[0];
      float2 s = make_float2(0.f, 0.f);
      int t = 0;
      for (; t + 8 <= S.T; t += 8) {
        float2 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = part[(int64_t)(t + u) * C + cc];
#pragma unroll
        for (int u = 0; u < 8; ++u) { s.x += v[u].x; s.y += v[u].y; }
      }
      for (; t < S.T; ++t) { const float2 v = part[(int64_t)t * C + cc]; s.x += v.x; s.y += v.y; }
      const float sc = (q ? S.fold1[1] : S.fold1[0])[cc].x * inv_p;
      k = make_float2(__fmaf_rn(sc, s.x, k.x), __fmaf_rn(sc, s.y, k.y));
      if (blockIdx.y == 0 && ch < C) {
        (q ? S.dbeta[1] : S.dbeta[0])[ch] = s.x;
        (q ? S.dgamma[1] : S.dgamma[0])[ch] = s.y;
      }
    }
    co[0][threadIdx.x] = k.x;
    co[1][threadIdx.x] = k.y * istd[cc];
    co[2][threadIdx.x] = mean[cc];
  }
  __syncthreads();
  const int cvl = threadIdx.x & 31, pr = threadIdx.x >> 5, ch0 = cb + cvl * 8;
  if (ch0 >= C) return;
  float a[8], b[8], mu[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) { a[e] = co[0][cvl * 8 + e]; b[e] = co[1][cvl * 8 + e]; mu[e] = co[2][cvl * 8 + e]; }
  const int64_t p0 = (int64_t)blockIdx.y * ppb, p1 = min(P, p0 + ppb);
  for (int64_t pb = p0 + pr; pb < p1; pb += 32) {
    V8 xv[4];
    float4 ga[4], gb[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t p = min(pb + 8 * u, p1 - 1);
      xv[u].q = *reinterpret_cast<const uint4*>(x + p * x_ld + ch0);
      ga[u] = *reinterpret_cast<const float4*>(G + p * g_ld + ch0);
      gb[u] = *reinterpret_cast<const float4*>(G + p * g_ld + ch0 + 4);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t p = pb + 8 * u;
      if (p < p1) {
        const float gf[8] = {ga[u].x, ga[u].y, ga[u].z, ga[u].w, gb[u].x, gb[u].y, gb[u].z, gb[u].w};
        V8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o.h[e] = f2bf(gf[e] - a[e] - b[e] * (bf2f(xv[u].h[e]) - mu[e]));
        *reinterpret_cast<uint4*>(dx0 + p * C + ch0) = o.q;
      }
    }
  }
}

// Tile plan.  Growth rates up to 64 take k_dgrad3s: groups of up to eight M-tiles, at most one workgroup per CU,
// as even a number of 64-pixel tiles each as that gives.  Wider ones k_dgrad3.  NT: the largest tile (64*NT pixels of one image: less halo per pixel)
// that leaves at most 15 % of its pixels unused, else the one that leaves the fewest, within 64 KB
// of LDS.  MT: two M-tiles per workgroup where that still gives one workgroup per CU (each M group
// stages the tile again; four need more than 256 registers).  T2: workgroups per M group; one per
// tile up to 256, beyond that each takes several.  bypass: the slice's coefficients stay in LDS up to 512
// channels (6 KB); wider slices form those of a 64-channel pass before it, so that LDS does not grow with k
// and every width of a row that dnb_block_create takes fits 64 KB.
struct Dgrad3Plan {
  int NT, MT, tpi, tiles, gy, T2;
  bool bypass;
  int ks, u;  // k_dgrad3s: K-steps, vectors per thread; tiles = pixels there
  size_t lds;
};
Dgrad3Plan plan_dgrad3(int n, int h, int w, int k, int B) {
  Dgrad3Plan p{};
  const int hw = h * w, mtiles = (B + 15) / 16;
  const int64_t P = (int64_t)n * hw;
  if (k <= 64 && P < ((int64_t)1 << 30)) {
    p.ks = (k + 31) / 32;
    const int seg = 64 + 2 * (w + 1), T = (int)((P + 63) / 64);
    p.u = (seg + (512 >> (p.ks == 2 ? 3 : 2)) - 1) / (512 >> (p.ks == 2 ? 3 : 2));
    p.lds = (size_t)2 * (seg + 1) * (32 * p.ks + 8) * sizeof(u16);
    p.gy = (mtiles + 7) / 8;
    p.tiles = (int)P;
    // workgroups per XCD, not per chip: the gy of a tile share one, and with 85 x 3 five XCDs had 33 for their 32 CUs
    // (10800 pixels, 8 to 288 channels: 19.5 us a launch for 10)
    int most = 32 / p.gy * 8;
    if (most < 1) most = 1;
    const int per = (T + most - 1) / most;
    p.T2 = (T + per - 1) / per;
    if (p.u <= 2 * p.ks) return p;
    p = Dgrad3Plan{};
  }
  int best = 0;
  p.bypass = k > 512;
  for (int nt : {4, 2, 1}) {
    const size_t lds = (size_t)(64 * nt + 2 * (w + 1)) * 72 * sizeof(u16) + (size_t)3 * (p.bypass ? 64 : k) * sizeof(float);
    if (lds > 60 * 1024 && nt > 1) continue;
    const int used = (hw + 64 * nt - 1) / (64 * nt) * 64 * nt;
    if (best == 0 || used < best) { best = used; p.NT = nt; p.lds = lds; }
    if (used * 100 <= 115 * hw) break;
  }
  p.tpi = (hw + 64 * p.NT - 1) / (64 * p.NT);
  p.tiles = n * p.tpi;
  p.MT = mtiles >= 2 && (int64_t)p.tiles * ((mtiles + 1) / 2) >= 256 ? 2 : 1;
  p.gy = (mtiles + p.MT - 1) / p.MT;
  const int per = (p.tiles + 255) / 256;
  p.T2 = (p.tiles + per - 1) / per;
  return p;
}

}  // namespace

// Splits of the upper layer's share of the lower one's slice: its partials are added by every workgroup of the
// next launch, and it runs beside the weight gradients.
constexpr int kNearSplits = 64;
constexpr int kFarSplits = 256;

size_t bwd_partial1_floats(int64_t P, int C, int layers) {
  int ppw;
  return (size_t)2 * layers * C * dgrad1_splits(P, C, kFarSplits, &ppw);
}
size_t bwd_partial1_near_floats(int64_t P, int k) {
  int ppw;
  return (size_t)2 * k * dgrad1_splits(P, k, kNearSplits, &ppw);
}
size_t bwd_partial2_floats(int n, int h, int w, int k, int B) {
  return (size_t)2 * B * (plan_dgrad3(n, h, w, k, B).T2 + 1);
}

int bwd_near_splits() { return kNearSplits; }
int bwd_far_splits() { return kFarSplits; }

hipError_t bwd_dgrad3(const BwdLayer& L, hipStream_t st) {
  const Dgrad3Plan p = plan_dgrad3(L.n, L.h, L.w, L.k, L.B);
  const int64_t P = (int64_t)L.n * L.h * L.w;
  Dgrad3Args A{};
  A.dy = L.last ? (const u16*)L.dy + L.c : nullptr;
  A.G = L.G + L.c; A.g_ld = L.ld;
  A.x = (const u16*)L.y + L.c; A.x_ld = L.ld;
  A.k = L.k;
  A.mean = L.mean_y + L.c; A.istd = L.istd_y + L.c;
  A.inv_p = 1.0f / (float)P;
  A.gl = (u16*)L.gl;
  A.M16 = (L.B + 15) & ~15; A.K32 = (L.k + 31) & ~31;
  A.W = (const u16*)L.pk3t;
  A.b = (const u16*)L.b; A.fold2 = L.fold2; A.mean_b = L.mean_b; A.istd_b = L.istd_b; A.B = L.B;
  A.dz = (u16*)L.db;
  A.part2 = (float2*)L.part2; A.T2 = p.T2;
  A.H = L.h; A.Wd = L.w; A.tpi = p.tpi; A.tiles = p.tiles; A.gy = p.gy;
  A.S = L.above;
  A.c = L.c;
  A.K = L.K; A.K_set = L.K_set;
  const int fin = L.above.n ? (L.above.width + 63) / 64 : 0;
  const dim3 grid((unsigned)(p.T2 * p.gy + fin));
  if (p.ks) {
    auto by = [](unsigned d) {
      int c = 0;
      while ((1u << c) < d) ++c;
      return DivBy{(unsigned)((((unsigned long long)1 << (31 + c)) + d - 1) / d), 31 + c};
    };
    const dim3 gs((unsigned)((p.T2 + 7) / 8 * 8 * p.gy + fin));
    const int T = (int)((P + 63) / 64);
    const DivBy dhw = by((unsigned)(L.h * L.w)), dw = by((unsigned)L.w);
#define DNB_D3S(KS, U) hipLaunchKernelGGL((k_dgrad3s<KS, U>), gs, dim3(512), p.lds, st, A, T, dhw, dw)
    if (p.ks == 1) { if (p.u == 1) DNB_D3S(1, 1); else DNB_D3S(1, 2); }
    else if (p.u <= 2) DNB_D3S(2, 2); else if (p.u == 3) DNB_D3S(2, 3); else DNB_D3S(2, 4);
#undef DNB_D3S
  } else {
#define DNB_D3(NT, MT)                                                                             \
  do {                                                                                             \
    if (p.bypass) hipLaunchKernelGGL((k_dgrad3<NT, MT, true>), grid, dim3(256), p.lds, st, A);     \
    else hipLaunchKernelGGL((k_dgrad3<NT, MT, false>), grid, dim3(256), p.lds, st, A);             \
  } while (0)
#define DNB_D3M(NT)                                   \
  do {                                                \
    if (p.MT == 2) DNB_D3(NT, 2); else DNB_D3(NT, 1); \
  } while (0)
  if (p.NT == 4) DNB_D3M(4); else if (p.NT == 2) DNB_D3M(2); else DNB_D3M(1);
#undef DNB_D3M
#undef DNB_D3
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // BN2's element-wise pass.  Up to 128 partials per channel are added by its own workgroups (98 take them 1 us,
  // a launch 4.5); more (large images, where a launch weighs little) are first brought down to one.
  const float2* part = (const float2*)L.part2;
  int T = p.T2;
  if (T > 128) {
    float2* one = (float2*)L.part2 + (int64_t)T * L.B;
    hipLaunchKernelGGL(k_sum_pairs, dim3((unsigned)((L.B + 63) / 64)), dim3(256), 0, st, part, T, L.B, one);
    part = one;
    T = 1;
  }
  const int cv = L.B / 8;
  int lsh = 5;
  for (int s = 4; s >= 2; --s)
    if (((cv + (1 << s) - 1) >> s << s) < ((cv + (1 << lsh) - 1) >> lsh << lsh)) lsh = s;
  const int rows = 256 >> lsh;
  int64_t ppb = (int64_t)rows * 2;
  while ((P + ppb - 1) / ppb > 2048) ppb *= 2;
  const dim3 ga((unsigned)((P + ppb - 1) / ppb), (unsigned)((cv + (1 << lsh) - 1) >> lsh));
  hipLaunchKernelGGL(k_bn2_apply, ga, dim3(256), 0, st, (u16*)L.db, (const u16*)L.b, P, L.B, (int)ppb, lsh, A.inv_p,
                     L.fold2, L.mean_b, L.istd_b, part, T, L.dgamma2, L.dbeta2);
  return hipGetLastError();
}

hipError_t bwd_dgrad1(const BwdLayer& L, float2* part, int* Tp, hipStream_t st) {
  const int64_t P = (int64_t)L.n * L.h * L.w;
  Dgrad1Args A{};
  A.db = (const u16*)L.db; A.B = L.B;
  A.W = (const u16*)L.pk1t; A.C16 = (L.c + 15) & ~15; A.B32 = (L.B + 31) & ~31;
  A.x = (const u16*)L.x; A.x_ld = L.x_ld;
  A.dy = (const u16*)L.dy; A.G = L.G; A.g_ld = L.ld;
  A.fold1 = L.fold1; A.mean = L.mean_y; A.istd = L.istd_y;
  A.part1 = part; A.C = L.c; A.P = P;
  const int T = dgrad1_splits(P, L.c, kFarSplits, &A.ppw);
  *Tp = T;
  const dim3 grid((unsigned)((L.c + 31) / 32), (unsigned)T);
  if (L.last) hipLaunchKernelGGL(k_dgrad1<true>, grid, dim3(256), 0, st, A);
  else hipLaunchKernelGGL(k_dgrad1<false>, grid, dim3(256), 0, st, A);
  return hipGetLastError();
}

hipError_t bwd_dx0(const BwdLayer& L, void* dx0, hipStream_t st) {
  const int64_t P = (int64_t)L.n * L.h * L.w;
  int64_t ppb = 64;
  while ((P + ppb - 1) / ppb * ((L.c + 255) / 256) > 2048) ppb *= 2;
  hipLaunchKernelGGL(k_dx0, dim3((unsigned)((L.c + 255) / 256), (unsigned)((P + ppb - 1) / ppb)), dim3(256), 0, st, L.G, L.ld,
                     (const u16*)L.y, L.ld, (u16*)dx0, P, L.c, (int)ppb, 1.0f / (float)P, L.K_set ? L.K : nullptr, L.above,
                     L.mean_y, L.istd_y);
  return hipGetLastError();
}

}  // namespace nhwc
}  // namespace dnb
