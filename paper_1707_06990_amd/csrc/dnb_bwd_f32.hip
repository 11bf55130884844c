// fp32 / NCHW backward chain of a bottleneck layer, the part behind the 3x3 data gradient:
//
//   k_dgrad3_v4 / _wpm / _v3  (dnb_conv_f32_fast.hip) 3x3 data gradient, BN2's mask and sums
//   k_bn_bwd_apply            gradient of b_l, element-wise on P x B
//   k_dgrad1 / s / p          1x1 data gradient; BN1+ReLU backward and the concatenation's backward
//                             (accumulate into the slab G) in the epilogue, with BN1's two sums.  Where the slab
//                             is large, layers go in pairs: layer l-1 needs of layer l only its own slice, so
//                             after layer l's b_l gradient only those k channels are formed, and after layer
//                             l-1's the channels below, of both layers, in one pass (k_dgrad1p)
//   k_wgrad_pair              both weight gradients, the end of this BN1 (bn1_finish_body) and the sums of
//                             the previous layer's weight-gradient partials
//
// BN1's backward is  du = s*(dz - dbeta/P - xhat*dgamma/P),  dz = the masked gradient, s = gamma*istd.
// Its first term needs no sum, so it is added into the slab where dz is formed; the other two are
// constants per channel times 1 and xhat, and xhat does not depend on the layer.  They are collected per
// channel, K0 = sum_l s_l*dbeta_l/P and K1 = sum_l s_l*dgamma_l/P, and taken off once, where a slice of
// the slab is finally read:  g = G - K0 - K1*xhat.  Per layer that is 12 bytes per element of the
// concatenated input (x, G read, G write) instead of 36 (gradient written; read with x by the reduction;
// read with x and G by the element-wise pass, G written), and five launches per layer instead of six or seven.
// DenseNet-BC-100 step 5.25 -> 4.92 ms (fused), 6.54 -> 6.20 ms (shared), DenseNet-BC-250 45.0 -> 42.5 ms, before
// k_dgrad1s.  What is left: the 3x3 data gradient, 20 us with the correction and BN2's sums against 15 without on
// the first block of BC-100 (its 108 weight registers leave none for prefetching).
#include "dnb_f32_dev.h"
#include "dnb_internal.h"
#include "dnb_stats.h"

namespace dnb {

namespace {

struct Dgrad1Args {
  const float* db; int64_t db_stride; int B;  // gradient of b_l
  const float* W; int C16, B16;               // packed weights [C16][B16]
  const float* x; int64_t x_stride;           // concatenated features
  const float* dy; float* G; int64_t g_stride;  // slab; dy replaces its first read (FIRST)
  const float *gamma, *beta, *mean, *istd;
  float2* part1; int lo, C, T;                // channels lo..C-1; out [C - lo][T]
  int hw, tpi, tiles, nwm;
};
// The lower layer of a pair (k_dgrad1p); Dgrad1Args holds the upper one.
struct Dgrad1Lower {
  const float *db, *W; int C16;
  const float *gamma, *beta;
  float2* part1;
};

// Output channels on M, pixels on N; bound by the slab's traffic (12 bytes per element against 2*B
// flops).  A wave owns 32 channels (two M-tiles) and walks over 64-pixel tiles T apart: a lane holds 4
// consecutive pixels of 8 channels, so x and the slab move in 16-byte pieces, 256 contiguous bytes per
// channel.  The waves of a workgroup take neighbouring channels of the same tile (the db rows they share
// come from L1) or, where there are few channels, other tiles; they share nothing else, the sums stay in
// registers until a wave's last tile.
// NCH: 16-channel chunks of b_l whose weights stay in registers; 0: read in the loop.
template <int NCH, bool FIRST, bool SLICE>
__global__ __launch_bounds__(256, 2) void k_dgrad1(Dgrad1Args A) {
  const int lo = SLICE ? A.lo : 0;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, j = lane & 15, g = lane >> 4;
  const int wm = wave % A.nwm, wp = wave / A.nwm, nwp = 4 / A.nwm;
  const int m0 = (lo & ~15) + ((int)blockIdx.y * A.nwm + wm) * 32, t0 = (int)blockIdx.x * nwp + wp;
  if (m0 >= A.C || t0 >= A.T) return;
  const int HW = A.hw, nch = A.B16 >> 4;
  const int mt[2] = {m0 >> 4, min((m0 >> 4) + 1, (A.C16 >> 4) - 1)};
  constexpr int KR = NCH > 0 ? NCH : 1;
  float4 w[2][KR];
  if (NCH > 0) {
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int c = 0; c < KR; ++c) w[a][c] = ldg4(wfrag(A.W, A.B16, mt[a], c));
  }
  float sc[2][4], sf[2][4], mu[2][4], s0[2][4], s1[2][4];
  auto ch = [&](int a, int r) { return min(m0 + a * 16 + 4 * g + r, A.C - 1); };
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int c = ch(a, r);
      mu[a][r] = A.mean[c];
      bn_fold(A.gamma[c], A.beta[c], mu[a][r], A.istd[c], sc[a][r], sf[a][r]);
      s0[a][r] = s1[a][r] = 0.f;
    }

  for (int tile = t0; tile < A.tiles; tile += A.T) {
    const int img = tile / A.tpi, q = (tile - img * A.tpi) * 64 + 4 * j;
    const bool ok = q < HW;  // HW % 4 == 0: a lane's four pixels are in or out together
    const int qc = ok ? q : 0;
    const float* dbp = A.db + (int64_t)img * A.db_stride + qc;
    const float* xp = A.x + (int64_t)img * A.x_stride + qc;
    const float* rp = (FIRST ? A.dy : A.G) + (int64_t)img * A.g_stride + qc;
    float4 d[KR][4], x4[2][4], g4[2][4];
    if (NCH > 0) {
#pragma unroll
      for (int c = 0; c < KR; ++c)
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) d[c][ks] = ldg4(dbp + (int64_t)min(c * 16 + 4 * ks + g, A.B - 1) * HW);
    }
    auto load_slab = [&](int a) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        x4[a][r] = ldg4(xp + (int64_t)ch(a, r) * HW);
        g4[a][r] = ldg4(rp + (int64_t)ch(a, r) * HW);
      }
    };
    load_slab(0);
    if (NCH > 0) load_slab(1);  // (beside the chunk ring of the other form there are registers for one half)
    f32x4 acc[2][4];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[a][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    auto products = [&](const float4(&dd)[4], const float4& w0, const float4& w1) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          acc[0][t] = mfma16(elem(w0, ks), elem(dd[ks], t), acc[0][t]);
          acc[1][t] = mfma16(elem(w1, ks), elem(dd[ks], t), acc[1][t]);
        }
    };
    if (NCH > 0) {
#pragma unroll
      for (int c = 0; c < KR; ++c) products(d[c], w[0][c], w[1][c]);
    } else {
      float4 da[2][4], wa[2][2];  // two chunks in flight
      auto load = [&](int c, float4(&dd)[4], float4(&ww)[2]) {
        c = min(c, nch - 1);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) dd[ks] = ldg4(dbp + (int64_t)min(c * 16 + 4 * ks + g, A.B - 1) * HW);
        ww[0] = ldg4(wfrag(A.W, A.B16, mt[0], c));
        ww[1] = ldg4(wfrag(A.W, A.B16, mt[1], c));
      };
      load(0, da[0], wa[0]);
      load(1, da[1], wa[1]);
      for (int c = 0; c < nch; c += 2) {
        products(da[0], wa[0][0], wa[0][1]);
        load(c + 2, da[0], wa[0]);
        if (c + 1 < nch) products(da[1], wa[1][0], wa[1][1]);
        load(c + 3, da[1], wa[1]);
      }
      load_slab(1);
    }
    if (ok) {
      float* op = A.G + (int64_t)img * A.g_stride + q;
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float o[4];
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const float xv = elem(x4[a][r], t), dz = __fmaf_rn(xv, sc[a][r], sf[a][r]) > 0.f ? acc[a][t][r] : 0.f;
            o[t] = __fmaf_rn(sc[a][r], dz, elem(g4[a][r], t));
            s0[a][r] += dz;
            s1[a][r] = __fmaf_rn(dz, xv - mu[a][r], s1[a][r]);
          }
          if (m0 + a * 16 + 4 * g + r < A.C && (!SLICE || m0 + a * 16 + 4 * g + r >= lo))
            *reinterpret_cast<float4*>(op + (int64_t)ch(a, r) * HW) = make_float4(o[0], o[1], o[2], o[3]);
        }
    }
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float u = row16_sum(s0[a][r]), v = row16_sum(s1[a][r]);
      const int m = m0 + a * 16 + 4 * g + r;
      if (j == 0 && m < A.C && (!SLICE || m >= lo)) A.part1[(int64_t)(m - lo) * A.T + t0] = make_float2(u, v * A.istd[m]);
    }
}

// The same where a workgroup's four waves have four groups of 32 channels to share a tile among: the tile
// of db sits in LDS, staged one tile ahead, so that the products wait for no load of their own; x and the
// slab, requested before them, arrive under them.  (Read by every wave for itself, the db rows of a tile
// queued behind the slab's loads: loads return in order.)  DenseNet-BC-250 step 42.4 -> 39.95 ms, BC-100 4.96 -> 4.83.
template <int NCH, bool FIRST>
__global__ __launch_bounds__(256, 2) void k_dgrad1s(Dgrad1Args A) {
  __shared__ __attribute__((aligned(16))) float tile_db[NCH * 16 * 64];
  __shared__ float4 cst[128];  // scale, shift, mean, 1/std of the workgroup's channels
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, j = lane & 15, g = lane >> 4;
  const int mw = (int)blockIdx.y * 128, m0 = mw + wave * 32, HW = A.hw, t0 = blockIdx.x;
  if (tid < 128) {
    const int c = min(mw + tid, A.C - 1);
    float sc, sf;
    bn_fold(A.gamma[c], A.beta[c], A.mean[c], A.istd[c], sc, sf);
    cst[tid] = make_float4(sc, sf, A.mean[c], A.istd[c]);
  }
  const int mtl = (A.C16 >> 4) - 1;
  float4 w[2][NCH];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int c = 0; c < NCH; ++c) w[a][c] = ldg4(wfrag(A.W, A.B16, min((m0 >> 4) + a, mtl), c));
  auto ch = [&](int a, int r) { return min(m0 + a * 16 + 4 * g + r, A.C - 1); };
  float s0[2][4], s1[2][4];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int r = 0; r < 4; ++r) s0[a][r] = s1[a][r] = 0.f;

  float4 st[NCH];  // thread: row 16u + tid/16, pixels 4*(tid%16)..+3
  const int srow = tid >> 4, scol = 4 * (tid & 15);
  auto request = [&](int tile) {
    const int img = tile / A.tpi, q = min((tile - img * A.tpi) * 64 + scol, HW - 4);
    const float* p = A.db + (int64_t)img * A.db_stride + q;
#pragma unroll
    for (int u = 0; u < NCH; ++u) st[u] = ldg4(p + (int64_t)min(u * 16 + srow, A.B - 1) * HW);
  };
  request(t0);
  for (int tile = t0; tile < A.tiles; tile += A.T) {
    __syncthreads();  // the previous tile's reads are done
#pragma unroll
    for (int u = 0; u < NCH; ++u) *reinterpret_cast<float4*>(&tile_db[(u * 16 + srow) * 64 + scol]) = st[u];
    __syncthreads();
    const int img = tile / A.tpi, q = (tile - img * A.tpi) * 64 + 4 * j;
    const bool ok = q < HW;  // HW % 4 == 0: a lane's four pixels are in or out together
    const int qc = ok ? q : 0;
    const float* xp = A.x + (int64_t)img * A.x_stride + qc;
    const float* rp = (FIRST ? A.dy : A.G) + (int64_t)img * A.g_stride + qc;
    float4 x4[2][4], g4[2][4];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        x4[a][r] = ldg4(xp + (int64_t)ch(a, r) * HW);
        g4[a][r] = ldg4(rp + (int64_t)ch(a, r) * HW);
      }
    request(min(tile + A.T, A.tiles - 1));
    __builtin_amdgcn_sched_barrier(0);  // all of these are in flight before the products
    f32x4 acc[2][4];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[a][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < NCH; ++c)
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const float4 d = *reinterpret_cast<const float4*>(&tile_db[(c * 16 + 4 * ks + g) * 64 + 4 * j]);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          acc[0][t] = mfma16(elem(w[0][c], ks), elem(d, t), acc[0][t]);
          acc[1][t] = mfma16(elem(w[1][c], ks), elem(d, t), acc[1][t]);
        }
      }
    __builtin_amdgcn_sched_barrier(0);
    if (ok) {
      float* op = A.G + (int64_t)img * A.g_stride + q;
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float4 k = cst[wave * 32 + a * 16 + 4 * g + r];
          float o[4];
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const float xv = elem(x4[a][r], t), dz = __fmaf_rn(xv, k.x, k.y) > 0.f ? acc[a][t][r] : 0.f;
            o[t] = __fmaf_rn(k.x, dz, elem(g4[a][r], t));
            s0[a][r] += dz;
            s1[a][r] = __fmaf_rn(dz, xv - k.z, s1[a][r]);
          }
          if (m0 + a * 16 + 4 * g + r < A.C)
            *reinterpret_cast<float4*>(op + (int64_t)ch(a, r) * HW) = make_float4(o[0], o[1], o[2], o[3]);
        }
    }
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float u = row16_sum(s0[a][r]), v = row16_sum(s1[a][r]);
      const int m = m0 + a * 16 + 4 * g + r;
      if (j == 0 && m < A.C) A.part1[(int64_t)m * A.T + t0] = make_float2(u, v * cst[wave * 32 + a * 16 + 4 * g + r].w);
    }
}

// Two layers at once, on the channels that both read: x and the slab move once for the two, 12 bytes per element
// instead of 24.  Eight waves of 16 channels each; both layers' weights stay in registers, both tiles of db sit in
// LDS, in two buffers: the next pixel tile is put down between the two layers' products, one barrier a tile.  65536
// pixels, 1000 channels, 96 outputs: 232 us (283 with one buffer and operands read as they are needed) and 13 for the
// slice between, against 2 x 240; 786 MB and 25.8 GFLOP, 111 TFLOP/s.
template <int NCH, bool FIRST>
__global__ __launch_bounds__(512) void k_dgrad1p(Dgrad1Args A, Dgrad1Lower B) {
  extern __shared__ __attribute__((aligned(16))) float tile_db[];  // two buffers of [2][NCH*16][64]
  __shared__ float4 cst[2][128];  // scale, shift, mean, 1/std of the workgroup's channels
  constexpr int TS = NCH * 16 * 64, SU = (NCH + 1) / 2;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, j = lane & 15, g = lane >> 4;
  const int mw = (int)blockIdx.y * 128, m0 = mw + wave * 16, HW = A.hw, t0 = blockIdx.x;
  if (tid < 256) {
    const int li = tid >> 7, c = min(mw + (tid & 127), A.C - 1);
    float sc, sf;
    bn_fold((li ? B.gamma : A.gamma)[c], (li ? B.beta : A.beta)[c], A.mean[c], A.istd[c], sc, sf);
    cst[li][tid & 127] = make_float4(sc, sf, A.mean[c], A.istd[c]);
  }
  float4 w[2][NCH];
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    w[0][c] = ldg4(wfrag(A.W, A.B16, min(m0 >> 4, (A.C16 >> 4) - 1), c));
    w[1][c] = ldg4(wfrag(B.W, A.B16, min(m0 >> 4, (B.C16 >> 4) - 1), c));
  }
  auto ch = [&](int r) { return min(m0 + 4 * g + r, A.C - 1); };
  float s0[2][4], s1[2][4];
#pragma unroll
  for (int li = 0; li < 2; ++li)
#pragma unroll
    for (int r = 0; r < 4; ++r) s0[li][r] = s1[li][r] = 0.f;

  float4 st[2][SU];  // thread: rows 32u + tid/16, pixels 4*(tid%16)..+3
  const int srow = tid >> 4, scol = 4 * (tid & 15);
  auto request = [&](int tile) {
    const int img = tile / A.tpi, q = min((tile - img * A.tpi) * 64 + scol, HW - 4);
#pragma unroll
    for (int u = 0; u < SU; ++u) {
      const int64_t o = (int64_t)img * A.db_stride + q + (int64_t)min(u * 32 + srow, A.B - 1) * HW;
      st[0][u] = ldg4(A.db + o);
      st[1][u] = ldg4(B.db + o);
    }
  };
  auto deposit = [&](int buf) {
#pragma unroll
    for (int u = 0; u < SU; ++u) {
      const int row = u * 32 + srow;
      if (NCH % 2 == 0 || row < NCH * 16) {
        lds_st4(&tile_db[buf + row * 64 + scol], st[0][u]);
        lds_st4(&tile_db[buf + TS + row * 64 + scol], st[1][u]);
      }
    }
  };
  request(t0);
  deposit(0);
  request(min(t0 + A.T, A.tiles - 1));
  __syncthreads();
  for (int tile = t0, buf = 0; tile < A.tiles; tile += A.T, buf ^= 2 * TS) {
    const int img = tile / A.tpi, q = (tile - img * A.tpi) * 64 + 4 * j;
    const bool ok = q < HW;  // HW % 4 == 0: a lane's four pixels are in or out together
    const int qc = ok ? q : 0;
    const float* xp = A.x + (int64_t)img * A.x_stride + qc;
    const float* rp = (FIRST ? A.dy : A.G) + (int64_t)img * A.g_stride + qc;
    float4 x4[4], g4[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      x4[r] = ldg4(xp + (int64_t)ch(r) * HW);
      g4[r] = ldg4(rp + (int64_t)ch(r) * HW);
    }
    __builtin_amdgcn_sched_barrier(0);  // all of these are in flight before the products
    // operands two steps ahead of their products, held there by scheduling barriers (left alone, the compiler reads two
    // and waits for them)
    constexpr int S = NCH * 4;
    float4 d[3];
    auto operand = [&](int s) { return lds_ld4(&tile_db[buf + s / S * TS + (4 * (s % S) + g) * 64 + 4 * j]); };
    d[0] = operand(0);
    d[1] = operand(1);
#pragma unroll
    for (int li = 0; li < 2; ++li) {
      f32x4 acc[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[t] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < S; ++i) {
        const int s = li * S + i;
        if (s + 2 < 2 * S) d[(s + 2) % 3] = operand(s + 2);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = mfma16(elem(w[li][i / 4], i % 4), elem(d[s % 3], t), acc[t]);
        __builtin_amdgcn_sched_barrier(0);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float4 k = cst[li][wave * 16 + 4 * g + r];
        float o[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const float xv = elem(x4[r], t), dz = ok && __fmaf_rn(xv, k.x, k.y) > 0.f ? acc[t][r] : 0.f;
          o[t] = __fmaf_rn(k.x, dz, elem(g4[r], t));
          s0[li][r] += dz;
          s1[li][r] = __fmaf_rn(dz, xv - k.z, s1[li][r]);
        }
        g4[r] = make_float4(o[0], o[1], o[2], o[3]);
      }
      if (li == 0) {  // the next tile to the other buffer, whose reads ended before the last barrier
        deposit(buf ^ (2 * TS));
        request(min(tile + 2 * A.T, A.tiles - 1));
      }
    }
    if (ok) {
      float* op = A.G + (int64_t)img * A.g_stride + q;
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (m0 + 4 * g + r < A.C) *reinterpret_cast<float4*>(op + (int64_t)ch(r) * HW) = g4[r];
    }
    __syncthreads();
  }
#pragma unroll
  for (int li = 0; li < 2; ++li)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float u = row16_sum(s0[li][r]), v = row16_sum(s1[li][r]);
      const int m = m0 + 4 * g + r;
      if (j == 0 && m < A.C) (li ? B.part1 : A.part1)[(int64_t)m * A.T + t0] = make_float2(u, v * cst[li][wave * 16 + 4 * g + r].w);
    }
}

// dx0 = G - K0 - K1*xhat on the block input's channels.  grid (channels, image ranges), 16-byte accesses.
__global__ __launch_bounds__(256) void k_dx0(const float* __restrict__ G, int64_t g_stride, const float* __restrict__ x,
                                             int64_t x_stride, float* __restrict__ dx0, int64_t d_stride, int n, int hw,
                                             int ipb, const float2* __restrict__ K, const float* __restrict__ mean,
                                             const float* __restrict__ istd) {
  const int ch = blockIdx.x, n0 = blockIdx.y * ipb, ni = min(n, n0 + ipb) - n0;
  const float k0 = K[ch].x, k1 = K[ch].y * istd[ch], mu = mean[ch];
  const int64_t inner = (int64_t)ch * hw;
  for (RowIter it(hw / 4, threadIdx.x, 256); it.img < ni; it.next()) {
    const int64_t im = n0 + it.img, q = inner + (int64_t)it.q * 4;
    const float4 gv = ldg4(G + im * g_stride + q), xv = ldg4(x + im * x_stride + q);
    *reinterpret_cast<float4*>(dx0 + im * d_stride + q) =
        make_float4((gv.x - k0) - k1 * (xv.x - mu), (gv.y - k0) - k1 * (xv.y - mu), (gv.z - k0) - k1 * (xv.z - mu),
                    (gv.w - k0) - k1 * (xv.w - mu));
  }
}

__global__ __launch_bounds__(256) void k_bn1_finish(Bn1Finish f) { bn1_finish_body(f, blockIdx.x); }

}  // namespace

// Pixel ranges of k_dgrad1 (= partial pairs per channel): about 2048 waves in all (two per SIMD), at most
// one tile each.
int bwd32_dgrad1_splits(int n, int hw, int c) {
  const int64_t tiles = (int64_t)((hw + 63) / 64) * n, groups = (c + 31) / 32;
  int64_t t = 2048 / groups;
  if (t > 512) t = 512;
  if (t > tiles) t = tiles;
  return t < 1 ? 1 : (int)t;
}
// ... of a pair's k channels between its layers: a tile per wave where there are up to 1024 (with two, the loads of
// a second tile waited out behind the first's products: 13.5 us a launch on the first block of BC-100)
static int near_splits(int n, int hw) {
  const int64_t tiles = (int64_t)((hw + 63) / 64) * n;
  return tiles < 1024 ? (int)tiles : 1024;
}
// ... of k_dgrad1p: one workgroup of 128 channels per CU.
static int dgrad1p_splits(int n, int hw, int c) {
  const int64_t tiles = (int64_t)((hw + 63) / 64) * n, groups = (c + 127) / 128;
  int64_t t = 256 / groups;
  if (t > tiles) t = tiles;
  return t < 1 ? 1 : (int)t;
}
size_t bwd32_partial1_floats(int n, int hw, int c) { return 2 * (size_t)c * bwd32_dgrad1_splits(n, hw, c); }
size_t bwd32_partial1_pair_floats(int n, int hw, int c) { return 4 * (size_t)c * dgrad1p_splits(n, hw, c); }
size_t bwd32_partial1_near_floats(int n, int hw, int k) { return 2 * (size_t)k * near_splits(n, hw); }

// Whether a layer over c channels and the one above it share their pass over the slab.  What that saves is half
// the slab's traffic, what it costs a launch for the k channels between them: from about 56 MB a layer on
// (16384 pixels x 216 channels: 17 + 9 us against 2 x 12; 65536 x 96: 26 + 9 against 18 + 20; x 180: 46 + 9
// against 2 x 36).
bool bwd32_pair_ok(int n, int hw, int c, int B) {
  const int B16 = (B + 15) & ~15;
  return B16 >= 48 && B16 <= 128 && c > 64 && (int64_t)12 * c * n * hw >= (int64_t)56 << 20;
}

hipError_t bwd32_dgrad1(const Bwd32Layer& L, hipStream_t st) {
  Dgrad1Args A{};
  const int hw = L.h * L.w;
  A.db = L.db; A.db_stride = (int64_t)L.B * hw; A.B = L.B;
  A.W = L.pk1t; A.C16 = (L.cw + 15) & ~15; A.B16 = (L.B + 15) & ~15;
  A.x = L.x; A.x_stride = L.x_stride;
  A.dy = L.dy; A.G = L.G; A.g_stride = L.ys;
  A.gamma = L.g1; A.beta = L.b1; A.mean = L.mean_y; A.istd = L.istd_y;
  A.part1 = L.part1; A.lo = L.lo; A.C = L.c;
  A.hw = hw; A.tpi = (hw + 63) / 64; A.tiles = A.tpi * L.n;
  if (L.up_db) {  // with the layer above
    const Dgrad1Lower B{L.db, L.pk1t, A.C16, L.g1, L.b1, L.part1 + (int64_t)L.c * dgrad1p_splits(L.n, hw, L.c)};
    A.db = L.up_db; A.W = L.up_pk1t; A.C16 = (L.c + L.k + 15) & ~15; A.gamma = L.up_g1; A.beta = L.up_b1;
    A.T = dgrad1p_splits(L.n, hw, L.c);
    const dim3 grid((unsigned)A.T, (unsigned)((L.c + 127) / 128));
#define DNB_L(NCH)                                                                                            \
  do {                                                                                                        \
    const size_t lds = (size_t)4 * NCH * 16 * 64 * sizeof(float);                                             \
    if (L.first) hipLaunchKernelGGL((k_dgrad1p<NCH, true>), grid, dim3(512), lds, st, A, B);                  \
    else hipLaunchKernelGGL((k_dgrad1p<NCH, false>), grid, dim3(512), lds, st, A, B);                         \
  } while (0)
    switch (A.B16 >> 4) {
      case 3: DNB_L(3); break; case 4: DNB_L(4); break; case 5: DNB_L(5); break; case 6: DNB_L(6); break;
      case 7: DNB_L(7); break; default: DNB_L(8); break;
    }
#undef DNB_L
    return hipGetLastError();
  }
  const int groups = (L.c - (L.lo & ~15) + 31) / 32;
  A.T = L.lo ? near_splits(L.n, hw) : bwd32_dgrad1_splits(L.n, hw, L.c);
  A.nwm = groups >= 3 ? 4 : groups;
  const int nwp = 4 / A.nwm;
  // (fewer chunks: the products are too few to hide anything; more: no registers for their weights)
  if (A.nwm == 4 && A.B16 >= 48 && A.B16 <= 128 && L.lo == 0) {
    const dim3 grid((unsigned)A.T, (unsigned)((groups + 3) / 4));
#define DNB_L(NCH)                                                                       \
  do {                                                                                   \
    if (L.first) hipLaunchKernelGGL((k_dgrad1s<NCH, true>), grid, dim3(256), 0, st, A);   \
    else hipLaunchKernelGGL((k_dgrad1s<NCH, false>), grid, dim3(256), 0, st, A);         \
  } while (0)
    switch (A.B16 >> 4) {
      case 3: DNB_L(3); break; case 4: DNB_L(4); break; case 5: DNB_L(5); break; case 6: DNB_L(6); break;
      case 7: DNB_L(7); break; default: DNB_L(8); break;
    }
#undef DNB_L
    return hipGetLastError();
  }
  const dim3 grid((unsigned)((A.T + nwp - 1) / nwp), (unsigned)((groups + A.nwm - 1) / A.nwm));
#define DNB_LF(NCH, SLICE)                                                                      \
  do {                                                                                          \
    if (L.first) hipLaunchKernelGGL((k_dgrad1<NCH, true, SLICE>), grid, dim3(256), 0, st, A);   \
    else hipLaunchKernelGGL((k_dgrad1<NCH, false, SLICE>), grid, dim3(256), 0, st, A);          \
  } while (0)
#define DNB_L(NCH)                                                                              \
  do {                                                                                          \
    if (L.lo) DNB_LF(NCH, true); else DNB_LF(NCH, false);                                       \
  } while (0)
  switch (A.B16 >> 4) {
    case 1: DNB_LF(1, false); break; case 2: DNB_LF(2, false); break; case 3: DNB_L(3); break; default: DNB_L(0); break;
  }
#undef DNB_LF
#undef DNB_L
  return hipGetLastError();
}

void bwd32_bn1_finish(const Bwd32Layer& L, Bn1Finish* out) {
  const int hw = L.h * L.w, W = L.c - L.lo;
  const int T = L.up_db ? dgrad1p_splits(L.n, hw, L.c) : L.lo ? near_splits(L.n, hw) : bwd32_dgrad1_splits(L.n, hw, L.c);
  *out = Bn1Finish{};
  out->n = L.up_db ? 2 : 1;
  out->T = T; out->C = W; out->lo = L.lo; out->wgs = (W + 3) / 4;
  for (int q = 0; q < out->n; ++q) {
    const bool up = L.up_db && q == 0;
    out->part[q] = L.part1 + (int64_t)q * W * T;
    out->gamma[q] = up ? L.up_g1 : L.g1;
    out->dgamma[q] = up ? L.up_dgamma1 : L.dgamma1;
    out->dbeta[q] = up ? L.up_dbeta1 : L.dbeta1;
  }
  out->istd = L.istd_y;
  out->inv_p = 1.0f / ((float)L.n * (float)hw);
  out->K = L.K; out->first = L.first ? 1 : 0;
}
hipError_t launch_bn1_finish(const Bn1Finish& f, hipStream_t st) {
  if (f.wgs == 0) return hipSuccess;
  hipLaunchKernelGGL(k_bn1_finish, dim3((unsigned)f.wgs), dim3(256), 0, st, f);
  return hipGetLastError();
}

hipError_t bwd32_dx0(const Bwd32Layer& L, float* dx0, hipStream_t st) {
  const int hw = L.h * L.w;
  int s = 1024 / L.c, cap = (L.n * (hw / 4) + 255) / 256;  // at least one position per thread
  if (s > cap) s = cap;
  if (s > L.n) s = L.n;
  if (s < 1) s = 1;
  const int ipb = (L.n + s - 1) / s;
  hipLaunchKernelGGL(k_dx0, dim3((unsigned)L.c, (unsigned)((L.n + ipb - 1) / ipb)), dim3(256), 0, st, L.G, L.ys, L.y, L.ys, dx0,
                     (int64_t)L.c * hw, L.n, hw, ipb, (const float2*)L.K, L.mean_y, L.istd_y);
  return hipGetLastError();
}

}  // namespace dnb
