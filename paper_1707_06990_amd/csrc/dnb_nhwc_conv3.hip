// bf16 / NHWC 3x3 convolution (stride 1, zero padding) with BN statistics of its output (forward pass):
//
//   out[q][m] = sum_{t,c} W(t,m,c) * act(in[q + shift(t)][c]),  act = BN+ReLU prologue or identity.
//
// The bottleneck's width fits LDS, so a tile's input is staged whole: one round of loads, BN+ReLU applied
// once per element (coefficients in registers: a thread keeps its 8 channels), one barrier, then only LDS
// reads, weight loads (a 64-channel chunk ahead) and MFMAs.  k_conv walks the channels in chunks, with a
// wait for memory and a barrier per chunk, and gives its workgroup 64 outputs of which a growth rate of 32
// fills half.  What is left is a launch, one memory latency, the staging (56x56: 2.8 rows staged per row
// computed) and about 2300 cycles per tile each of LDS reads, weight loads and MFMAs.
// us a launch against k_conv's: 32 images of 14x14, 128 -> 32 channels 5.8 (11.5), 192 -> 48 9.0 (17);
// 7x7 5.6 (10.5) and 6.2 (14); 28x28 9.1 (13.6) and 14.1 (25); 56x56 34 (47) and 49 (66).
// Where its partials are few it folds BN2 itself (FOLD): 6.5 -> 9.5 us a launch at 14x14 with 98 partials of 128
// channels, for a k_bn_fold of 4.8 us and its place in the stream; DenseNet-264-shaped forward 4.60 -> 4.15 ms with the
// 1x1's.
// Each output's K order (chunk, tap, K-step), its rounding and the statistics' 64-pixel groups are those of
// k_conv (same bits).
#include "dnb_internal.h"
#include "dnb_nhwc_dev.h"
#include "dnb_stats.h"

namespace dnb {
namespace nhwc {

namespace {

struct Conv3Args {
  const u16* in; int64_t in_ld;
  const u16* W; int M16, K32;        // packed weights, nine taps of [M16][K32]
  u16* out; int64_t out_ld;
  int cin, cout, H, Wd;
  int tpi, tiles, gy;                // 64-pixel tiles per image, in all; groups of MG M-tiles
  const float2* fold;
  float* spart;
  FoldIn F; int cap;                 // FOLD: BN2 folded here; channels, rounded up to a power of two
};

constexpr int kFoldMax = 256;  // most channels folded inside (512 threads, two lanes a channel)

// A workgroup owns 64 pixels of one image (with a row and a pixel of halo on either side) and MG M-tiles;
// wave w < 2*MG forms M-tile w / 2 of two of the tile's four pixel tiles, all eight waves stage.
// (Two workgroups a CU asked for where tiles are many: 56x56 45 -> 34 us, 28x28 11.6 -> 9.1 us.)
template <int MG, bool PRO, bool FOLD>
__global__ __launch_bounds__(512, (MG > 1 && !FOLD ? 4 : 2)) void k_conv3(Conv3Args A) {
  extern __shared__ __attribute__((aligned(16))) u16 lds[];
  __shared__ uint2 xch[MG][4][64];
  __shared__ float2 cfl[FOLD ? kFoldMax : 1], table[FOLD ? 127 : 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), j = lane & 15, g = lane >> 4;
  const int slot = blockIdx.x >> 3, grp = slot % A.gy, tile = (slot / A.gy) * 8 + (blockIdx.x & 7);
  if (tile >= A.tiles) return;
  const int W = A.Wd, HW = A.H * W, img = tile / A.tpi, q0 = (tile - img * A.tpi) * 64;
  const int halo = W + 1, seg = 64 + 2 * halo;
  const int nch = (A.cin + 63) / 64, PITCH = nch * 64 + 8, NV = nch * 8;
  const int rpp = 512 / NV;                        // rows per pass
  const int v = tid % NV, r = tid / NV;
  const bool act = r < rpp;                        // threads past the last whole row repeat it
  const int passes = (seg + rpp - 1) / rpp;
  const u16* ib = A.in + (int64_t)img * HW * A.in_ld + min(8 * v, A.cin - 8);
  const bool cok = 8 * v < A.cin;
  float2 f[8];
  auto request = [&](int p0, uint4(&q)[4]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int s = min((p0 + u) * rpp + r, seg - 1);
      q[u] = *reinterpret_cast<const uint4*>(ib + (int64_t)min(max(q0 - halo + s, 0), HW - 1) * A.in_ld);
    }
  };
  auto deposit = [&](int p0, const uint4(&q)[4]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int s = (p0 + u) * rpp + r, px = q0 - halo + s;
      V8 x;
      x.q = q[u];
      if (PRO) {
#pragma unroll
        for (int e = 0; e < 8; ++e) x.h[e] = f2bf(fmaxf(__fmaf_rn(bf2f(x.h[e]), f[e].x, f[e].y), 0.f));
      }
      if (px < 0 || px >= HW || !cok) x.q = make_uint4(0u, 0u, 0u, 0u);
      if (act && s < seg) *reinterpret_cast<uint4*>(lds + s * PITCH + 8 * v) = x.q;
    }
  };
  auto rest = [&]() {
    for (int p = 4; p < passes; p += 4) {
      uint4 q[4];
      request(p, q);
      deposit(p, q);
    }
    if (tid < PITCH / 8) *reinterpret_cast<uint4*>(lds + seg * PITCH + 8 * tid) = make_uint4(0u, 0u, 0u, 0u);  // a row of zeros
    __syncthreads();
  };
  uint4 q[4];
  request(0, q);
  if (PRO) {
    const int cf = min(8 * v, A.cin - 8);
    if (FOLD) {  // every workgroup folds the BN of its input for itself, the first keeps the result
      float2* sh = reinterpret_cast<float2*>(lds);  // [2][512], before the tile
      const int ch = tid & (A.cap - 1), ql = tid / A.cap, cc = min(ch, A.cin - 1);
      stat_table(StatRuns{A.F.T, A.F.per, A.F.tpr}, table, tid);
      __syncthreads();
      if (A.cap == 64) stat_merge_runs<8>(A.F.part, A.F.T, A.cin, cc, ql, table, sh, 512, tid);
      else if (A.cap == 128) stat_merge_runs<4>(A.F.part, A.F.T, A.cin, cc, ql, table, sh, 512, tid);
      else stat_merge_runs<2>(A.F.part, A.F.T, A.cin, cc, ql, table, sh, 512, tid);
      __syncthreads();
      if (tid < A.cin) {
        const float ga = A.F.gamma[tid], be = A.F.beta[tid];
        const float2 m = A.cap == 64 ? stat_merge_finish<8>(sh, A.F.T, table, 64, 512, tid)
                         : A.cap == 128 ? stat_merge_finish<4>(sh, A.F.T, table, 128, 512, tid)
                                        : stat_merge_finish<2>(sh, A.F.T, table, 256, 512, tid);
        const float is = bn_istd(m.y, A.F.count, A.F.eps);
        float2 o;
        bn_fold(ga, be, m.x, is, o.x, o.y);
        cfl[tid] = o;
        if (tile == 0 && grp == 0) { A.F.mean[tid] = m.x; A.F.istd[tid] = is; A.F.fold[tid] = o; }
      }
      __syncthreads();
#pragma unroll
      for (int e = 0; e < 8; ++e) f[e] = cfl[cf + e];
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) f[e] = A.fold[cf + e];
    }
  }

  const int mt = grp * MG + (wave >> 1), tp = (wave & 1) * 2;
  const int left = min(64, HW - q0);               // pixels of the tile
  if (wave < 2 * MG) {
    // weights of a 64-channel chunk: nine taps x two K-steps, each requested a chunk ahead
    const int nk = A.K32 >> 5;
    const char* wb = reinterpret_cast<const char*>(A.W) + (int64_t)min(mt, A.M16 / 16 - 1) * nk * 1024;
    const int64_t ts = (int64_t)A.M16 * A.K32 * 2;
    uint4 w[9][2];
    auto wload = [&](int c, int t9) {
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
        w[t9][kk] = *reinterpret_cast<const uint4*>(wb + t9 * ts + (int64_t)min(2 * c + kk, nk - 1) * 1024 + (unsigned)lane * 16);
    };
#pragma unroll
    for (int t9 = 0; t9 < 9; ++t9) wload(0, t9);
    deposit(0, q);
    rest();
    f32x4 acc[2];
    int row[2], zero = seg * PITCH + 8 * g;
    bool lok[2], rok[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      acc[t] = (f32x4){0.f, 0.f, 0.f, 0.f};
      const int i = (tp + t) * 16 + j, wc = (q0 + i) % W;
      row[t] = (i + halo) * PITCH + 8 * g;
      lok[t] = wc != 0;
      rok[t] = wc != W - 1;
    }
    auto tap = [&](int c, int t9, int kk) {
      const int di = t9 / 3 - 1, dj = t9 % 3 - 1, off = (di * W + dj) * PITCH;
      V8 wv;
      wv.q = w[t9][kk];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int a = ((dj < 0 && !lok[t]) || (dj > 0 && !rok[t]) ? zero : row[t] + off) + c * 64;
        V8 x;
        x.q = *reinterpret_cast<const uint4*>(lds + a + kk * 32);
        acc[t] = mfma_bf16(wv, x, acc[t]);
      }
    };
    for (int c = 0; c < nk >> 1; ++c) {
#pragma unroll
      for (int t9 = 0; t9 < 9; ++t9) {
        tap(c, t9, 0);
        tap(c, t9, 1);
        wload(min(c + 1, nch - 1), t9);
      }
    }
    // the last chunk's one K-step by itself (beside it lie zeros, but an infinite weight times zero is not zero)
    if (nk & 1) {
#pragma unroll
      for (int t9 = 0; t9 < 9; ++t9) tap(nch - 1, t9, 0);
    }
    const int m = mt * 16 + 4 * g;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      uint2 pk;
      pk.x = (unsigned)f2bf(acc[t][0]) | ((unsigned)f2bf(acc[t][1]) << 16);
      pk.y = (unsigned)f2bf(acc[t][2]) | ((unsigned)f2bf(acc[t][3]) << 16);
      xch[wave >> 1][tp + t][lane] = pk;
      const int i = (tp + t) * 16 + j;
      if (i < left && m < A.cout) *reinterpret_cast<uint2*>(A.out + ((int64_t)img * HW + q0 + i) * A.out_ld + m) = pk;  // cout % 4 == 0
    }
  } else {
    deposit(0, q);
    rest();
  }
  __syncthreads();
  // statistics of what is stored, in k_conv's order of additions: wave w forms M-tile w
  const int ms = (grp * MG + wave) * 16 + 4 * g;
  if (wave >= MG || ms >= A.cout) return;
  uint2 h[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) h[t] = xch[wave][t][lane];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float x[4], sum = 0.f, m2 = 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const unsigned p = e < 2 ? h[t].x : h[t].y;
      x[t] = __uint_as_float((e & 1) ? p & 0xffff0000u : p << 16);
      sum += (t * 16 + j < left) ? x[t] : 0.f;
    }
    sum = row16_sum(sum);
    const float mu = sum / (float)left;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const float d = x[t] - mu;
      m2 += (t * 16 + j < left) ? d * d : 0.f;
    }
    m2 = row16_sum(m2);
    if (j == 0) {
      float* o = A.spart + stat_at(A.tiles, A.cout, tile, ms + e);
      o[0] = (float)left; o[1] = mu; o[2] = m2;
    }
  }
}

}  // namespace

// The 3x3 with statistics; false (nothing launched) if the shape is not taken: a staged tile of more than
// 76 KB, or more than one workgroup per CU of which no two share a CU's LDS (six layers' forward at batch 16, 192
// channels: 62x62 to 48 of them 454 us against k_conv's 434, 60x60 to 64 466 against 438; 61x61 to 48, the last
// that share, 389 against 431).  M-tiles per workgroup: as few as keep the launch within
// a workgroup per CU, each staging the tile again (14x14, 192 -> 48: one 12.3 us, two 8.6, three 9.4), and all
// of them, up to four, where tiles alone fill the chip.  Wp: packed weights, nine taps
// of [M16][K32]; *sT = partials per channel.
bool conv3_stats(const void* in, int64_t in_ld, const void* Wp, void* out, int64_t out_ld, int n, int cin, int cout, int h, int w,
                 const float2* fold, float* spart, int* sT, const FoldIn* F, hipStream_t st) {
  const int hw = h * w, nch = (cin + 63) / 64;
  const int64_t tpi = (hw + 63) / 64, tiles = tpi * n;
  size_t lds = (size_t)(64 + 2 * (w + 1) + 1) * (nch * 64 + 8) * sizeof(u16);
  if (lds > 76 * 1024 || nch * 8 > 512 || tiles > (1 << 24)) return false;
  Conv3Args A{};
  A.in = (const u16*)in; A.in_ld = in_ld;
  A.W = (const u16*)Wp; A.M16 = (cout + 15) & ~15; A.K32 = (cin + 31) & ~31;
  A.out = (u16*)out; A.out_ld = out_ld;
  A.cin = cin; A.cout = cout; A.H = h; A.Wd = w;
  A.tpi = (int)tpi; A.tiles = (int)tiles;
  A.fold = fold; A.spart = spart;
  if (F) {
    if (F->T > kRowStats || cin > kFoldMax) return false;
    A.F = *F;
    A.cap = cin <= 64 ? 64 : cin <= 128 ? 128 : 256;
    if (A.cap * F->T > 16384) return false;  // 32 partials a thread: at 49 a launch of k_bn_fold is faster again
    if (lds < 2 * 512 * sizeof(float2)) lds = 2 * 512 * sizeof(float2);
  }
  const int mtiles = A.M16 / 16;
  int mg = 1;
  const int most = mtiles < 4 ? mtiles : mtiles % 3 == 0 ? 3 : 4;
  while (mg < most && tiles * ((mtiles + mg - 1) / mg) > 256) ++mg;
  A.gy = (mtiles + mg - 1) / mg;
  if (tiles * A.gy > 256 && (A.gy > 1 || 2 * (lds + (size_t)mg * 4 * 64 * sizeof(uint2)) > 160 * 1024)) return false;
  if (sT) *sT = A.tiles;
  const dim3 grid((unsigned)((A.tiles + 7) / 8 * 8 * A.gy));
#define DNB_C3(MG)                                                                              \
  do {                                                                                          \
    if (F) hipLaunchKernelGGL((k_conv3<MG, true, true>), grid, dim3(512), lds, st, A);          \
    else if (fold) hipLaunchKernelGGL((k_conv3<MG, true, false>), grid, dim3(512), lds, st, A); \
    else hipLaunchKernelGGL((k_conv3<MG, false, false>), grid, dim3(512), lds, st, A);          \
  } while (0)
  switch (mg) { case 1: DNB_C3(1); break; case 2: DNB_C3(2); break; case 3: DNB_C3(3); break; default: DNB_C3(4); break; }
#undef DNB_C3
  return true;
}

}  // namespace nhwc
}  // namespace dnb
