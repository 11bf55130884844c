// bf16 / NHWC 1x1 convolution with BN statistics of its output, for few pixels (forward pass):
//
//   out[p][m] = sum_c W[m][c] * act(in[p][c]),  act = BN+ReLU prologue or identity.
//
// The 14x14 and 7x7 blocks have fewer 64-pixel tiles x output groups than the chip has CUs: one workgroup
// per CU at most, which has nothing but its own waves to cover its latencies.  In k_conv's form, four waves
// that load, transform and multiply a 64-channel chunk in turn, a chunk took 0.9 us (22 us a launch at 98
// tiles x 1300 channels x 128 outputs), most of it waiting.  Here the waves have two roles: NP producers
// load the features D steps ahead, apply BN+ReLU and put them into LDS; NC consumers, an M-tile of 16
// outputs each, take their weights from L2 D steps ahead and do only LDS reads and MFMAs.  A step is 128
// channels with one barrier, 0.65 us: about 900 cycles of LDS traffic (the consumers' fragments 512, the
// tile 128, the coefficients 256) beside 600 of the producers' vector work.  At 6272 pixels x 128 outputs,
// 1024 channels 18 -> 9.1 us, 2272 channels 31 -> 14.9 us; DenseNet-264-shaped forward 6.61 -> 5.60 ms.
// Tried: two M-tiles x two pixel tiles a consumer (half the LDS reads, twice the weight loads): 16.4 us;
// 256-channel steps: spills; four producers: 16.9 us.
// Each output's K order, its rounding and the statistics' 64-pixel groups are those of k_conv (same bits).
#include "dnb_internal.h"
#include "dnb_nhwc_dev.h"
#include "dnb_stats.h"

namespace dnb {
namespace nhwc {

namespace {

struct Conv1Args {
  const u16* in; int64_t in_ld;
  const u16* W; int nk;              // packed weights, K-steps of 32
  u16* out; int64_t out_ld;
  int cin, cout, M16;
  int64_t P;
  const float2* fold;
  float* spart; int T;               // partials per channel = tiles of 64 pixels
  int gy;                            // groups of NC M-tiles
  FoldIn F; int cap;                 // FOLD: BN1 folded here; fresh channels, rounded up to a power of two
};
constexpr int kFresh = 64;           // most fresh channels folded inside

// D: steps in flight.  Tiles are dealt to the XCDs in turn, the gy workgroups of a tile to one XCD (they
// read the same features).  Both roles run whole groups of D steps, every step with the same loads (at
// clamped addresses) and one barrier, so that a use waits for its own load and not for all of them; past
// the last step only the products are skipped.
// FOLD: BN1 is folded here: the producers form a step's pairs from the channels' statistics; those of the fresh
// channels (the last layer's output) are merged by the consumers before the first step, who have nothing else to
// do then.  The first workgroup keeps what the backward pass needs.
template <int NC, int NP, int D, bool PRO, bool FOLD>
__global__ __launch_bounds__((NC + NP) * 64) void k_conv1(Conv1Args A) {
  constexpr int KC = 128, PITCH = KC + 8, BUFE = 64 * PITCH;
  constexpr int RS = NP * 4, U = 64 / RS;  // 64 pixels x 16 vectors of 8 channels over NP waves
  __shared__ __attribute__((aligned(16))) u16 lds[2 * BUFE];
  // (scale, shift) of a step's channels: pair e of the 8-channel vectors v side by side, [e][v][4] (a lane's
  // four reads at 64-byte strides met on a quarter of the banks: 16.2 -> 14.4 us a launch)
  __shared__ __attribute__((aligned(16))) float cof[2][2 * KC];
  __shared__ float2 fresh[FOLD ? kFresh : 1];
  __shared__ float2 runs[FOLD ? 2 * 256 : 1], table[FOLD ? 127 : 1];
  const int slot = blockIdx.x >> 3, grp = slot % A.gy, tile = (slot / A.gy) * 8 + (blockIdx.x & 7);
  if (tile >= A.T) return;
  const bool keep = FOLD && tile == 0 && grp == 0;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nst = (A.cin + KC - 1) / KC, steps = (nst + D - 1) / D * D;
  const int tile_px = (int)min((int64_t)64, A.P - (int64_t)tile * 64);

  if (wave >= NC) {
    // ---- producer: vector v of rows r, r + RS, ...; a scalar base and 32-bit offsets (64 rows)
    const int pid = (wave - NC) * 64 + lane, v = pid & 15, r = pid >> 4;
    // coefficient of a step (FOLD: channel, both its coefficients) that this thread brings, its place in cof
    const int ci = pid & ((FOLD ? 1 : 2) * KC - 1), c2 = FOLD ? 2 * ci : ci, cw = ((c2 >> 2) & 3) * 64 + (c2 >> 4) * 4 + (c2 & 3);
    const bool cwr = (wave - NC) * 64 < (FOLD ? 1 : 2) * KC;
    const char* tb = reinterpret_cast<const char*>(A.in + (int64_t)tile * 64 * A.in_ld);
    unsigned ro[U];
#pragma unroll
    for (int u = 0; u < U; ++u) ro[u] = (unsigned)min(r + u * RS, tile_px - 1) * (unsigned)(2 * A.in_ld);
    uint4 ring[D][U];
    struct Coef { float a, b, m, i; };  // FOLD: gamma, beta, mean, 1/std
    Coef cr[D];
    auto request = [&](int s, uint4(&q)[U], Coef& c) {
      const unsigned co = min(s * 2 * KC + 16 * v, 2 * A.cin - 16);  // cin % 8 == 0
#pragma unroll
      for (int u = 0; u < U; ++u) q[u] = *reinterpret_cast<const uint4*>(tb + (ro[u] + co));
      if (FOLD) {
        const int ch = min(s * KC + ci, A.cin - 1);
        c = Coef{A.F.gamma[ch], A.F.beta[ch], A.F.mean[ch], A.F.istd[ch]};
      } else if (PRO) {
        c.a = reinterpret_cast<const float*>(A.fold)[min(s * 2 * KC + ci, 2 * A.cin - 1)];
      }
    };
    auto coefs = [&](int s, const Coef& c) {  // of step s, to its buffer
      if (FOLD) {
        const int ch = s * KC + ci;
        float2 o;
        bn_fold(c.a, c.b, c.m, c.i, o.x, o.y);
        if (ch >= A.F.lo && ch < A.cin) o = fresh[ch - A.F.lo];
        *reinterpret_cast<float2*>(&cof[s & 1][cw]) = o;
        if (keep && ch < A.cin) A.F.fold[ch] = o;
      } else {
        cof[s & 1][cw] = c.a;
      }
    };
    auto deposit = [&](int s, const uint4(&q)[U], int buf) {
      u16* o = lds + buf * BUFE + r * PITCH + 8 * v;
      float4 f[4];
      if (PRO) {
#pragma unroll
        for (int e = 0; e < 4; ++e) f[e] = *reinterpret_cast<const float4*>(&cof[buf][64 * e + 4 * v]);
      }
      V8 x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        x[u].q = q[u];
        if (PRO) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            x[u].h[2 * e] = f2bf(fmaxf(__fmaf_rn(bf2f(x[u].h[2 * e]), f[e].x, f[e].y), 0.f));
            x[u].h[2 * e + 1] = f2bf(fmaxf(__fmaf_rn(bf2f(x[u].h[2 * e + 1]), f[e].z, f[e].w), 0.f));
          }
        }
      }
      if ((s + 1) * KC > A.cin || tile_px < 64) {  // uniform: channels past the last, rows past the last
        const bool cok = s * KC + 8 * v < A.cin;
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (!cok || r + u * RS >= tile_px) x[u].q = make_uint4(0u, 0u, 0u, 0u);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) *reinterpret_cast<uint4*>(o + u * RS * PITCH) = x[u].q;
    };
#pragma unroll
    for (int s = 0; s < D; ++s) request(s, ring[s], cr[s]);
    if (FOLD) {  // the fresh channels' pairs
      __syncthreads();
      __syncthreads();
      __syncthreads();
    }
    if (PRO && cwr) { coefs(0, cr[0]); coefs(1, cr[1]); }
    __syncthreads();
    // step s: coefficients of step s + 1 into the buffer that step s - 1 has left, deposit of step s, request
    // of step s + D into the registers that frees.  The consumers read step s - 1.
    for (int sb = 0; sb < steps; sb += D) {
#pragma unroll
      for (int u = 0; u < D; ++u) {
        const int s = sb + u, par = s & 1;
        if (PRO && cwr) coefs(s + 1, cr[(u + 1) % D]);
        deposit(s, ring[u], par);
        request(s + D, ring[u], cr[u]);
        __syncthreads();
      }
    }
    __syncthreads();
    return;
  }

  // ---- consumer: M-tile grp*NC + wave
  const int mt = grp * NC + wave, j = lane & 15, g = lane >> 4;
  const char* wb = reinterpret_cast<const char*>(A.W) + (int64_t)min(mt, A.M16 / 16 - 1) * A.nk * 1024;  // a K-step is 1 KB
  const unsigned lo = lane * 16;
  uint4 ring[D][4];
  auto wload = [&](int s, uint4(&q)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) q[i] = *reinterpret_cast<const uint4*>(wb + (int64_t)min(s * 4 + i, A.nk - 1) * 1024 + lo);
  };
  f32x4 acc[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) acc[t] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < D; ++s) wload(s, ring[s]);
  if (FOLD) {
    const int tid = threadIdx.x, nf = A.F.hi - A.F.lo;  // (the first 256 threads)
    stat_table(StatRuns{A.F.T, A.F.per, A.F.tpr}, table, tid);
    __syncthreads();
    if (tid < 256) {
      const int ch = min(tid & (A.cap - 1), nf - 1), ql = tid / A.cap;
      if (A.cap == 16) stat_merge_runs<16>(A.F.part, A.F.T, nf, ch, ql, table, runs, 256, tid);
      else if (A.cap == 32) stat_merge_runs<8>(A.F.part, A.F.T, nf, ch, ql, table, runs, 256, tid);
      else stat_merge_runs<4>(A.F.part, A.F.T, nf, ch, ql, table, runs, 256, tid);
    }
    __syncthreads();
    if (tid < nf) {
      const float ga = A.F.gamma[A.F.lo + tid], be = A.F.beta[A.F.lo + tid];
      const float2 m = A.cap == 16 ? stat_merge_finish<16>(runs, A.F.T, table, 16, 256, tid)
                      : A.cap == 32 ? stat_merge_finish<8>(runs, A.F.T, table, 32, 256, tid)
                                    : stat_merge_finish<4>(runs, A.F.T, table, 64, 256, tid);
      const float is = bn_istd(m.y, A.F.count, A.F.eps);
      float2 o;
      bn_fold(ga, be, m.x, is, o.x, o.y);
      fresh[tid] = o;
      if (keep) { A.F.mean[A.F.lo + tid] = m.x; A.F.istd[A.F.lo + tid] = is; }
    }
    __syncthreads();
  }
  __syncthreads();
  __syncthreads();  // step 0 is in LDS
  for (int sb = 0; sb < steps; sb += D) {
#pragma unroll
    for (int u = 0; u < D; ++u) {
      const int s = sb + u;
      if (s < nst) {
        // K-steps past the last one meet zeros in LDS
        const u16* b = lds + (s & 1) * BUFE + j * PITCH + 8 * g;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          V8 w, x[4];
          w.q = ring[u][i];
#pragma unroll
          for (int t = 0; t < 4; ++t) x[t].q = *reinterpret_cast<const uint4*>(b + t * 16 * PITCH + i * 32);
#pragma unroll
          for (int t = 0; t < 4; ++t) acc[t] = mfma_bf16(w, x[t], acc[t]);
        }
      }
      wload(s + D, ring[u]);
      __syncthreads();
    }
  }
  // rounded to bf16 first: statistics describe exactly what is stored
  const int m = mt * 16 + 4 * g;
  if (m >= A.cout) return;  // cout % 4 == 0
  u16 h[4][4];
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) h[t][e] = f2bf(acc[t][e]);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float sum = 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t) sum += (t * 16 + j < tile_px) ? bf2f(h[t][e]) : 0.f;
    sum = row16_sum(sum);
    const float mu = sum / (float)tile_px;
    float m2 = 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const float d = bf2f(h[t][e]) - mu;
      m2 += (t * 16 + j < tile_px) ? d * d : 0.f;
    }
    m2 = row16_sum(m2);
    if (j == 0) {
      float* o = A.spart + stat_at(A.T, A.cout, tile, m + e);
      o[0] = (float)tile_px; o[1] = mu; o[2] = m2;
    }
  }
  u16* const ob = A.out + (int64_t)tile * 64 * A.out_ld + m;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int q = t * 16 + j;
    if (q < tile_px) {
      uint2 pk;
      pk.x = (unsigned)h[t][0] | ((unsigned)h[t][1] << 16);
      pk.y = (unsigned)h[t][2] | ((unsigned)h[t][3] << 16);
      *reinterpret_cast<uint2*>(ob + (int64_t)q * A.out_ld) = pk;
    }
  }
}

}  // namespace

// Output M-tiles per workgroup, 0 if the shape is not taken: 4 or 6, whichever first gives at most one
// workgroup per CU, counted on the XCD that gets most (tiles are dealt to the eight in turn, all groups of a tile to
// one; with 83 tiles x 3 groups, 249 workgroups, three XCDs had 33 for 32 CUs: 384 + 48 l channels, 192 outputs, eight
// layers' forward 281 us, with two groups 233).  More tiles: several of k_conv's smaller workgroups share a CU and
// cover one another's latencies (25088 pixels x 320 channels x 128 outputs 11 us there, 14.6 us here; 83 tiles, 288
// outputs, which are three groups at the least, eight layers' forward from 104 channels 350 us there, 375 here).
static int conv1_group(int64_t P, int64_t in_ld, int cout) {
  const int64_t T = (P + 63) / 64;
  const int mtiles = (cout + 15) / 16;
  if (in_ld >= (1 << 24)) return 0;  // 32-bit offsets inside a tile
  for (int nc : {4, 6})
    if ((T + 7) / 8 * ((mtiles + nc - 1) / nc) <= 32) return nc;
  return 0;
}

// The 1x1 with statistics; false (nothing launched) if the shape is not taken.  Wp: packed weights
// [M16][K32]; *sT = partials per channel.
bool conv1_stats(const void* in, int64_t in_ld, const void* Wp, void* out, int64_t out_ld, int64_t P, int cin, int cout,
                 const float2* fold, float* spart, int* sT, const FoldIn* F, hipStream_t st) {
  const int nc = conv1_group(P, in_ld, cout);
  if (!nc) return false;
  if (F && (F->T > kRowStats || F->hi != cin || F->hi - F->lo > kFresh)) return false;
  Conv1Args A{};
  A.in = (const u16*)in; A.in_ld = in_ld;
  A.W = (const u16*)Wp; A.nk = (cin + 31) / 32;
  A.out = (u16*)out; A.out_ld = out_ld;
  A.cin = cin; A.cout = cout; A.M16 = (cout + 15) & ~15;
  A.P = P; A.fold = fold; A.spart = spart;
  A.T = (int)((P + 63) / 64);
  A.gy = (A.M16 / 16 + nc - 1) / nc;
  if (F) {
    A.F = *F;
    A.cap = F->hi - F->lo <= 16 ? 16 : F->hi - F->lo <= 32 ? 32 : 64;
  }
  if (sT) *sT = A.T;
  const dim3 grid((unsigned)((A.T + 7) / 8 * 8 * A.gy));
#define DNB_C1(NC)                                                                                             \
  do {                                                                                                         \
    if (F) hipLaunchKernelGGL((k_conv1<NC, 8, 3, true, true>), grid, dim3((NC + 8) * 64), 0, st, A);           \
    else if (fold) hipLaunchKernelGGL((k_conv1<NC, 8, 3, true, false>), grid, dim3((NC + 8) * 64), 0, st, A);  \
    else hipLaunchKernelGGL((k_conv1<NC, 8, 3, false, false>), grid, dim3((NC + 8) * 64), 0, st, A);           \
  } while (0)
  if (nc == 4) DNB_C1(4); else DNB_C1(6);
#undef DNB_C1
  return true;
}

}  // namespace nhwc
}  // namespace dnb
