// fp32 NCHW 3x3 convolution (forward and data gradient) for what the whole-K LDS tiles of
// dnb_conv_f32_fast.hip do not take: any image width up to 31 (up to 60 where rows are 16-byte
// friendly) and any number of input channels -- a block without a bottleneck convolves its whole
// concatenation, ragged images have rows of 14 or 7 pixels.
//
// A workgroup owns 64 consecutive pixels of one image; its waves split K (chunks of 16 input
// channels, taken in turn) or the output channels.  Every wave stages the chunks it needs into LDS of
// its own (16 channels of its pixels plus a halo of a row and a pixel on both sides), so there is no
// barrier in the loop: the next chunk's loads are in flight during the 36*MT*4 matrix instructions of
// the current one, and waves drift apart.  A tap is the staged tile at
// an offset; taps left and right of the image are masked, above and below are staged zeros.
// Bound by the matrix pipe (9*16*MT*4 instructions of 32 cycles per chunk) once a wave has two chunks;
// the kernel before it (16-pixel tiles, weights re-packed by every workgroup, two barriers a chunk)
// took 83 us per launch on the 160..292-channel layers of a 16x16 block at batch 64, this one 20: the
// 12-layer block without bottleneck 2.13 -> 1.20 ms; the 28x28 DenseNet-BC-40 step at batch 37, with the
// weight gradient of dnb_conv_f32.hip, 2.86 -> 1.96 ms.  (On the shapes the whole-K tiles take it is within
// 1 % of them on a DenseNet-BC-250 step for k = 24 outputs, and slower as their data gradient.)
#include <hip/hip_ext.h>

#include "dnb_f32_dev.h"
#include "dnb_internal.h"
#include "dnb_stats.h"

namespace dnb {

namespace {

// VEC: 16-byte loads (W % 4 == 0 and aligned operands).  WN: column groups of 16 lanes per channel row.
template <int MT, bool VEC, int WN, bool STATS>
__global__ __launch_bounds__(512, 2) void k_conv3x3_v5(const float* __restrict__ in, int64_t in_stride,
                                                       const float* __restrict__ Wp, int Mpad, int Kpad,
                                                       float* __restrict__ out, int64_t out_stride, int cin, int cout, int H,
                                                       int W, int wk, float* __restrict__ spart, int sT) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  constexpr int V = VEC ? 4 : 1, COLS = 16 * WN * V;
  constexpr int CS = COLS <= 144 ? 144 : 208;  // channel pitch: 16 (mod 64) floats, the four rows of an operand read on disjoint banks
  static_assert(COLS <= CS, "channel pitch");
  constexpr int WD = MT == 1 ? 9 : 3;  // weights requested this many taps ahead
  const int HW = H * W, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, j = lane & 15, g = lane >> 4;
  const int ks_ = wave % wk, ms_ = wave / wk, mslots = (int)(blockDim.x >> 6) / wk;
  const int q0 = blockIdx.x * 64, img = blockIdx.z;
  const int mt0 = (blockIdx.y * mslots + ms_) * MT;  // first M-tile of this wave
  const int nchunks = Kpad >> 4, halo = VEC ? W + 4 : W + 1;
  const float* inb = in + (int64_t)img * in_stride;
  float* my = lds + wave * (16 * CS);
  const int nmy = mt0 * 16 < Mpad && ks_ < nchunks ? (nchunks - ks_ + wk - 1) / wk : 0;

  // staging: lane (j, g) takes rows g + 4v, column groups j + 16w
  const int seg = (64 + 2 * halo) / V;
  float st[4][WN][V];
  auto request = [&](int i) {  // i-th chunk of this wave, clamped
    const int c0 = (ks_ + min(i, nmy - 1) * wk) * 16;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int ch = min(c0 + g + 4 * v, cin - 1);
#pragma unroll
      for (int w = 0; w < WN; ++w) {
        const float* p = inb + (int64_t)ch * HW + min(max(q0 - halo + V * (j + 16 * w), 0), HW - V);
        if (VEC) {
          const float4 t = ldg4(p);
          st[v][w][0] = t.x; st[v][w][1 % V] = t.y; st[v][w][2 % V] = t.z; st[v][w][3 % V] = t.w;
        } else {
          st[v][w][0] = *p;
        }
      }
    }
  };
  auto deposit = [&](int i) {
    const int c0 = (ks_ + i * wk) * 16;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const bool cok = c0 + g + 4 * v < cin;
#pragma unroll
      for (int w = 0; w < WN; ++w) {
        const int col = j + 16 * w, q = q0 - halo + V * col;
        float x[V];
#pragma unroll
        for (int e = 0; e < V; ++e) {
          x[e] = st[v][w][e];
          if (!(cok && q >= 0 && q < HW)) x[e] = 0.f;  // (HW % V == 0: a vector is in or out)
        }
        if (col < seg) {
          float* d = my + (g + 4 * v) * CS + V * col;
          if (VEC) *reinterpret_cast<float4*>(d) = make_float4(x[0], x[1 % V], x[2 % V], x[3 % V]);
          else *d = x[0];
        }
      }
    }
  };
  // one wave reads what its other lanes wrote: LDS operations of a wave complete in order; the fence
  // keeps the compiler from moving them across
  auto wave_sync = [] {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };

  float4 w4[WD][MT];
  auto wload = [&](int i, int t9, float4(&w)[MT]) {
    const int ci = ks_ + min(i, nmy - 1) * wk;
#pragma unroll
    for (int a = 0; a < MT; ++a)  // M-tiles past the padded rows repeat the last, never stored
      w[a] = ldg4(wfrag(Wp + (int64_t)t9 * Mpad * Kpad, Kpad, min(mt0 + a, (Mpad >> 4) - 1), ci));
  };

  f32x4 acc[MT][4];
#pragma unroll
  for (int a = 0; a < MT; ++a)
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[a][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
  bool lok[4], rok[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int wc = (q0 + t * 16 + j) % W;
    lok[t] = wc != 0;
    rok[t] = wc != W - 1;
  }

  if (nmy > 0) {
    request(0);
#pragma unroll
    for (int t9 = 0; t9 < WD; ++t9) wload(0, t9, w4[t9]);
    for (int i = 0; i < nmy; ++i) {
      wave_sync();  // the previous chunk's reads are issued
      deposit(i);
      wave_sync();
      request(i + 1);
      if constexpr (!VEC && MT == 1) {
        // the products of the loop below, with operands two steps ahead of them, held there by scheduling barriers (left
        // alone, the compiler reads a step's four and waits for them): with the packing of the weights 14.8 -> 13.5 us for
        // 96 -> 16 channels on 37 images of 7x7, 19.0 -> 18.2 for 160 -> 12 on 64 of 14x14, 15.1 -> 13.7 for 100 -> 12 on 4.
        // Not with 16-byte rows, where the other wave of a SIMD covers that.
        float b[3][4];
        auto operand = [&](int s, float(&o)[4]) {
          const float* base = my + g * CS + j + halo + (s / 12 - 1) * W + s / 4 % 3 - 1 + 4 * (s % 4) * CS;
#pragma unroll
          for (int t = 0; t < 4; ++t) o[t] = base[16 * t];
        };
        operand(0, b[0]);
        operand(1, b[1]);
#pragma unroll
        for (int s = 0; s < 36; ++s) {
          const int t9 = s / 4, ks = s % 4;
          if (s + 2 < 36) operand(s + 2, b[(s + 2) % 3]);
          __builtin_amdgcn_sched_barrier(0);
          float x[4];
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            x[t] = b[s % 3][t];
            if (t9 % 3 == 0 && !lok[t]) x[t] = 0.f;
            if (t9 % 3 == 2 && !rok[t]) x[t] = 0.f;
          }
#pragma unroll
          for (int t = 0; t < 4; ++t) acc[0][t] = mfma16(elem(w4[t9 % WD][0], ks), x[t], acc[0][t]);
          __builtin_amdgcn_sched_barrier(0);
          if (ks == 3) wload(i + (t9 + WD >= 9 ? 1 : 0), (t9 + WD) % 9, w4[t9 % WD]);
        }
        continue;
      }
#pragma unroll
      for (int t9 = 0; t9 < 9; ++t9) {
        const float* base = my + g * CS + j + halo + (t9 / 3 - 1) * W + t9 % 3 - 1;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          float b[4];
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            b[t] = base[4 * ks * CS + 16 * t];
            if (t9 % 3 == 0 && !lok[t]) b[t] = 0.f;
            if (t9 % 3 == 2 && !rok[t]) b[t] = 0.f;
          }
#pragma unroll
          for (int a = 0; a < MT; ++a)
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[a][t] = mfma16(elem(w4[t9 % WD][a], ks), b[t], acc[a][t]);
        }
        wload(i + (t9 + WD >= 9 ? 1 : 0), (t9 + WD) % 9, w4[t9 % WD]);
      }
    }
  }
  if (wk > 1) ksplit_reduce<MT, 4>(acc, lds + (size_t)ms_ * (MT * 4 * (wk - 1) * 256), ks_, lane, wk);

  const int px = min(64, HW - q0);
#pragma unroll
  for (int a = 0; a < MT; ++a) {
    if (a % wk != ks_ || (mt0 + a) * 16 >= Mpad) continue;  // M-tile a lives in wave a % wk of the group
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = (mt0 + a) * 16 + 4 * g + r;
      if (STATS) {
        float s = 0.f, m2 = 0.f;
#pragma unroll
        for (int t = 0; t < 4; ++t) s += t * 16 + j < px ? acc[a][t][r] : 0.f;
        const float mu = row16_sum(s) / (float)px;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const float d = acc[a][t][r] - mu;
          m2 += t * 16 + j < px ? d * d : 0.f;
        }
        m2 = row16_sum(m2);
        if (j == 0 && m < cout) {
          float* p = spart + ((int64_t)m * sT + img * gridDim.x + blockIdx.x) * 3;
          p[0] = (float)px; p[1] = mu; p[2] = m2;
        }
      }
      if (m < cout) {
        float* o = out + (int64_t)img * out_stride + (int64_t)m * HW + q0 + j;
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if (t * 16 + j < px) o[16 * t] = acc[a][t][r];
      }
    }
  }
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace

bool launch_conv3x3_any(const float* in, int64_t in_stride, const float* packed, float* out, int64_t out_stride, int n,
                        int cin, int cout, int h, int w, float* spart, int* sT, hipStream_t st,
                        hipEvent_t ev0, hipEvent_t ev1) {
  const int hw = h * w, mtiles = (cout + 15) / 16, M16 = mtiles * 16, K16 = (cin + 15) & ~15, nchunks = K16 / 16;
  const bool vec = w % 4 == 0 && in_stride % 4 == 0 && aligned16(in);
  int wn;
  if (vec) {
    const int seg4 = (64 + 2 * w + 8) / 4;
    if (seg4 > 48) return false;
    wn = seg4 <= 32 ? 2 : 3;
  } else {
    const int seg = 64 + 2 * (w + 1);
    if (seg > 128) return false;
    wn = seg <= 96 ? 6 : 8;
  }
  const int tiles = (hw + 63) / 64;
  // K split over the waves where there are chunks for it (three or four, whichever they divide by) and few
  // M-tiles; else the M-tiles are split, as many per wave as leave a workgroup per CU.  Eight where no CU gets more
  // than one workgroup: the other wave of a SIMD then multiplies while one waits for its staging (batch 64, 16x16
  // rows, 256 channels to 12: 24.9 -> 22.0 us, to 40: 43.8 -> 39.6).  With more, several workgroups of four waves do
  // that for each other and twice the LDS and waves to add only cost (32x32 rows, 512 workgroups, 128 channels to 12:
  // 1.33 times four waves' time, 256 to 40: 1.10; 16x16 rows, one M-tile: 0.95 to 1.03).
  int nw = 4, wk = 1, mt = 1;
  if (mtiles <= 3 && nchunks >= 2) {
    wk = nw = nchunks <= 4 ? nchunks : (nchunks % 4 != 0 && nchunks % 3 == 0 && nchunks <= 9 ? 3 : nchunks >= 8 && (int64_t)tiles * n <= 256 ? 8 : 4);
    mt = mtiles;
  } else {
    if (mtiles < 4) nw = mtiles;
    for (mt = 3; mt > 1; --mt)
      if ((int64_t)tiles * n * ((mtiles + nw * mt - 1) / (nw * mt)) >= 256 && nw * mt < mtiles + nw) break;
  }
  const int mslots = nw / wk, gy = (mtiles + mslots * mt - 1) / (mslots * mt);
  const size_t cs = (vec && wn == 3) ? 208 : 144, stage = (size_t)nw * 16 * cs,
               red = wk > 1 ? (size_t)mslots * mt * 4 * (wk - 1) * 256 : 0;
  const size_t lds = (stage > red ? stage : red) * sizeof(float);
  const dim3 grid((unsigned)tiles, (unsigned)gy, (unsigned)n);
  const int T = tiles * n;
  if (sT) *sT = T;
#define DNB_L(MT, VEC, WN, STATS)                                                                                     \
  hipExtLaunchKernelGGL((k_conv3x3_v5<MT, VEC, WN, STATS>), grid, dim3(64 * nw), lds, st, ev0, ev1, 0, in, in_stride,  \
                        packed, M16, K16, out, out_stride, cin, cout, h, w, wk, spart, T)
#define DNB_L3(MT, VEC, WN)                                                                  \
  do {                                                                                       \
    if (spart) DNB_L(MT, VEC, WN, true); else DNB_L(MT, VEC, WN, false);                     \
  } while (0)
#define DNB_L2(MT)                                                                     \
  do {                                                                                 \
    if (vec) { if (wn == 2) DNB_L3(MT, true, 2); else DNB_L3(MT, true, 3); }            \
    else { if (wn == 6) DNB_L3(MT, false, 6); else DNB_L3(MT, false, 8); }              \
  } while (0)
  if (mt == 3) DNB_L2(3); else if (mt == 2) DNB_L2(2); else DNB_L2(1);
#undef DNB_L2
#undef DNB_L3
#undef DNB_L
  return true;
}

}  // namespace dnb
