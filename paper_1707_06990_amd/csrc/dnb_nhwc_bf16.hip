// bf16 / NHWC kernels of the dense block (feature maps stored as bf16, channels contiguous;
// fp32 accumulation, fp32 BN statistics, fp32 parameters and parameter gradients, fp32 gradient
// slab).  Every step of the fused schedule, built around v_mfma_f32_16x16x32_bf16 with output
// channels on M and pixels on N, so a lane's operand is 8 consecutive channels of one pixel
// (16 bytes of NHWC) and an accumulator holds 4 consecutive channels of one pixel (one 8-byte
// NHWC store).
//
// Convolutions (forward / data gradient): the workgroup stages a 64-pixel tile (+ one image row
// of halo for 3x3) of a 64-channel chunk in LDS, double-buffered, applying the BN+ReLU prologue
// once per element; its four waves split the output-channel tiles and take packed bf16 weights
// from L2 through register rings.  The backward chain is in dnb_nhwc_bwd.hip, the weight gradients in
// dnb_nhwc_wgrad.hip; here only the one for rows wider than those take (both operands transposed on
// their way into LDS, one staging per tap).
#include "dnb_internal.h"
#include "dnb_nhwc_dev.h"
#include "dnb_stats.h"

namespace dnb {
namespace nhwc {

namespace {

// ----------------------------------------------------------------------------- small kernels

// dst[p][0:c] = src[p][0:c] (bf16, c % 8 == 0), pixel strides in elements
__global__ __launch_bounds__(256) void k_copy_rows(const u16* __restrict__ src, int64_t sld,
                                                   u16* __restrict__ dst, int64_t dld, int64_t P, int cv) {
  const int64_t total = P * cv;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
    const int64_t p = i / cv;
    const int v = (int)(i - p * cv);
    *reinterpret_cast<uint4*>(dst + p * dld + 8 * v) = *reinterpret_cast<const uint4*>(src + p * sld + 8 * v);
  }
}

// out[p][0:c] = bf16(max(0, fma(x[p][ch], scale_ch, shift_ch))) with (scale, shift) = fold[ch]: BN+ReLU
// into shared storage 2 exactly as the fused schedule's convolutions apply it in their operand
// loads; copy (may be null) receives the raw features (the concatenation into shared storage 1).  One launch may hold two
// (the storages that the backward pass re-populates).  Bound by launch, memory round trip and copy rate: a thread requests two vectors
// together, and only its first position costs a division.
struct RowsArgs {
  const u16* x; int64_t ld;
  const float2* fold;
  u16* out; int64_t old;
  u16* copy; int64_t cld;
  int total, cv, wgs;  // 8-channel vectors (P * cv < 2^28), of a pixel; workgroups
};
template <bool TWO>
__global__ __launch_bounds__(256) void k_bn_relu_rows(RowsArgs A, RowsArgs B) {
  const bool second = TWO && (int)blockIdx.x >= A.wgs;
  // (field by field: chosen as a whole, the second's arguments would be read after the first's)
  const RowsArgs R{second ? B.x : A.x, second ? B.ld : A.ld, second ? B.fold : A.fold, second ? B.out : A.out,
                   second ? B.old : A.old, second ? B.copy : A.copy, second ? B.cld : A.cld, second ? B.total : A.total,
                   second ? B.cv : A.cv, second ? B.wgs : A.wgs};
  const int step = R.wgs * 256, dp = step / R.cv, dv = step - dp * R.cv;
  int i = ((int)blockIdx.x - (second ? A.wgs : 0)) * 256 + (int)threadIdx.x;
  int p = i / R.cv, v = i - p * R.cv;
  for (; i < R.total; ) {
    V8 r[2];
    int pp[2], vv[2];
    bool ok[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      ok[u] = i < R.total;
      pp[u] = ok[u] ? p : 0; vv[u] = ok[u] ? v : 0;
      r[u].q = *reinterpret_cast<const uint4*>(R.x + (int64_t)pp[u] * R.ld + 8 * vv[u]);
      i += step; p += dp; v += dv;
      if (v >= R.cv) { v -= R.cv; ++p; }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const float4* f4 = reinterpret_cast<const float4*>(R.fold + 8 * vv[u]);
      V8 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float4 f = f4[e];  // two channels' (scale, shift)
        o.h[2 * e] = f2bf(fmaxf(__fmaf_rn(bf2f(r[u].h[2 * e]), f.x, f.y), 0.f));
        o.h[2 * e + 1] = f2bf(fmaxf(__fmaf_rn(bf2f(r[u].h[2 * e + 1]), f.z, f.w), 0.f));
      }
      if (!ok[u]) continue;
      *reinterpret_cast<uint4*>(R.out + (int64_t)pp[u] * R.old + 8 * vv[u]) = o.q;
      if (R.copy) *reinterpret_cast<uint4*>(R.copy + (int64_t)pp[u] * R.cld + 8 * vv[u]) = r[u].q;
    }
  }
}

// Statistics partials of c channels over pixel range split s: part[(ch*S + s)*3] = (count, mean, M2).
// Thread = (8-channel vector, pixel row): 32 vectors x 8 rows per workgroup, 16-byte loads.  Each
// thread sums deviations from its first value (no cancellation for |mean| >> std), converts to
// (count, mean, M2) and the 8 rows are combined in row order.  grid (vector groups, splits).
__global__ __launch_bounds__(256) void k_stats_partial(const u16* __restrict__ x, int64_t ld, int64_t P,
                                                       int c, int ppb, float* __restrict__ part) {
  __shared__ float red[3][8][256];
  const int cvl = threadIdx.x & 31, pr = threadIdx.x >> 5;
  const int ch0 = (blockIdx.x * 32 + cvl) * 8, s = blockIdx.y, S = gridDim.y;
  const int64_t p0 = (int64_t)s * ppb, p1 = min(P, p0 + ppb);
  const bool ok = ch0 < c;
  float K[8], sd[8], sq[8];
  float cnt = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) K[e] = sd[e] = sq[e] = 0.f;
  if (ok) {
    int64_t p = p0 + pr;
    if (p < p1) {
      V8 v;
      v.q = *reinterpret_cast<const uint4*>(x + p * ld + ch0);
#pragma unroll
      for (int e = 0; e < 8; ++e) K[e] = bf2f(v.h[e]);
      cnt = 1.f;
      p += 8;
    }
    // eight rows requested before the first is added (in row order; a load per row waited out its latency:
    // 74 us for the 401408 x 64 features of a stem)
    for (; p + 8 * 15 < p1; p += 128) {  // sixteen while there are as many: 401408 x 64 features 46 -> 20 us
      V8 v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u].q = *reinterpret_cast<const uint4*>(x + (p + 8 * u) * ld + ch0);
#pragma unroll
      for (int u = 0; u < 16; ++u) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float d = bf2f(v[u].h[e]) - K[e];
          sd[e] += d;
          sq[e] = __fmaf_rn(d, d, sq[e]);
        }
        cnt += 1.f;
      }
    }
    for (; p < p1; p += 64) {
      V8 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u].q = *reinterpret_cast<const uint4*>(x + min(p + 8 * u, p1 - 1) * ld + ch0);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (p + 8 * u < p1) {
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float d = bf2f(v[u].h[e]) - K[e];
            sd[e] += d;
            sq[e] = __fmaf_rn(d, d, sq[e]);
          }
          cnt += 1.f;
        }
      }
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float md = cnt > 0.f ? sd[e] / cnt : 0.f;
    red[0][e][threadIdx.x] = cnt;
    red[1][e][threadIdx.x] = K[e] + md;
    red[2][e][threadIdx.x] = fmaxf(0.f, __fmaf_rn(-sd[e], md, sq[e]));
  }
  __syncthreads();
  // a thread a channel (32 threads with eight each took 7 us to form the quotients)
  const int e = threadIdx.x & 7, cv = threadIdx.x >> 3, ch = blockIdx.x * 256 + (int)threadIdx.x;
  if (ch < c) {
    Stat3 a{red[0][e][cv], red[1][e][cv], red[2][e][cv]};
    for (int r = 1; r < 8; ++r)
      a = stat_combine(a, Stat3{red[0][e][r * 32 + cv], red[1][e][r * 32 + cv], red[2][e][r * 32 + cv]});
    float* o = part + ((int64_t)ch * S + s) * 3;
    o[0] = a.c; o[1] = a.m; o[2] = a.m2;
  }
}

// Packed bf16 weights: per tap [M16][K32] (zero filled) in fragment order, see wfrag.
__global__ __launch_bounds__(256) void k_pack_block_weights(const float* __restrict__ params,
                                                            u16* __restrict__ packed, int c0, int k, int B) {
  const int l = blockIdx.y + 1;
  const int B16 = (B + 15) & ~15, k16 = (k + 15) & ~15, B32 = (B + 31) & ~31, k32 = (k + 31) & ~31;
  // the sizes of the layers before this one, a lane each (one after the other they were 3 us of every workgroup at the
  // 64th layer)
  int64_t poff = 0, koff = 0;
  for (int i = 1 + (int)(threadIdx.x & 63); i < l; i += 64) {
    const int c = c0 + (i - 1) * k, c16 = (c + 15) & ~15, c32 = (c + 31) & ~31;
    poff += 2 * (int64_t)c + (int64_t)B * c + 2 * B + 9 * (int64_t)k * B;
    koff += (int64_t)B16 * c32 + (int64_t)c16 * B32 + 9 * (int64_t)k16 * B32 + 9 * (int64_t)B16 * k32;
  }
  poff = wave_sum_i64(poff);
  koff = wave_sum_i64(koff);
  const int C = c0 + (l - 1) * k, C16 = (C + 15) & ~15, C32 = (C + 31) & ~31;
  const float* W1 = params + poff + 2 * C;
  const float* W3 = W1 + (int64_t)B * C + 2 * B;
  u16* A = packed + koff;
  const int64_t n1 = (int64_t)B16 * C32, n2 = (int64_t)C16 * B32, n3 = 9 * (int64_t)k16 * B32,
                n4 = 9 * (int64_t)B16 * k32, total = n1 + n2 + n3 + n4;
  // A thread makes a lane's fragment, eight K indexes of one row: eight loads in flight and one 16-byte store
  // (an element at a time took 180 us for the 64 layers of 14x14 features of the DenseNet-264-shaped network).
  for (int64_t i8 = (int64_t)blockIdx.x * 256 + threadIdx.x; i8 * 8 < total; i8 += (int64_t)gridDim.x * 256) {
    const int64_t idx = i8 * 8;
    const float* src;  // of K index 0 of the row
    int64_t step;
    int k0, kn;        // first K index of the fragment, K indexes of the row (0: a padding row)
    if (idx < n1) {                       // 1x1 forward  [B16][C32]
      int m;
      wunfrag((int)idx, C32, m, k0);
      src = W1 + (int64_t)min(m, B - 1) * C; step = 1; kn = m < B ? C : 0;
    } else if (idx < n1 + n2) {           // 1x1 dgrad    [C16][B32]
      int cc;
      wunfrag((int)(idx - n1), B32, cc, k0);
      src = W1 + min(cc, C - 1); step = C; kn = cc < C ? B : 0;
    } else if (idx < n1 + n2 + n3) {      // 3x3 forward  [9][k16][B32]
      const int e = (int)(idx - n1 - n2), t = e / (k16 * B32);
      int mm;
      wunfrag(e - t * (k16 * B32), B32, mm, k0);
      src = W3 + (int64_t)min(mm, k - 1) * B * 9 + t; step = 9; kn = mm < k ? B : 0;
    } else {                              // 3x3 dgrad    [9][B16][k32], transposed and flipped
      const int e = (int)(idx - n1 - n2 - n3), t = e / (B16 * k32);
      int cc;
      wunfrag(e - t * (B16 * k32), k32, cc, k0);
      src = W3 + (int64_t)min(cc, B - 1) * 9 + (8 - t); step = (int64_t)B * 9; kn = cc < B ? k : 0;
    }
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = src[min(k0 + e, max(kn - 1, 0)) * step];
    V8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o.h[e] = f2bf(k0 + e < kn ? v[e] : 0.f);
    *reinterpret_cast<uint4*>(A + idx) = o.q;
  }
}

// One convolution's weights: [taps][M16][K32] from element (m, c, t) at w[m*sm + c*sc + (flip ? taps-1-t : t)].
__global__ __launch_bounds__(256) void k_pack_weights(const float* __restrict__ w, int64_t sm, int64_t sc, int flip,
                                                      int cout, int cin, int taps, u16* __restrict__ outp) {
  const int M16 = (cout + 15) & ~15, K32 = (cin + 31) & ~31;
  const int64_t total = (int64_t)taps * M16 * K32;
  for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (int64_t)gridDim.x * 256) {
    const int t = (int)(idx / (M16 * K32));
    int m, c;
    wunfrag((int)(idx - (int64_t)t * (M16 * K32)), K32, m, c);
    const float v = (m < cout && c < cin) ? w[(int64_t)m * sm + (int64_t)c * sc + (flip ? taps - 1 - t : t)] : 0.f;
    outp[idx] = f2bf(v);
  }
}

// ----------------------------------------------------------------------------- conv fwd / dgrad

// out[q][m] = sum_{t,c} W(t,m,c) * act(in[q+shift(t)][c]),  act = BN+ReLU prologue or identity.
// 256 threads; a workgroup owns 64 pixels -- for the 1x1 a flat range of all n*h*w pixels (grid.x
// tiles, grid.z = 1), for the 3x3 a range of one image (grid.z = images) plus one image row and
// one pixel of halo on both sides -- and the four waves split the output channels (MT M-tiles
// each).  Input channels are walked in chunks of 64 through two LDS buffers: the next chunk is
// requested from HBM before the current chunk's MFMAs are issued and written to the other
// buffer (BN+ReLU applied, rounded to bf16) after them: one barrier per chunk, load latency
// under the matrix work.  TIN = u16 (bf16) or float (the gradient slab).  STATS: per-tile
// (count, mean, M2) of the rounded outputs, at stat_at.
template <int TAPS, int MT, typename TIN, bool PRO, bool STATS, bool RING>
__global__ __launch_bounds__(256) void k_conv(
    const TIN* __restrict__ in, int64_t in_ld, const u16* __restrict__ Wp, int M16, int K32,
    u16* __restrict__ out, int64_t out_ld, int cin, int cout, int H, int W, int64_t Ptot,
    const float2* __restrict__ fold, float* __restrict__ spart, int sT) {
  extern __shared__ u16 lds[];
  constexpr int KC = 64, PITCH = KC + 8;  // elements per staged pixel (144 bytes: spreads banks)
  constexpr int U = TAPS == 9 ? 8 : 2;    // 16-byte vectors per thread and chunk (3x3: W <= 95)
  const int HW = H * W;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int j = lane & 15, g = lane >> 4;
  const int img = TAPS == 9 ? blockIdx.z : 0;
  const int64_t q0 = (int64_t)blockIdx.x * 64;
  const int64_t limit = TAPS == 9 ? (int64_t)HW : Ptot;  // pixels of the range q0 indexes
  const int halo = (TAPS == 9) ? W + 1 : 0;
  const int seg = 64 + 2 * halo, nvec = seg * 8, BUFE = seg * PITCH;
  const TIN* inb = in + (int64_t)img * HW * in_ld;
  const int mbase = (blockIdx.y * 4 + wave) * (MT * 16);
  const bool m_ok = mbase < M16;

  f32x4 acc[MT][4];
#pragma unroll
  for (int a = 0; a < MT; ++a)
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[a][t] = (f32x4){0.f, 0.f, 0.f, 0.f};

  bool lok[4], rok[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int wc = (int)((q0 + t * 16 + j) % W);
    lok[t] = wc != 0;
    rok[t] = wc != W - 1;
  }

  // PRO: the folded BN (scale, shift) of all input channels is copied to LDS once, behind the two
  // tile buffers (the staging reads it for every vector it transforms)
  // Inside a chunk pair e of the eight 8-channel vectors lies side by side, [e][v][4]: a thread keeps one vector
  // per chunk, and its reads at 64-byte strides met on a quarter of the banks.
  float* flds = reinterpret_cast<float*>(lds + 2 * BUFE);  // 2*BUFE*2 bytes is a multiple of 16
  auto fpos = [](int c) { return ((c >> 1) & 3) * 32 + (c >> 3) * 4 + (c & 1) * 2; };
  if (PRO) {
    for (int i = tid; i < cin; i += 256) {
      const float2 fl = fold[i];
      float* o = flds + (i & ~(KC - 1)) * 2 + fpos(i & (KC - 1));
      o[0] = fl.x; o[1] = fl.y;
    }
    __syncthreads();
  }

  struct Raw { uint4 a, b; };  // bf16: a only; float: 8 floats
  // Every load of the main loop is unconditional, at an address clamped into the tensor: the
  // number of loads in flight at each point is then the same on every path, and a use waits only
  // for its own load instead of for all of them.
  auto request = [&](int c0, Raw(&v)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int idx = min(u * 256 + tid, nvec - 1);
      const int s = idx >> 3, ch = min(c0 + 8 * (idx & 7), cin - 8);  // cin % 8 == 0
      const int64_t q = min(max(q0 - halo + s, (int64_t)0), limit - 1);
      if (sizeof(TIN) == 2) {
        v[u].a = *reinterpret_cast<const uint4*>(reinterpret_cast<const u16*>(inb) + q * in_ld + ch);
      } else {
        const float* pf = reinterpret_cast<const float*>(inb) + q * in_ld + ch;
        v[u].a = *reinterpret_cast<const uint4*>(pf);
        v[u].b = *reinterpret_cast<const uint4*>(pf + 4);
      }
    }
  };
  auto deposit = [&](int c0, const Raw(&v)[U], int boff) {
    float4 fl[4];
    if (PRO) {
      const int vv = tid & 7;
#pragma unroll
      for (int e = 0; e < 4; ++e) fl[e] = *reinterpret_cast<const float4*>(&flds[2 * c0 + e * 32 + vv * 4]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int idx = u * 256 + tid;
      if (idx < nvec) {
        const int s = idx >> 3, vv = idx & 7, ch = c0 + 8 * vv;
        const int64_t q = q0 - halo + s;
        V8 o;
        o.q = make_uint4(0u, 0u, 0u, 0u);
        if (q >= 0 && q < limit && ch < cin) {  // a vector is entirely in or out
          float f[8];
          if (sizeof(TIN) == 2) {
            V8 r;
            r.q = v[u].a;
#pragma unroll
            for (int e = 0; e < 8; ++e) f[e] = bf2f(r.h[e]);
          } else {
            f[0] = __uint_as_float(v[u].a.x); f[1] = __uint_as_float(v[u].a.y);
            f[2] = __uint_as_float(v[u].a.z); f[3] = __uint_as_float(v[u].a.w);
            f[4] = __uint_as_float(v[u].b.x); f[5] = __uint_as_float(v[u].b.y);
            f[6] = __uint_as_float(v[u].b.z); f[7] = __uint_as_float(v[u].b.w);
          }
          if (PRO) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              f[2 * e] = fmaxf(__fmaf_rn(f[2 * e], fl[e].x, fl[e].y), 0.f);
              f[2 * e + 1] = fmaxf(__fmaf_rn(f[2 * e + 1], fl[e].z, fl[e].w), 0.f);
            }
          }
#pragma unroll
          for (int e = 0; e < 8; ++e) o.h[e] = f2bf(f[e]);
        }
        *reinterpret_cast<uint4*>(&lds[boff + s * PITCH + 8 * vv]) = o.q;
      }
    }
  };

  // packed weights of one (chunk, tap): MT M-tiles x 2 K-steps, 16 bytes per lane each.  They
  // come from L2 at best and, early in a launch, from HBM, so they are requested before their use, into
  // a ring of register sets indexed statically: the 1x1 one chunk ahead or (RING) four, the 3x3 nine taps
  // (MT == 1) or three.  Rows past M16 and K-steps past K32 are clamped: their products are never formed or
  // never stored.
  struct WSet { uint4 w[MT][2]; };
  auto wload = [&](int c0, int t9, WSet& ws) {
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
        ws.w[a][kk] = *reinterpret_cast<const uint4*>(
            wfrag(Wp + (int64_t)t9 * M16 * K32, K32, min(mbase + a * 16, M16 - 16) >> 4, min(c0 + kk * 32, K32 - 32) >> 5));
  };
  // the MFMAs of one (chunk, tap) on the tile staged at boff
  auto mm = [&](int c0, int t9, int boff, const WSet& ws) {
    const int di = (TAPS == 9) ? t9 / 3 - 1 : 0, dj = (TAPS == 9) ? t9 % 3 - 1 : 0;
    const int ksteps = min(2, (K32 - c0) >> 5);
    if (m_ok) {
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        if (kk < ksteps) {
          V8 bfrag[4];
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            bfrag[t].q = *reinterpret_cast<const uint4*>(
                &lds[boff + (t * 16 + j + halo + di * W + dj) * PITCH + kk * 32 + 8 * g]);
            if ((dj < 0 && !lok[t]) || (dj > 0 && !rok[t])) bfrag[t].q = make_uint4(0u, 0u, 0u, 0u);
          }
#pragma unroll
          for (int a = 0; a < MT; ++a) {
            V8 w;
            w.q = ws.w[a][kk];
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[a][t] = mfma_bf16(w, bfrag[t], acc[a][t]);
          }
        }
      }
    }
  };

  const int clast = ((cin - 1) / KC) * KC;  // start of the last chunk
  if (RING) {  // 1x1 with many chunks
    // chunk x lives in ring slot x % 4 (activations and weights alike): step s multiplies chunk
    // c, requests chunk c+4 into the slots it has just freed and deposits chunk c+1
    Raw r[4][U];
    WSet wt[4];
    request(0, r[0]);
    wload(0, 0, wt[0]);
#pragma unroll
    for (int x = 1; x < 4; ++x) {
      wload(min(x * KC, clast), 0, wt[x]);
      request(min(x * KC, clast), r[x]);
    }
    deposit(0, r[0], 0);
    __syncthreads();
    // The loop always runs whole groups of four steps: steps past the last chunk load (clamped),
    // deposit and synchronise like the others and only skip the MFMAs, so the sequence of loads
    // and of waits for them is the same on every path.
    for (int cb = 0; cb < cin; cb += 4 * KC) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int c0 = cb + s * KC, cn = min(c0 + 4 * KC, clast);
        if (c0 < cin) mm(c0, 0, (s & 1) * BUFE, wt[s]);
        wload(cn, 0, wt[s]);
        request(cn, r[s]);
        deposit(min(c0 + KC, clast), r[(s + 1) & 3], ((s & 1) ^ 1) * BUFE);
        __syncthreads();
      }
    }
  } else {
    constexpr int WD = TAPS == 1 ? 1 : (MT == 1 ? 9 : 3);
    Raw va[U];
    {
      Raw v[U];
      request(0, v);
      request(min(KC, clast), va);
      deposit(0, v, 0);
    }
    WSet wt[WD];
#pragma unroll
    for (int s = 0; s < WD; ++s) wload(0, s, wt[s]);
    __syncthreads();
    int it = 0;
    for (int c0 = 0; c0 < cin; c0 += KC, ++it) {
      const int boff = (it & 1) * BUFE;
      const int cn = min(c0 + KC, clast);
#pragma unroll
      for (int t9 = 0; t9 < TAPS; ++t9) {
        mm(c0, t9, boff, wt[t9 % WD]);
        if (t9 + WD < TAPS) wload(c0, t9 + WD, wt[t9 % WD]);
        else wload(cn, t9 + WD - TAPS, wt[t9 % WD]);
      }
      if (c0 + KC < cin) deposit(c0 + KC, va, ((it & 1) ^ 1) * BUFE);
      request(min(c0 + 2 * KC, clast), va);  // in flight across the barrier and the next chunk's MFMAs
      __syncthreads();
    }
  }

  if (!m_ok) return;
  const int tile_px = (int)min((int64_t)64, limit - q0);
  const int tile_id = TAPS == 9 ? img * gridDim.x + blockIdx.x : blockIdx.x;
#pragma unroll
  for (int a = 0; a < MT; ++a) {
    if (mbase + a * 16 >= M16) continue;
    // round to bf16 first: statistics describe exactly what is stored
    float rv[4][4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) rv[t][r] = bf2f(f2bf(acc[a][t][r]));
    if (STATS) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float s = 0.f;
#pragma unroll
        for (int t = 0; t < 4; ++t) s += (q0 + t * 16 + j < limit) ? rv[t][r] : 0.f;
        s = row16_sum(s);
        const float mu = s / (float)tile_px;
        float m2 = 0.f;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const float d = rv[t][r] - mu;
          m2 += (q0 + t * 16 + j < limit) ? d * d : 0.f;
        }
        m2 = row16_sum(m2);
        const int m = mbase + a * 16 + 4 * g + r;
        if (j == 0 && m < cout) {
          float* p = spart + stat_at(sT, cout, tile_id, m);
          p[0] = (float)tile_px; p[1] = mu; p[2] = m2;
        }
      }
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int64_t q = q0 + t * 16 + j;
      const int m = mbase + a * 16 + 4 * g;
      if (q < limit && m < cout) {  // cout % 4 == 0 on this path
        u16* o = out + ((int64_t)img * HW + q) * out_ld + m;
        uint2 pk;
        pk.x = (unsigned)f2bf(acc[a][t][0]) | ((unsigned)f2bf(acc[a][t][1]) << 16);
        pk.y = (unsigned)f2bf(acc[a][t][2]) | ((unsigned)f2bf(acc[a][t][3]) << 16);
        *reinterpret_cast<uint2*>(o) = pk;
      }
    }
  }
}

// ----------------------------------------------------------------------------- weight gradient

// dW[m][c][t] = sum_{img,q} g[q][m] * act(a[q+shift(t)][c]).  grid (pixel splits, c groups of 64,
// m groups of 64).  Per 64-pixel tile and tap the workgroup stages gT[m][pixel] and aT[c][pixel]
// (transposed, prologue and edge masks applied) in LDS; wave w owns m-tile w of the group and
// all four c-tiles.  part[split][m][c][t] fp32.
template <int TAPS, typename TG, bool PRO>
__global__ __launch_bounds__(256) void k_wgrad(
    const u16* __restrict__ a, int64_t a_ld, const TG* __restrict__ gout, int64_t g_ld,
    float* __restrict__ part, int cin, int cout, int n, int H, int W, int tiles_per_img,
    int tiles_per_split, const float2* __restrict__ fold) {
  __shared__ u16 gT[64 * 72];  // [m][pixel], pitch 72 elements (144 bytes)
  __shared__ u16 aT[64 * 72];  // [c][pixel]
  constexpr int PT = 72;
  const int HW = H * W;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int j = lane & 15, g = lane >> 4;
  const int c0 = blockIdx.y * 64, m0 = blockIdx.z * 64;
  const int total_tiles = n * tiles_per_img;
  const int t_begin = blockIdx.x * tiles_per_split, t_end = min(total_tiles, t_begin + tiles_per_split);

  f32x4 acc[TAPS][4];
#pragma unroll
  for (int t = 0; t < TAPS; ++t)
#pragma unroll
    for (int y = 0; y < 4; ++y) acc[t][y] = (f32x4){0.f, 0.f, 0.f, 0.f};

  for (int tile = t_begin; tile < t_end; ++tile) {
    const int img = tile / tiles_per_img, q0 = (tile - img * tiles_per_img) * 64;
    const u16* ab = a + (int64_t)img * HW * a_ld;
    const TG* gb = gout + (int64_t)img * HW * g_ld;
    __syncthreads();
    // gT: thread = (pixel s, 8-channel vector v of the 64 m's)
    for (int idx = tid; idx < 64 * 8; idx += 256) {
      const int s = idx >> 3, v = idx & 7;
      const int q = q0 + s, m = m0 + 8 * v;
      u16 h[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) h[e] = 0;
      if (q < HW && m < cout) {  // cout % 8 == 0
        if (sizeof(TG) == 2) {
          V8 r;
          r.q = *reinterpret_cast<const uint4*>(reinterpret_cast<const u16*>(gb) + (int64_t)q * g_ld + m);
#pragma unroll
          for (int e = 0; e < 8; ++e) h[e] = r.h[e];
        } else {
          const float* pf = reinterpret_cast<const float*>(gb) + (int64_t)q * g_ld + m;
          const float4 x = *reinterpret_cast<const float4*>(pf), y = *reinterpret_cast<const float4*>(pf + 4);
          h[0] = f2bf(x.x); h[1] = f2bf(x.y); h[2] = f2bf(x.z); h[3] = f2bf(x.w);
          h[4] = f2bf(y.x); h[5] = f2bf(y.y); h[6] = f2bf(y.z); h[7] = f2bf(y.w);
        }
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) gT[(8 * v + e) * PT + s] = h[e];
    }
#pragma unroll
    for (int t9 = 0; t9 < TAPS; ++t9) {  // unrolled: acc[t9] must stay in registers
      const int di = (TAPS == 9) ? t9 / 3 - 1 : 0, dj = (TAPS == 9) ? t9 % 3 - 1 : 0;
      if (t9 > 0) __syncthreads();
      for (int idx = tid; idx < 64 * 8; idx += 256) {
        const int s = idx >> 3, v = idx & 7;
        const int q = q0 + s, ch = c0 + 8 * v;
        const int wc = q % W, qq = q + di * W + dj;
        u16 h[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) h[e] = 0;
        const bool ok = q < HW && ch < cin && qq >= 0 && qq < HW && !(dj < 0 && wc == 0) && !(dj > 0 && wc == W - 1);
        if (ok) {
          V8 r;
          r.q = *reinterpret_cast<const uint4*>(ab + (int64_t)qq * a_ld + ch);
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            if (PRO) {
              const float2 fl = fold[ch + e];
              h[e] = f2bf(fmaxf(__fmaf_rn(bf2f(r.h[e]), fl.x, fl.y), 0.f));
            } else {
              h[e] = r.h[e];
            }
          }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) aT[(8 * v + e) * PT + s] = h[e];
      }
      __syncthreads();
      // 64 pixels = 2 K-steps of 32
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        V8 af;
        af.q = *reinterpret_cast<const uint4*>(&gT[(wave * 16 + j) * PT + ks * 32 + 8 * g]);
#pragma unroll
        for (int y = 0; y < 4; ++y) {
          V8 bf;
          bf.q = *reinterpret_cast<const uint4*>(&aT[(y * 16 + j) * PT + ks * 32 + 8 * g]);
          acc[t9][y] = mfma_bf16(af, bf, acc[t9][y]);
        }
      }
    }
  }

  float* pb = part + (int64_t)blockIdx.x * cout * cin * TAPS;
#pragma unroll
  for (int t9 = 0; t9 < TAPS; ++t9)
#pragma unroll
    for (int y = 0; y < 4; ++y) {
      const int c = c0 + y * 16 + j;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + wave * 16 + 4 * g + r;
        if (m < cout && c < cin) pb[((int64_t)m * cin + c) * TAPS + t9] = acc[t9][y][r];
      }
    }
}

// ----------------------------------------------------------------------------- BN + ReLU backward

// Thread = (pixel row pr, 8-channel vector cv); workgroup = 256 threads covering `rows` pixels per
// step x CV vectors (CV*rows = 256).  grid (channel-vector groups, pixel splits).
// part[(ch*S + s)*2] = (sum dz, sum dz*xhat) over the split's pixels.
__global__ __launch_bounds__(256) void k_bn_bwd_partial(
    const u16* __restrict__ x, int64_t x_ld, const u16* __restrict__ dact, int64_t d_ld, int64_t P,
    int c, int ppb, int lsh, const float* __restrict__ gamma, const float* __restrict__ beta,
    const float* __restrict__ mean, const float* __restrict__ istd, float* __restrict__ part) {
  __shared__ float red[2][8][256];
  // L = 1 << lsh channel vectors x 256/L pixel rows; four pixels per thread in flight
  const int L = 1 << lsh, rows = 256 >> lsh;
  const int cvl = threadIdx.x & (L - 1), pr = threadIdx.x >> lsh;
  const int ch0 = (blockIdx.x * L + cvl) * 8, s = blockIdx.y, S = gridDim.y;
  const int64_t p0 = (int64_t)s * ppb, p1 = min(P, p0 + ppb);
  float sb[8], sg[8], sc[8], sf[8], mu[8], is[8];
  const bool ok = ch0 < c;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    sb[e] = sg[e] = 0.f;
    if (ok) {
      mu[e] = mean[ch0 + e]; is[e] = istd[ch0 + e];
      bn_fold(gamma[ch0 + e], beta[ch0 + e], mu[e], is[e], sc[e], sf[e]);
    }
  }
  if (ok) {
    const u16* xp = x + ch0;
    const u16* dp = dact + ch0;
    for (int64_t pb = p0 + pr; pb < p1; pb += 4 * rows) {
      V8 xv[4], dv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {  // rows past the split are clamped here and skipped below
        const int64_t p = min(pb + u * rows, p1 - 1);
        xv[u].q = *reinterpret_cast<const uint4*>(xp + p * x_ld);
        dv[u].q = *reinterpret_cast<const uint4*>(dp + p * d_ld);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (pb + u * rows < p1) {
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float xf = bf2f(xv[u].h[e]);
            const float dz = __fmaf_rn(xf, sc[e], sf[e]) > 0.f ? bf2f(dv[u].h[e]) : 0.f;
            sb[e] += dz;
            sg[e] = __fmaf_rn(dz, (xf - mu[e]) * is[e], sg[e]);
          }
        }
      }
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) { red[0][e][threadIdx.x] = sb[e]; red[1][e][threadIdx.x] = sg[e]; }
  __syncthreads();
  // one thread per (sum, channel of the vector, vector): adds its 256/L pixel rows in order
  for (int q = threadIdx.x; q < 16 * L; q += 256) {
    const int cv = q & (L - 1), e = (q >> lsh) & 7, which = q >> (lsh + 3);
    const int ch = (blockIdx.x * L + cv) * 8 + e;
    if (ch < c) {
      float acc = 0.f;
      for (int r = 0; r < rows; ++r) acc += red[which][e][r * L + cv];
      part[((int64_t)ch * S + s) * 2 + which] = acc;
    }
  }
}

// dgamma/dbeta = sum of the S partials, one wave per channel: lane i adds partials i, i+64, ...
// in order, then a butterfly over the lanes (fixed order, every lane the same bits).
// (Measured alternative: with at most 32 partials per channel, every workgroup of the
// element-wise pass added them itself and this launch was left out for slabs of up to 8192
// pixels.  The reduction pass with fewer splits and the element-wise pass with that prologue
// each took 3-5 us longer, more than the 3 us launch they replaced: config 4 went from 15.0
// to 15.2 ms.)
__global__ __launch_bounds__(256) void k_bn_bwd_finalize(const float* __restrict__ part, int c, int S,
                                                         float* __restrict__ dgamma, float* __restrict__ dbeta) {
  const int ch = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (ch >= c) return;
  const float2* pp = reinterpret_cast<const float2*>(part) + (int64_t)ch * S;
  float b = 0.f, g = 0.f;
  for (int s = lane; s < S; s += 64) { const float2 v = pp[s]; b += v.x; g += v.y; }
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) { b += __shfl_xor(b, off, 64); g += __shfl_xor(g, off, 64); }
  if (lane == 0) { dbeta[ch] = b; dgamma[ch] = g; }
}

// du = scale*(dz - dbeta/P - xhat*dgamma/P).  ACC: added into the fp32 slab G (BN1, concat
// backward); else written as bf16 over dact (BN2: gradient of b_l).
template <bool ACC>
__global__ __launch_bounds__(256) void k_bn_bwd_apply(
    const u16* __restrict__ x, int64_t x_ld, const u16* dact, int64_t d_ld, u16* du_bf, int64_t du_ld,
    float* __restrict__ G, int64_t g_ld, int64_t P, int c, int ppb, int lsh, float inv_p,
    const float* __restrict__ gamma, const float* __restrict__ beta, const float* __restrict__ mean,
    const float* __restrict__ istd, const float* __restrict__ dgamma, const float* __restrict__ dbeta) {
  // same thread map as k_bn_bwd_partial: a thread keeps its eight channels' coefficients in
  // registers and walks pixels, four in flight
  const int L = 1 << lsh, rows = 256 >> lsh;
  const int cvl = threadIdx.x & (L - 1), pr = threadIdx.x >> lsh;
  const int ch0 = (blockIdx.x * L + cvl) * 8;
  if (ch0 >= c) return;
  const int64_t p0 = (int64_t)blockIdx.y * ppb, p1 = min(P, p0 + ppb);
  float sc[8], sf[8], mu[8], is[8], db[8], dg[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    mu[e] = mean[ch0 + e]; is[e] = istd[ch0 + e];
    bn_fold(gamma[ch0 + e], beta[ch0 + e], mu[e], is[e], sc[e], sf[e]);
    db[e] = dbeta[ch0 + e] * inv_p;
    dg[e] = dgamma[ch0 + e] * inv_p;
  }
  const u16* xp = x + ch0;
  const u16* dp = dact + ch0;
  for (int64_t pb = p0 + pr; pb < p1; pb += 4 * rows) {
    V8 xv[4], dv[4];
    float4 ga[4], gb[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {  // rows past the split are clamped here and skipped below
      const int64_t p = min(pb + u * rows, p1 - 1);
      xv[u].q = *reinterpret_cast<const uint4*>(xp + p * x_ld);
      dv[u].q = *reinterpret_cast<const uint4*>(dp + p * d_ld);
      if (ACC) {
        const float* gp = G + p * g_ld + ch0;
        ga[u] = *reinterpret_cast<const float4*>(gp);
        gb[u] = *reinterpret_cast<const float4*>(gp + 4);
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t p = pb + u * rows;
      if (p < p1) {
        float r[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float xf = bf2f(xv[u].h[e]);
          const float dz = __fmaf_rn(xf, sc[e], sf[e]) > 0.f ? bf2f(dv[u].h[e]) : 0.f;
          r[e] = sc[e] * (dz - db[e] - (xf - mu[e]) * is[e] * dg[e]);
        }
        if (ACC) {
          float* gp = G + p * g_ld + ch0;
          float4 a = ga[u], b = gb[u];
          a.x += r[0]; a.y += r[1]; a.z += r[2]; a.w += r[3]; b.x += r[4]; b.y += r[5]; b.z += r[6]; b.w += r[7];
          *reinterpret_cast<float4*>(gp) = a;
          *reinterpret_cast<float4*>(gp + 4) = b;
        } else {
          V8 ov;
#pragma unroll
          for (int e = 0; e < 8; ++e) ov.h[e] = f2bf(r[e]);
          *reinterpret_cast<uint4*>(du_bf + p * du_ld + ch0) = ov.q;
        }
      }
    }
  }
}

inline unsigned grid1d(int64_t items, int per, unsigned cap) {
  int64_t g = (items + per - 1) / per;
  if (g < 1) g = 1;
  if (g > (int64_t)cap) g = cap;
  return (unsigned)g;
}

}  // namespace

// ============================================================================ launchers

hipError_t copy_rows(const void* src, int64_t sld, void* dst, int64_t dld, int64_t P, int c, hipStream_t st) {
  hipLaunchKernelGGL(k_copy_rows, dim3(grid1d(P * (c / 8), 512, 16384)), dim3(256), 0, st, (const u16*)src, sld,
                     (u16*)dst, dld, P, c / 8);
  return hipGetLastError();
}

static RowsArgs rows_args(const BnReluRows& r, int64_t P) {
  RowsArgs A{(const u16*)r.x, r.ld, r.fold, (u16*)r.out, r.old, (u16*)r.copy, r.cld, (int)(P * (r.c / 8)), r.c / 8, 0};
  A.wgs = (int)grid1d(A.total, 512, 16384);  // two vectors a thread
  return A;
}
hipError_t bn_relu_rows(const BnReluRows& a, const BnReluRows* b, int64_t P, hipStream_t st) {
  const RowsArgs A = rows_args(a, P), B = b ? rows_args(*b, P) : RowsArgs{};
  const dim3 grid((unsigned)(A.wgs + B.wgs));
  if (b) hipLaunchKernelGGL(k_bn_relu_rows<true>, grid, dim3(256), 0, st, A, B);
  else hipLaunchKernelGGL(k_bn_relu_rows<false>, grid, dim3(256), 0, st, A, B);
  return hipGetLastError();
}

int stats_splits(int64_t P, int c) {
  const int groups = (c / 8 + 31) / 32;
  int s = 1024 / groups;
  if (s > 256) s = 256;
  const int64_t cap = (P + 63) / 64;
  if (s > cap) s = (int)cap;
  return s < 1 ? 1 : s;
}
size_t stats_partial_floats(int64_t P, int c) { return (size_t)c * stats_splits(P, c) * 3; }

hipError_t stats_partial(const void* x, int64_t ld, int64_t P, int c, float* part, int* T, hipStream_t st) {
  const int S = stats_splits(P, c);
  const int ppb = (int)((P + S - 1) / S);
  const int gs = (int)((P + ppb - 1) / ppb);
  *T = gs;
  hipLaunchKernelGGL(k_stats_partial, dim3((unsigned)((c / 8 + 31) / 32), (unsigned)gs), dim3(256), 0, st,
                     (const u16*)x, ld, P, c, ppb, part);
  return hipGetLastError();
}

size_t packed_layer_elems(int c, int k, int B) {
  const size_t B16 = (B + 15) & ~15, k16 = (k + 15) & ~15, B32 = (B + 31) & ~31, k32 = (k + 31) & ~31;
  const size_t c16 = (c + 15) & ~15, c32 = (c + 31) & ~31;
  return B16 * c32 + c16 * B32 + 9 * k16 * B32 + 9 * B16 * k32;
}

hipError_t pack_block_weights(const float* params, void* packed, int c0, int k, int B, int m, hipStream_t st) {
  const size_t most = packed_layer_elems(c0 + (m - 1) * k, k, B);
  unsigned gx = (unsigned)((most / 8 + 255) / 256);  // (a layer's elements are a multiple of 512)
  const unsigned cap = 8192 / m < 16 ? 16 : (unsigned)(8192 / m);  // (2048 in all: 50 and 47 us for DenseNet-264's last blocks; 44, 43)
  if (gx > cap) gx = cap;
  if (gx < 1) gx = 1;
  hipLaunchKernelGGL(k_pack_block_weights, dim3(gx, (unsigned)m), dim3(256), 0, st, params, (u16*)packed, c0, k, B);
  return hipGetLastError();
}

size_t packed_weight_elems(int cout, int cin, int taps) {
  return (size_t)taps * ((cout + 15) & ~15) * ((cin + 31) & ~31);
}

hipError_t pack_weights(WeightView wv, int cout, int cin, int taps, void* packed, hipStream_t st) {
  const size_t total = packed_weight_elems(cout, cin, taps);
  unsigned grid = (unsigned)((total + 255) / 256);
  if (grid > 4096) grid = 4096;
  hipLaunchKernelGGL(k_pack_weights, dim3(grid), dim3(256), 0, st, wv.w, wv.sm, wv.sc, wv.flip, cout, cin, taps,
                     (u16*)packed);
  return hipGetLastError();
}

size_t conv_stats_partial_floats(int n, int cout, int h, int w) {
  return (size_t)cout * n * ((h * w + 63) / 64) * 3;
}

// taps 1 or 9; in_f32: input is the fp32 gradient slab.  fold: BN+ReLU prologue (or null).
// spart: epilogue statistics (or null), *sT = partials per channel.
hipError_t conv(const void* in, int64_t in_ld, bool in_f32, const void* Wp, void* out, int64_t out_ld, int n,
                int cin, int cout, int h, int w, int taps, const float2* fold, float* spart, int* sT,
                hipStream_t st) {
  const int hw = h * w, M16 = (cout + 15) & ~15, K32 = (cin + 31) & ~31, mtiles = M16 / 16;
  const int64_t P = (int64_t)n * hw;
  // 1x1: flat 64-pixel tiles over all images; 3x3: tiles of one image
  const int64_t ptiles = taps == 9 ? (int64_t)((hw + 63) / 64) * n : (P + 63) / 64;
  if ((fold != nullptr) != (spart != nullptr) && fold) return hipErrorInvalidValue;
  if (taps == 1 && spart && !in_f32 && conv1_stats(in, in_ld, Wp, out, out_ld, P, cin, cout, fold, spart, sT, nullptr, st))
    return hipGetLastError();
  if (taps == 9 && spart && !in_f32 && conv3_stats(in, in_ld, Wp, out, out_ld, n, cin, cout, h, w, fold, spart, sT, nullptr, st))
    return hipGetLastError();
  int mt = (mtiles + 3) / 4;
  if (mt > 3) mt = 3;
  // few pixel tiles: split the output channels over more workgroups (each repeats the staging,
  // on compute units that would otherwise idle) so that a chunk costs each of them less
  while (mt > 1 && ptiles * ((mtiles + 4 * mt - 1) / (4 * mt)) < 256) --mt;
  const int gy = (mtiles + 4 * mt - 1) / (4 * mt);
  dim3 grid(taps == 9 ? (unsigned)((hw + 63) / 64) : (unsigned)ptiles, (unsigned)gy, taps == 9 ? (unsigned)n : 1u);
  const int T = (int)ptiles;
  if (sT) *sT = T;
  const int halo = taps == 9 ? w + 1 : 0;
  const size_t lds = (size_t)2 * (64 + 2 * halo) * 72 * sizeof(u16) + (fold ? (size_t)((cin + 63) & ~63) * 8 : 0);
  if (lds > 64 * 1024 + (fold ? 56 * 8 : 0) || (taps == 9 && (64 + 2 * halo) * 8 > 8 * 256)) return hipErrorInvalidValue;
  // Four chunks in flight with eight or more of them and about one workgroup per compute unit: 392 pixels x 2112
  // channels x 1056 outputs 30.9 -> 26.4 us, 1568 x 2208 x 192 27.0 -> 21.8.  With several workgroups a unit their
  // phases already cover one another's latencies and the ring's extra loads only cost (1568 x 1056 x 2112 27.1 -> 30.5),
  // with few at all the weights come fast enough without (49 x 1056 x 128 12.0 -> 12.8).  With statistics k_conv1 takes
  // these.
  const bool ring = taps == 1 && !spart && cin >= 512 && mt == 1 && ptiles * gy >= 64 && ptiles * gy <= 320;
#define DNB_K(TAPS, MT, TIN, PRO, STATS, RING)                                                                  \
  hipLaunchKernelGGL((k_conv<TAPS, MT, TIN, PRO, STATS, RING>), grid, dim3(256), lds, st, (const TIN*)in, in_ld, \
                     (const u16*)Wp, M16, K32, (u16*)out, out_ld, cin, cout, h, w, P, fold, spart, T)
#define DNB_K2(TAPS, MT)                                                                                          \
  do {                                                                                                            \
    if (in_f32) DNB_K(TAPS, MT, float, false, false, false);                                                 \
    else if (fold) DNB_K(TAPS, MT, u16, true, true, false);                                                       \
    else if (spart) DNB_K(TAPS, MT, u16, false, true, false);                                                     \
    else DNB_K(TAPS, MT, u16, false, false, false);                                                               \
  } while (0)
#define DNB_K3(TAPS)                                                                  \
  do {                                                                                \
    if (mt == 3) DNB_K2(TAPS, 3); else if (mt == 2) DNB_K2(TAPS, 2); else DNB_K2(TAPS, 1); \
  } while (0)
  if (ring && in_f32) DNB_K(1, 1, float, false, false, true);
  else if (ring) DNB_K(1, 1, u16, false, false, true);
  else if (taps == 9) DNB_K3(9);
  else DNB_K3(1);
#undef DNB_K3
#undef DNB_K2
#undef DNB_K
  return hipGetLastError();
}

// The any-shape weight gradient k_wgrad: what dnb_nhwc_wgrad.hip's kernels do not take (rows of more
// than 95 pixels on the 3x3, 2^30 pixels and more).
static int wgrad_splits(int n, int cin, int cout, int h, int w) {
  const int64_t tiles = (int64_t)n * (((int64_t)h * w + 63) / 64);
  int64_t s = 1024 / (((cin + 63) / 64) * ((cout + 63) / 64));
  if (s < 1) s = 1;
  if (s > tiles) s = tiles;
  if (s > 128) s = 128;
  const int64_t tps = (tiles + s - 1) / s;
  return (int)((tiles + tps - 1) / tps);
}
size_t wgrad_partial_floats(int n, int cin, int cout, int h, int w, int taps, bool carrying) {
  const size_t f = wgrad_fast_partial_floats(n, cin, cout, h, w, taps, carrying);
  return f ? f : (size_t)wgrad_splits(n, cin, cout, h, w) * cin * cout * taps;
}

// g_f32: the gradient operand is an fp32 tensor, else bf16.  Writes the partials and adds them into dw.
hipError_t wgrad(const void* a, int64_t a_ld, const void* g, int64_t g_ld, bool g_f32, float* part, float* dw, int n,
                 int cin, int cout, int h, int w, int taps, const float2* fold, hipStream_t st) {
  if (g_f32 && fold) return hipErrorInvalidValue;  // the block's gradient operands are bf16
  WgradSum own{};
  if (wgrad_fast(WgradIn{a, a_ld, g, g_ld, part, dw, cin, cout, fold}, g_f32, n, h, w, taps, &own, st)) {
    const hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : wgrad_finish(taps == 1 ? &own : nullptr, taps == 1 ? nullptr : &own, st);
  }
  const int tpi = (int)(((int64_t)h * w + 63) / 64), tiles = n * tpi;
  const int S = wgrad_splits(n, cin, cout, h, w);
  const int tps = (tiles + S - 1) / S;
  dim3 grid((unsigned)S, (unsigned)((cin + 63) / 64), (unsigned)((cout + 63) / 64));
#define DNB_W(TAPS, TG, PRO)                                                                              \
  hipLaunchKernelGGL((k_wgrad<TAPS, TG, PRO>), grid, dim3(256), 0, st, (const u16*)a, a_ld, (const TG*)g, \
                     g_ld, part, cin, cout, n, h, w, tpi, tps, fold)
#define DNB_W2(TAPS)                                                                                      \
  do {                                                                                                    \
    if (g_f32) DNB_W(TAPS, float, false);                                                                 \
    else if (fold) DNB_W(TAPS, u16, true);                                                                \
    else DNB_W(TAPS, u16, false);                                                                         \
  } while (0)
  if (taps == 9) DNB_W2(9); else DNB_W2(1);
#undef DNB_W2
#undef DNB_W
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_sum_partials(part, S, (int64_t)cin * cout * taps, dw, st);
}

// channel vectors side by side in a workgroup of the BN backward kernels: 4, 8, 16 or 32
// (the count among 8, 16, 32 that leaves the fewest lanes without a vector; 4 for tiny c)
static int bn_bwd_lsh(int c) {
  const int cv = c / 8;
  if (cv <= 4) return 2;
  int best = 5, waste = ((cv + 31) / 32) * 32 - cv;
  for (int lsh = 4; lsh >= 3; --lsh) {
    const int L = 1 << lsh, w = ((cv + L - 1) / L) * L - cv;
    if (w < waste) { waste = w; best = lsh; }
  }
  return best;
}
int bn_bwd_splits(int64_t P, int c) {
  const int lsh = bn_bwd_lsh(c), L = 1 << lsh, rows = 256 >> lsh;
  const int groups = (c / 8 + L - 1) / L;
  int s = 1024 / groups;
  if (s > 256) s = 256;
  const int64_t cap = (P + 8 * rows - 1) / (8 * rows);  // at least two batches of four pixels per thread
  if (s > cap) s = (int)cap;
  return s < 1 ? 1 : s;
}
size_t bn_bwd_partial_floats(int64_t P, int c) { return (size_t)c * bn_bwd_splits(P, c) * 2; }

// BN+ReLU backward, reduction pass: dgamma / dbeta over (P, c).
static hipError_t bn_relu_bwd_reduce(const void* x, int64_t x_ld, const void* dact, int64_t d_ld, int64_t P, int c,
                              const float* gamma, const float* beta, const float* mean, const float* istd,
                              float* dgamma, float* dbeta, float* part, hipStream_t st) {
  const int S = bn_bwd_splits(P, c), lsh = bn_bwd_lsh(c), L = 1 << lsh;
  const int ppb = (int)((P + S - 1) / S);
  const int gs = (int)((P + ppb - 1) / ppb);
  const dim3 grid((unsigned)((c / 8 + L - 1) / L), (unsigned)gs);
  hipLaunchKernelGGL(k_bn_bwd_partial, grid, dim3(256), 0, st, (const u16*)x, x_ld, (const u16*)dact, d_ld, P, c, ppb,
                     lsh, gamma, beta, mean, istd, part);
  hipLaunchKernelGGL(k_bn_bwd_finalize, dim3((unsigned)((c + 3) / 4)), dim3(256), 0, st, part, c, gs, dgamma, dbeta);
  return hipGetLastError();
}

// BN+ReLU backward, element-wise pass over (P, c) with dgamma / dbeta given.  G != null: du is
// accumulated into the fp32 slab (row stride g_ld); else du is written as bf16 to du_bf (may
// alias dact).  A channel sub-range of a wider BN is this call with every pointer moved to the
// range's first channel (a multiple of 8) and `c` its length; `P` is the BN's pixel count.
static hipError_t bn_relu_bwd_apply(const void* x, int64_t x_ld, const void* dact, int64_t d_ld, void* du_bf, int64_t du_ld,
                             float* G, int64_t g_ld, int64_t P, int c, const float* gamma, const float* beta,
                             const float* mean, const float* istd, const float* dgamma, const float* dbeta,
                             hipStream_t st) {
  if (c <= 0) return hipSuccess;
  const int S = bn_bwd_splits(P, c), lsh = bn_bwd_lsh(c), L = 1 << lsh;
  const int ppb = (int)((P + S - 1) / S);
  const float inv_p = 1.0f / (float)P;
  // the element-wise pass wants more, shorter workgroups than the reduction
  const int ppa = (int)min((int64_t)ppb, (int64_t)(256 >> lsh) * 16);
  const dim3 grida((unsigned)((c / 8 + L - 1) / L), (unsigned)((P + ppa - 1) / ppa));
  if (G)
    hipLaunchKernelGGL((k_bn_bwd_apply<true>), grida, dim3(256), 0, st, (const u16*)x, x_ld, (const u16*)dact, d_ld,
                       (u16*)nullptr, (int64_t)0, G, g_ld, P, c, ppa, lsh, inv_p, gamma, beta, mean, istd, dgamma, dbeta);
  else
    hipLaunchKernelGGL((k_bn_bwd_apply<false>), grida, dim3(256), 0, st, (const u16*)x, x_ld, (const u16*)dact, d_ld,
                       (u16*)du_bf, du_ld, (float*)nullptr, (int64_t)0, P, c, ppa, lsh, inv_p, gamma, beta, mean, istd,
                       dgamma, dbeta);
  return hipGetLastError();
}

// Both passes over the same (P, c).
hipError_t bn_relu_bwd(const void* x, int64_t x_ld, const void* dact, int64_t d_ld, void* du_bf, int64_t du_ld,
                       float* G, int64_t g_ld, int64_t P, int c, const float* gamma, const float* beta,
                       const float* mean, const float* istd, float* dgamma, float* dbeta, float* part,
                       hipStream_t st) {
  hipError_t e = bn_relu_bwd_reduce(x, x_ld, dact, d_ld, P, c, gamma, beta, mean, istd, dgamma, dbeta, part, st);
  if (e != hipSuccess) return e;
  return bn_relu_bwd_apply(x, x_ld, dact, d_ld, du_bf, du_ld, G, g_ld, P, c, gamma, beta, mean, istd, dgamma, dbeta, st);
}

}  // namespace nhwc
}  // namespace dnb
