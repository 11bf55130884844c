// bf16 / NHWC weight gradients.
//
//   1x1:  dW[m][c]    = sum_p g[p][m] * act(a[p][c])
//   3x3:  dW[m][c][t] = sum_p g[p][m] * act(a[p + shift(t)][c])     (taps outside the image are zero)
//
// Both contract over pixels, while memory has channels contiguous.  Tiles are staged in LDS as they
// lie in memory, one row per pixel (16-byte stores, BN+ReLU applied on the way), and the operand
// fragments are taken with the transposing LDS read (ds_read_b64_tr_b16: sixteen lanes read four
// rows of sixteen channels and each gets one channel of the four rows).  A tap of the 3x3 is then
// the same tile read at other row addresses, and a tap outside the image a read of a row of zeros:
// one flat pixel axis over all images, no padding of ragged rows, no shifts in registers.
//
// What bounds them: at the 14x14 and 7x7 blocks of the ImageNet-shaped networks there are some 10^3
// pixels to contract over for 10^5 weights, so the launch is the ramp, a few staged tiles per
// workgroup and the partial sums (written once, read once; smaller output tiles mean fewer splits and
// fewer of those bytes, and the gradient rows they read again come from L2).  So: 64 input channels
// x all output channels (up to 192) per workgroup, pixels split until the chip is full; a layer's
// two weight gradients in one launch, which also carries the sums of the layer before.  The earlier
// kernels (transposed staging by 2-byte stores, 256 x 192 tiles, some 96 workgroups each, two
// launches and two sums per layer) took 50 us per layer of the DenseNet-264-shaped step at batch 32.
#include "dnb_internal.h"
#include "dnb_nhwc_dev.h"
#include "dnb_stats.h"

namespace dnb {
namespace nhwc {

namespace {

typedef short s16x4 __attribute__((ext_vector_type(4)));

// Pitch of a staged row of 64 channels.  The sixteen-lane groups of a wave read 32-byte pieces of rows
// 4g..4g+3; with row pitches of 32 or 160 (mod 256) bytes the eight pieces of two groups lie on
// disjoint banks.
constexpr int AP = 80;
__host__ __device__ constexpr int gpitch(int mtiles) { return mtiles == 12 ? 208 : mtiles == 8 ? 144 : mtiles > 2 ? 80 : 48; }

// rows r0..r3 (this lane's address is row (lane>>2)&3, channels 4*(lane&3)) -> one channel, 4 rows
__device__ __forceinline__ uint2 tr_read(const u16* p) {
  return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p));
}
// K index 8g + e of the matrix instruction = pixel 4g + e (e < 4) or 16 + 4g + e - 4 of a step of 32,
// for both operands
__device__ __forceinline__ V8 tr_frag(const u16* lo, const u16* hi) {
  const uint2 a = tr_read(lo), b = tr_read(hi);
  V8 v;
  v.q = make_uint4(a.x, a.y, b.x, b.y);
  return v;
}

template <typename TG>
struct GVec {  // 8 channels of the gradient operand as loaded
  uint4 q;
};
template <>
struct GVec<float> {
  float4 lo, hi;
};
__device__ __forceinline__ void gload(GVec<u16>& v, const u16* p) { v.q = *reinterpret_cast<const uint4*>(p); }
__device__ __forceinline__ void gload(GVec<float>& v, const float* p) {
  v.lo = *reinterpret_cast<const float4*>(p);
  v.hi = *reinterpret_cast<const float4*>(p + 4);
}
__device__ __forceinline__ uint4 gbf(const GVec<u16>& v) { return v.q; }
__device__ __forceinline__ uint4 gbf(const GVec<float>& v) {
  V8 t;
  t.h[0] = f2bf(v.lo.x); t.h[1] = f2bf(v.lo.y); t.h[2] = f2bf(v.lo.z); t.h[3] = f2bf(v.lo.w);
  t.h[4] = f2bf(v.hi.x); t.h[5] = f2bf(v.hi.y); t.h[6] = f2bf(v.hi.z); t.h[7] = f2bf(v.hi.w);
  return t.q;
}

__device__ __forceinline__ uint4 bnrelu8(uint4 q, const float2 (&f)[8]) {
  V8 t;
  t.q = q;
#pragma unroll
  for (int e = 0; e < 8; ++e) t.h[e] = f2bf(fmaxf(__fmaf_rn(bf2f(t.h[e]), f[e].x, f[e].y), 0.f));
  return t.q;
}

// A finished launch's partial sums, to be added up by a later launch.  Partials are in accumulator
// order, [S][block of (c group, m group)][wave][tile][lane][4].
struct SumArgs {
  const float* part;
  float* out;
  int taps, S, gy, gz, mt, cin, cout;  // mt: M-tiles of a block; taps 0: nothing to do
  int wgs;
};

struct Wg1Args {
  const u16* a; int64_t a_ld;
  const void* g; int64_t g_ld;
  float* part;
  int cin, cout, P, S, tps, gy, gz, n;  // n: workgroups
  const float2* fold;
};
struct Wg3Args {
  const u16* a; int64_t a_ld;
  const void* g; int64_t g_ld;
  float* part;
  int cin, cout, P, H, W, R, S, tps, gy, gz, n;
  const float2* fold;
};

// ---------------------------------------------------------------- 1x1

// 64 input channels x 16*MG output channels over tps tiles of 64 pixels.  Wave (wave & 1, wave >> 1)
// holds two c-tiles x MG/2 m-tiles.  The next tile's loads are in flight during the products of the
// current one; loads are unconditional at clamped addresses, rows past the last pixel become zeros.
// Workgroups go to the eight XCDs in turn; each XCD takes an equal, consecutive share of the (range, column) items, so that
// its L2 holds the gradient rows that a range's columns share (whole ranges per XCD left XCDs idle where ranges are few:
// 12 to 6 of them at 14x14 and 7x7).
template <int MG, bool PRO, typename TG>
__device__ __forceinline__ void wgrad1_body(const Wg1Args& A, int id, u16* lds) {
  const int cols = A.gy * A.gz, item = (id & 7) * (A.n >> 3) + (id >> 3), bx = item / cols, col = item - bx * cols;
  if (bx >= A.S) return;
  const int cg = col / A.gz, mg = col % A.gz;
  constexpr int GP = gpitch(MG), GV = 2 * MG, GU = MG / 2;
  u16* gS = lds + 64 * AP;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4;
  const int c0 = cg * 64, m0 = mg * MG * 16;
  const int tiles = (A.P + 63) >> 6, t_begin = bx * A.tps, t_end = min(tiles, t_begin + A.tps);

  const int av = tid & 7, ar = tid >> 3;
  const int ch = min(c0 + 8 * av, A.cin - 8);  // cin, cout % 8 == 0
  const u16* asrc = A.a + ch;
  float2 f[8];
  if (PRO) {
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = A.fold[ch + e];
  }
  const TG* gsrc[GU];
  int gr[GU];
#pragma unroll
  for (int u = 0; u < GU; ++u) {
    const int idx = tid + 256 * u;
    gr[u] = idx / GV;
    gsrc[u] = (const TG*)A.g + min(m0 + 8 * (idx % GV), A.cout - 8);
  }
  uint4 ra[2];
  GVec<TG> rg[GU];
  auto issue = [&](int t) {
#pragma unroll
    for (int u = 0; u < 2; ++u) ra[u] = *reinterpret_cast<const uint4*>(asrc + (int64_t)min(t * 64 + ar + 32 * u, A.P - 1) * A.a_ld);
#pragma unroll
    for (int u = 0; u < GU; ++u) gload(rg[u], gsrc[u] + (int64_t)min(t * 64 + gr[u], A.P - 1) * A.g_ld);
  };

  f32x4 acc[2][GU];
#pragma unroll
  for (int y = 0; y < 2; ++y)
#pragma unroll
    for (int x = 0; x < GU; ++x) acc[y][x] = (f32x4){0.f, 0.f, 0.f, 0.f};
  const int row = 4 * g + ((lane >> 2) & 3), cc = 4 * (lane & 3);
  const u16* af = lds + row * AP + (wave & 1) * 32 + cc;
  const u16* gf = gS + row * GP + (wave >> 1) * (GU * 16) + cc;

  if (t_begin < t_end) issue(t_begin);
  for (int t = t_begin; t < t_end; ++t) {
    __syncthreads();  // the previous tile's fragment reads are done
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      uint4 q = ra[u];
      if (PRO) q = bnrelu8(q, f);
      if (t * 64 + ar + 32 * u >= A.P) q = make_uint4(0u, 0u, 0u, 0u);
      *reinterpret_cast<uint4*>(lds + (ar + 32 * u) * AP + 8 * av) = q;
    }
#pragma unroll
    for (int u = 0; u < GU; ++u) {
      uint4 q = gbf(rg[u]);
      if (t * 64 + gr[u] >= A.P) q = make_uint4(0u, 0u, 0u, 0u);
      *reinterpret_cast<uint4*>(gS + gr[u] * GP + 8 * ((tid + 256 * u) % GV)) = q;
    }
    __syncthreads();
    issue(min(t + 1, t_end - 1));
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      V8 b[2], w[GU];
#pragma unroll
      for (int y = 0; y < 2; ++y) b[y] = tr_frag(af + ks * 32 * AP + y * 16, af + (ks * 32 + 16) * AP + y * 16);
#pragma unroll
      for (int x = 0; x < GU; ++x) w[x] = tr_frag(gf + ks * 32 * GP + x * 16, gf + (ks * 32 + 16) * GP + x * 16);
#pragma unroll
      for (int x = 0; x < GU; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) acc[y][x] = mfma_bf16(w[x], b[y], acc[y][x]);
    }
  }
  float* pb = A.part + ((int64_t)bx * cols + col) * (64 * MG * 16) + wave * (MG * 256) + lane * 4;
#pragma unroll
  for (int y = 0; y < 2; ++y)
#pragma unroll
    for (int x = 0; x < GU; ++x)
      *reinterpret_cast<float4*>(pb + (x * 2 + y) * 256) = make_float4(acc[y][x][0], acc[y][x][1], acc[y][x][2], acc[y][x][3]);
}

// ---------------------------------------------------------------- 3x3

// 64 input channels x 16*MT output channels x 9 taps over tps tiles of 64 consecutive pixels of the
// flat axis (images follow one another; a 9-bit mask per pixel says which taps are inside its image).
// The activations sit in a ring of R rows (R a power of two, at least 64 pixels plus a halo of a row
// and a pixel on both sides): each tile stages the 64 pixels that are new, so a pixel is loaded and
// normalised once per workgroup.  Row R of the ring is zero.  Wave w holds c-tile w, all taps and
// m-tiles.
template <int MT, bool PRO, typename TG>
__device__ __forceinline__ void wgrad3_body(const Wg3Args& A, int id, u16* lds) {
  const int cols = A.gy * A.gz, col = id % cols, bx = id / cols;
  if (bx >= A.S) return;
  const int cg = col / A.gz, mg = col % A.gz;
  constexpr int GP = gpitch(MT), GV = 2 * MT, GU = MT == 3 ? 2 : 1;  // 64 * GV vectors over 256 threads
  const int R = A.R, RM = R - 1;
  u16* gS = lds + (R + 1) * AP;
  unsigned* mask = reinterpret_cast<unsigned*>(gS + 64 * GP);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4;
  const int c0 = cg * 64, m0 = mg * MT * 16, W = A.W, HW = A.H * W, lead = W + 1;
  const int tiles = (A.P + 63) >> 6, t_begin = bx * A.tps, t_end = min(tiles, t_begin + A.tps);

  const int av = tid & 7, ar = tid >> 3;
  const int ch = min(c0 + 8 * av, A.cin - 8);
  const u16* asrc = A.a + ch;
  float2 f[8];
  if (PRO) {
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = A.fold[ch + e];
  }
  const TG* gsrc[GU];
  int gr[GU];
#pragma unroll
  for (int u = 0; u < GU; ++u) {
    const int idx = min(tid + 256 * u, 64 * GV - 1);  // threads past the tile repeat its last vector
    gr[u] = idx / GV;
    gsrc[u] = (const TG*)A.g + min(m0 + 8 * (idx % GV), A.cout - 8);
  }
  uint4 ra[2];
  GVec<TG> rg[GU];
  auto issue = [&](int t) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int p = t * 64 + lead + ar + 32 * u;
      ra[u] = *reinterpret_cast<const uint4*>(asrc + (int64_t)min(max(p, 0), A.P - 1) * A.a_ld);
    }
#pragma unroll
    for (int u = 0; u < GU; ++u) gload(rg[u], gsrc[u] + (int64_t)min(t * 64 + gr[u], A.P - 1) * A.g_ld);
  };
  auto put = [&](int p, uint4 q) {  // pixels outside [0, P) are never read: their taps are masked
    if (PRO) q = bnrelu8(q, f);
    *reinterpret_cast<uint4*>(lds + (p & RM) * AP + 8 * av) = q;
  };

  f32x4 acc[9][MT];
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int x = 0; x < MT; ++x) acc[t][x] = (f32x4){0.f, 0.f, 0.f, 0.f};
  const int row = 4 * g + ((lane >> 2) & 3), cc = 4 * (lane & 3), acol = wave * 16 + cc;
  const u16* gf = gS + row * GP + cc;
  const int zrow = R * AP + acol;

  if (t_begin < t_end) {
    issue(t_begin);
    const int pf = t_begin * 64 - lead;  // the pixels before the first chunk
    for (int r = ar; r < 2 * lead; r += 32) {
      const int p = pf + r;
      put(p, *reinterpret_cast<const uint4*>(asrc + (int64_t)min(max(p, 0), A.P - 1) * A.a_ld));
    }
    if (tid < AP / 8) *reinterpret_cast<uint4*>(lds + R * AP + 8 * tid) = make_uint4(0u, 0u, 0u, 0u);
  }
  for (int t = t_begin; t < t_end; ++t) {
    __syncthreads();  // the previous tile's fragment reads are done
#pragma unroll
    for (int u = 0; u < 2; ++u) put(t * 64 + lead + ar + 32 * u, ra[u]);
#pragma unroll
    for (int u = 0; u < GU; ++u) {
      uint4 q = gbf(rg[u]);
      if (t * 64 + gr[u] >= A.P) q = make_uint4(0u, 0u, 0u, 0u);
      *reinterpret_cast<uint4*>(gS + gr[u] * GP + 8 * (min(tid + 256 * u, 64 * GV - 1) % GV)) = q;
    }
    if (tid < 64) {
      const int p = t * 64 + tid, q = p % HW, y = q / W, x = q - y * W;
      unsigned b = 0;
      if (p < A.P) {
        const unsigned r3 = (x > 0 ? 1u : 0u) | 2u | (x < W - 1 ? 4u : 0u);
        b = (y > 0 ? r3 : 0u) | (r3 << 3) | (y < A.H - 1 ? r3 << 6 : 0u);
      }
      mask[tid] = b;
    }
    __syncthreads();
    issue(min(t + 1, t_end - 1));
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int r0 = ks * 32 + row, r1 = r0 + 16;
      const unsigned k0 = mask[r0], k1 = mask[r1];
      const int p0 = t * 64 + r0, p1 = t * 64 + r1;
      V8 w[MT];
#pragma unroll
      for (int x = 0; x < MT; ++x) w[x] = tr_frag(gf + ks * 32 * GP + x * 16, gf + (ks * 32 + 16) * GP + x * 16);
#pragma unroll
      for (int t9 = 0; t9 < 9; ++t9) {
        const int off = (t9 / 3 - 1) * W + t9 % 3 - 1;
        const int a0 = (k0 >> t9) & 1 ? ((p0 + off) & RM) * AP + acol : zrow;
        const int a1 = (k1 >> t9) & 1 ? ((p1 + off) & RM) * AP + acol : zrow;
        const V8 b = tr_frag(lds + a0, lds + a1);
#pragma unroll
        for (int x = 0; x < MT; ++x) acc[t9][x] = mfma_bf16(w[x], b, acc[t9][x]);
      }
    }
  }
  float* pb = A.part + ((int64_t)bx * cols + col) * (4 * 9 * MT * 256) + wave * (9 * MT * 256) + lane * 4;
#pragma unroll
  for (int t9 = 0; t9 < 9; ++t9)
#pragma unroll
    for (int x = 0; x < MT; ++x)
      *reinterpret_cast<float4*>(pb + (t9 * MT + x) * 256) = make_float4(acc[t9][x][0], acc[t9][x][1], acc[t9][x][2], acc[t9][x][3]);
}

// ---------------------------------------------------------------- sums of partials

// Workgroup wg adds the S partials of 64 accumulator quads: four 64-thread groups take every fourth
// split (loads four deep), their results are added in group order.  red: 3*64 float4.
__device__ __forceinline__ void sum_body(const SumArgs& s, int wg, float4* red) {
  const int t = threadIdx.x & 63, sg = threadIdx.x >> 6;
  const int block = 4 * 256 * s.mt * (s.taps == 9 ? 9 : 1);
  const int64_t per_split = (int64_t)s.gy * s.gz * block;
  const int64_t i = ((int64_t)wg * 64 + t) * 4;  // one (block, wave, tile) per workgroup
  const int blk = (int)(i / block), rem = (int)(i - (int64_t)blk * block);
  const int cg = blk / s.gz, mg = blk - cg * s.gz;
  const int tile = rem >> 8, per_wave = s.mt * (s.taps == 9 ? 9 : 1), wave = tile / per_wave, tt = tile - wave * per_wave;
  int mb, cb, t9 = 0;  // first output / input channel of the tile, tap
  if (s.taps == 9) {
    t9 = tt / s.mt;
    mb = (mg * s.mt + tt - t9 * s.mt) * 16;
    cb = cg * 64 + wave * 16;
  } else {
    mb = (mg * s.mt + (wave >> 1) * (s.mt / 2) + (tt >> 1)) * 16;
    cb = cg * 64 + (wave & 1) * 32 + (tt & 1) * 16;
  }
  if (mb >= s.cout || cb >= s.cin) return;  // uniform
  float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
  const float* p = s.part + i;
  int k = sg;
  for (; k + 12 < s.S; k += 16) {
    float4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = *reinterpret_cast<const float4*>(p + (int64_t)(k + 4 * u) * per_split);
#pragma unroll
    for (int u = 0; u < 4; ++u) { sum.x += v[u].x; sum.y += v[u].y; sum.z += v[u].z; sum.w += v[u].w; }
  }
  for (; k < s.S; k += 4) {
    const float4 v = *reinterpret_cast<const float4*>(p + (int64_t)k * per_split);
    sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
  }
  if (sg > 0) red[(sg - 1) * 64 + t] = sum;
  __syncthreads();
  if (sg > 0) return;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const float4 o = red[q * 64 + t];
    sum.x += o.x; sum.y += o.y; sum.z += o.z; sum.w += o.w;
  }
  const int c = cb + (t & 15), m = mb + 4 * (t >> 4);
  if (c >= s.cin) return;
  const float o4[4] = {sum.x, sum.y, sum.z, sum.w};
#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (m + r < s.cout) s.out[((int64_t)(m + r) * s.cin + c) * s.taps + t9] = o4[r];
}

// ---------------------------------------------------------------- 1x1 data gradient + BN1 backward

// du_c = W_c . db (over the B outputs), masked by BN1's ReLU, scaled and added into the slab, with BN1's sums
// of dz and dz*(x - mean): see dnb_nhwc_bwd.hip.  Bound by the slab's traffic: 10 bytes per element (x 2, G 4 + 4)
// against 2*B flops, so two layers that both read a channel are done in one pass (the upper one's share of the
// lower one's own slice goes first, beside the upper one's weight gradients, and only that delays the chain):
// 5 bytes per element and layer, and no launch of its own.
struct D1Args {
  int nl, n, cols, T, nk;         // layers; workgroups (cols x T); K-steps of 32 outputs
  const u16* db[2]; const u16* W[2];
  int mtiles[2];
  const float2* fold[2];
  float2* part[2];
  const u16* x; int64_t x_ld;
  const u16* dy; float* G; int64_t ld;
  int first;
  const float *mean, *istd;
  int B, cb, ce;
  int P, ppw;                     // pixels per wave, a multiple of 32
};

// Output channels on M, pixels on N.  A workgroup owns 32 channels (two M-tiles, weights and coefficients of
// both layers in LDS) and a range of pixels, of which each wave walks a quarter in steps of 32 (two N-tiles); a
// lane then holds 4 consecutive channels of a pixel: the slab is read and written in 16-byte pieces, 128
// contiguous bytes per pixel and wave.  Waves share nothing until the sums at the end.
template <int KS>
__device__ __forceinline__ void dgrad1_body(const D1Args& A, int id, u16* lds) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, j = lane & 15, g = lane >> 4;
  const int col = id % A.cols, ty = id / A.cols, c00 = (A.cb & ~15) + col * 32;
  float* cf = reinterpret_cast<float*>(lds + A.nl * 2 * A.nk * 512);  // [nl][32][2]
  for (int i = tid; i < A.nl * 2 * A.nk * 64; i += 256) {
    const int f = i >> 6, s = f % A.nk, a = (f / A.nk) & 1, li = f / (2 * A.nk);
    const int mt = min((c00 >> 4) + a, (li ? A.mtiles[1] : A.mtiles[0]) - 1);
    *reinterpret_cast<uint4*>(lds + i * 8) =
        *reinterpret_cast<const uint4*>((li ? A.W[1] : A.W[0]) + ((int64_t)mt * A.nk + s) * 512 + (i & 63) * 8);
  }
  if (tid < 32 * A.nl) {
    const float2 f = (tid < 32 ? A.fold[0] : A.fold[1])[min(c00 + (tid & 31), A.ce - 1)];
    cf[2 * tid] = f.x; cf[2 * tid + 1] = f.y;
  }
  float mu[2][4], s0[2][2][4], s1[2][2][4];
  int ch[2];
  bool cok[2];
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const int c = c00 + a * 16 + 4 * g;  // cb, ce % 8 == 0: a lane's four channels are in or out together
    cok[a] = c >= A.cb && c < A.ce;
    ch[a] = min(c, A.ce - 4);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      mu[a][r] = A.mean[ch[a] + r];
#pragma unroll
      for (int li = 0; li < 2; ++li) s0[li][a][r] = s1[li][a][r] = 0.f;
    }
  }
  __syncthreads();
  const int pw0 = (ty * 4 + wave) * A.ppw, pw1 = min(A.P, pw0 + A.ppw);
  for (int pb = pw0; pb < pw1; pb += 32) {
    int p[2];
    uint2 xr[2][2];
    float gv[2][2][4];
    V8 d[2][KS];
    auto dload = [&](const u16* db, int s0) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int s = 0; s < KS; ++s)
          d[t][s].q = *reinterpret_cast<const uint4*>(db + (int64_t)p[t] * A.B + min(32 * (s0 + s) + 8 * g, A.B - 8));
    };
#pragma unroll
    for (int t = 0; t < 2; ++t) p[t] = min(pb + t * 16 + j, pw1 - 1);  // clamped: masked below
    dload(A.db[0], 0);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int a = 0; a < 2; ++a) xr[t][a] = *reinterpret_cast<const uint2*>(A.x + (int64_t)p[t] * A.x_ld + ch[a]);
    if (A.first) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          const uint2 v = *reinterpret_cast<const uint2*>(A.dy + (int64_t)p[t] * A.ld + ch[a]);
          gv[t][a][0] = bf2f((u16)v.x); gv[t][a][1] = bf2f((u16)(v.x >> 16));
          gv[t][a][2] = bf2f((u16)v.y); gv[t][a][3] = bf2f((u16)(v.y >> 16));
        }
    } else {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          const float4 v = *reinterpret_cast<const float4*>(A.G + (int64_t)p[t] * A.ld + ch[a]);
          gv[t][a][0] = v.x; gv[t][a][1] = v.y; gv[t][a][2] = v.z; gv[t][a][3] = v.w;
        }
    }
#pragma unroll
    for (int li = 0; li < 2; ++li) {
      if (li < A.nl) {
        f32x4 acc[2][2];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int a = 0; a < 2; ++a) acc[t][a] = (f32x4){0.f, 0.f, 0.f, 0.f};
        for (int sb = 0; sb < A.nk; sb += KS) {
          if (li > 0 || sb > 0) dload(A.db[li], sb);
#pragma unroll
          for (int s = 0; s < KS; ++s) {
            if (sb + s < A.nk) {
              V8 w[2];
#pragma unroll
              for (int a = 0; a < 2; ++a) w[a].q = *reinterpret_cast<const uint4*>(lds + ((li * 2 + a) * A.nk + sb + s) * 512 + lane * 8);
#pragma unroll
              for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int a = 0; a < 2; ++a) acc[t][a] = mfma_bf16(w[a], d[t][s], acc[t][a]);
            }
          }
        }
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          const float4* fp = reinterpret_cast<const float4*>(cf + (li * 32 + a * 16 + 4 * g) * 2);
          const float4 f0 = fp[0], f1 = fp[1];
          const float sc[4] = {f0.x, f0.z, f1.x, f1.z}, sf[4] = {f0.y, f0.w, f1.y, f1.w};
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            const bool ok = pb + t * 16 + j < pw1 && cok[a];
            const float xf[4] = {bf2f((u16)xr[t][a].x), bf2f((u16)(xr[t][a].x >> 16)), bf2f((u16)xr[t][a].y),
                                 bf2f((u16)(xr[t][a].y >> 16))};
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float dz = ok && __fmaf_rn(xf[r], sc[r], sf[r]) > 0.f ? acc[t][a][r] : 0.f;
              gv[t][a][r] = __fmaf_rn(sc[r], dz, gv[t][a][r]);
              s0[li][a][r] += dz;
              s1[li][a][r] = __fmaf_rn(dz, xf[r] - mu[a][r], s1[li][a][r]);
            }
          }
        }
      }
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int a = 0; a < 2; ++a)
        if (pb + t * 16 + j < pw1 && cok[a])
          *reinterpret_cast<float4*>(A.G + (int64_t)p[t] * A.ld + ch[a]) = make_float4(gv[t][a][0], gv[t][a][1], gv[t][a][2], gv[t][a][3]);
  }
  __syncthreads();  // the weights are read
  float* red = reinterpret_cast<float*>(lds);  // [2][4][32][2]
#pragma unroll
  for (int li = 0; li < 2; ++li)
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float u = row16_sum(s0[li][a][r]), v = row16_sum(s1[li][a][r]);
        if (j == 0) {
          float* o = red + ((li * 4 + wave) * 32 + a * 16 + 4 * g + r) * 2;
          o[0] = u; o[1] = v;
        }
      }
  __syncthreads();
  const int li = tid >> 5, c = c00 + (tid & 31);
  if (li < A.nl && c >= A.cb && c < A.ce) {
    float u = 0.f, v = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q) { u += red[((li * 4 + q) * 32 + (tid & 31)) * 2]; v += red[((li * 4 + q) * 32 + (tid & 31)) * 2 + 1]; }
    (li ? A.part[1] : A.part[0])[(int64_t)ty * (A.ce - A.cb) + c - A.cb] = make_float2(u, v * A.istd[c]);
  }
}

// ---------------------------------------------------------------- kernels

// A layer's two weight gradients, the pending sums of the layer before it and a data gradient (which reads the
// gradient of b_l as the 1x1's does and writes only the slab and its sums).  The 3x3's workgroups first: they are
// the fewer and the longer ones.
// (Waves per SIMD asked for: left alone the allocator takes 200 registers where 168 hold the code.)
template <int MG, int MT, bool PRO>
__global__ __launch_bounds__(256, (MT == 3 ? 2 : 3)) void k_wgrad_pair(Wg1Args A1, Wg3Args A3, SumArgs s1, SumArgs s3, D1Args D) {
  extern __shared__ __attribute__((aligned(16))) u16 lds[];
  int id = blockIdx.x;
  if (id < A3.n) { wgrad3_body<MT, PRO, u16>(A3, id, lds); return; }
  id -= A3.n;
  if (id < D.n) { dgrad1_body<MG / 2>(D, id, lds); return; }
  id -= D.n;
  if (id < A1.n) { wgrad1_body<MG, PRO, u16>(A1, id, lds); return; }
  id -= A1.n;
  if (id < s1.wgs) { sum_body(s1, id, reinterpret_cast<float4*>(lds)); return; }
  id -= s1.wgs;
  if (id < s3.wgs) sum_body(s3, id, reinterpret_cast<float4*>(lds));
}
template <int MG, bool PRO, typename TG>
__global__ __launch_bounds__(256) void k_wgrad1(Wg1Args A) {
  extern __shared__ __attribute__((aligned(16))) u16 lds[];
  wgrad1_body<MG, PRO, TG>(A, blockIdx.x, lds);
}
template <int MT, bool PRO, typename TG>
__global__ __launch_bounds__(256, (MT == 3 ? 2 : 3)) void k_wgrad3(Wg3Args A) {
  extern __shared__ __attribute__((aligned(16))) u16 lds[];
  wgrad3_body<MT, PRO, TG>(A, blockIdx.x, lds);
}
__global__ __launch_bounds__(256) void k_wgrad_sums(SumArgs s1, SumArgs s3) {
  __shared__ float4 red[192];
  int id = blockIdx.x;
  if (id < s1.wgs) { sum_body(s1, id, red); return; }
  id -= s1.wgs;
  if (id < s3.wgs) sum_body(s3, id, red);
}

// ---------------------------------------------------------------- plans

// Workgroups of the 1x1 and of the 3x3.  A split costs a partial of the whole weight tensor: the
// lower bounds fill the chip, the upper ones apply where a split still has eight tiles (large images,
// small partials).  Not sharp: lower bounds of 192..512 and 64..256, upper ones of 512..1024 and
// 256..768 moved the DenseNet-264-shaped step between 16.03 and 16.35 ms; beside a data gradient, whose workgroups
// fill the chip too, 512 at most for the 1x1 (a transition's gradient by itself: 260 us with 512, 111 with 1024; blocks
// of more than 256 outputs, whose data gradient has a launch of its own: 2 to 5 % of a step).
constexpr int WG1_MIN = 256, WG1_MAX = 1024, WG1_CARRYING_MAX = 512, WG3_MIN = 128, WG3_MAX = 256, LONG_TILES = 8;

int splits_for(int tiles, int cols, int lo, int hi) {
  int s = lo / cols, s2 = hi / cols;
  if (s2 > tiles / LONG_TILES) s2 = tiles / LONG_TILES;
  if (s < s2) s = s2;
  if (s > tiles) s = tiles;
  if (s < 1) s = 1;
  const int tps = (tiles + s - 1) / s;
  return (tiles + tps - 1) / tps;
}

struct Plan1 {
  int mg, gy, gz, S, tps, n;
  size_t lds, floats;
};
Plan1 plan1(int P, int cin, int cout, int most) {
  Plan1 p{};
  const int mt = (cout + 15) / 16;
  int best = 0;
  for (int mg : {12, 8, 4}) {  // the largest group, unless a smaller one saves an eighth of the tiles
    const int pad = (mt + mg - 1) / mg * mg;
    if (best == 0 || pad * 8 < best * 7) { best = pad; p.mg = mg; }
  }
  p.gy = (cin + 63) / 64;
  p.gz = (mt + p.mg - 1) / p.mg;
  const int tiles = (P + 63) / 64;
  p.S = splits_for(tiles, p.gy * p.gz, WG1_MIN, most);
  p.tps = (tiles + p.S - 1) / p.S;
  p.n = (p.S * p.gy * p.gz + 7) / 8 * 8;
  p.lds = (size_t)64 * (AP + gpitch(p.mg)) * sizeof(u16);
  p.floats = (size_t)p.S * p.gy * p.gz * 64 * p.mg * 16;
  return p;
}
struct Plan3 {
  bool ok;
  int mt, R, gy, gz, S, tps, n;
  size_t lds, floats;
};
Plan3 plan3(int P, int w, int cin, int cout) {
  Plan3 p{};
  const int need = 64 + 2 * (w + 1);
  if (need > 256) return p;  // wider rows: the tap-by-tap kernel
  p.ok = true;
  p.R = need <= 128 ? 128 : 256;
  const int mt = (cout + 15) / 16;
  p.mt = mt <= 3 ? mt : (mt + 2) / 3 * 3 <= (mt + 1) / 2 * 2 ? 3 : 2;  // (four would need more than 256 registers)
  p.gy = (cin + 63) / 64;
  p.gz = (mt + p.mt - 1) / p.mt;
  const int tiles = (P + 63) / 64;
  p.S = splits_for(tiles, p.gy * p.gz, WG3_MIN, WG3_MAX);
  p.tps = (tiles + p.S - 1) / p.S;
  p.n = p.S * p.gy * p.gz;
  p.lds = ((size_t)(p.R + 1) * AP + 64 * gpitch(p.mt)) * sizeof(u16) + 64 * sizeof(unsigned);
  p.floats = (size_t)p.S * p.gy * p.gz * 4 * 9 * p.mt * 256;
  return p;
}

Wg1Args args1(const Plan1& p, const WgradIn& w, int P) {
  return Wg1Args{(const u16*)w.a, w.a_ld, w.g, w.g_ld, w.part, w.cin, w.cout, P, p.S, p.tps, p.gy, p.gz, p.n, w.fold};
}
Wg3Args args3(const Plan3& p, const WgradIn& w, int P, int h, int wd) {
  return Wg3Args{(const u16*)w.a, w.a_ld, w.g, w.g_ld, w.part, w.cin, w.cout, P, h, wd, p.R, p.S, p.tps, p.gy, p.gz, p.n, w.fold};
}
SumArgs sum_args(WgradSum* s) {
  SumArgs a{};
  if (!s || s->taps == 0) return a;
  a = SumArgs{s->part, s->out, s->taps, s->S, s->gy, s->gz, s->mt, s->cin, s->cout, 0};
  a.wgs = s->gy * s->gz * 4 * s->mt * (s->taps == 9 ? 9 : 1);
  s->taps = 0;
  return a;
}

}  // namespace

// pixel indexes (with a halo) are 32-bit in these kernels
static bool fits(int n, int h, int w) { return (int64_t)n * h * w < (int64_t)1 << 30; }

size_t wgrad_fast_partial_floats(int n, int cin, int cout, int h, int w, int taps, bool carrying) {
  if (!fits(n, h, w)) return 0;
  const int P = n * h * w;
  if (taps == 1) return plan1(P, cin, cout, carrying ? WG1_CARRYING_MAX : WG1_MAX).floats;
  const Plan3 p = plan3(P, w, cin, cout);
  return p.ok ? p.floats : 0;
}

hipError_t wgrad_finish(WgradSum* s1, WgradSum* s3, hipStream_t st) {
  const SumArgs a1 = sum_args(s1), a3 = sum_args(s3);
  if (a1.wgs + a3.wgs == 0) return hipSuccess;
  hipLaunchKernelGGL(k_wgrad_sums, dim3((unsigned)(a1.wgs + a3.wgs)), dim3(256), 0, st, a1, a3);
  return hipGetLastError();
}

bool wgrad_fast(const WgradIn& in, bool g_f32, int n, int h, int w, int taps, WgradSum* own, hipStream_t st) {
  if ((g_f32 && in.fold) || !fits(n, h, w)) return false;
  const int P = n * h * w;
  if (taps == 1) {
    const Plan1 p = plan1(P, in.cin, in.cout, WG1_MAX);
    const Wg1Args A = args1(p, in, P);
#define DNB_L(MG)                                                                                                 \
  do {                                                                                                            \
    if (g_f32) hipLaunchKernelGGL((k_wgrad1<MG, false, float>), dim3((unsigned)p.n), dim3(256), p.lds, st, A);      \
    else if (in.fold) hipLaunchKernelGGL((k_wgrad1<MG, true, u16>), dim3((unsigned)p.n), dim3(256), p.lds, st, A);  \
    else hipLaunchKernelGGL((k_wgrad1<MG, false, u16>), dim3((unsigned)p.n), dim3(256), p.lds, st, A);              \
  } while (0)
    if (p.mg == 12) DNB_L(12); else if (p.mg == 8) DNB_L(8); else DNB_L(4);
#undef DNB_L
    *own = WgradSum{in.part, in.dw, 1, p.S, p.gy, p.gz, p.mg, in.cin, in.cout};
    return true;
  }
  const Plan3 p = plan3(P, w, in.cin, in.cout);
  if (!p.ok) return false;
  const Wg3Args A = args3(p, in, P, h, w);
#define DNB_L(MT)                                                                                                 \
  do {                                                                                                            \
    if (g_f32) hipLaunchKernelGGL((k_wgrad3<MT, false, float>), dim3((unsigned)p.n), dim3(256), p.lds, st, A);      \
    else if (in.fold) hipLaunchKernelGGL((k_wgrad3<MT, true, u16>), dim3((unsigned)p.n), dim3(256), p.lds, st, A);  \
    else hipLaunchKernelGGL((k_wgrad3<MT, false, u16>), dim3((unsigned)p.n), dim3(256), p.lds, st, A);              \
  } while (0)
  switch (p.mt) { case 1: DNB_L(1); break; case 2: DNB_L(2); break; default: DNB_L(3); break; }
#undef DNB_L
  *own = WgradSum{in.part, in.dw, 9, p.S, p.gy, p.gz, p.mt, in.cin, in.cout};
  return true;
}

// About 1024 workgroups over the slab, at most `most` splits; each wave takes at least one step of 32 pixels.
int dgrad1_splits(int64_t P, int C, int most, int* ppw) {
  const int64_t cols = (C + 31) / 32;
  int64_t t = 1024 / cols;
  if (t > most) t = most;
  if (t > (P + 127) / 128) t = (P + 127) / 128;
  if (t < 1) t = 1;
  const int64_t px = ((P + 4 * t - 1) / (4 * t) + 31) / 32 * 32;
  *ppw = (int)px;
  return (int)((P + 4 * px - 1) / (4 * px));
}

bool wgrad_pair(const WgradIn& w1, const WgradIn& w3, int n, int h, int w, WgradSum* s1, WgradSum* s3, const Dgrad1In& d1,
                int most_splits, int* T1, hipStream_t st) {
  if (!fits(n, h, w)) return false;
  const int P = n * h * w;
  const Plan1 p1 = plan1(P, w1.cin, w1.cout, d1.nl ? WG1_CARRYING_MAX : WG1_MAX);
  const Plan3 p3 = plan3(P, w, w3.cin, w3.cout);
  if (!p3.ok || (w1.fold != nullptr) != (w3.fold != nullptr)) return false;
  const Wg1Args A1 = args1(p1, w1, P);
  const Wg3Args A3 = args3(p3, w3, P, h, w);
  const SumArgs a1 = sum_args(s1), a3 = sum_args(s3);
  size_t lds = p1.lds > p3.lds ? p1.lds : p3.lds;
  D1Args D{};
  if (d1.nl) {
    if (d1.B > kDgrad1MaxB) return false;
    D.nl = d1.nl;
    D.nk = (d1.B + 31) / 32;
    D.cols = (d1.ce - (d1.cb & ~15) + 31) / 32;
    D.T = dgrad1_splits(P, d1.ce - d1.cb, most_splits, &D.ppw);
    D.n = D.cols * D.T;
    for (int i = 0; i < 2; ++i) {
      D.db[i] = (const u16*)d1.db[i]; D.W[i] = (const u16*)d1.W[i]; D.mtiles[i] = d1.C16[i] / 16;
      D.fold[i] = d1.fold1[i]; D.part[i] = d1.part[i];
    }
    D.x = (const u16*)d1.x; D.x_ld = d1.x_ld; D.dy = (const u16*)d1.dy; D.G = d1.G; D.ld = d1.ld; D.first = d1.first;
    D.mean = d1.mean; D.istd = d1.istd; D.B = d1.B; D.cb = d1.cb; D.ce = d1.ce; D.P = P;
    *T1 = D.T;
    const size_t need = (size_t)D.nl * 2 * D.nk * 1024 + (size_t)D.nl * 256;  // (the sums' 2 KB reuse it)
    if (need > lds) lds = need;
  }
  const dim3 grid((unsigned)(A1.n + A3.n + D.n + a1.wgs + a3.wgs));
#define DNB_L(MG, MT)                                                                                               \
  do {                                                                                                              \
    if (w1.fold) hipLaunchKernelGGL((k_wgrad_pair<MG, MT, true>), grid, dim3(256), lds, st, A1, A3, a1, a3, D);         \
    else hipLaunchKernelGGL((k_wgrad_pair<MG, MT, false>), grid, dim3(256), lds, st, A1, A3, a1, a3, D);                \
  } while (0)
#define DNB_L2(MG)                                                                                                  \
  switch (p3.mt) { case 1: DNB_L(MG, 1); break; case 2: DNB_L(MG, 2); break; default: DNB_L(MG, 3); break; }
  if (p1.mg == 12) { DNB_L2(12) } else if (p1.mg == 8) { DNB_L2(8) } else { DNB_L2(4) }
#undef DNB_L2
#undef DNB_L
  *s1 = WgradSum{w1.part, w1.dw, 1, p1.S, p1.gy, p1.gz, p1.mg, w1.cin, w1.cout};
  *s3 = WgradSum{w3.part, w3.dw, 9, p3.S, p3.gy, p3.gz, p3.mt, w3.cin, w3.cout};
  return true;
}

}  // namespace nhwc
}  // namespace dnb
