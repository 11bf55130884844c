// Device helpers shared by the kernel files: BN's folded affine map and the deterministic
// merging of (count, mean, M2) partial statistics.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dnb {

// The one place BN's affine map is folded into (scale, shift); forward, recomputation
// and backward all call it so the ReLU mask is reproduced bit for bit.
__device__ __forceinline__ void bn_fold(float gamma, float beta, float mean, float istd,
                                        float& scale, float& shift) {
  scale = __fmul_rn(gamma, istd);
  shift = __fmaf_rn(-mean, scale, beta);
}

__device__ __forceinline__ float bn_istd(float m2, float cnt, float eps) {
  return __fdiv_rn(1.0f, __fsqrt_rn(__fadd_rn(__fdiv_rn(m2, cnt), eps)));
}

template <int CTRL>
__device__ __forceinline__ float row16_from(float v) {  // the value of another lane of the row of 16
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}

// Sum over each row of 16 lanes, every lane gets it: four vector additions whose second operand comes
// from another lane of the row.  The order of additions (and the bits) is that of a butterfly over
// lane distances 1, 2, 4, 8: after two steps the lanes of a quad agree, so the mirrored lane 7 - i holds
// what lane i ^ 4 does, then 15 - i what i ^ 8 does.  That needs every step to round: a product passed in
// must not be fused into the first addition (the lanes of a pair would differ), hence no contraction here.
// Through __shfl_xor each step goes to the LDS crossbar and back; with two such sums per output channel
// that was 3 us of a convolution's launch.
__device__ __forceinline__ float row16_sum(float v) {
#pragma clang fp contract(off)
  v = v + row16_from<0xB1>(v);   // quad_perm [1,0,3,2]
  v = v + row16_from<0x4E>(v);   // quad_perm [2,3,0,1]
  v = v + row16_from<0x141>(v);  // row_half_mirror
  v = v + row16_from<0x140>(v);  // row_mirror
  return v;
}

// Sum of squares over each row of 16 lanes, for the row's lane 0 only.  Lane 0 adds as the butterfly
// does, d0*d0 entering unrounded: ((d0^2 + d1^2) + (d2^2 + d3^2)) + ..., its partners at distances 4 and 8
// taken by rotation (the lanes of a quad differ in the last place here, so a mirrored lane would not do).
__device__ __forceinline__ float row16_sumsq0(float d) {
#pragma clang fp contract(off)
  float v = __fmaf_rn(d, d, row16_from<0xB1>(__fmul_rn(d, d)));
  v = v + row16_from<0x4E>(v);
  v = v + row16_from<0x12C>(v);  // row_ror 12: lane i takes lane i + 4
  v = v + row16_from<0x128>(v);  // row_ror 8
  return v;
}

// Sum over the 64 lanes, the same in every lane.
__device__ __forceinline__ int64_t wave_sum_i64(int64_t v) {
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) v += (int64_t)__shfl_xor((long long)v, off, 64);
  return v;
}

struct Stat3 {
  float c, m, m2;  // count, mean, sum of squared deviations from the mean
};

// Pairwise update: statistics of the union of two disjoint sets (a first, then b).
__device__ __forceinline__ Stat3 stat_combine(Stat3 a, Stat3 b) {
  if (b.c == 0.f) return a;
  if (a.c == 0.f) return b;
  const float tot = __fadd_rn(a.c, b.c), d = __fsub_rn(b.m, a.m);
  Stat3 r;
  r.c = tot;
  r.m = __fmaf_rn(d, __fdiv_rn(b.c, tot), a.m);
  r.m2 = __fadd_rn(__fadd_rn(a.m2, b.m2), __fmul_rn(__fmul_rn(d, d), __fdiv_rn(__fmul_rn(a.c, b.c), tot)));
  return r;
}

// Butterfly over the 64 lanes; both lanes of a pair evaluate combine(lower lane, upper lane),
// so every lane ends with the same bits.
__device__ __forceinline__ Stat3 stat_merge_wave(Stat3 v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    Stat3 o;
    o.c = __shfl_xor(v.c, off, 64); o.m = __shfl_xor(v.m, off, 64); o.m2 = __shfl_xor(v.m2, off, 64);
    v = (lane & off) ? stat_combine(o, v) : stat_combine(v, o);
  }
  return v;
}

// Merges T partials of three floats each, st apart, with the whole workgroup (blockDim a multiple of
// 64, at most 1024): thread t folds partials t, t+blockDim, ... in order, then waves, then the
// per-wave results in wave order.  `sh` needs 3 floats per wave.  Result in every thread.
__device__ __forceinline__ Stat3 stat_merge_block(const float* __restrict__ p, int T, float* sh, int st = 3) {
  Stat3 v{0.f, 0.f, 0.f};
  // four of the thread's partials are requested before the first is folded in (a fold per load
  // would wait out one memory latency per partial); loads past T repeat the last partial and
  // enter as empty sets, which stat_combine passes through unchanged
  const int bd = blockDim.x;
  for (int i = threadIdx.x; i < T; i += 4 * bd) {
    Stat3 o[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int q = min(i + u * bd, T - 1);
      const float* e = p + (int64_t)q * st;
      o[u] = Stat3{e[0], e[1], e[2]};
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (i + u * bd >= T) o[u] = Stat3{0.f, 0.f, 0.f};
      v = stat_combine(v, o[u]);
    }
  }
  v = stat_merge_wave(v);
  const int wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) { sh[3 * wave] = v.c; sh[3 * wave + 1] = v.m; sh[3 * wave + 2] = v.m2; }
  __syncthreads();
  Stat3 r{sh[0], sh[1], sh[2]};
  for (int w = 1; w < nw; ++w) r = stat_combine(r, Stat3{sh[3 * w], sh[3 * w + 1], sh[3 * w + 2]});
  return r;
}


// Where partials of (count, mean, M2) are few they lie [T][C][3], else [C][T][3]: the kernels that merge the few
// have a lane per channel (one of [C][T][3] read 64 cache lines at a time: 18 us for 128 channels x 98).
constexpr int kRowStats = 128;
__host__ __device__ __forceinline__ int64_t stat_at(int T, int C, int t, int ch) {
  return T <= kRowStats ? ((int64_t)t * C + ch) * 3 : ((int64_t)ch * T + t) * 3;
}

// Merging T <= kRowStats partials ([T][C][3]) of many channels inside a kernel, in the order and with the bits of
// stat_merge_block with 256 threads: per 64 partials a balanced tree, then those in order.  The counts (tiles of 64
// pixels of runs of `per` pixels, tpr tiles each) are the same for every channel, so the two quotients of each
// node, the only slow part, are formed once: table[node] = (nb / (na + nb), na * nb / (na + nb)); an empty right side
// is marked by 0.  Threads: table by the first 127; after a barrier thread tid takes channel tid % cap and one of
// Q = NT / cap runs of 64 / Q leaves, to sh[2][NT]; after another the first cap threads finish a channel each.  For
// kernels that fold the BN they apply themselves: a launch of k_bn_fold is two memory latencies and a kernel boundary.
struct StatRuns { int T, per, tpr; };
__device__ __forceinline__ int stat_pixels(const StatRuns& R, int t) {  // of the first t tiles
  t = min(t, R.T);
  return (t / R.tpr) * R.per + min((t % R.tpr) * 64, R.per);
}
__device__ __forceinline__ void stat_table(const StatRuns& R, float2* table, int tid) {
  if (tid >= 127) return;
  int lo = 0, half = 64;  // the node that joins the two groups of 64
  if (tid < 126) {
    int i = tid % 63, n = 32;
    half = 1;
    while (i >= n) { i -= n; n >>= 1; half <<= 1; }
    lo = (tid / 63) * 64 + i * 2 * half;
  }
  const int m = stat_pixels(R, lo + half);
  const float na = (float)(m - stat_pixels(R, lo)), nb = (float)(stat_pixels(R, lo + 2 * half) - m), tot = __fadd_rn(na, nb);
  table[tid] = nb > 0.f ? make_float2(__fdiv_rn(nb, tot), __fdiv_rn(__fmul_rn(na, nb), tot)) : make_float2(0.f, 0.f);
}
__device__ __forceinline__ float2 stat_join(float2 a, float2 b, float2 w) {  // (mean, M2)
  const float d = __fsub_rn(b.x, a.x);
  const float m = __fmaf_rn(d, w.x, a.x), m2 = __fadd_rn(__fadd_rn(a.y, b.y), __fmul_rn(__fmul_rn(d, d), w.y));
  return w.x > 0.f ? make_float2(m, m2) : a;
}
// S leaves a group: 64, or 16 or 32 where T is no more than that (the joins left out meet empty sets only).
template <int Q, int S>
__device__ __forceinline__ void stat_runs(const float* __restrict__ p, int T, int C, int ch, int q, const float2* table,
                                          float2* sh, int NT, int tid) {
  constexpr int L = S / Q;
  for (int w = 0; w < 2; ++w) {
    float2 v[L];
#pragma unroll
    for (int i = 0; i < L; ++i) {
      const float* e = p + ((int64_t)min(w * 64 + q * L + i, T - 1) * C + ch) * 3;
      v[i] = make_float2(e[1], e[2]);
    }
    int off = w * 63;
#pragma unroll
    for (int h = 1; h < L; h <<= 1) {  // pairs h leaves apart
#pragma unroll
      for (int i = 0; i < L; i += 2 * h) v[i] = stat_join(v[i], v[i + h], table[off + (q * L + i) / (2 * h)]);
      off += 32 / h;
    }
    sh[w * NT + tid] = v[0];
    if (T <= 64) break;
  }
}
template <int Q, int S>
__device__ __forceinline__ float2 stat_finish(const float2* sh, int T, const float2* table, int cap, int NT, int ch) {
  float2 g[2];
  for (int w = 0; w < 2; ++w) {
    float2 v[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) v[q] = sh[w * NT + q * cap + ch];
    int off = w * 63 + 64 - 64 / (S / Q);  // the levels above S / Q leaves
#pragma unroll
    for (int h = 1; h < Q; h <<= 1) {
#pragma unroll
      for (int i = 0; i < Q; i += 2 * h) v[i] = stat_join(v[i], v[i + h], table[off + i / (2 * h)]);
      off += 32 / (S / Q) / h;
    }
    if (T <= 64) return v[0];
    if (w == 0) g[0] = v[0]; else g[1] = v[0];
  }
  return stat_join(g[0], g[1], table[126]);
}
template <int Q>
__device__ __forceinline__ void stat_merge_runs(const float* __restrict__ p, int T, int C, int ch, int q, const float2* table,
                                                float2* sh, int NT, int tid) {
  if (T <= 16) stat_runs<Q, 16>(p, T, C, ch, q, table, sh, NT, tid);
  else if (T <= 32) stat_runs<Q, 32>(p, T, C, ch, q, table, sh, NT, tid);
  else stat_runs<Q, 64>(p, T, C, ch, q, table, sh, NT, tid);
}
template <int Q>
__device__ __forceinline__ float2 stat_merge_finish(const float2* sh, int T, const float2* table, int cap, int NT, int ch) {
  return T <= 16 ? stat_finish<Q, 16>(sh, T, table, cap, NT, ch)
         : T <= 32 ? stat_finish<Q, 32>(sh, T, table, cap, NT, ch) : stat_finish<Q, 64>(sh, T, table, cap, NT, ch);
}

// What k_bn_fold does for channels lo..hi-1, given to a kernel that folds by itself.
struct FoldIn {
  const float *gamma, *beta;
  float *mean, *istd;          // of all channels; lo..hi-1 are written by one workgroup
  const float* part; int T;    // partials of lo..hi-1, [T][hi - lo][3] (T <= kRowStats)
  int per, tpr;                // pixels and tiles of 64 pixels of a run of tiles (an image, or all pixels)
  float count;                 // pixels in all
  int lo, hi;
  float eps;
  float2* fold;                // out: folded pairs, by one workgroup
};

// ---- pieces of the fp32 BN+ReLU backward reduction shared by its own kernel and by the launch
// that carries it beside the weight gradients (same code, same bits)

__device__ __forceinline__ float bnb_wave_sum(float v) {
  // butterfly over the 64 lanes of a wavefront: every lane ends with the same total
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Sum over the workgroup; the result is returned to every thread.  `red` holds one
// float per wave.  Safe to call repeatedly (barrier before reuse).
__device__ __forceinline__ float bnb_block_sum(float v, float* red) {
  v = bnb_wave_sum(v);
  const int wave = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[wave] = v;
  __syncthreads();
  float t = 0.f;
  for (int i = 0; i < nw; ++i) t += red[i];
  return t;
}

// rows of hw contiguous floats, one per image: walks (image, vector-in-row) pairs with a stride
// of blockDim threads without a division per element
struct RowIter {
  int img, q, dimg, dq, hwv;
  __device__ __forceinline__ RowIter(int hwv_, int tid, int nthr) : hwv(hwv_) {
    img = tid / hwv_; q = tid - img * hwv_;
    dimg = nthr / hwv_; dq = nthr - dimg * hwv_;
  }
  __device__ __forceinline__ void next() {
    img += dimg; q += dq;
    if (q >= hwv) { q -= hwv; ++img; }
  }
};

// ---- the end of a layer's BN1 in the fp32 backward chain: sums of the partial pairs [ch][T], parameter
// gradients and the running constants K (see dnb_bwd_f32.hip).  Carried by the layer's weight-gradient
// launch; a wave per channel.
struct Bn1Finish {
  int n;                       // layers whose sums these are (two where they shared the pass over the slab)
  const float2* part[2];
  int T, lo, C, wgs;           // C channels from lo on; wgs = 0: nothing to do
  const float *gamma[2], *istd;
  float inv_p;
  float2* K;
  int first;                   // K is set, not added to
  float *dgamma[2], *dbeta[2];
};
template <int N>  // of a layer by itself nothing of a second one is loaded, added or waited for
__device__ __forceinline__ void bn1_finish_layers(const Bn1Finish& A, int wg) {
  const int i = wg * (int)(blockDim.x >> 6) + (int)(threadIdx.x >> 6);
  if (i >= A.C) return;
  const int ch = A.lo + i;
  float2 s[N];
#pragma unroll
  for (int q = 0; q < N; ++q) {
    s[q] = make_float2(0.f, 0.f);
    const float2* p = A.part[q] + (int64_t)i * A.T;
    for (int t = threadIdx.x & 63; t < A.T; t += 64) { const float2 v = p[t]; s[q].x += v.x; s[q].y += v.y; }
  }
#pragma unroll
  for (int q = 0; q < N; ++q) {
    s[q].x = bnb_wave_sum(s[q].x);
    s[q].y = bnb_wave_sum(s[q].y);
  }
  if ((threadIdx.x & 63) == 0) {
    float2 k = A.first ? make_float2(0.f, 0.f) : A.K[ch];
#pragma unroll
    for (int q = 0; q < N; ++q) {
      const float sc = __fmul_rn(A.gamma[q][ch], A.istd[ch]) * A.inv_p;
      k = make_float2(__fmaf_rn(sc, s[q].x, k.x), __fmaf_rn(sc, s[q].y, k.y));
      A.dbeta[q][ch] = s[q].x;
      A.dgamma[q][ch] = s[q].y;
    }
    A.K[ch] = k;
  }
}
__device__ __forceinline__ void bn1_finish_body(const Bn1Finish& A, int wg) {
  if (A.n == 1) bn1_finish_layers<1>(A, wg);
  else bn1_finish_layers<2>(A, wg);
}

struct BnBwdPartialArgs {
  const float* x; int64_t x_stride; const float* dact; int64_t dact_stride;
  int n, hw, ipb;
  const float *gamma, *beta, *mean, *istd;
  float* part;
  int c, splits;  // grid of the reduction: channels x image splits
};

// Workgroup (ch, s): partial sums of dz and dz*xhat over images [s*ipb, (s+1)*ipb) of channel ch,
// 16-byte accesses (hw and the strides multiples of 4, 16-byte aligned), 256 threads.
__device__ __forceinline__ void bn_bwd_partial_body4(const BnBwdPartialArgs& A, int ch, int s) {
  __shared__ float red[4];
  const int n0 = s * A.ipb, ni = min(A.n, n0 + A.ipb) - n0;
  const int hwv = A.hw / 4;
  float scale, shift;
  const float mu = A.mean[ch], is = A.istd[ch];
  bn_fold(A.gamma[ch], A.beta[ch], mu, is, scale, shift);
  const int64_t inner = (int64_t)ch * A.hw;
  const float* xp = A.x + (int64_t)n0 * A.x_stride + inner;
  const float* gp = A.dact + (int64_t)n0 * A.dact_stride + inner;
  float sb = 0.f, sg = 0.f;
  // four positions per pass: all eight loads are issued (unconditionally; a position past the
  // range repeats the last image's) before the first is consumed
  for (RowIter it(hwv, threadIdx.x, blockDim.x); it.img < ni;) {
    float4 t[4], g[4];
    bool ok[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      ok[u] = it.img < ni;
      const int im = ok[u] ? it.img : ni - 1;
      t[u] = *reinterpret_cast<const float4*>(xp + (int64_t)im * A.x_stride + (int64_t)it.q * 4);
      g[u] = *reinterpret_cast<const float4*>(gp + (int64_t)im * A.dact_stride + (int64_t)it.q * 4);
      it.next();
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (ok[u]) {
        const float tv[4] = {t[u].x, t[u].y, t[u].z, t[u].w}, gv[4] = {g[u].x, g[u].y, g[u].z, g[u].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float dz = __fmaf_rn(tv[e], scale, shift) > 0.f ? gv[e] : 0.f;
          sb += dz;
          sg = __fmaf_rn(dz, (tv[e] - mu) * is, sg);
        }
      }
    }
  }
  sb = bnb_block_sum(sb, red);
  sg = bnb_block_sum(sg, red);
  if (threadIdx.x == 0) {
    float* p = A.part + ((int64_t)ch * A.splits + s) * 2;
    p[0] = sb; p[1] = sg;
  }
}

}  // namespace dnb
