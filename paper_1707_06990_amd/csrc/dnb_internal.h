// Internal declarations shared by the host orchestration and the kernel files of
// the dense-block library (fp32 NCHW path).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/dnb.h"

struct dnb_block;

namespace dnb {

// dnb_block_create for a caller that has `spare` bytes anyway for the scratch that starts at block_tail_offset
int block_create(const dnb_block_desc* desc, size_t spare, dnb_block** out);

// (dnb_block.hip) where a block's call-local scratch starts in its workspace, and moving it elsewhere
size_t block_tail_offset(const dnb_block* b);
bool block_layers_in_pairs(const dnb_block* b);
void block_move_tail(dnb_block* b, size_t to);

// ---- element-wise and reduction kernels (HBM-bound) -------------------------------------

// dst[i][0:len] = src[i][0:len] for i < n; strides in elements.
hipError_t launch_copy_slab(const float* src, int64_t src_stride, float* dst, int64_t dst_stride,
                            int n, int64_t len, hipStream_t st);

// Per-channel batch statistics of x (n, c, hw; image stride `stride`): mean and
// 1/sqrt(biased var + eps).  The reduction is split over image ranges: launch_bn_stats_partial
// writes (count, mean, M2) per (channel, split) -- bn_stats_partial_floats(n, c, hw) floats --
// and the first kernel that needs the statistics merges them (StatsSrc below), so the forward
// chain has no separate finalisation launch.  launch_bn_stats = partials + a finalise kernel.
size_t bn_stats_partial_floats(int n, int c, int hw);
hipError_t launch_bn_stats_partial(const float* x, int64_t stride, int n, int c, int hw,
                                   float* partials, int* splits, hipStream_t st);
hipError_t launch_bn_stats(const float* x, int64_t stride, int n, int c, int hw, float eps,
                           float* mean, float* istd, float* partials, hipStream_t st);

// Where a kernel finds BN statistics: finalised arrays indexed by channel, except channels in
// [fresh_lo, fresh_hi), whose partials (index ch - fresh_lo) it merges itself and stores back.
struct StatsSrc {
  float* mean;
  float* istd;
  const float* part;
  int splits, fresh_lo, fresh_hi;
  float eps;
};

// out = max(0, fma(x, gamma*istd, beta - mean*gamma*istd)); if copy_out != nullptr the raw x
// is also written there (concatenation and BN+ReLU of the same data in one pass).
hipError_t launch_bn_relu(const float* x, int64_t x_stride, float* out, int64_t out_stride,
                          float* copy_out, int64_t copy_stride, int n, int c, int hw,
                          const float* gamma, const float* beta, StatsSrc s, hipStream_t st);

// Two of them with finished statistics in one launch: a with its copy, b without.
hipError_t launch_bn_relu_two(const float* xa, int64_t xa_stride, float* outa, int64_t outa_stride, float* copya,
                              int64_t copya_stride, int ca, const float* gammaa, const float* betaa, float* meana, float* istda,
                              const float* xb, int64_t xb_stride, float* outb, int64_t outb_stride, int cb,
                              const float* gammab, const float* betab, float* meanb, float* istdb, int n, int hw, hipStream_t st);

// BN+ReLU backward.  Pass 1 reduces dbeta = sum dz, dgamma = sum dz*xhat with
// dz = dact * [fma(x,scale,shift) > 0]; pass 2 writes
// du = gamma*istd*(dz - dbeta/P - xhat*dgamma/P), overwriting or accumulating.
// `partials` needs bn_bwd_partial_floats(n, c, hw) floats.
size_t bn_bwd_partial_floats(int n, int c, int hw);
// Describes the reduction pass (passes & 1) of launch_bn_relu_bwd for another launch to carry
// (launch_conv_wgrad_pair); false when the 16-byte form does not apply to these operands.
struct BnBwdPartialArgs;
struct PendingSum;
bool bn_bwd_partial_plan(const float* x, int64_t x_stride, const float* dact, int64_t dact_stride, int n, int c,
                         int hw, const float* gamma, const float* beta, const float* mean, const float* istd,
                         float* partials, BnBwdPartialArgs* out);
hipError_t launch_bn_relu_bwd(const float* x, int64_t x_stride, const float* dact,
                              int64_t dact_stride, float* du, int64_t du_stride, bool accumulate,
                              int n, int c, int hw, const float* gamma, const float* beta,
                              const float* mean, const float* istd, float* dgamma, float* dbeta,
                              float* partials, hipStream_t st, int passes = 3 /*1 reduce | 2 apply*/,
                              hipEvent_t ev_start = nullptr, hipEvent_t ev_stop = nullptr,
                              PendingSum* absorb = nullptr /*a pending sum for the reduction to carry; cleared*/);

// The element-wise pass alone, from `psplits` partial pairs per channel in [c][psplits] order.
hipError_t launch_bn_bwd_apply(const float* x, int64_t x_stride, const float* dact, int64_t dact_stride, float* du,
                               int64_t du_stride, int n, int c, int hw, const float* gamma, const float* beta,
                               const float* mean, const float* istd, float* dgamma, float* dbeta, const float* partials,
                               int psplits, hipStream_t st);

// One bottleneck layer of the fp32 backward chain (dnb_conv_f32_fast.hip: the 3x3; dnb_bwd_f32.hip: the
// rest).  c = C_l input channels; image strides in elements.
struct Bwd32Layer {
  int n, h, w, c, k, B;
  bool last;                             // l = m: the slab is not written yet, dy stands in for it
  const float *y, *dy; int64_t ys;       // features and gradient of the output
  const float* x; int64_t x_stride;      // concatenated input of the layer: y in place, or storage 1
  const float* b;                        // b_l
  float *G, *gl, *db;                    // slab (stride ys), corrected slice [n][k][hw], gradient of b_l
  const float *pk1t, *pk3t;              // packed data-gradient weights
  const float *g1, *b1, *g2, *b2;
  const float *mean_y, *istd_y, *mean_b, *istd_b;
  float *dgamma1, *dbeta1;
  float2 *part1, *part2, *K;
  // what bwd32_dgrad1 and bwd32_bn1_finish take: channels lo..c-1 (c: of the slice's upper end) of a layer of cw
  // channels, by itself or (up_db) with the layer above, whose c + k channels include these
  int lo, cw;
  bool first;                            // nothing has been added to these channels of the slab yet
  const float *up_db, *up_pk1t, *up_g1, *up_b1;
  float *up_dgamma1, *up_dbeta1;
};
bool bwd32_pair_ok(int n, int hw, int c, int B);
bool bwd32_ok(int n, int h, int w, int k, int B);
size_t bwd32_partial1_floats(int n, int hw, int c);       // of a layer by itself
size_t bwd32_partial1_pair_floats(int n, int hw, int c);  // of two layers in one pass
size_t bwd32_partial1_near_floats(int n, int hw, int k);  // of a pair's k channels between its layers
size_t bwd32_partial2_floats(int n, int h, int w, int k, int B);
int bwd32_dgrad1_splits(int n, int hw, int c);
// 3x3 data gradient of the corrected slice, masked by BN2's ReLU, with BN2's sums.  *T2: partial pairs per channel.
hipError_t bwd32_dgrad3(const Bwd32Layer& L, int* T2, hipStream_t st);
// 1x1 data gradient, BN1 backward and concat backward into the slab
hipError_t bwd32_dgrad1(const Bwd32Layer& L, hipStream_t st);
// the end of the layer's BN1, for launch_conv_wgrad_pair to carry (or launch_bn1_finish on its own)
struct Bn1Finish;
void bwd32_bn1_finish(const Bwd32Layer& L, Bn1Finish* out);
hipError_t launch_bn1_finish(const Bn1Finish& f, hipStream_t st);
// gradient of the block input, after every layer's BN1 is finished
hipError_t bwd32_dx0(const Bwd32Layer& L, float* dx0, hipStream_t st);

// out[(img*c + ch)*hw + q] = 1 if fma(u[img*stride + ch*hw + q], scale, shift) > 0 else 0, with
// (scale, shift) = bn_fold(gamma, beta, mean, istd): the ReLU decision exactly as every kernel takes it.
hipError_t launch_relu_decisions(const float* u, int64_t stride, int n, int c, int hw, const float* gamma,
                                 const float* beta, const float* mean, const float* istd, unsigned char* out,
                                 hipStream_t st);

// the same for a bf16 tensor of P rows of c channels (pixel stride ld): out[p*c + ch]
hipError_t launch_relu_decisions_rows(const void* u, int64_t ld, int64_t P, int c, const float* gamma, const float* beta,
                                      const float* mean, const float* istd, unsigned char* out, hipStream_t st);

// ---- the classifier head of the network steps (fp32): linear + mean softmax cross-entropy, and its backward
hipError_t launch_head_forward(const float* pooled, const float* wl, const float* bl, const int32_t* labels, float* logits,
                               float* dlogits, float* terms, float* loss, int n, int c, int classes, hipStream_t st);
hipError_t launch_head_backward(const float* dlogits, const float* pooled, const float* wl, float* dpooled, float* dwl,
                                float* dbl, int n, int c, int classes, hipStream_t st);

// ---- convolutions (MFMA implicit GEMM, fp32) -----------------------------------------------

// Weight addressing for the implicit-GEMM kernel: element (m = output channel, c = input
// channel, t = tap) lives at w[m*sm + c*sc + (flip ? taps-1-t : t)].
struct WeightView {
  const float* w;
  int64_t sm, sc;
  int flip;
};

// Packed weights for the fast kernels: [taps][cout16 x cin16], zero padded to multiples of 16,
// in fragment order (see dnb_conv_f32_fast.hip).
size_t packed_weight_floats(int cout, int cin, int taps);
hipError_t launch_pack_weights(WeightView wv, int cout, int cin, int taps, float* packed, hipStream_t st);
// All layers of a block in one launch.  Layer l (input width c) occupies packed_layer_floats
// floats: 1x1 forward [B16][c16], 1x1 dgrad [c16][B16], 3x3 forward [9][k16][B16],
// 3x3 dgrad [9][B16][k16], in that order.
size_t packed_layer_floats(int c, int k, int B);
hipError_t launch_pack_block_weights(const float* params, float* packed, int c0, int k, int B, int m,
                                     hipStream_t st);

// out[n][m][q] = sum_{c,t} W(m,c,t) * in[n][c][q + shift(t)], zero outside the image.
// taps = 1 or 9.  Used for forward (W = OIHW as is) and data gradient (transposed, flipped).
// `packed` (may be null) is the same weight view packed by launch_pack_weights; with it, shapes
// whose pixel counts and strides are multiples of 4 take the fast kernels.
// Optional extras of the fast kernels:
//   fold        BN+ReLU prologue: the input is max(0, fma(x, fold[c].x, fold[c].y)) (fast path only)
//   stats_part  epilogue statistics of the output: [cout][stats_T][3] partials (count, mean, M2),
//               conv_stats_partial_floats floats; stats_T is set by the launcher
//   used_fast   set by the launcher; false = generic kernel ran, no statistics were written
//   ev_start / ev_stop  optional events stamped at the fast kernel's own start and end
struct ConvExtras {
  const float2* fold;
  float* stats_part;
  int stats_T;
  bool used_fast;
  hipEvent_t ev_start = nullptr, ev_stop = nullptr;
};
size_t conv_stats_partial_floats(int n, int cout, int h, int w);
hipError_t launch_conv_igemm(const float* in, int64_t in_stride, WeightView wv, const float* packed,
                             float* out, int64_t out_stride, int n, int cin, int cout, int h, int w,
                             int taps, ConvExtras* ex, hipStream_t st);
// whether the any-shape kernels (forward, data gradient, weight gradient) have LDS for this shape: they
// are the fallback wherever an operand is not 16-byte friendly, so a plan must not count on the fast ones
bool conv3x3_generic_fits(int n, int cin, int cout, int h, int w);
bool conv_fast_ok(const float* in, int64_t in_stride, const float* out, int64_t out_stride, int h,
                  int w, int taps);

// fold[ch] = BN's affine map folded to (scale, shift) for nch channels; channels in
// [fresh_lo, fresh_hi) are first finalised from their [T][3] partial statistics.
hipError_t launch_bn_fold(const float* gamma, const float* beta, float* mean, float* istd,
                          const float* part, int T, int fresh_lo, int fresh_hi, float eps, int nch,
                          float2* fold, hipStream_t st, bool rows = false);

// dW[m][c][t] = sum_{n,q} g[n][m][q] * in[n][c][q + shift(t)]  (OIHW result).
// alone: the launch holds nothing else; most: floats that the partials of a 1x1 may take where fewer will do (0: the fewest).
// The launch is to be given the same two.
size_t conv_wgrad_partial_floats(int n, int cin, int cout, int h, int w, int taps, bool alone = false, size_t most = SIZE_MAX);
// partial floats of the fast (16-byte-vector) weight-gradient kernel for this shape, 0 if its tile plan does not fit
size_t conv_wgrad_fast_partial_floats(int n, int cin, int cout, int h, int w, int taps, bool alone = false, size_t most = SIZE_MAX);
// A sum of weight-gradient partials that a launch has left for later.  In a chain of weight
// gradients on one stream the next weight-gradient launch carries it out with extra workgroups
// (the partials are complete when that launch starts), which saves a launch per layer; what is
// left at the end of the chain is summed by launch_pending_sum.
struct PendingSum {
  int kind = 0;  // 0 nothing pending; 1 out[e] = sum_s part[s][e]; 2 the 3x3 fast kernel's accumulator-order partials
  const float* part = nullptr;
  float* out = nullptr;
  int splits = 0;
  int64_t count = 0;                                      // elements of one partial
  int gy = 0, gz = 0, mtw = 0, ctw = 0, cin = 0, cout = 0;  // kind 2: how a partial maps to OIHW
};
hipError_t launch_pending_sum(PendingSum* p, hipStream_t st);  // no-op for kind 0; clears *p
// fold != null applies the BN+ReLU prologue to `in` (fast path only).
// absorb: a pending sum (of another partial buffer) to carry out in this launch, or before it
// when the fast path does not apply; cleared.  defer: if given, this call's own sum is not
// launched when it can be deferred and is described there instead (kind 0 if it was launched).
hipError_t launch_conv_wgrad(const float* in, int64_t in_stride, const float* g, int64_t g_stride,
                             float* dw, int n, int cin, int cout, int h, int w, int taps,
                             float* partials, const float2* fold, hipStream_t st, hipEvent_t ev_start = nullptr,
                             hipEvent_t ev_stop = nullptr /*stamped around the fast kernel (not the sum)*/,
                             bool* used_fast = nullptr, PendingSum* absorb = nullptr, PendingSum* defer = nullptr, bool alone = false,
                             size_t most = SIZE_MAX);

// Both weight gradients of a bottleneck layer on one stream: the 1x1 (in1: C_l channels, g1: the
// gradient of b_l, B channels) and the 3x3 (in3: B channels, g3: the gradient of x_l, k
// channels).  One launch when the fast pair applies, else two launch_conv_wgrad calls.  *pend1 /
// *pend3: in, the previous layer's pending sums (carried out here); out, this layer's.
struct Bn1Finish;
hipError_t launch_conv_wgrad_pair(const float* in1, int64_t in1_stride, const float* g1, int64_t g1_stride,
                                  float* dw1, int cin1, float* part1, const float2* fold1, const float* in3,
                                  int64_t in3_stride, const float* g3, int64_t g3_stride, float* dw3, int cout3,
                                  float* part3, const float2* fold3, int n, int B, int h, int w, hipStream_t st,
                                  PendingSum* pend1, PendingSum* pend3, const BnBwdPartialArgs* bn = nullptr,
                                  bool* bn_done = nullptr, hipEvent_t ev_start = nullptr, hipEvent_t ev_stop = nullptr,
                                  bool* paired = nullptr, const Bn1Finish* fin = nullptr, size_t most1 = SIZE_MAX);
// (fin: the end of a layer's BN1, always carried out;  most1: floats that the 1x1's partials may take;
//  bn: a BN backward reduction to carry in the same launch, *bn_done says whether it was;
//  ev_start / ev_stop are stamped around the shared launch, *paired says whether there was one)

// out[e] = sum over splits of partials[split][e] (fixed order).
hipError_t launch_sum_partials(const float* partials, int splits, int64_t count, float* out, hipStream_t st);

// ---- bf16 / NHWC path (dnb_nhwc_bf16.hip): feature maps bf16 with channels contiguous, row
// strides ("ld") in elements; parameters, statistics, gradient slab and partials fp32.
struct FoldIn;
namespace nhwc {
hipError_t copy_rows(const void* src, int64_t sld, void* dst, int64_t dld, int64_t P, int c, hipStream_t st);
// out = bf16(max(0, fma(x, fold.x, fold.y))) per channel; copy (may be null) = x  (storage 2 / storage 1)
struct BnReluRows { const void* x; int64_t ld; const float2* fold; void* out; int64_t old; void* copy; int64_t cld; int c; };
hipError_t bn_relu_rows(const BnReluRows& a, const BnReluRows* b /* null, or a second in the same launch */, int64_t P, hipStream_t st);
size_t stats_partial_floats(int64_t P, int c);
hipError_t stats_partial(const void* x, int64_t ld, int64_t P, int c, float* part, int* T, hipStream_t st);
// per layer, in order: 1x1 forward [B16][c32], 1x1 dgrad [c16][B32], 3x3 forward [9][k16][B32],
// 3x3 dgrad [9][B16][k32]  (bf16 elements; 16 / 32 = rounded up to that multiple)
size_t packed_layer_elems(int c, int k, int B);
hipError_t pack_block_weights(const float* params, void* packed, int c0, int k, int B, int m, hipStream_t st);
size_t packed_weight_elems(int cout, int cin, int taps);
hipError_t pack_weights(WeightView wv, int cout, int cin, int taps, void* packed, hipStream_t st);
size_t conv_stats_partial_floats(int n, int cout, int h, int w);
hipError_t conv(const void* in, int64_t in_ld, bool in_f32, const void* Wp, void* out, int64_t out_ld, int n,
                int cin, int cout, int h, int w, int taps, const float2* fold, float* spart, int* sT,
                hipStream_t st);
// (dnb_nhwc_conv1.hip) The 1x1 with statistics of its output, few pixels; false (nothing launched) if the shape is not taken.
// F (may be null): the BN of the input is folded by the kernel itself (fold is then an output).
bool conv1_stats(const void* in, int64_t in_ld, const void* Wp, void* out, int64_t out_ld, int64_t P, int cin, int cout,
                 const float2* fold, float* spart, int* sT, const FoldIn* F, hipStream_t st);
// (dnb_nhwc_conv3.hip) The 3x3 with statistics of its output; false (nothing launched) if the shape is not taken.
bool conv3_stats(const void* in, int64_t in_ld, const void* Wp, void* out, int64_t out_ld, int n, int cin, int cout, int h, int w,
                 const float2* fold, float* spart, int* sT, const FoldIn* F, hipStream_t st);
// One weight gradient: dw[m][c][t] = sum_p g[p][m] * act(a[p + shift(t)][c]), fold = BN+ReLU of a (or null).
struct WgradIn {
  const void* a; int64_t a_ld;
  const void* g; int64_t g_ld;
  float *part, *dw;
  int cin, cout;
  const float2* fold;
};
// The sum of a launch's partials, left for a later launch on the same stream (taps 0: nothing pending).
struct WgradSum {
  const float* part;
  float* out;
  int taps, S, gy, gz, mt, cin, cout;
};
// (dnb_nhwc_wgrad.hip) Partial floats of the kernels there, 0 if they do not take the shape.
size_t wgrad_fast_partial_floats(int n, int cin, int cout, int h, int w, int taps, bool carrying);
// Launches the partials and describes their sum in *own; false (nothing launched) if the shape is not taken.
bool wgrad_fast(const WgradIn& in, bool g_f32, int n, int h, int w, int taps, WgradSum* own, hipStream_t st);
// 1x1 data gradient with BN1 + concat backward on channels cb..ce-1, for one layer or for two at once (layer 0 the
// upper one): partial sums [T][ce - cb] per layer.
struct Dgrad1In {
  int nl;                        // layers, 0: nothing to do
  const void *db[2], *W[2];      // gradient of b_l [P][B]; packed weights [C16][B32]
  int C16[2];
  const float2* fold1[2];
  float2* part[2];
  const void* x; int64_t x_ld;   // concatenated features
  const void* dy; float* G; int64_t ld;  // the slab; dy replaces its first read
  bool first;
  const float *mean, *istd;      // of y's channels
  int B, cb, ce;
};
// ... carried by the weight-gradient launch if B <= dgrad1_max_b; pixel splits T and pixels per wave
constexpr int kDgrad1MaxB = 256;
int dgrad1_splits(int64_t P, int C, int most, int* ppw);
// A layer's 1x1 and 3x3 weight gradients in one launch (bf16 gradient operands).  *s1 / *s3: in, the sums
// pending from the layer before (of other partial buffers), carried out in this launch; out, this layer's.
// d1: a data gradient carried beside them (nl 0: none); *T1 = its splits.
bool wgrad_pair(const WgradIn& w1, const WgradIn& w3, int n, int h, int w, WgradSum* s1, WgradSum* s3, const Dgrad1In& d1,
                int most_splits, int* T1, hipStream_t st);
// Carries out what is pending (either may be null).
hipError_t wgrad_finish(WgradSum* s1, WgradSum* s3, hipStream_t st);
size_t wgrad_partial_floats(int n, int cin, int cout, int h, int w, int taps, bool carrying = false);  // carrying: of wgrad_pair with a data gradient
// writes per-split partials to `part` and their sum to dw ([cout][cin][taps])
hipError_t wgrad(const void* a, int64_t a_ld, const void* g, int64_t g_ld, bool g_f32, float* part, float* dw, int n,
                 int cin, int cout, int h, int w, int taps, const float2* fold, hipStream_t st);
size_t bn_bwd_partial_floats(int64_t P, int c);
hipError_t bn_relu_bwd(const void* x, int64_t x_ld, const void* dact, int64_t d_ld, void* du_bf, int64_t du_ld,
                       float* G, int64_t g_ld, int64_t P, int c, const float* gamma, const float* beta,
                       const float* mean, const float* istd, float* dgamma, float* dbeta, float* part,
                       hipStream_t st);

// BN1 sums still to be turned into parameter gradients and K0 / K1: of one layer or two, over channels
// base .. base + width - 1, partials [T][width] each.  n = 0: none.
struct BwdSums {
  int n, T, width, base;
  const float2* part[2];
  const float2* fold1[2];
  float *dgamma[2], *dbeta[2];
};
// One layer of the backward chain (dnb_nhwc_bwd.hip).  c = C_l input channels, ld = C_out.
struct BwdLayer {
  int n, h, w, c, k, B;
  int64_t ld;
  bool last;                     // l = m: the slab is not written yet, dy stands in for it
  bool K_set;                    // K0 / K1 hold something
  BwdSums above;                 // the sums the launches since the last dgrad3 left
  const void *y, *dy, *b;        // features, gradient of the output, b_l
  const void* x; int64_t x_ld;   // concatenated input of the layer: y in place, or storage 1
  float* G;                      // gradient slab
  void *gl, *db;                 // g_l in bf16 [P][k] (l < m), gradient of b_l [P][B]
  const void *pk1t, *pk3t;       // packed data-gradient weights
  const float2 *fold1, *fold2;
  const float *mean_y, *istd_y, *mean_b, *istd_b;
  float *dgamma1, *dbeta1, *dgamma2, *dbeta2;
  float* part2;                  // partial sums of BN2
  float2* K;                     // per channel of y: K0, K1
};
// partial sums of BN1: of one layer or two over C channels; of a pair's upper layer over the lower one's k
size_t bwd_partial1_floats(int64_t P, int C, int layers);
size_t bwd_partial1_near_floats(int64_t P, int k);
int bwd_near_splits();  // most splits of the latter, of the former
int bwd_far_splits();
size_t bwd_partial2_floats(int n, int h, int w, int k, int B);
// 3x3 data gradient and BN2 backward: db, g_l, BN2's parameter gradients, and what L.above holds
hipError_t bwd_dgrad3(const BwdLayer& L, hipStream_t st);
// B > kDgrad1MaxB: 1x1 data gradient, BN1 backward and concat backward into the slab, one layer; *T = splits
hipError_t bwd_dgrad1(const BwdLayer& L, float2* part, int* T, hipStream_t st);
// gradient of the block input and the last BN1 sums (L.above over exactly its channels)
hipError_t bwd_dx0(const BwdLayer& L, void* dx0, hipStream_t st);
}  // namespace nhwc

}  // namespace dnb
