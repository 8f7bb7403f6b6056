// Internal interfaces between the convolution front end (conv_api.hip) and its kernel families.
#pragma once
#include "common.h"

struct ConvGeom {
  int N, H, W, Cin, Cout, R, S, stride, pad, Ho, Wo;
};

static inline ConvGeom make_geom(const cnnk_conv_desc* d) {
  ConvGeom g;
  g.N = d->N; g.H = d->H; g.W = d->W; g.Cin = d->Cin; g.Cout = d->Cout;
  g.R = d->R; g.S = d->S; g.stride = d->stride; g.pad = d->pad;
  g.Ho = conv_out(d->H, d->pad, d->R, d->stride);
  g.Wo = conv_out(d->W, d->pad, d->S, d->stride);
  return g;
}

// What a forward kernel does with its fp32 accumulators before it rounds and stores them, for the validation
// pass: an inference-mode batch norm (gamma null: none), a residual added to the rounded value, a ReLU.
// The convolution's own output is then never stored.
struct ConvTail {
  const float* gamma;
  const float* beta;
  const float* mean;
  const float* var;
  float eps;
  const bf16_t* res;   // nullable: same shape as the output
  int relu;
};
// y = act(sc * acc + bi) per channel, the coefficients of channel c
__device__ __forceinline__ void tail_coef(const ConvTail& t, int c, bool ok, float* sc, float* bi) {
  *sc = 1.f;
  *bi = 0.f;
  if (t.gamma && ok) {
    *sc = t.gamma[c] * (1.f / sqrtf(t.var[c] + t.eps));
    *bi = fmaf(-t.mean[c], *sc, t.beta[c]);
  }
}
// one accumulator (16 pixels of one channel) through the batch norm and, unless a residual follows, the ReLU
__device__ __forceinline__ f32x16_t tail_acc(f32x16_t v, float sc, float bi, bool relu) {
  f32x16_t o;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const float t = fmaf(v[r], sc, bi);
    o[r] = relu && !(t > 0.f) ? 0.f : t;
  }
  return o;
}
// residual and ReLU on eight stored channels
__device__ __forceinline__ uint4 tail_residual(const ConvTail& t, uint4 v, uint4 res) {
  float x[8], r[8];
  unpack8(v, x);
  unpack8(res, r);
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    x[e] += r[e];
    if (t.relu) x[e] = x[e] > 0.f ? x[e] : 0.f;
  }
  return uint4{pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(x[4], x[5]), pack_bf16x2(x[6], x[7])};
}

// direct kernels (any shape, both dtypes)
size_t conv_direct_wgrad_ws(const ConvGeom& g);
int conv_direct_fwd(const ConvGeom& g, int dtype, const void* x, const void* w, void* y, hipStream_t st);
int conv_direct_dgrad(const ConvGeom& g, int dtype, const void* dy, const void* w, void* dx, int accumulate,
                      hipStream_t st);
int conv_direct_wgrad(const ConvGeom& g, int dtype, const void* x, const void* dy, float* dw, void* ws,
                      hipStream_t st);
int reduce_partials(const float* part, float* out, int n, int P, hipStream_t st);

// bf16 MFMA implicit-GEMM kernels
bool conv_mfma_supported(const ConvGeom& g, int pass);
size_t conv_mfma_ws(const ConvGeom& g, int pass, bool want_stats);
int conv_mfma_fwd(const ConvGeom& g, const bf16_t* x, const bf16_t* w, bf16_t* y, float* ch_sum,
                  float* ch_sumsq, void* ws, hipStream_t st, const ConvTail* tail = nullptr);
int conv_mfma_dgrad(const ConvGeom& g, const bf16_t* dy, const bf16_t* w, bf16_t* dx, int accumulate,
                    void* ws, hipStream_t st);
int conv_mfma_wgrad(const ConvGeom& g, const bf16_t* x, const bf16_t* dy, float* dw, void* ws,
                    hipStream_t st);
// The same without the final reduction: *part points at *P partial gradients (each Cout*R*S*Cin
// floats; dw itself with *P = 1 when the reduction was not split), for a caller that reduces them
// in its own way.
int conv_mfma_wgrad_partials(const ConvGeom& g, const bf16_t* x, const bf16_t* dy, float* dw, void* ws,
                             const float** part, int* P, hipStream_t st);
// what it runs for all shapes but those of conv_wgrad_patch (conv_wgrad_gemm.hip)
size_t conv_wgrad_gemm_ws(const ConvGeom& g);
int conv_wgrad_gemm(const ConvGeom& g, const bf16_t* x, const bf16_t* dy, float* dw, void* ws, const float** part, int* P,
                    hipStream_t st);

// data gradient with weights already transposed to [Cin][R*S][Cout], and the batched transposition
constexpr int kMaxTranspose = 32;
struct TransposeTable {
  int count;
  int block_begin[kMaxTranspose + 1];
  const bf16_t* src[kMaxTranspose];
  bf16_t* dst[kMaxTranspose];
  int Cout[kMaxTranspose], T[kMaxTranspose], Cin[kMaxTranspose];
};
int conv_transpose_weights_multi(TransposeTable& t, hipStream_t st);
int conv_mfma_dgrad_pt(const ConvGeom& g, const bf16_t* dy, const bf16_t* wt, bf16_t* dx, int accumulate,
                       hipStream_t st);

// implicit GEMM with the operands loaded straight into LDS (conv_gemm.hip); the data gradient takes the weights as
// they are.  stats: [2][Cout][conv_gemm_stat_rows].
bool conv_gemm_supported(const ConvGeom& g, int pass);
int conv_gemm_stat_rows(const ConvGeom& g);
int conv_gemm_fwd(const ConvGeom& g, const bf16_t* x, const bf16_t* w, bf16_t* y, float* stats, hipStream_t st, const ConvTail* tail);
int conv_gemm_dgrad(const ConvGeom& g, const bf16_t* dy, const bf16_t* w, bf16_t* dx, int accumulate, hipStream_t st);

// 3x3 stride-1 kernels with the input patch resident in LDS (forward, data gradient)
bool conv_patch_supported(const ConvGeom& g, int pass);
int conv_patch_stat_rows(const ConvGeom& g);
int conv_patch_fwd(const ConvGeom& g, const bf16_t* x, const bf16_t* w, bf16_t* y, float* stats, hipStream_t st,
                   const ConvTail* tail = nullptr);
int conv_patch_dgrad(const ConvGeom& g, const bf16_t* dy, const bf16_t* wt, bf16_t* dx, int accumulate,
                     hipStream_t st);

// 3x3 stride-1 weight gradient from LDS patches with transposing LDS loads
bool conv_wgrad_patch_supported(const ConvGeom& g);
size_t conv_wgrad_patch_ws(const ConvGeom& g);
int conv_wgrad_patch(const ConvGeom& g, const bf16_t* x, const bf16_t* dy, float* dw, void* ws, hipStream_t st);
// the same partial sums with the operand tiles loaded straight into LDS (conv_wgrad_dma.hip)
int conv_wgrad_dma_launch(const ConvGeom& g, const bf16_t* x, const bf16_t* dy, float* part, int TI, int TH, int ctiles,
                          int tiles_per_block, int mtiles, int nw, int otiles, int splits, hipStream_t st);

// fewer than 8 input channels: zero-pad to 8 in the workspace, then the MFMA kernels
bool conv_pad_supported(const ConvGeom& g);
size_t conv_pad_ws(const ConvGeom& g, int pass, bool want_stats);
int conv_pad_fwd(const ConvGeom& g, const bf16_t* x, const bf16_t* w, bf16_t* y, float* ch_sum, float* ch_sumsq,
                 void* ws, hipStream_t st, const ConvTail* tail = nullptr);
int conv_pad_wgrad(const ConvGeom& g, const bf16_t* x, const bf16_t* dy, float* dw, void* ws, hipStream_t st);
// Hook 1 of 4 (see "Hooks between cnnk_train_step and the convolution entry points" below).
// The forward and the weight-gradient call of such a layer both need the 8-channel copy of x.  When
// set (per host thread), the forward call writes it to buf and sets valid, and a weight-gradient
// call that finds valid set reads it there instead of padding x again (the caller vouches that x
// and buf are unchanged in between).
size_t conv_pad_x8_bytes(const ConvGeom& g);
struct X8Cache {
  bf16_t* buf;
  bool valid;
};
extern thread_local X8Cache* t_cnnk_x8_cache;

// first layer (3 input channels, 3x3, stride 1, pad 1, at most 64 output channels): forward on MFMA
// without operand staging
bool conv_first_supported(const ConvGeom& g);
size_t conv_first_ws(const ConvGeom& g);
int conv_first_fwd(const ConvGeom& g, const bf16_t* x, const bf16_t* w, bf16_t* y, float* ch_sum, float* ch_sumsq,
                   void* ws, hipStream_t st, const ConvTail* tail = nullptr);
bool conv_first_wgrad_supported(const ConvGeom& g);   // additionally W % 16 == 0
size_t conv_first_wgrad_ws(const ConvGeom& g);
int conv_first_wgrad(const ConvGeom& g, const bf16_t* x, const bf16_t* dy, float* dw, void* ws, hipStream_t st);

// ch_sum[c] = sum_b part[b][0][c], ch_sumsq[c] = sum_b part[b][1][c]  (double accumulation)
int channel_sums_finalize(const float* part, int nb, int C, float* ch_sum, float* ch_sumsq, hipStream_t st);

// ---- Hooks between cnnk_train_step and the convolution entry points -----------------------------
// cnnk_train_step calls the public entry points (cnnk_conv2d_fwd / _wgrad) and passes four extra
// pieces of context through the per-thread pointers below (t_cnnk_x8_cache above, t_cnnk_sgd_fuse,
// t_cnnk_wgrad_cus, t_cnnk_part_sums).  Contract, the same for all four: the step sets the pointer immediately
// before ONE entry-point call on the same host thread and resets it to its neutral value (nullptr /
// 256) right after that call returns, whatever the call's status.  Hooks 1 to 3 are read once, at the entry point's
// entry; hook 4 is read where a forward path adds up its channel sums, by its last launch helper (channel_sums_finalize,
// called at most once and with the workspace left alone from there on).  Outside cnnk_train_step the values are always neutral, so a direct caller of the C ABI
// never sees them, and calls from other host threads are unaffected (thread_local).  The library
// keeps no other state between calls except two process-wide tables that are written once or by
// an explicit call: the "dynamic LDS size already raised" flag of each kernel launcher (set on the
// first launch; harmless to set twice, so unsynchronised first launches from two threads are
// benign) and the cnnk_tune table (explicitly documented as not thread-safe).
//
// Hook 2 of 4.  When set (per host thread), the next split-K reduction of a weight gradient also applies the
// SGD-momentum update of that parameter in the same launch (out = sum of partials is still
// written as the gradient): g' = g + wd*w; v <- mu*v + g'; w <- w - lr*v; optional bf16 copy.
// wait (nullable): an event the stream waits for between the weight-gradient kernel and the
// reduction (the last reader of the old weights).  done is set when the fused launch was made;
// callers fall back to a separate update otherwise (unsplit reductions, other reducers).
// group (nullable): instead of being launched, the reduction and its update are appended to the group (while it has
// room; done is set all the same), whose one launch the step makes later; the partial sums stay until then.
constexpr int kReduceGroup = 16;
struct ReduceItem {
  const float* part;
  float* out;
  float* w;
  float* v;
  bf16_t* wlp;
  int n, P, block0;
};
struct ReduceGroup {
  int count;
  float lr, mu, wd;
  ReduceItem it[kReduceGroup];
};
int reduce_group(ReduceGroup& g, hipStream_t st);
struct SgdFuse {
  float* w;
  float* v;
  void* wlp;
  float lr, mu, wd;
  hipEvent_t wait;
  bool done;
  ReduceGroup* group;
};
extern thread_local SgdFuse* t_cnnk_sgd_fuse;

constexpr int kTuneKeys = 24;
extern int g_cnnk_tune[kTuneKeys];
// Hook 3 of 4.  Compute units the weight-gradient kernels size their grids for (256 = the whole device).  The
// training step lowers it for the weight gradients it runs on its second stream, beside the rest
// of the backward pass: fewer, longer-lived workgroups leave the other stream room to run.
// Workspace sizes are always computed for the whole device (the upper bound).
extern thread_local int t_cnnk_wgrad_cus;

// Hook 4 of 4.  When set, a forward convolution whose batch norm is the very next call on the same stream and workspace may leave
// its per-channel sums as partials part[2][C][nb] in the workspace (nb > 0) instead of adding them up in a launch of its own.
// They have to stay there until the batch norm's launch: nothing else may be enqueued on that workspace in between.
struct PartSums {
  const float* part;
  int nb;
  bool shifted;        // of add_stats: relative to the first row, any nb
};
extern thread_local PartSums* t_cnnk_part_sums;
// whether passes over 64 channels of every row, which is how partials are consumed, pay for m rows of C channels
bool bn_slabs_pay_for(size_t m, int C);

// Forward convolution with a tail (no per-channel sums), for the shapes a matrix-core kernel takes
// (conv_tail_supported); CNNK_ERR_UNSUPPORTED, and nothing launched, for the others.
bool conv_tail_supported(const cnnk_conv_desc* d);
int conv_fwd_tail(const cnnk_conv_desc* d, const void* x, const void* w, void* y, const ConvTail& tail, void* ws,
                  size_t ws_bytes, hipStream_t st);

// cnnk_bn_relu_fwd / _bwd with the ReLU mask kept from one to the other: a bit per element (NHWC order, the lowest bit
// of a byte first), m * C / 8 bytes.  Backward: with a mask, y is not read and may be null.  partials (nullable): where its nb is not
// 0 they stand in for ch_sum and ch_sumsq, whose contents are then not read.
int bn_relu_fwd(const cnnk_bn_desc* d, const void* x, const void* residual, const float* gamma, const float* beta, void* y,
                unsigned char* mask, float* save_mean, float* save_invstd, float* running_mean, float* running_var,
                const float* ch_sum, const float* ch_sumsq, const PartSums* partials, void* ws, size_t ws_bytes, void* stream);
int bn_relu_bwd(const cnnk_bn_desc* d, const void* dy, const void* x, const void* y, const unsigned char* mask, const float* gamma,
                const float* beta, const float* save_mean, const float* save_invstd, void* dx, void* dresidual, int flags,
                float* dgamma, float* dbeta, void* ws, size_t ws_bytes, void* stream);

// per-channel sum / sum of squares of a tensor with C channels (used when the conv kernel
// itself does not produce them)
size_t channel_stats_ws(size_t m, int C);
// y = a + b with the partial sums that the batch norm of y, the very next call, begins with (channel_stats_ws bytes of ws), and whether
// that is faster than the two passes
bool add_stats_pays(int dtype, size_t m, int C);
int add_stats(int dtype, const void* a, const void* b, void* y, size_t m, int C, PartSums* out, void* ws, hipStream_t st);
// d0 = src and d1 = src, or += where acc0, acc1 say so: cnnk_grad_route to two different tensors with one read
int grad_route2(size_t n, int dtype, const void* src, void* d0, int acc0, void* d1, int acc1, hipStream_t st);
int channel_stats(int dtype, const void* x, size_t m, int C, float* ch_sum, float* ch_sumsq, void* ws,
                  hipStream_t st);
