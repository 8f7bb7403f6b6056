// cnnk_vit_train_step: one training step of a pre-norm Vision Transformer classifier on one device
// (Section IV-A's second model; Algorithm 1's inner loop: forward pass, loss, backward pass, update).
// Host code: the order of the calls, the layout of the arena, the parameter table.  Everything runs
// through the entry points of cnnk_vit.h (and the classifier head and the residual sums through
// cnnk_fc_softmax_xent / cnnk_add of cnnk.h).
#include <stdio.h>
#include <string.h>
#include "common.h"
#include "sgd.h"
#include "gemm.h"
#include "vit.h"
#include "../../include/cnnk_vit.h"

int cnnk_fill_zero(void* p, size_t bytes, hipStream_t st);   // vit_ops.hip

namespace {
enum { P_WE = 0, P_BE, P_CLS, P_POS, P_BLOCK0 };                          // model parameters
enum { B_G1 = 0, B_B1, B_WQKV, B_BQKV, B_WO, B_BO, B_G2, B_B2, B_W1, B_C1, B_W2, B_C2, B_COUNT };
// internal tensors of the arena behind the public ones
enum { X_Z0 = CNNK_VIT_TENSORS, X_DZ0, X_STATS1, X_STATS2, X_LSE, X_STATSF, X_TENSORS };

struct Geo {
  int B, n, T, d, m, K0, L, classes, dtype, heads;
  size_t rows, es;
};

bool make_geo(const cnnk_vit_desc* v, Geo* g) {
  if (!v) return false;
  if (v->B <= 0 || v->image <= 0 || v->patch <= 0 || v->dim <= 0 || v->heads <= 0 || v->layers <= 0 || v->mlp <= 0 ||
      v->classes <= 0 || v->image % v->patch != 0 || v->dim % v->heads != 0)
    return false;
  g->B = v->B;
  g->n = (v->image / v->patch) * (v->image / v->patch);
  g->T = g->n + 1;
  g->d = v->dim;
  g->m = v->mlp;
  g->K0 = v->patch * v->patch * 3;
  g->L = v->layers;
  g->classes = v->classes;
  g->dtype = v->dtype;
  g->heads = v->heads;
  g->rows = (size_t)g->B * g->T;
  g->es = elem_size(v->dtype);
  return true;
}

int validate(const cnnk_vit_desc* v, Geo* g) {
  if (!v) return CNNK_ERR_NULL;
  if (!make_geo(v, g)) return CNNK_ERR_SHAPE;
  if (v->dtype != CNNK_F32 && v->dtype != CNNK_BF16) return CNNK_ERR_UNSUPPORTED;
  const int dh = v->dim / v->heads;
  if ((dh != 16 && dh != 32 && dh != 64) || (long long)g->T * dh > 16384) return CNNK_ERR_UNSUPPORTED;
  if (v->dim % 8 != 0 || v->mlp % 8 != 0 || g->K0 % 8 != 0 || v->dim > 2048 || v->mlp > 65536) return CNNK_ERR_UNSUPPORTED;
  if ((double)g->rows * (v->mlp > 3 * v->dim ? v->mlp : 3 * v->dim) > 2147483647.0) return CNNK_ERR_UNSUPPORTED;
  if (!(v->ln_eps >= 0.f)) return CNNK_ERR_SHAPE;
  return CNNK_OK;
}

// bytes of one instance of a tensor (0: not a per-layer tensor id / unused)
size_t tensor_bytes(const Geo& g, int id) {
  const size_t r = g.rows, es = g.es;
  switch (id) {
    case CNNK_VIT_PATCHES: return (size_t)g.B * g.n * g.K0 * es;
    case CNNK_VIT_TOK: case CNNK_VIT_DTOK: return r * g.d * es;
    case CNNK_VIT_H: case CNNK_VIT_O: case CNNK_VIT_XMID: case CNNK_VIT_H2: case CNNK_VIT_XOUT:
    case CNNK_VIT_DH: case CNNK_VIT_DO: case CNNK_VIT_DXMID: case CNNK_VIT_DH2: case CNNK_VIT_DXOUT:
      return r * g.d * es;
    case CNNK_VIT_QKV: case CNNK_VIT_DQKV: return r * 3 * g.d * es;
    case CNNK_VIT_U: case CNNK_VIT_G: case CNNK_VIT_DU: case CNNK_VIT_DG: return r * g.m * es;
    case CNNK_VIT_F: case CNNK_VIT_DF: return (size_t)g.B * g.d * es;
    case X_Z0: case X_DZ0: return (size_t)g.B * g.n * g.d * es;
    case X_STATS1: case X_STATS2: return r * 2 * sizeof(float);
    case X_LSE: return (size_t)g.B * g.heads * g.T * sizeof(float);
    case X_STATSF: return (size_t)g.B * 2 * sizeof(float);
    default: return 0;
  }
}
bool per_layer(int id) {
  switch (id) {
    case CNNK_VIT_H: case CNNK_VIT_QKV: case CNNK_VIT_O: case CNNK_VIT_XMID: case CNNK_VIT_H2: case CNNK_VIT_U:
    case CNNK_VIT_G: case CNNK_VIT_XOUT: case CNNK_VIT_DH: case CNNK_VIT_DQKV: case CNNK_VIT_DO: case CNNK_VIT_DXMID:
    case CNNK_VIT_DH2: case CNNK_VIT_DU: case CNNK_VIT_DG: case CNNK_VIT_DXOUT: case X_STATS1: case X_STATS2: case X_LSE:
      return true;
    default: return false;
  }
}

struct Arena {
  size_t off[X_TENSORS];      // offset of instance 0
  size_t size[X_TENSORS];     // bytes of one instance, rounded up to 256
  size_t total;
};

void layout(const Geo& g, Arena* a) {
  size_t at = 0;
  for (int id = 0; id < X_TENSORS; ++id) {
    const size_t b = tensor_bytes(g, id);
    a->size[id] = align_up(b, 256);
    a->off[id] = at;
    at += a->size[id] * (per_layer(id) ? (size_t)g.L : 1);
  }
  a->total = at;
}

size_t max_sz(size_t a, size_t b) { return a > b ? a : b; }

// Whether the backward pass runs with its weight gradients in groups: bf16, every product on the dense kernels.
bool grouped(const Geo& g) {
  const long long rows = (long long)g.rows;
  return g.dtype == CNNK_BF16 && linear_dense(rows, g.d, 3 * g.d, g.dtype) && linear_dense(rows, g.d, g.d, g.dtype) &&
         linear_dense(rows, g.d, g.m, g.dtype) && linear_dense(rows, g.m, g.d, g.dtype) && linear_dense((long long)g.B * g.n, g.K0, g.d, g.dtype);
}
// Blocks whose weight gradients share a launch.  On a second stream one where that gives every CU a workgroup (ViT-B/16,
// 288 a block: one block / two, step at batch 8 3.24 / 3.22 ms, 16 4.40 / 4.68, 32 6.95 / 7.12, 64 11.64 / 11.79), otherwise as
// many as give it about 400 (512 columns, 136 a block, 96 images of 65 tokens: one block 2.87, two 2.77, three 2.78; 384
// columns, 72 a block, 192 images of 257: one 3.54, four 3.40, six 3.42).  On one stream nothing runs beside the launch, and
// the more workgroups it has, the less of it is a last round that is nearly empty (one block / three / seven, ViT-B/16 at
// batch 8 3.57 / 3.31 / 3.28 ms, 64 12.82 / 11.58 / 11.50; 512 columns 3.08 / 2.92 / 2.83; 384 columns 3.70 / 3.64 / 3.34).
// At most seven (28 products and the embedding's fit the table).
constexpr int kMostBlocks = 7;
int group_blocks(const Geo& g, bool two) {
  if (!two) return kMostBlocks;
  const int t = gemm_bf16_wgrad_tiles(g.d, 3 * g.d) + gemm_bf16_wgrad_tiles(g.d, g.d) + gemm_bf16_wgrad_tiles(g.d, g.m) + gemm_bf16_wgrad_tiles(g.m, g.d);
  const int n = t >= 256 ? 1 : (400 + t - 1) / t;
  return n > kMostBlocks ? kMostBlocks : n;
}
// Shapes of the products of the group of `blocks` blocks that ends with block l (or up to the last one); block 0's
// group has the patch embedding as well.  Returns their number.
int fill_group(const Geo& g, int l, int blocks, GemmWgrad* p) {
  int n = 0;
  const int end = l + blocks < g.L ? l + blocks : g.L;
  for (int k = l; k < end; ++k) {
    const int kn[4][2] = {{g.m, g.d}, {g.d, g.m}, {g.d, g.d}, {g.d, 3 * g.d}};
    for (int q = 0; q < 4; ++q) p[n++] = GemmWgrad{nullptr, nullptr, nullptr, nullptr, (long long)g.rows, kn[q][0], kn[q][1]};
  }
  if (l == 0) p[n++] = GemmWgrad{nullptr, nullptr, nullptr, nullptr, (long long)g.B * g.n, g.K0, g.d};
  return n;
}

// Into how many parts the rows of every weight gradient are split: what fills the device best for a group of the step
// with two streams, and the same for every group of either, so that the sums are the same bits.
int group_splits(const Geo& g) {
  GemmWgrad p[32];
  const int n = fill_group(g, 0, group_blocks(g, true), p);
  return gemm_bf16_wgrad_group_splits(p, n);
}

// The workspace of a step on one stream, half of it on two: the scratch of a call, then the partial sums of the layer
// norms and of fc1's bias gradients of `blocks` blocks, which live until their group's final sums.  With a second
// stream those may come at any time before the join, so every block has partial sums of its own, in the two halves; on
// one stream the next group takes the last one's place.
struct Workspace {
  size_t scratch, ln, gelu, total;      // ln: of one layer norm; gelu: of one fc1
  int blocks;
  size_t block() const { return 2 * ln + gelu; }
};

Workspace workspace(const cnnk_vit_desc* v, const Geo& g) {
  Workspace ws{};
  size_t& w = ws.scratch;
  const long long shapes[5][3] = {{(long long)g.B * g.n, g.K0, g.d}, {(long long)g.rows, g.d, 3 * g.d}, {(long long)g.rows, g.d, g.d},
                                  {(long long)g.rows, g.d, g.m}, {(long long)g.rows, g.m, g.d}};
  for (int i = 0; i < 5; ++i) w = max_sz(w, cnnk_linear_workspace_bytes(shapes[i][0], (int)shapes[i][1], (int)shapes[i][2], g.dtype));
  cnnk_ln_desc ln = {(int)g.rows, g.d, g.dtype, v->ln_eps, 0};
  w = max_sz(w, cnnk_layernorm_workspace_bytes(&ln));
  w = max_sz(w, cnnk_bias_act_workspace_bytes((long long)g.rows, 3 * g.d));
  w = max_sz(w, cnnk_bias_act_workspace_bytes((long long)g.rows, g.m));
  cnnk_fc_desc fc = {g.B, g.d, g.classes, g.dtype};
  w = max_sz(w, cnnk_fc_workspace_bytes(&fc));
  if (grouped(g)) {
    for (int two = 0; two < 2; ++two) {
      const int group = group_blocks(g, two != 0);
      for (int l = 0; l < g.L; l += group) {
        GemmWgrad p[32];
        const int n = fill_group(g, l, group, p);
        w = max_sz(w, gemm_bf16_wgrad_group_ws(p, n, group_splits(g)));
      }
    }
    const int one = group_blocks(g, false), half = (g.L + 1) / 2;
    ws.blocks = one > half ? (one < g.L ? one : g.L) : half;
    ws.ln = align_up(cnnk_layernorm_workspace_bytes(&ln), 256);
    ws.gelu = align_up((size_t)gemm_bf16_dgrad_gelu_parts((long long)g.rows, g.m, g.d) * g.m * sizeof(float), 256);
  }
  w = align_up(w, 256);
  ws.total = w + (size_t)ws.blocks * ws.block();
  return ws;
}

// Walks the step's calls in order.  In enumeration mode nothing runs: the walk counts the calls and
// copies the name of call `want`.
struct Walk {
  bool run;
  int idx, want;
  char* name_out;
  int name_n;
  int rc;
  void** events;
  hipStream_t st;
  template <typename F>
  void call(int layer, const char* name, F&& f) {
    if (!run) {
      if (idx == want && name_out && name_n > 0) {
        if (layer >= 0) snprintf(name_out, (size_t)name_n, "block%d.%s", layer, name);
        else snprintf(name_out, (size_t)name_n, "%s", name);
      }
      ++idx;
      return;
    }
    if (rc != CNNK_OK) { ++idx; return; }
    if (events) (void)hipEventRecord((hipEvent_t)events[2 * idx], st);
    rc = f();
    if (events) (void)hipEventRecord((hipEvent_t)events[2 * idx + 1], st);
    ++idx;
  }
};

size_t param_elems(const Geo& g, int k) {
  const size_t d = (size_t)g.d, m = (size_t)g.m;
  const size_t blk[B_COUNT] = {d, d, 3 * d * d, 3 * d, d * d, d, d, d, m * d, m, d * m, d};
  const int p_tail = P_BLOCK0 + B_COUNT * g.L;
  if (k == P_WE) return d * g.K0;
  if (k == P_BE || k == P_CLS) return d;
  if (k == P_POS) return (size_t)g.T * d;
  if (k < p_tail) return blk[(k - P_BLOCK0) % B_COUNT];
  if (k == p_tail || k == p_tail + 1) return d;
  return k == p_tail + 2 ? (size_t)g.classes * d : (size_t)g.classes;
}

// SGD-momentum of parameters [k0, k1)
int update_params(const Geo& g, const cnnk_vit_buffers* buf, int k0, int k1, float lr, float mu, float wd, hipStream_t st) {
  SgdTable t;
  t.count = 0;
  int rc = CNNK_OK;
  for (int k = k0; k < k1 && rc == CNNK_OK; ++k) {
    const int i = t.count++;
    t.w[i] = (float*)buf->param[k]; t.v[i] = (float*)buf->mom[k]; t.g[i] = (const float*)buf->grad[k];
    t.wlp[i] = g.dtype == CNNK_BF16 ? buf->param_lp[k] : nullptr; t.n[i] = param_elems(g, k);
    if (t.count == kSgdMaxTensors || k == k1 - 1) { rc = sgd_multi(t, lr, mu, wd, st); t.count = 0; }
  }
  return rc;
}

// The backward pass and the update with the products that only the update waits for in groups: the data-gradient
// chain runs on `st`; the weight gradients of group_blocks() transformer blocks, with the bias gradients (column
// sums of an operand that those products load anyway), the final sums of the blocks' layer norms and of fc1's bias
// gradients and the update of the blocks' parameters follow as three launches, on the second stream if there is one.
// GELU's gradient is taken in the epilogue of fc2's data gradient, which leaves partial sums of the unrounded products
// for fc1's bias.  Per block of ViT-B/16 10 launches and one event pair instead of 24 and 7: at batch 8 the step was
// bound by enqueueing them, and at batch 64 split products for a fraction of the device each took 270 us a block.
int backward_grouped(const cnnk_vit_desc* v, const Geo& g, const cnnk_vit_buffers* buf, const Arena& A, float lr, float mu, float wd,
                     bool two, hipStream_t st) {
  const int d = g.d, m = g.m, T = g.T, G = group_blocks(g, two), p_tail = P_BLOCK0 + B_COUNT * g.L;
  const long long rows = (long long)g.rows, prow = (long long)g.B * g.n;
  const cnnk_ln_desc ln = {(int)g.rows, d, g.dtype, v->ln_eps, 0};
  const cnnk_ln_desc ln_cls = {g.B, d, g.dtype, v->ln_eps, (long long)T * d};
  const cnnk_attn_desc ad = {g.B, T, v->heads, d / v->heads, g.dtype};
  const cnnk_embed_desc ed = {g.B, v->image, v->patch, d, g.dtype};
  const Workspace W = workspace(v, g);
  char* const base = (char*)buf->arena;
  auto at = [&](int id, int l) -> bf16_t* { return (bf16_t*)(base + A.off[id] + A.size[id] * (size_t)(per_layer(id) ? l : 0)); };
  auto P = [&](int k) { return (float*)buf->param[k]; };
  auto Wm = [&](int k) { return (const bf16_t*)buf->param_lp[k]; };
  auto Gr = [&](int k) { return (float*)buf->grad[k]; };
  char* const ws = (char*)buf->ws;
  const size_t wsb = W.scratch;
  const hipStream_t side = two ? (hipStream_t)buf->aux_stream : st;
  char* const side_ws = two ? ws + buf->ws_bytes / 2 / 256 * 256 : ws;
  // partial sums of block l: of its two layer norms, then of fc1's bias gradient
  auto parts_of = [&](int l) -> char* {
    if (!two) return ws + W.scratch + (size_t)(l % G) * W.block();
    return (l < W.blocks ? ws + (size_t)l * W.block() : side_ws + (size_t)(l - W.blocks) * W.block()) + W.scratch;
  };
  int rc = cnnk_fill_zero(at(CNNK_VIT_DXOUT, g.L - 1), A.size[CNNK_VIT_DXOUT], st);
  if (rc == CNNK_OK)
    rc = cnnk_layernorm_bwd(&ln_cls, at(CNNK_VIT_DF, 0), at(CNNK_VIT_XOUT, g.L - 1), P(p_tail), (const float*)at(X_STATSF, 0), nullptr,
                            at(CNNK_VIT_DXOUT, g.L - 1), Gr(p_tail), Gr(p_tail + 1), ws, wsb, st);
  GemmWgrad pend[32];
  ColumnSums sums;
  const int splits = group_splits(g), ln_parts = ln_bwd_parts(&ln), gelu_parts = gemm_bf16_dgrad_gelu_parts(rows, m, d);
  int np = 0;
  sums.count = 0;
  auto defer = [&](const bf16_t* dy, const bf16_t* x, int kw, int kb, long long r, int K, int N) {
    pend[np++] = GemmWgrad{dy, x, Gr(kw), kb < 0 ? nullptr : Gr(kb), r, K, N};
  };
  auto norm_bwd = [&](int l, int second, const bf16_t* dy, const bf16_t* x, int kg, const void* stats, const bf16_t* dres, bf16_t* dx) -> int {
    float* part = (float*)(parts_of(l) + second * W.ln);
    sums.it[sums.count++] = {part, Gr(kg), Gr(kg + 1), ln_parts, d};
    return ln_bwd_rows_partial(&ln, dy, x, P(kg), (const float*)stats, dres, dx, part, st);
  };
  for (int l = g.L - 1; l >= 0 && rc == CNNK_OK; --l) {
    const int p0 = P_BLOCK0 + B_COUNT * l;
    const bf16_t* xin = l ? at(CNNK_VIT_XOUT, l - 1) : at(CNNK_VIT_TOK, 0);
    bf16_t* dxin = l ? at(CNNK_VIT_DXOUT, l - 1) : at(CNNK_VIT_DTOK, 0);
    const bf16_t *dxo = at(CNNK_VIT_DXOUT, l), *du = at(CNNK_VIT_DU, l), *dxm = at(CNNK_VIT_DXMID, l), *dqkv = at(CNNK_VIT_DQKV, l);
    float* const du_part = (float*)(parts_of(l) + 2 * W.ln);
    rc = gemm_bf16_dgrad_gelu(rows, m, d, dxo, Wm(p0 + B_W2), at(CNNK_VIT_U, l), at(CNNK_VIT_DG, l), at(CNNK_VIT_DU, l), du_part, st);
    sums.it[sums.count++] = {du_part, Gr(p0 + B_C1), Gr(p0 + B_C1) + m / 2, gelu_parts, m / 2};
    if (rc == CNNK_OK) rc = gemm_bf16_dgrad(rows, d, m, du, Wm(p0 + B_W1), at(CNNK_VIT_DH2, l), st);
    if (rc == CNNK_OK) rc = norm_bwd(l, 1, at(CNNK_VIT_DH2, l), at(CNNK_VIT_XMID, l), p0 + B_G2, at(X_STATS2, l), dxo, at(CNNK_VIT_DXMID, l));
    if (rc == CNNK_OK) rc = gemm_bf16_dgrad(rows, d, d, dxm, Wm(p0 + B_WO), at(CNNK_VIT_DO, l), st);
    if (rc == CNNK_OK) rc = cnnk_attention_bwd(&ad, at(CNNK_VIT_QKV, l), at(CNNK_VIT_O, l), at(CNNK_VIT_DO, l), (const float*)at(X_LSE, l), at(CNNK_VIT_DQKV, l), st);
    if (rc == CNNK_OK) rc = gemm_bf16_dgrad(rows, d, 3 * d, dqkv, Wm(p0 + B_WQKV), at(CNNK_VIT_DH, l), st);
    if (rc == CNNK_OK) rc = norm_bwd(l, 0, at(CNNK_VIT_DH, l), xin, p0 + B_G1, at(X_STATS1, l), dxm, dxin);
    defer(dxo, at(CNNK_VIT_G, l), p0 + B_W2, p0 + B_C2, rows, m, d);
    defer(du, at(CNNK_VIT_H2, l), p0 + B_W1, -1, rows, d, m);
    defer(dxm, at(CNNK_VIT_O, l), p0 + B_WO, p0 + B_BO, rows, d, d);
    defer(dqkv, at(CNNK_VIT_H, l), p0 + B_WQKV, p0 + B_BQKV, rows, d, 3 * d);
    if (l == 0 && rc == CNNK_OK) {
      rc = embed_bwd(&ed, at(CNNK_VIT_DTOK, 0), at(X_DZ0, 0), nullptr, Gr(P_CLS), Gr(P_POS), st);
      defer(at(X_DZ0, 0), at(CNNK_VIT_PATCHES, 0), P_WE, P_BE, prow, g.K0, d);
    }
    if (l % G != 0 || rc != CNNK_OK) continue;
    if (two && (hipEventRecord((hipEvent_t)buf->ev_fork, st) != hipSuccess || hipStreamWaitEvent(side, (hipEvent_t)buf->ev_fork, 0) != hipSuccess))
      return CNNK_ERR_HIP;
    rc = gemm_bf16_wgrad_group(pend, np, splits, side_ws, side);
    if (rc == CNNK_OK) rc = column_sums_group(sums, side);
    const int last = l + G < g.L ? l + G : g.L;
    if (rc == CNNK_OK) rc = update_params(g, buf, l ? p0 : 0, P_BLOCK0 + B_COUNT * last, lr, mu, wd, side);
    np = 0;
    sums.count = 0;
  }
  if (rc == CNNK_OK) rc = update_params(g, buf, p_tail, p_tail + 4, lr, mu, wd, st);
  if (two && rc == CNNK_OK && (hipEventRecord((hipEvent_t)buf->ev_join, side) != hipSuccess || hipStreamWaitEvent(st, (hipEvent_t)buf->ev_join, 0) != hipSuccess))
    rc = CNNK_ERR_HIP;
  return rc;
}

int walk(const cnnk_vit_desc* v, const Geo& g, const cnnk_vit_buffers* buf, float lr, float mu, float wd, Walk& w,
         bool forward_only = false) {
  Arena A;
  layout(g, &A);
  char* base = buf ? (char*)buf->arena : nullptr;
  auto at = [&](int id, int l) -> void* { return base ? base + A.off[id] + A.size[id] * (size_t)(per_layer(id) ? l : 0) : nullptr; };
  // Calls that only the update waits for go to the second stream when there is one: `st`, `ws` and
  // `wsb` are what the call lambdas below read, and forked() points them at the second stream and the
  // upper half of the workspace for the duration of one call.
  const bool two = w.run && buf && buf->aux_stream && buf->ev_fork && buf->ev_join && !w.events;
  void* const ws_main = buf ? buf->ws : nullptr;
  const size_t wsb_main = buf ? (two ? buf->ws_bytes / 2 / 256 * 256 : buf->ws_bytes) : 0;
  void* ws = ws_main;
  size_t wsb = wsb_main;
  hipStream_t st = w.st;
  auto forked = [&](int layer, const char* name, auto&& f) {
    if (!two) { w.call(layer, name, f); return; }
    if (w.rc != CNNK_OK) { ++w.idx; return; }
    hipStream_t aux = (hipStream_t)buf->aux_stream;
    if (hipEventRecord((hipEvent_t)buf->ev_fork, w.st) != hipSuccess || hipStreamWaitEvent(aux, (hipEvent_t)buf->ev_fork, 0) != hipSuccess) {
      w.rc = CNNK_ERR_HIP;
      ++w.idx;
      return;
    }
    st = aux; ws = (char*)ws_main + wsb_main; wsb = wsb_main;
    w.rc = f();
    st = w.st; ws = ws_main; wsb = wsb_main;
    ++w.idx;
  };
  const bool bf = g.dtype == CNNK_BF16;
  auto P = [&](int k) -> float* { return buf ? (float*)buf->param[k] : nullptr; };
  auto Wm = [&](int k) -> const void* { return buf ? (bf ? buf->param_lp[k] : buf->param[k]) : nullptr; };
  auto Gr = [&](int k) -> float* { return buf ? (float*)buf->grad[k] : nullptr; };
  const int d = g.d, m = g.m, T = g.T;
  const long long rows = (long long)g.rows;
  const cnnk_embed_desc ed = {g.B, v->image, v->patch, d, g.dtype};
  const long long prow = (long long)g.B * g.n;     // patch rows
  const int dt = g.dtype;
  const cnnk_ln_desc ln = {(int)g.rows, d, g.dtype, v->ln_eps, 0};
  const cnnk_ln_desc ln_cls = {g.B, d, g.dtype, v->ln_eps, (long long)T * d};
  const cnnk_attn_desc ad = {g.B, T, v->heads, d / v->heads, g.dtype};
  const cnnk_fc_desc fc = {g.B, d, g.classes, g.dtype};
  const int p_tail = P_BLOCK0 + B_COUNT * g.L;     // gf, bf, Wh, bh

  // ---- forward ----
  w.call(-1, "embed.patchify", [&] { return cnnk_vit_patchify(&ed, buf->x, at(CNNK_VIT_PATCHES, 0), st); });
  w.call(-1, "embed.gemm", [&] { return cnnk_linear_fwd(prow, g.K0, d, dt, at(CNNK_VIT_PATCHES, 0), Wm(P_WE), nullptr, nullptr, CNNK_ACT_NONE, nullptr, at(X_Z0, 0), ws, wsb, st); });
  w.call(-1, "embed.tokens", [&] { return cnnk_vit_embed_fwd(&ed, at(X_Z0, 0), P(P_BE), P(P_CLS), P(P_POS), at(CNNK_VIT_TOK, 0), st); });
  for (int l = 0; l < g.L; ++l) {
    const int p0 = P_BLOCK0 + B_COUNT * l;
    void* xin = l ? at(CNNK_VIT_XOUT, l - 1) : at(CNNK_VIT_TOK, 0);
    w.call(l, "ln1", [&] { return cnnk_layernorm_fwd(&ln, xin, P(p0 + B_G1), P(p0 + B_B1), at(CNNK_VIT_H, l), (float*)at(X_STATS1, l), st); });
    w.call(l, "qkv.gemm", [&] { return cnnk_linear_fwd(rows, d, 3 * d, dt, at(CNNK_VIT_H, l), Wm(p0 + B_WQKV), P(p0 + B_BQKV), nullptr, CNNK_ACT_NONE, nullptr, at(CNNK_VIT_QKV, l), ws, wsb, st); });
    w.call(l, "attn", [&] { return cnnk_attention_fwd(&ad, at(CNNK_VIT_QKV, l), at(CNNK_VIT_O, l), (float*)at(X_LSE, l), st); });
    w.call(l, "proj.gemm_res", [&] { return cnnk_linear_fwd(rows, d, d, dt, at(CNNK_VIT_O, l), Wm(p0 + B_WO), P(p0 + B_BO), xin, CNNK_ACT_NONE, nullptr, at(CNNK_VIT_XMID, l), ws, wsb, st); });
    w.call(l, "ln2", [&] { return cnnk_layernorm_fwd(&ln, at(CNNK_VIT_XMID, l), P(p0 + B_G2), P(p0 + B_B2), at(CNNK_VIT_H2, l), (float*)at(X_STATS2, l), st); });
    w.call(l, "fc1.gemm_gelu", [&] { return cnnk_linear_fwd(rows, d, m, dt, at(CNNK_VIT_H2, l), Wm(p0 + B_W1), P(p0 + B_C1), nullptr, CNNK_ACT_GELU, at(CNNK_VIT_U, l), at(CNNK_VIT_G, l), ws, wsb, st); });
    w.call(l, "fc2.gemm_res", [&] { return cnnk_linear_fwd(rows, m, d, dt, at(CNNK_VIT_G, l), Wm(p0 + B_W2), P(p0 + B_C2), at(CNNK_VIT_XMID, l), CNNK_ACT_NONE, nullptr, at(CNNK_VIT_XOUT, l), ws, wsb, st); });
  }
  void* xlast = at(CNNK_VIT_XOUT, g.L - 1);
  w.call(-1, "head.ln", [&] { return cnnk_layernorm_fwd(&ln_cls, xlast, P(p_tail), P(p_tail + 1), at(CNNK_VIT_F, 0), (float*)at(X_STATSF, 0), st); });
  if (forward_only) {
    w.call(-1, "head.loss", [&] {
      return cnnk_fc_softmax_xent(&fc, at(CNNK_VIT_F, 0), P(p_tail + 2), P(p_tail + 3), buf->labels, buf->loss, buf->pred,
                                  buf->probs, nullptr, nullptr, nullptr, ws, wsb, st);
    });
    return w.rc;
  }
  w.call(-1, "head.loss", [&] {
    return cnnk_fc_softmax_xent(&fc, at(CNNK_VIT_F, 0), P(p_tail + 2), P(p_tail + 3), buf->labels, buf->loss, buf->pred, buf->probs,
                                at(CNNK_VIT_DF, 0), Gr(p_tail + 2), Gr(p_tail + 3), ws, wsb, st);
  });
  // ---- backward ----
  if (w.run && buf && !w.events && grouped(g)) {
    bool ok = true;      // the grouped sums of split products store 16 bytes at a time
    for (int k = 0; k < p_tail; ++k) ok = ok && (((size_t)buf->grad[k]) & 15) == 0;
    if (ok) {
      if (w.rc == CNNK_OK) w.rc = backward_grouped(v, g, buf, A, lr, mu, wd, two, w.st);
      return w.rc;
    }
  }
  void* dxlast = at(CNNK_VIT_DXOUT, g.L - 1);
  w.call(-1, "head.zero", [&] { return cnnk_fill_zero(dxlast, A.size[CNNK_VIT_DXOUT], st); });
  w.call(-1, "head.ln.bwd", [&] {
    return cnnk_layernorm_bwd(&ln_cls, at(CNNK_VIT_DF, 0), xlast, P(p_tail), (const float*)at(X_STATSF, 0), nullptr, dxlast, Gr(p_tail),
                              Gr(p_tail + 1), ws, wsb, st);
  });
  for (int l = g.L - 1; l >= 0; --l) {
    const int p0 = P_BLOCK0 + B_COUNT * l;
    void* xin = l ? at(CNNK_VIT_XOUT, l - 1) : at(CNNK_VIT_TOK, 0);
    void* dxin = l ? at(CNNK_VIT_DXOUT, l - 1) : at(CNNK_VIT_DTOK, 0);
    void* dxo = at(CNNK_VIT_DXOUT, l);
    forked(l, "fc2.dbias", [&] { return cnnk_bias_act_bwd(rows, d, g.dtype, CNNK_ACT_NONE, dxo, nullptr, nullptr, Gr(p0 + B_C2), ws, wsb, st); });
    forked(l, "fc2.wgrad", [&] { return cnnk_linear_wgrad(rows, m, d, dt, at(CNNK_VIT_G, l), dxo, Gr(p0 + B_W2), ws, wsb, st); });
    w.call(l, "fc2.dgrad", [&] { return cnnk_linear_dgrad(rows, m, d, dt, dxo, Wm(p0 + B_W2), at(CNNK_VIT_DG, l), ws, wsb, st); });
    w.call(l, "fc1.gelu.bwd", [&] { return cnnk_bias_act_bwd(rows, m, g.dtype, CNNK_ACT_GELU, at(CNNK_VIT_DG, l), at(CNNK_VIT_U, l), at(CNNK_VIT_DU, l), Gr(p0 + B_C1), ws, wsb, st); });
    forked(l, "fc1.wgrad", [&] { return cnnk_linear_wgrad(rows, d, m, dt, at(CNNK_VIT_H2, l), at(CNNK_VIT_DU, l), Gr(p0 + B_W1), ws, wsb, st); });
    w.call(l, "fc1.dgrad", [&] { return cnnk_linear_dgrad(rows, d, m, dt, at(CNNK_VIT_DU, l), Wm(p0 + B_W1), at(CNNK_VIT_DH2, l), ws, wsb, st); });
    w.call(l, "ln2.bwd", [&] {
      return cnnk_layernorm_bwd(&ln, at(CNNK_VIT_DH2, l), at(CNNK_VIT_XMID, l), P(p0 + B_G2), (const float*)at(X_STATS2, l), dxo,
                                at(CNNK_VIT_DXMID, l), Gr(p0 + B_G2), Gr(p0 + B_B2), ws, wsb, st);
    });
    void* dxm = at(CNNK_VIT_DXMID, l);
    forked(l, "proj.dbias", [&] { return cnnk_bias_act_bwd(rows, d, g.dtype, CNNK_ACT_NONE, dxm, nullptr, nullptr, Gr(p0 + B_BO), ws, wsb, st); });
    forked(l, "proj.wgrad", [&] { return cnnk_linear_wgrad(rows, d, d, dt, at(CNNK_VIT_O, l), dxm, Gr(p0 + B_WO), ws, wsb, st); });
    w.call(l, "proj.dgrad", [&] { return cnnk_linear_dgrad(rows, d, d, dt, dxm, Wm(p0 + B_WO), at(CNNK_VIT_DO, l), ws, wsb, st); });
    w.call(l, "attn.bwd", [&] { return cnnk_attention_bwd(&ad, at(CNNK_VIT_QKV, l), at(CNNK_VIT_O, l), at(CNNK_VIT_DO, l), (const float*)at(X_LSE, l), at(CNNK_VIT_DQKV, l), st); });
    forked(l, "qkv.dbias", [&] { return cnnk_bias_act_bwd(rows, 3 * d, g.dtype, CNNK_ACT_NONE, at(CNNK_VIT_DQKV, l), nullptr, nullptr, Gr(p0 + B_BQKV), ws, wsb, st); });
    forked(l, "qkv.wgrad", [&] { return cnnk_linear_wgrad(rows, d, 3 * d, dt, at(CNNK_VIT_H, l), at(CNNK_VIT_DQKV, l), Gr(p0 + B_WQKV), ws, wsb, st); });
    w.call(l, "qkv.dgrad", [&] { return cnnk_linear_dgrad(rows, d, 3 * d, dt, at(CNNK_VIT_DQKV, l), Wm(p0 + B_WQKV), at(CNNK_VIT_DH, l), ws, wsb, st); });
    w.call(l, "ln1.bwd", [&] {
      return cnnk_layernorm_bwd(&ln, at(CNNK_VIT_DH, l), xin, P(p0 + B_G1), (const float*)at(X_STATS1, l), dxm, dxin, Gr(p0 + B_G1),
                                Gr(p0 + B_B1), ws, wsb, st);
    });
  }
  w.call(-1, "embed.tokens.bwd", [&] { return cnnk_vit_embed_bwd(&ed, at(CNNK_VIT_DTOK, 0), at(X_DZ0, 0), Gr(P_BE), Gr(P_CLS), Gr(P_POS), st); });
  forked(-1, "embed.wgrad", [&] { return cnnk_linear_wgrad(prow, g.K0, d, dt, at(CNNK_VIT_PATCHES, 0), at(X_DZ0, 0), Gr(P_WE), ws, wsb, st); });
  // ---- update ----
  if (two && w.rc == CNNK_OK) {
    if (hipEventRecord((hipEvent_t)buf->ev_join, (hipStream_t)buf->aux_stream) != hipSuccess ||
        hipStreamWaitEvent(w.st, (hipEvent_t)buf->ev_join, 0) != hipSuccess)
      w.rc = CNNK_ERR_HIP;
  }
  w.call(-1, "update", [&] {
    return update_params(g, buf, 0, p_tail + 4, lr, mu, wd, st);
  });
  return w.rc;
}
}  // namespace

extern "C" size_t cnnk_vit_arena_bytes(const cnnk_vit_desc* v) {
  Geo g;
  if (validate(v, &g) != CNNK_OK) return 0;
  Arena a;
  layout(g, &a);
  return a.total;
}

extern "C" size_t cnnk_vit_workspace_bytes(const cnnk_vit_desc* v) {
  Geo g;
  if (validate(v, &g) != CNNK_OK) return 0;
  return workspace(v, g).total;
}

extern "C" int cnnk_vit_tensor(const cnnk_vit_desc* v, int id, int layer, size_t* offset, size_t* bytes) {
  Geo g;
  const int rc = validate(v, &g);
  if (rc != CNNK_OK) return rc;
  if (!offset || !bytes) return CNNK_ERR_NULL;
  if (id < 0 || id >= CNNK_VIT_TENSORS) return CNNK_ERR_SHAPE;
  if (per_layer(id) && (layer < 0 || layer >= g.L)) return CNNK_ERR_SHAPE;
  Arena a;
  layout(g, &a);
  *offset = a.off[id] + a.size[id] * (size_t)(per_layer(id) ? layer : 0);
  *bytes = tensor_bytes(g, id);
  return CNNK_OK;
}

extern "C" int cnnk_vit_step_calls(const cnnk_vit_desc* v) {
  Geo g;
  if (validate(v, &g) != CNNK_OK) return 0;
  Walk w = {false, 0, -1, nullptr, 0, CNNK_OK, nullptr, nullptr};
  walk(v, g, nullptr, 0.f, 0.f, 0.f, w);
  return w.idx;
}

extern "C" int cnnk_vit_step_call_name(const cnnk_vit_desc* v, int i, char* out, int n) {
  Geo g;
  const int rc = validate(v, &g);
  if (rc != CNNK_OK) return rc;
  if (!out || n <= 0) return CNNK_ERR_NULL;
  out[0] = 0;
  Walk w = {false, 0, i, out, n, CNNK_OK, nullptr, nullptr};
  walk(v, g, nullptr, 0.f, 0.f, 0.f, w);
  return (i >= 0 && i < w.idx) ? CNNK_OK : CNNK_ERR_SHAPE;
}

static int check_buffers(const cnnk_vit_desc* v, const Geo& g, const cnnk_vit_buffers* buf, bool training) {
  if (!buf || !buf->param || !buf->x || !buf->labels || !buf->loss || !buf->pred || !buf->arena) return CNNK_ERR_NULL;
  if (training && (!buf->grad || !buf->mom)) return CNNK_ERR_NULL;
  const int np = P_BLOCK0 + B_COUNT * g.L + 4;
  if (buf->n_params != np) return CNNK_ERR_SHAPE;
  const bool bf = g.dtype == CNNK_BF16;
  if (bf && !buf->param_lp) return CNNK_ERR_NULL;
  for (int k = 0; k < np; ++k) {
    if (!buf->param[k] || (training && (!buf->grad[k] || !buf->mom[k]))) return CNNK_ERR_NULL;
    const int r = k >= P_BLOCK0 && k < np - 4 ? (k - P_BLOCK0) % B_COUNT : -1;
    const bool matrix = k == P_WE || r == B_WQKV || r == B_WO || r == B_W1 || r == B_W2;
    if (bf && matrix && !buf->param_lp[k]) return CNNK_ERR_NULL;
  }
  if (buf->arena_bytes < cnnk_vit_arena_bytes(v)) return CNNK_ERR_WORKSPACE;
  if ((((size_t)buf->arena) & 255) != 0 || (((size_t)buf->ws) & 255) != 0) return CNNK_ERR_UNSUPPORTED;
  return CNNK_OK;
}

extern "C" int cnnk_vit_eval_step(const cnnk_vit_desc* v, const cnnk_vit_buffers* buf, int* n_correct, void* stream) {
  Geo g;
  int rc = validate(v, &g);
  if (rc != CNNK_OK) return rc;
  rc = check_buffers(v, g, buf, false);
  if (rc != CNNK_OK) return rc;
  if (!buf->ws || buf->ws_bytes < workspace(v, g).total) return CNNK_ERR_WORKSPACE;
  cnnk_vit_buffers b = *buf;          // one stream, no per-call events
  b.events = nullptr; b.n_events = 0; b.aux_stream = nullptr;
  Walk w = {true, 0, -1, nullptr, 0, CNNK_OK, nullptr, (hipStream_t)stream};
  rc = walk(v, g, &b, 0.f, 0.f, 0.f, w, true);
  if (rc != CNNK_OK || !n_correct) return rc;
  return cnnk_count_correct(g.B, buf->pred, buf->labels, n_correct, stream);
}

extern "C" int cnnk_vit_train_step(const cnnk_vit_desc* v, const cnnk_vit_buffers* buf, float lr, float momentum,
                                   float weight_decay, void* stream) {
  Geo g;
  const int rc = validate(v, &g);
  if (rc != CNNK_OK) return rc;
  const int rcb = check_buffers(v, g, buf, true);
  if (rcb != CNNK_OK) return rcb;
  const bool two_streams = buf->aux_stream && buf->ev_fork && buf->ev_join && !buf->events;
  if (!buf->ws || buf->ws_bytes < workspace(v, g).total * (two_streams ? 2 : 1)) return CNNK_ERR_WORKSPACE;
  if ((((size_t)buf->arena) & 255) != 0 || (((size_t)buf->ws) & 255) != 0) return CNNK_ERR_UNSUPPORTED;
  Walk w = {true, 0, -1, nullptr, 0, CNNK_OK, nullptr, (hipStream_t)stream};
  if (buf->events) {
    Walk c = {false, 0, -1, nullptr, 0, CNNK_OK, nullptr, nullptr};
    walk(v, g, nullptr, 0.f, 0.f, 0.f, c);
    if (buf->n_events < 2 * c.idx) return CNNK_ERR_WORKSPACE;
    w.events = buf->events;
  }
  return walk(v, g, buf, lr, momentum, weight_decay, w);
}
