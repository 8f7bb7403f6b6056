// cnnk_train_step: forward over a layer list, loss, backward over the reversed list, SGD-momentum
// update of every parameter (the inner mini-batch loop of the paper's Algorithm 1 for one
// data-parallel replica).  Host code only: it validates the whole list first, then enqueues the
// kernels of the other entry points on one stream, with no host synchronisation in between.
#include <algorithm>
#include <utility>
#include <vector>
#include "common.h"
#include "sgd.h"
#include "conv.h"

namespace {

// grid budget (in compute units) of a weight gradient that runs beside the backward pass: measured
// optimum on ResNet-18 b256 (96..128 are within 1 %, 64 and 192 are 3 % slower)
constexpr int kAuxWgradCus = 112;
// Work for the second stream from which a step uses it: the flops of the convolutions, forward and backward, and 4500 for
// every element of their weights (their gradient, momentum and update move about 24 bytes each).  Below, the step is a
// chain of launches of a few us, and the events between the streams (50 to 80 us a step) cost more than the overlap
// gives.  us per step with one stream / two, by GF and million weights: tiny CNN b512 0.9 GF 640 / 663; 6-layer ResNet
// 0.3 M b16 13 GF 302 / 347, b48 39 GF 366 / 372, b64 52 GF 380 / 376; VGG-style 1.1 M b16 15 GF 350 / 360, b32 29 GF
// 370 / 384, b48 44 GF 397 / 404, b64 58 GF 412 / 416, b96 88 GF 482 / 448; twelve 3x3 layers 1.6 M b16 40 GF 663 / 604;
// 24 1x1 layers 1.5 M 37 GF 958 / 1112; ResNet-18 11 M b1 3 GF 1062 / 1024, b8 27 GF 1114 / 1056; ResNet-50 24 M b1 8 GF
// 2512 / 2385; WRN-28-10 36 M b1 31 GF 2362 / 2202.
constexpr double kAuxMinWork = 46e9, kAuxWorkPerWeight = 4500;
constexpr int kStatSlots = 4;   // convolutions whose per-channel sums may be pending at once
constexpr size_t kStatBytes = kStatSlots * 2 * 2048 * sizeof(float);

struct Walk {
  std::vector<size_t> slot_elems;   // 0 = not seen yet
  std::vector<size_t> param_elems;
  size_t ws = 0;
  size_t wt_bytes = 0;               // transposed bf16 weights of every conv whose data gradient runs on MFMA
  std::vector<size_t> wt_off;        // per layer: offset into that region, or (size_t)-1
  int x8_layer = -1;                 // first-layer convolution with fewer than 8 input channels, if any:
  size_t x8_off = 0;                 // its 8-channel copy of the network input lives in the same region
  std::vector<size_t> mask_off;      // per layer: offset of its ReLU mask, or (size_t)-1
  size_t mask_bytes = 0;             // ReLU masks (a bit per element) of the batch norms with a residual input
  bool shared_read = false;          // a weight of several layers is read by a data gradient, not copied before
  double flops = 0;                  // of the convolutions, forward and backward
  double weights = 0;                // their elements
  int convs = 0;
  int dtype = -1;
};

// what one stream of a training step needs
size_t step_workspace(const Walk& w) { return ((w.ws + 255) / 256 * 256 + kStatBytes + w.wt_bytes + w.mask_bytes + 255) / 256 * 256; }

// Whether a layer's data gradient takes a copy of the weights made before the backward pass.  The kernels of
// conv_gemm.hip read the weights themselves, which the second stream updates as soon as their own layer's data gradient
// is done: not where a layer that comes later in the backward pass has the same weights.
bool dgrad_pretransposed(const cnnk_layer& l, bool shared) {
  if (l.op != CNNK_OP_CONV || l.in0 == 0 || l.d.conv.dtype != CNNK_BF16) return false;
  const ConvGeom g = make_geom(&l.d.conv);
  return conv_mfma_supported(g, CNNK_PASS_DGRAD) && (shared || !conv_gemm_supported(g, CNNK_PASS_DGRAD));
}

bool set_elems(std::vector<size_t>& v, int id, size_t n) {
  if (id < 0 || id >= (int)v.size()) return false;
  if (v[id] == 0) { v[id] = n; return true; }
  return v[id] == n;
}

// Layers whose weight gradients share a fork of the second stream, and the launch of their reductions and updates.
// Small steps are bound by enqueueing (ResNet-18 at batch 32: 1305 of 1334 us; a fork and its events cost as much as
// several launches), so they take two at a time; large ones lose, because a weight gradient starts later and less of it
// runs beside the data gradients.  us per step one by one / in pairs, by flops per convolution (forward and backward):
// ResNet-50 b16 2.3 GF 3539 / 2623, ResNet-18 b32 5.3 GF 1212 / 1095, VGG-style b64 9.7 GF 415 / 403, ResNet-18 b64 10.7 GF
// 1297 / 1219, b77 12.8 GF 1360 / 1363, VGG-style b128 19 GF 460 / 485, WRN-28-10 b64 72 GF 4119 / 4223.  Three to
// sixteen at a time are slower than two everywhere but below 3 GF, where three and four are even.
constexpr double kPairFlops = 11e9;
int wgrad_group(const Walk& w) {
  if (g_cnnk_tune[17] > 0) return g_cnnk_tune[17] < kReduceGroup ? g_cnnk_tune[17] : kReduceGroup;
  return w.flops < kPairFlops * w.convs ? 2 : 1;
}

size_t max_sz(size_t a, size_t b) { return a > b ? a : b; }

// whether two tensors of `bytes` bytes share memory
bool share(const void* a, const void* b, size_t bytes) {
  const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
  return x < y + bytes && y < x + bytes;
}

// Checks every layer and gathers tensor sizes and the workspace need.  n_slots/n_params < 0:
// sizes are unknown (workspace query), ids are only checked for being non-negative.
int walk_layers(const cnnk_layer* L, int n, int n_slots, int n_params, Walk* w) {
  if (!L) return CNNK_ERR_NULL;
  if (n <= 0) return CNNK_ERR_SHAPE;
  int max_slot = 0, max_param = 0;
  for (int i = 0; i < n; ++i) {
    const int ids[3] = {L[i].in0, L[i].in1, L[i].out};
    for (int k = 0; k < 3; ++k) if (ids[k] > max_slot) max_slot = ids[k];
    if (L[i].p0 > max_param) max_param = L[i].p0;
    if (L[i].p1 > max_param) max_param = L[i].p1;
  }
  if (n_slots >= 0 && max_slot >= n_slots) return CNNK_ERR_SHAPE;
  if (n_params >= 0 && max_param >= n_params) return CNNK_ERR_SHAPE;
  w->slot_elems.assign(max_slot + 1, 0);
  w->param_elems.assign(max_param + 1, 0);
  w->wt_off.assign(n, (size_t)-1);
  w->mask_off.assign(n, (size_t)-1);
  std::vector<int> conv_uses(max_param + 1, 0);
  for (int i = 0; i < n; ++i)
    if (L[i].op == CNNK_OP_CONV && L[i].p0 >= 0) ++conv_uses[L[i].p0];
  for (int i = 0; i < n; ++i) {
    const cnnk_layer& l = L[i];
    int dt = -1;
    bool ok = true;
    switch (l.op) {
      case CNNK_OP_CONV: {
        const cnnk_conv_desc& d = l.d.conv;
        int rc = cnnk_validate_conv(&d);
        if (rc != CNNK_OK) return rc;
        dt = d.dtype;
        const int Ho = conv_out(d.H, d.pad, d.R, d.stride), Wo = conv_out(d.W, d.pad, d.S, d.stride);
        ok = l.in0 >= 0 && l.out > 0 && l.p0 >= 0 &&
             set_elems(w->slot_elems, l.in0, (size_t)d.N * d.H * d.W * d.Cin) &&
             set_elems(w->slot_elems, l.out, (size_t)d.N * Ho * Wo * d.Cout) &&
             set_elems(w->param_elems, l.p0, (size_t)d.Cout * d.R * d.S * d.Cin);
        ++w->convs;
        w->weights += (double)d.Cout * d.R * d.S * d.Cin;
        w->flops += 2.0 * d.N * Ho * Wo * d.Cout * d.R * d.S * d.Cin * (l.in0 == 0 ? 2 : 3);
        for (int p = 0; p < 3; ++p) w->ws = max_sz(w->ws, cnnk_conv2d_workspace_bytes(&d, p));
        if (!ok) break;
        if (dgrad_pretransposed(l, conv_uses[l.p0] > 1)) {
          w->wt_off[i] = w->wt_bytes;
          w->wt_bytes += align_up((size_t)d.Cout * d.R * d.S * d.Cin * sizeof(bf16_t), 256);
        } else if (l.in0 != 0 && conv_uses[l.p0] > 1) {
          w->shared_read = true;
        }
        if (w->x8_layer < 0 && l.in0 == 0 && d.dtype == CNNK_BF16 && conv_pad_supported(make_geom(&d))) {
          w->x8_layer = i;
          w->x8_off = w->wt_bytes;
          w->wt_bytes += conv_pad_x8_bytes(make_geom(&d));
        }
        break;
      }
      case CNNK_OP_BN: {
        const cnnk_bn_desc& d = l.d.bn;
        const size_t e = (size_t)d.N * d.H * d.W * d.C;
        dt = d.dtype;
        if (d.N <= 0 || d.H <= 0 || d.W <= 0 || d.C <= 0) return CNNK_ERR_SHAPE;
        if (d.C % 8 != 0 || d.C > 2048) return CNNK_ERR_UNSUPPORTED;
        if (l.in0 == 0) return CNNK_ERR_UNSUPPORTED;  // batch norm directly on the network input
        ok = l.in0 > 0 && l.out > 0 && l.p0 >= 0 && l.p1 >= 0 && set_elems(w->slot_elems, l.in0, e) &&
             set_elems(w->slot_elems, l.out, e) && (l.in1 < 0 || set_elems(w->slot_elems, l.in1, e)) &&
             set_elems(w->param_elems, l.p0, d.C) && set_elems(w->param_elems, l.p1, d.C);
        w->ws = max_sz(w->ws, cnnk_bn_workspace_bytes(&d));
        if (d.relu && l.in1 >= 0) {
          w->mask_off[i] = w->mask_bytes;
          w->mask_bytes += align_up(e / 8, 256);
        }
        break;
      }
      case CNNK_OP_POOL: {
        const cnnk_pool_desc& d = l.d.pool;
        dt = d.dtype;
        if (d.N <= 0 || d.H <= 0 || d.W <= 0 || d.C <= 0) return CNNK_ERR_SHAPE;
        if (d.C % 8 != 0) return CNNK_ERR_UNSUPPORTED;
        size_t eo;
        if (d.mode == CNNK_POOL_MAX2) {
          if ((d.H & 1) || (d.W & 1)) return CNNK_ERR_SHAPE;
          eo = (size_t)d.N * (d.H / 2) * (d.W / 2) * d.C;
        } else if (d.mode == CNNK_POOL_GAP) {
          eo = (size_t)d.N * d.C;
        } else {
          return CNNK_ERR_UNSUPPORTED;
        }
        ok = l.in0 >= 0 && l.out > 0 && set_elems(w->slot_elems, l.in0, (size_t)d.N * d.H * d.W * d.C) &&
             set_elems(w->slot_elems, l.out, eo);
        break;
      }
      case CNNK_OP_ADD: {
        const cnnk_pool_desc& d = l.d.pool;
        dt = d.dtype;
        if (d.N <= 0 || d.H <= 0 || d.W <= 0 || d.C <= 0) return CNNK_ERR_SHAPE;
        const size_t e = (size_t)d.N * d.H * d.W * d.C;
        ok = l.in0 >= 0 && l.in1 >= 0 && l.out > 0 && set_elems(w->slot_elems, l.in0, e) &&
             set_elems(w->slot_elems, l.in1, e) && set_elems(w->slot_elems, l.out, e);
        break;
      }
      case CNNK_OP_FC_LOSS: {
        const cnnk_fc_desc& d = l.d.fc;
        dt = d.dtype;
        if (i != n - 1) return CNNK_ERR_UNSUPPORTED;
        if (d.N <= 0 || d.F <= 0 || d.classes <= 0) return CNNK_ERR_SHAPE;
        if (d.classes > 4096 || d.N > 65535) return CNNK_ERR_UNSUPPORTED;
        ok = l.in0 > 0 && l.p0 >= 0 && l.p1 >= 0 && set_elems(w->slot_elems, l.in0, (size_t)d.N * d.F) &&
             set_elems(w->param_elems, l.p0, (size_t)d.classes * d.F) && set_elems(w->param_elems, l.p1, d.classes);
        w->ws = max_sz(w->ws, cnnk_fc_workspace_bytes(&d));
        break;
      }
      default:
        return CNNK_ERR_UNSUPPORTED;
    }
    if (!ok) return CNNK_ERR_SHAPE;
    if (dt != CNNK_F32 && dt != CNNK_BF16) return CNNK_ERR_UNSUPPORTED;
    if (w->dtype < 0) w->dtype = dt;
    if (dt != w->dtype) return CNNK_ERR_UNSUPPORTED;
  }
  if (L[n - 1].op != CNNK_OP_FC_LOSS) return CNNK_ERR_UNSUPPORTED;
  return CNNK_OK;
}

}  // namespace

extern "C" int cnnk_train_step_event_groups(int n_layers) { return n_layers > 0 ? 3 * n_layers - 1 : 0; }

namespace {
// Records the caller's events around one group of launches when timing was requested.
struct GroupTimer {
  void** ev;
  hipStream_t st;
  GroupTimer(const cnnk_buffers* B, int n_layers, void* stream) : ev(nullptr), st((hipStream_t)stream) {
    if (B->events && B->n_events >= 2 * cnnk_train_step_event_groups(n_layers)) ev = B->events;
  }
  void begin(int g) { if (ev) (void)hipEventRecord((hipEvent_t)ev[2 * g], st); }
  void end(int g) { if (ev) (void)hipEventRecord((hipEvent_t)ev[2 * g + 1], st); }
};
}  // namespace

extern "C" size_t cnnk_train_step_workspace_bytes(const cnnk_layer* layers, int n_layers) {
  Walk w;
  if (walk_layers(layers, n_layers, -1, -1, &w) != CNNK_OK) return 0;
  return step_workspace(w);
}

extern "C" int cnnk_train_step(const cnnk_layer* L, int n, const cnnk_buffers* B, const int* labels, float lr,
                               float momentum, float weight_decay, float* loss, int* pred, void* stream) {
  if (!B || !labels || !loss || !pred) return CNNK_ERR_NULL;
  if (!B->act || !B->dact || !B->param || !B->grad || !B->mom || !B->bn_save || !B->pool_idx) return CNNK_ERR_NULL;
  Walk w;
  int rc = walk_layers(L, n, B->n_slots, B->n_params, &w);
  if (rc != CNNK_OK) return rc;
  if (!B->ws || B->ws_bytes < step_workspace(w)) return CNNK_ERR_WORKSPACE;
  const bool bf16 = w.dtype == CNNK_BF16;
  const size_t elem = bf16 ? sizeof(bf16_t) : sizeof(float);
  for (size_t s = 0; s < w.slot_elems.size(); ++s) {
    if (w.slot_elems[s] == 0) continue;
    if (!B->act[s] || (s != 0 && !B->dact[s])) return CNNK_ERR_NULL;
  }
  for (size_t p = 0; p < w.param_elems.size(); ++p) {
    if (w.param_elems[p] == 0) continue;
    if (!B->param[p] || !B->grad[p] || !B->mom[p]) return CNNK_ERR_NULL;
  }
  for (int i = 0; i < n; ++i) {
    if (L[i].op == CNNK_OP_CONV && bf16 && (!B->param_lp || !B->param_lp[L[i].p0])) return CNNK_ERR_NULL;
    if (L[i].op == CNNK_OP_BN && !B->bn_save[i]) return CNNK_ERR_NULL;
    if (L[i].op == CNNK_OP_POOL && L[i].d.pool.mode == CNNK_POOL_MAX2 && !B->pool_idx[i]) return CNNK_ERR_NULL;
  }
  // every tensor that the backward pass reads a gradient from must receive one
  {
    std::vector<char> has(w.slot_elems.size(), 0);
    for (int i = n - 1; i >= 0; --i) {
      const cnnk_layer& l = L[i];
      if (l.op != CNNK_OP_FC_LOSS && !has[l.out]) return CNNK_ERR_SHAPE;
      has[l.in0] = 1;
      if ((l.op == CNNK_OP_BN || l.op == CNNK_OP_ADD) && l.in1 >= 0) has[l.in1] = 1;
    }
  }

  // The first kStatBytes of the workspace carry the per-channel sums from a convolution to the
  // batch norm that follows it; the calls themselves get the rest.
  float* const stat_base = reinterpret_cast<float*>(B->ws);
  int stat_slot[kStatSlots];   // tensor slot whose sums each buffer holds, -1 = free
  for (int k = 0; k < kStatSlots; ++k) stat_slot[k] = -1;
  // second stream for the weight gradients (off while per-call timing is requested)
  const bool timing = B->events && B->n_events >= 2 * cnnk_train_step_event_groups(n);
  const size_t ws_one = step_workspace(w);
  hipStream_t aux = nullptr;
  if (B->aux_stream && B->ev_fork && B->ev_join && !timing) {
    if (B->ws_bytes < 2 * ws_one) return CNNK_ERR_WORKSPACE;
    if (w.flops + kAuxWorkPerWeight * w.weights >= kAuxMinWork && !w.shared_read) aux = (hipStream_t)B->aux_stream;
  }
  void* const aux_ws = static_cast<char*>(B->ws) + ws_one;
  const size_t aux_wsb = aux ? B->ws_bytes - ws_one : 0;
  char* const wt_region = static_cast<char*>(B->ws) + kStatBytes;
  // A batch norm with a residual input keeps its ReLU mask as one bit per element for the backward pass, which
  // read the whole output for it (a third of the first pass's reads: 45.5 -> 37.9 us per layer of ResNet-50 b256, where
  // these are the widest tensors, step 8.03 -> 7.98 ms; ResNet-18 b256 unchanged).
  unsigned char* const masks = reinterpret_cast<unsigned char*>(wt_region) + w.wt_bytes;
  auto mask_of = [&](int i) { return w.mask_off[i] != (size_t)-1 && g_cnnk_tune[9] >= 0 ? masks + w.mask_off[i] : nullptr; };
  void* ws = masks + w.mask_bytes;
  const size_t wsb = (aux ? ws_one : B->ws_bytes) - kStatBytes - w.wt_bytes - w.mask_bytes;
  GroupTimer timer(B, n, stream);
  // Side branches of the forward pass: a convolution i whose output goes through a plain batch norm
  // (i+1: no ReLU, no residual) into nothing but the residual input of a later batch norm j - the
  // projection shortcut of a residual block.  With a second stream the pair runs there, launched
  // when the main stream reaches the first other reader a < i of the same input, and joined in
  // front of j.
  std::vector<int> side_of(n, -1);     // side_of[a] = i: launch the branch that starts at i before layer a
  std::vector<char> on_side(n, 0), join_before(n, 0);
  if (aux && bf16) {
    for (int i = 0; i + 1 < n; ++i) {
      const cnnk_layer& c = L[i];
      const cnnk_layer& b = L[i + 1];
      if (c.op != CNNK_OP_CONV || b.op != CNNK_OP_BN || b.in0 != c.out || b.in1 >= 0 || b.d.bn.relu) continue;
      int readers_c = 0, readers_b = 0, j = -1, a = -1;
      for (int k = 0; k < n; ++k) {
        if (L[k].op == CNNK_OP_FC_LOSS) { if (L[k].in0 == c.out || L[k].in0 == b.out) readers_b = 99; continue; }
        const bool two = L[k].op == CNNK_OP_BN || L[k].op == CNNK_OP_ADD;
        if (L[k].in0 == c.out || (two && L[k].in1 == c.out)) ++readers_c;
        if (L[k].in0 == b.out) readers_b = 99;
        if (two && L[k].in1 == b.out) { ++readers_b; j = (L[k].op == CNNK_OP_BN) ? k : -1; }
        if (a < 0 && k < i && (L[k].in0 == c.in0 || (two && L[k].in1 == c.in0))) a = k;
      }
      if (readers_c != 1 || readers_b != 1 || j <= i + 1 || a < 0 || side_of[a] >= 0) continue;
      side_of[a] = i;
      on_side[i] = on_side[i + 1] = 1;
      join_before[j] = 1;
    }
  }
  float* const aux_stat = reinterpret_cast<float*>(aux_ws);              // sums hand-off of a side branch
  void* const aux_scratch = static_cast<char*>(aux_ws) + 2 * 2048 * sizeof(float);
  const size_t aux_scratch_b = aux ? aux_wsb - 2 * 2048 * sizeof(float) : 0;
  // All weight transpositions of the data-gradient kernels in one launch (per 32 layers).  With a
  // second stream they run there beside the classifier head, whose few small launches leave the
  // device almost idle (tune key 12 = -1 keeps them on the main stream).
  auto transpose_all = [&](hipStream_t s_) -> int {
    TransposeTable t;
    t.count = 0;
    int r = CNNK_OK;
    for (int i = 0; i < n; ++i) {
      if (w.wt_off[i] == (size_t)-1) continue;
      const cnnk_conv_desc& d = L[i].d.conv;
      const int k = t.count++;
      t.src[k] = static_cast<const bf16_t*>(B->param_lp[L[i].p0]);
      t.dst[k] = reinterpret_cast<bf16_t*>(wt_region + w.wt_off[i]);
      t.Cout[k] = d.Cout; t.T[k] = d.R * d.S; t.Cin[k] = d.Cin;
      if (t.count == kMaxTranspose) {
        r = conv_transpose_weights_multi(t, s_);
        if (r != CNNK_OK) return r;
        t.count = 0;
      }
    }
    if (t.count > 0) r = conv_transpose_weights_multi(t, s_);
    return r;
  };
  // Whether convolution i may leave its channel sums as partials in the workspace: its batch norm is the next call there.
  auto takes_partials = [&](int i) {
    return i + 1 < n && L[i + 1].op == CNNK_OP_BN && L[i + 1].in0 == L[i].out && L[i + 1].d.bn.C == L[i].d.conv.Cout &&
           bn_slabs_pay_for((size_t)L[i + 1].d.bn.N * L[i + 1].d.bn.H * L[i + 1].d.bn.W, L[i + 1].d.bn.C);
  };
  PartSums handed{nullptr, 0, false};     // the last layer's
  bool wt_forked = false;
  bool x8_valid = false;   // the forward pass left the first layer's 8-channel input copy in place
  // ---- forward pass and loss ---------------------------------------------------------------
  for (int i = 0; i < n; ++i) {
    const cnnk_layer& l = L[i];
    if (side_of[i] >= 0) {
      const int s0 = side_of[i];
      const cnnk_layer& c = L[s0];
      const cnnk_layer& b = L[s0 + 1];
      if (hipEventRecord((hipEvent_t)B->ev_fork, (hipStream_t)stream) != hipSuccess ||
          hipStreamWaitEvent(aux, (hipEvent_t)B->ev_fork, 0) != hipSuccess)
        return CNNK_ERR_HIP;
      const bool sums = c.d.conv.Cout % 8 == 0 && c.d.conv.Cout <= 2048;
      PartSums ps{nullptr, 0, false};
      if (sums && takes_partials(s0)) t_cnnk_part_sums = &ps;
      rc = cnnk_conv2d_fwd(&c.d.conv, B->act[c.in0], B->param_lp[c.p0], B->act[c.out], sums ? aux_stat : nullptr,
                           sums ? aux_stat + 2048 : nullptr, aux_scratch, aux_scratch_b, aux);
      t_cnnk_part_sums = nullptr;
      if (rc != CNNK_OK) return rc;
      float* run = B->bn_running ? B->bn_running[s0 + 1] : nullptr;
      rc = bn_relu_fwd(&b.d.bn, B->act[b.in0], nullptr, B->param[b.p0], B->param[b.p1], B->act[b.out], nullptr,
                       B->bn_save[s0 + 1], B->bn_save[s0 + 1] + b.d.bn.C, run, run ? run + b.d.bn.C : nullptr,
                       sums ? aux_stat : nullptr, sums ? aux_stat + 2048 : nullptr, &ps, aux_scratch, aux_scratch_b, aux);
      if (rc != CNNK_OK) return rc;
      if (hipEventRecord((hipEvent_t)B->ev_join, aux) != hipSuccess) return CNNK_ERR_HIP;
    }
    if (on_side[i]) continue;
    if (join_before[i] && hipStreamWaitEvent((hipStream_t)stream, (hipEvent_t)B->ev_join, 0) != hipSuccess)
      return CNNK_ERR_HIP;
    timer.begin(i);
    switch (l.op) {
      case CNNK_OP_CONV: {
        const void* wt = bf16 ? B->param_lp[l.p0] : (const void*)B->param[l.p0];
        // hand the per-channel sums to the batch norm that consumes this output, if one does and
        // a buffer is free
        int sb = -1;
        if (bf16 && l.d.conv.Cout % 8 == 0 && l.d.conv.Cout <= 2048) {
          bool wanted = false;
          for (int j = i + 1; j < n && !wanted; ++j) wanted = L[j].op == CNNK_OP_BN && L[j].in0 == l.out;
          for (int k = 0; wanted && k < kStatSlots && sb < 0; ++k)
            if (stat_slot[k] < 0) sb = k;
        }
        float* ssum = sb >= 0 ? stat_base + (size_t)sb * 4096 : nullptr;
        // the 8-channel copy of the network input is kept for this layer's weight gradient
        X8Cache x8c{reinterpret_cast<bf16_t*>(wt_region + w.x8_off), false};
        if (i == w.x8_layer) t_cnnk_x8_cache = &x8c;
        handed = {nullptr, 0, false};
        if (ssum && takes_partials(i)) t_cnnk_part_sums = &handed;
        rc = cnnk_conv2d_fwd(&l.d.conv, B->act[l.in0], wt, B->act[l.out], ssum, ssum ? ssum + 2048 : nullptr, ws, wsb,
                             stream);
        t_cnnk_part_sums = nullptr;
        t_cnnk_x8_cache = nullptr;
        if (i == w.x8_layer) x8_valid = x8c.valid;
        if (sb >= 0) stat_slot[sb] = l.out;
        break;
      }
      case CNNK_OP_BN: {
        const int C = l.d.bn.C;
        float* run = B->bn_running ? B->bn_running[i] : nullptr;
        int sb = -1;
        for (int k = 0; k < kStatSlots; ++k)
          if (stat_slot[k] == l.in0) sb = k;
        const float* ssum = sb >= 0 ? stat_base + (size_t)sb * 4096 : nullptr;
        rc = bn_relu_fwd(&l.d.bn, B->act[l.in0], l.in1 >= 0 ? B->act[l.in1] : nullptr, B->param[l.p0], B->param[l.p1],
                         B->act[l.out], mask_of(i), B->bn_save[i], B->bn_save[i] + C, run, run ? run + C : nullptr, ssum,
                         ssum ? ssum + 2048 : nullptr, &handed, ws, wsb, stream);
        handed = {nullptr, 0, false};
        if (sb >= 0) stat_slot[sb] = -1;
        break;
      }
      case CNNK_OP_POOL:
        rc = cnnk_pool_fwd(&l.d.pool, B->act[l.in0], B->act[l.out], B->pool_idx[i], stream);
        break;
      case CNNK_OP_ADD:
        // A batch norm of the sum that comes next starts from partial sums made here; not of a sum in place, whose first row (what
        // the partial sums are relative to) every workgroup reads from both summands while others store
        if (i + 1 < n && L[i + 1].op == CNNK_OP_BN && L[i + 1].in0 == l.out && g_cnnk_tune[20] >= 0 &&
            add_stats_pays(w.dtype, w.slot_elems[l.out] / L[i + 1].d.bn.C, L[i + 1].d.bn.C) &&
            !share(B->act[l.out], B->act[l.in0], w.slot_elems[l.out] * elem) && !share(B->act[l.out], B->act[l.in1], w.slot_elems[l.out] * elem)) {
          const size_t rows = w.slot_elems[l.out] / L[i + 1].d.bn.C;
          rc = add_stats(w.dtype, B->act[l.in0], B->act[l.in1], B->act[l.out], rows, L[i + 1].d.bn.C, &handed, ws, (hipStream_t)stream);
        } else {
          rc = cnnk_add(w.slot_elems[l.out], w.dtype, B->act[l.in0], B->act[l.in1], B->act[l.out], stream);
        }
        break;
      case CNNK_OP_FC_LOSS:
        if (aux && g_cnnk_tune[12] >= 0) {
          if (hipEventRecord((hipEvent_t)B->ev_fork, (hipStream_t)stream) != hipSuccess ||
              hipStreamWaitEvent(aux, (hipEvent_t)B->ev_fork, 0) != hipSuccess)
            return CNNK_ERR_HIP;
          rc = transpose_all(aux);
          if (rc != CNNK_OK) return rc;
          if (hipEventRecord((hipEvent_t)B->ev_join, aux) != hipSuccess) return CNNK_ERR_HIP;
          wt_forked = true;
        }
        rc = cnnk_fc_softmax_xent(&l.d.fc, B->act[l.in0], B->param[l.p0], B->param[l.p1], labels, loss, pred,
                                  B->probs, B->dact[l.in0], B->grad[l.p0], B->grad[l.p1], ws, wsb, stream);
        break;
    }
    timer.end(i);
    if (rc != CNNK_OK) return rc;
  }
  // ---- backward pass ---------------------------------------------------------------------------
  if (!wt_forked) {
    rc = transpose_all((hipStream_t)stream);
    if (rc != CNNK_OK) return rc;
  } else if (hipStreamWaitEvent((hipStream_t)stream, (hipEvent_t)B->ev_join, 0) != hipSuccess) {
    return CNNK_ERR_HIP;
  }
  std::vector<char> written(w.slot_elems.size(), 0);
  std::vector<char> updated(w.param_elems.size(), 0);   // parameters already updated on the second stream
  written[L[n - 1].in0] = 1;
  // Second stream, several layers at a time: one fork, their weight gradients, and one launch for all their
  // reductions and updates.
  const int group = aux && bf16 ? wgrad_group(w) : 1;
  std::vector<int> pending;
  auto flush = [&]() -> int {
    if (pending.empty()) return CNNK_OK;
    if (hipEventRecord((hipEvent_t)B->ev_fork, (hipStream_t)stream) != hipSuccess ||
        hipStreamWaitEvent(aux, (hipEvent_t)B->ev_fork, 0) != hipSuccess)
      return CNNK_ERR_HIP;
    ReduceGroup rg;
    rg.count = 0;
    rg.lr = lr; rg.mu = momentum; rg.wd = weight_decay;
    SgdTable rest;
    rest.count = 0;
    size_t used = 0;
    int r = CNNK_OK;
    for (int i : pending) {
      const cnnk_layer& l = L[i];
      // the partial sums of a layer stay until the group's launch: the next layer's follow them
      if (used + cnnk_conv2d_workspace_bytes(&l.d.conv, CNNK_PASS_WGRAD) > aux_wsb) {
        r = reduce_group(rg, aux);
        if (r != CNNK_OK) return r;
        used = 0;
      }
      void* const lp = B->param_lp ? B->param_lp[l.p0] : nullptr;
      SgdFuse fuse{B->param[l.p0], B->mom[l.p0], lp, lr, momentum, weight_decay, nullptr, false, &rg};
      X8Cache x8c{reinterpret_cast<bf16_t*>(wt_region + w.x8_off), x8_valid};
      const int before = rg.count;
      t_cnnk_sgd_fuse = &fuse;
      t_cnnk_wgrad_cus = kAuxWgradCus;
      if (i == w.x8_layer && x8_valid) t_cnnk_x8_cache = &x8c;
      r = cnnk_conv2d_wgrad(&l.d.conv, B->act[l.in0], B->dact[l.out], B->grad[l.p0], static_cast<char*>(aux_ws) + used, aux_wsb - used, aux);
      t_cnnk_x8_cache = nullptr;
      t_cnnk_wgrad_cus = 256;
      t_cnnk_sgd_fuse = nullptr;
      if (r != CNNK_OK) return r;
      if (rg.count > before) {
        const ReduceItem& t = rg.it[before];
        used = (size_t)(reinterpret_cast<const char*>(t.part + (size_t)t.n * t.P) - static_cast<const char*>(aux_ws));
        used = (used + 255) / 256 * 256;
      } else if (!fuse.done) {      // nothing to reduce
        const int k = rest.count++;
        rest.w[k] = B->param[l.p0]; rest.v[k] = B->mom[l.p0]; rest.g[k] = B->grad[l.p0];
        rest.wlp[k] = lp; rest.n[k] = w.param_elems[l.p0];
      }
    }
    pending.clear();
    r = reduce_group(rg, aux);
    if (r == CNNK_OK && rest.count) r = sgd_multi(rest, lr, momentum, weight_decay, aux);
    return r;
  };
  // Tried and dropped (ResNet-18 b256, same-box A/B): (1) the backward pass of a projection shortcut
  // on the second stream - queued behind the weight gradients there it made the main stream wait,
  // 2.45 vs 2.37 ms; (2) per-channel sums through exact 64-bit integer atomics (three fixed-point
  // limbs, 8 replicas) instead of partials + a finalising launch - same-address atomics serialise
  // in L2 at 10-20 ns each: 3.29 ms with one copy, 2.42 vs 2.40 ms with eight; (3) the finalising
  // reduction inside the consuming batch-norm launch (its first workgroups reduce and publish, all
  // wait on flags with device-scope release / acquire) - the cache write-back and invalidate of
  // those fences cost far more than the launch they save: 2.68 vs 2.33 ms; (4) the weight
  // transpositions on the second stream beside the forward pass: no change (2.334 vs 2.334 ms).
  for (int i = n - 2; i >= 0; --i) {
    const cnnk_layer& l = L[i];
    const int g0 = n + 2 * (n - 2 - i);
    timer.begin(g0);
    switch (l.op) {
      case CNNK_OP_CONV: {
        // data gradient of this layer (main stream); with a second stream it is enqueued first so
        // that the event behind it exists when the weight gradient's reduction needs it
        auto dgrad = [&]() -> int {
          if (l.in0 == 0) return CNNK_OK;
          int r;
          if (w.wt_off[i] != (size_t)-1) {
            r = conv_mfma_dgrad_pt(make_geom(&l.d.conv), static_cast<const bf16_t*>(B->dact[l.out]),
                                   reinterpret_cast<const bf16_t*>(wt_region + w.wt_off[i]),
                                   static_cast<bf16_t*>(B->dact[l.in0]), written[l.in0], (hipStream_t)stream);
          } else {
            const void* wt = bf16 ? B->param_lp[l.p0] : (const void*)B->param[l.p0];
            r = cnnk_conv2d_dgrad(&l.d.conv, B->dact[l.out], wt, B->dact[l.in0], written[l.in0], ws, wsb, stream);
          }
          written[l.in0] = 1;
          return r;
        };
        if (!aux) {
          X8Cache x8c{reinterpret_cast<bf16_t*>(wt_region + w.x8_off), x8_valid};
          if (i == w.x8_layer && x8_valid) t_cnnk_x8_cache = &x8c;
          rc = cnnk_conv2d_wgrad(&l.d.conv, B->act[l.in0], B->dact[l.out], B->grad[l.p0], ws, wsb, stream);
          t_cnnk_x8_cache = nullptr;
          timer.end(g0);
          timer.begin(g0 + 1);
          if (rc == CNNK_OK) rc = dgrad();
          break;
        }
        if (group > 1) {
          rc = dgrad();
          if (rc != CNNK_OK) return rc;
          for (int k : pending)        // layers that share their weights are not updated in one launch
            if (L[k].p0 == l.p0) { rc = flush(); break; }
          if (rc != CNNK_OK) return rc;
          pending.push_back(i);
          updated[l.p0] = 1;
          if ((int)pending.size() == group) rc = flush();
          break;
        }
        // dy and x are final here: fork the weight gradient onto the second stream
        if (hipEventRecord((hipEvent_t)B->ev_fork, (hipStream_t)stream) != hipSuccess ||
            hipStreamWaitEvent(aux, (hipEvent_t)B->ev_fork, 0) != hipSuccess)
          return CNNK_ERR_HIP;
        rc = dgrad();
        if (rc != CNNK_OK) return rc;
        // The update of this layer's weights follows its weight gradient on the second stream, in the
        // split-K reduction's launch (a separate launch where nothing is reduced).  A data gradient that
        // reads the weights themselves must be done by then: the event is re-recorded behind it and the
        // update waits for it.  The matrix-core kernels read the transposed copies made before the backward
        // pass, so nothing waits for them.
        const bool after_dgrad = l.in0 != 0 && w.wt_off[i] == (size_t)-1;
        if (after_dgrad && hipEventRecord((hipEvent_t)B->ev_fork, (hipStream_t)stream) != hipSuccess)
          return CNNK_ERR_HIP;
        SgdFuse fuse{B->param[l.p0], B->mom[l.p0], (bf16 && B->param_lp) ? B->param_lp[l.p0] : nullptr,
                     lr, momentum, weight_decay, after_dgrad ? (hipEvent_t)B->ev_fork : nullptr, false, nullptr};
        t_cnnk_sgd_fuse = &fuse;
        t_cnnk_wgrad_cus = kAuxWgradCus;
        X8Cache x8c{reinterpret_cast<bf16_t*>(wt_region + w.x8_off), x8_valid};
        if (i == w.x8_layer && x8_valid) t_cnnk_x8_cache = &x8c;
        rc = cnnk_conv2d_wgrad(&l.d.conv, B->act[l.in0], B->dact[l.out], B->grad[l.p0], aux_ws, aux_wsb, aux);
        t_cnnk_x8_cache = nullptr;
        t_cnnk_wgrad_cus = 256;
        t_cnnk_sgd_fuse = nullptr;
        if (rc != CNNK_OK) return rc;
        if (!fuse.done) {
          if (after_dgrad && hipStreamWaitEvent(aux, (hipEvent_t)B->ev_fork, 0) != hipSuccess) return CNNK_ERR_HIP;
          SgdTable t1;
          t1.count = 1;
          t1.w[0] = B->param[l.p0];
          t1.v[0] = B->mom[l.p0];
          t1.g[0] = B->grad[l.p0];
          t1.wlp[0] = (bf16 && B->param_lp) ? B->param_lp[l.p0] : nullptr;
          t1.n[0] = w.param_elems[l.p0];
          rc = sgd_multi(t1, lr, momentum, weight_decay, aux);
        }
        updated[l.p0] = 1;
        break;
      }
      case CNNK_OP_BN: {
        const int C = l.d.bn.C;
        const bool res = l.in1 > 0;
        const int flags = (written[l.in0] ? 1 : 0) | ((res && written[l.in1]) ? 2 : 0);
        // without a residual branch the ReLU mask is recomputed from x (y is not read)
        const void* ymask = (l.d.bn.relu && !res && g_cnnk_tune[9] >= 0) ? nullptr : B->act[l.out];
        rc = bn_relu_bwd(&l.d.bn, B->dact[l.out], B->act[l.in0], ymask, mask_of(i), B->param[l.p0], B->param[l.p1],
                         B->bn_save[i], B->bn_save[i] + C, B->dact[l.in0], res ? B->dact[l.in1] : nullptr, flags,
                         B->grad[l.p0], B->grad[l.p1], ws, wsb, stream);
        written[l.in0] = 1;
        if (res) written[l.in1] = 1;
        break;
      }
      case CNNK_OP_POOL:
        if (l.in0 != 0) {
          rc = cnnk_pool_bwd(&l.d.pool, B->dact[l.out], B->pool_idx[i], B->dact[l.in0], written[l.in0], stream);
          written[l.in0] = 1;
        }
        break;
      case CNNK_OP_ADD: {
        const int ins[2] = {l.in0, l.in1};
        const size_t bytes = w.slot_elems[l.out] * elem;
        if (l.in0 != 0 && l.in1 != 0 && g_cnnk_tune[20] >= 0 && !share(B->dact[l.in0], B->dact[l.in1], bytes) &&
            !share(B->dact[l.in0], B->dact[l.out], bytes) && !share(B->dact[l.in1], B->dact[l.out], bytes)) {
          rc = grad_route2(w.slot_elems[l.out], w.dtype, B->dact[l.out], B->dact[l.in0], written[l.in0], B->dact[l.in1], written[l.in1], (hipStream_t)stream);
          written[l.in0] = written[l.in1] = 1;
          break;
        }
        for (int k = 0; k < 2 && rc == CNNK_OK; ++k) {
          if (ins[k] == 0) continue;
          rc = cnnk_grad_route(w.slot_elems[l.out], w.dtype, B->dact[l.out], B->dact[ins[k]], written[ins[k]], stream);
          written[ins[k]] = 1;
        }
        break;
      }
      default:
        break;
    }
    if (l.op != CNNK_OP_CONV) {
      timer.end(g0);
      timer.begin(g0 + 1);
    }
    timer.end(g0 + 1);
    if (rc != CNNK_OK) return rc;
  }
  rc = flush();
  if (rc != CNNK_OK) return rc;
  // ---- parameter update -----------------------------------------------------------------------
  // With a second stream the parameters that are left (batch-norm and classifier parameters: their
  // gradients were computed on this stream) are updated first; the wait for the tail of the other
  // stream (the first layer's weight gradient and update) comes last, so the two overlap.
  const int g_upd = cnnk_train_step_event_groups(n) - 1;
  timer.begin(g_upd);
  SgdTable t;
  t.count = 0;
  for (size_t p = 0; p < w.param_elems.size(); ++p) {
    if (w.param_elems[p] == 0 || updated[p]) continue;
    const int k = t.count++;
    t.w[k] = B->param[p];
    t.v[k] = B->mom[p];
    t.g[k] = B->grad[p];
    t.wlp[k] = (bf16 && B->param_lp) ? B->param_lp[p] : nullptr;
    t.n[k] = w.param_elems[p];
    if (t.count == kSgdMaxTensors) {
      rc = sgd_multi(t, lr, momentum, weight_decay, (hipStream_t)stream);
      if (rc != CNNK_OK) return rc;
      t.count = 0;
    }
  }
  if (t.count > 0) rc = sgd_multi(t, lr, momentum, weight_decay, (hipStream_t)stream);
  timer.end(g_upd);
  if (aux && rc == CNNK_OK) {
    if (hipEventRecord((hipEvent_t)B->ev_join, aux) != hipSuccess ||
        hipStreamWaitEvent((hipStream_t)stream, (hipEvent_t)B->ev_join, 0) != hipSuccess)
      return CNNK_ERR_HIP;
  }
  return rc;
}

// Validation pass: the forward half of the step in inference mode.
extern "C" int cnnk_eval_step(const cnnk_layer* L, int n, const cnnk_buffers* B, const int* labels, float* loss,
                              int* pred, int* n_correct, void* stream) {
  if (!B || !labels || !loss || !pred) return CNNK_ERR_NULL;
  if (!B->act || !B->param || !B->bn_running || !B->pool_idx) return CNNK_ERR_NULL;
  Walk w;
  int rc = walk_layers(L, n, B->n_slots, B->n_params, &w);
  if (rc != CNNK_OK) return rc;
  if (!B->ws || B->ws_bytes < align_up(w.ws, 256) + kStatBytes + w.wt_bytes) return CNNK_ERR_WORKSPACE;
  const bool bf16 = w.dtype == CNNK_BF16;
  for (size_t s = 0; s < w.slot_elems.size(); ++s)
    if (w.slot_elems[s] != 0 && !B->act[s]) return CNNK_ERR_NULL;
  for (size_t p = 0; p < w.param_elems.size(); ++p)
    if (w.param_elems[p] != 0 && !B->param[p]) return CNNK_ERR_NULL;
  for (int i = 0; i < n; ++i) {
    if (L[i].op == CNNK_OP_CONV && bf16 && (!B->param_lp || !B->param_lp[L[i].p0])) return CNNK_ERR_NULL;
    if (L[i].op == CNNK_OP_BN && !B->bn_running[i]) return CNNK_ERR_NULL;
    if (L[i].op == CNNK_OP_POOL && L[i].d.pool.mode == CNNK_POOL_MAX2 && !B->pool_idx[i]) return CNNK_ERR_NULL;
  }
  void* ws = static_cast<char*>(B->ws) + kStatBytes + w.wt_bytes;
  const size_t wsb = B->ws_bytes - kStatBytes - w.wt_bytes;
  // A convolution whose output goes into nothing but one batch norm (or one sum) is run when the walk
  // reaches that layer, which then is the tail of the convolution's own launch: the pass over the
  // convolution's output is saved (ResNet-50 at batch 200: 0.7 of 2.2 ms).  Only where every tensor has one
  // writer and memory of its own, so that the convolution's input is what it was, also while it is read.
  std::vector<int> tail_of(n, -1);    // tail_of[j] = i: layer j runs as the tail of convolution i
  std::vector<char> deferred(n, 0);
  if (bf16) {
    std::vector<int> readers(w.slot_elems.size(), 0), writers(w.slot_elems.size(), 0), conv_of(w.slot_elems.size(), -1);
    for (int i = 0; i < n; ++i) {
      const cnnk_layer& l = L[i];
      ++readers[l.in0];
      if ((l.op == CNNK_OP_BN || l.op == CNNK_OP_ADD) && l.in1 >= 0) ++readers[l.in1];
      if (l.op != CNNK_OP_FC_LOSS) ++writers[l.out];
      if (l.op == CNNK_OP_CONV) conv_of[l.out] = i;
    }
    bool single = writers[0] == 0;
    std::vector<std::pair<const char*, size_t>> mem;
    for (size_t s = 0; s < writers.size(); ++s) {
      single = single && writers[s] <= 1;
      if (w.slot_elems[s] != 0) mem.emplace_back(static_cast<const char*>(B->act[s]), w.slot_elems[s] * sizeof(bf16_t));
    }
    std::sort(mem.begin(), mem.end());
    for (size_t k = 0; k + 1 < mem.size(); ++k) single = single && mem[k].first + mem[k].second <= mem[k + 1].first;
    auto alone = [&](int slot) { return slot >= 0 && conv_of[slot] >= 0 && readers[slot] == 1 ? conv_of[slot] : -1; };
    for (int j = 0; j < n && single; ++j) {
      const cnnk_layer& l = L[j];
      int i = -1;
      if (l.op == CNNK_OP_BN) i = alone(l.in0);
      if (l.op == CNNK_OP_ADD && l.in0 != l.in1) i = alone(l.in0) >= 0 ? alone(l.in0) : alone(l.in1);
      if (i < 0 || i > j || !conv_tail_supported(&L[i].d.conv)) continue;
      if (l.op == CNNK_OP_BN && l.d.bn.C != L[i].d.conv.Cout) continue;
      tail_of[j] = i;
      deferred[i] = 1;
    }
  }
  for (int i = 0; i < n && rc == CNNK_OK; ++i) {
    const cnnk_layer& l = L[i];
    if (deferred[i]) continue;
    if (tail_of[i] >= 0) {
      const cnnk_layer& c = L[tail_of[i]];
      ConvTail t{};
      if (l.op == CNNK_OP_BN) {
        t.gamma = B->param[l.p0]; t.beta = B->param[l.p1];
        t.mean = B->bn_running[i]; t.var = B->bn_running[i] + l.d.bn.C;
        t.eps = l.d.bn.eps; t.relu = l.d.bn.relu;
        t.res = l.in1 >= 0 ? static_cast<const bf16_t*>(B->act[l.in1]) : nullptr;
      } else {
        t.res = static_cast<const bf16_t*>(B->act[l.in0 == c.out ? l.in1 : l.in0]);
      }
      rc = conv_fwd_tail(&c.d.conv, B->act[c.in0], B->param_lp[c.p0], B->act[l.out], t, ws, wsb, (hipStream_t)stream);
      continue;
    }
    switch (l.op) {
      case CNNK_OP_CONV: {
        const void* wt = bf16 ? B->param_lp[l.p0] : (const void*)B->param[l.p0];
        rc = cnnk_conv2d_fwd(&l.d.conv, B->act[l.in0], wt, B->act[l.out], nullptr, nullptr, ws, wsb, stream);
        break;
      }
      case CNNK_OP_BN: {
        const float* run = B->bn_running[i];
        rc = cnnk_bn_relu_infer(&l.d.bn, B->act[l.in0], l.in1 >= 0 ? B->act[l.in1] : nullptr, B->param[l.p0],
                                B->param[l.p1], run, run + l.d.bn.C, B->act[l.out], stream);
        break;
      }
      case CNNK_OP_POOL:
        rc = cnnk_pool_fwd(&l.d.pool, B->act[l.in0], B->act[l.out], B->pool_idx[i], stream);
        break;
      case CNNK_OP_ADD:
        rc = cnnk_add(w.slot_elems[l.out], w.dtype, B->act[l.in0], B->act[l.in1], B->act[l.out], stream);
        break;
      case CNNK_OP_FC_LOSS:
        rc = cnnk_fc_softmax_xent(&l.d.fc, B->act[l.in0], B->param[l.p0], B->param[l.p1], labels, loss, pred,
                                  B->probs, nullptr, nullptr, nullptr, ws, wsb, stream);
        if (rc == CNNK_OK && n_correct) rc = cnnk_count_correct(l.d.fc.N, pred, labels, n_correct, stream);
        break;
    }
  }
  return rc;
}
