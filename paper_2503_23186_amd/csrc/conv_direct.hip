// Direct (non-MFMA) convolution kernels: the fp32 mode, and bf16 shapes the MFMA engine does
// not take (channel counts that are not multiples of 8, e.g. the 3-channel stem).
// One thread per output element, fp32 accumulation in a fixed order.
#include "common.h"
#include "conv.h"

namespace {

template <typename T, int Q>
__global__ void __launch_bounds__(256) direct_fwd_kernel(ConvGeom g, const T* __restrict__ x,
                                                         const T* __restrict__ w, T* __restrict__ y) {
  const size_t total = (size_t)g.N * g.Ho * g.Wo * g.Cout;
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= total) return;
  int k, wo, ho, n;
  if (total <= 0xffffffffu) {        // 32-bit divisions: a 64-bit one is over a hundred instructions, and nothing loads before them
    unsigned m = (unsigned)idx / (unsigned)g.Cout;
    k = (int)((unsigned)idx - m * (unsigned)g.Cout);
    const unsigned q = m / (unsigned)g.Wo;
    wo = (int)(m - q * (unsigned)g.Wo);
    n = (int)(q / (unsigned)g.Ho);
    ho = (int)(q - (unsigned)n * (unsigned)g.Ho);
  } else {
    k = (int)(idx % g.Cout);
    size_t m = idx / g.Cout;
    wo = (int)(m % g.Wo); m /= g.Wo;
    ho = (int)(m % g.Ho);
    n = (int)(m / g.Ho);
  }
  // The taps of a filter row are S * Cin consecutive elements of the image and of the filter; those inside the image
  // are [t0, t1).  Q at a time, all loads issued before the first product (tap by tap a 3x3 filter over three channels was nine memory
  // latencies; 8 x 32 x 32 positions of 16 channels 7.6 -> 6.9 us); past the end the last one is read again and not used, which only the last
  // group has to look at (in every group it keeps the loads one element wide: 512 x 16 x 16
  // positions, 16 -> 32 channels, 1148 us, so 195; 32 x 32 of three channels, eight images, 5.7 and 4.3).
  const int wi0 = wo * g.stride - g.pad;
  const int t0 = (wi0 < 0 ? -wi0 : 0) * g.Cin, t1 = min(g.S, g.W - wi0) * g.Cin;
  float acc = 0.f;
  for (int r = 0; r < g.R; ++r) {
    const int hi = ho * g.stride + r - g.pad;
    if (hi < 0 || hi >= g.H || t0 >= t1) continue;
    const T* xp = x + (((long)n * g.H + hi) * g.W + wi0) * g.Cin;
    const T* wp = w + ((size_t)k * g.R + r) * g.S * g.Cin;
    int t = t0;
    for (; t + Q <= t1; t += Q) {
      float xv[Q], wv[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        xv[q] = Elem<T>::ld(xp + t + q);
        wv[q] = Elem<T>::ld(wp + t + q);
      }
#pragma unroll
      for (int q = 0; q < Q; ++q) acc = fmaf(xv[q], wv[q], acc);
    }
    if (t < t1) {
      float xv[Q], wv[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int u = min(t + q, t1 - 1);
        xv[q] = Elem<T>::ld(xp + u);
        wv[q] = Elem<T>::ld(wp + u);
      }
#pragma unroll
      for (int q = 0; q < Q; ++q)
        if (t + q < t1) acc = fmaf(xv[q], wv[q], acc);
    }
  }
  Elem<T>::st(y + idx, acc);
}

template <typename T>
__global__ void __launch_bounds__(256) direct_dgrad_kernel(ConvGeom g, const T* __restrict__ dy,
                                                           const T* __restrict__ w, T* __restrict__ dx,
                                                           int accumulate) {
  const size_t total = (size_t)g.N * g.H * g.W * g.Cin;
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= total) return;
  const int c = (int)(idx % g.Cin);
  size_t m = idx / g.Cin;
  const int wi = (int)(m % g.W); m /= g.W;
  const int hi = (int)(m % g.H);
  const int n = (int)(m / g.H);
  float acc = 0.f;
  for (int r = 0; r < g.R; ++r) {
    const int th = hi + g.pad - r;
    if (th < 0 || th % g.stride != 0) continue;
    const int ho = th / g.stride;
    if (ho >= g.Ho) continue;
    for (int s = 0; s < g.S; ++s) {
      const int tw = wi + g.pad - s;
      if (tw < 0 || tw % g.stride != 0) continue;
      const int wo = tw / g.stride;
      if (wo >= g.Wo) continue;
      const T* dyp = dy + (((size_t)n * g.Ho + ho) * g.Wo + wo) * g.Cout;
      const T* wp = w + ((size_t)r * g.S + s) * g.Cin + c;
      const size_t wk = (size_t)g.R * g.S * g.Cin;
      for (int k = 0; k < g.Cout; ++k) acc = fmaf(Elem<T>::ld(dyp + k), Elem<T>::ld(wp + k * wk), acc);
    }
  }
  if (accumulate) acc += Elem<T>::ld(dx + idx);
  Elem<T>::st(dx + idx, acc);
}

// Partial weight gradient over the output positions [p*chunk, (p+1)*chunk) into part[p][i].  H threads share a sum, a run of the
// positions each, Q positions a round (see below).
template <typename T, int H, int Q>
__global__ void __launch_bounds__(256) direct_wgrad_kernel(ConvGeom g, const T* __restrict__ x,
                                                           const T* __restrict__ dy,
                                                           float* __restrict__ part, int chunk) {
  __shared__ float other[H > 1 ? 256 / H : 1];
  const int nw = g.Cout * g.R * g.S * g.Cin;
  const int col = threadIdx.x % (256 / H), run = H == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / (256 / H));     // whole wavefronts
  const int mine = blockIdx.x * (256 / H) + col;
  if (H == 1 && mine >= nw) return;
  const int i = H == 1 ? mine : min(mine, nw - 1);
  const int c = i % g.Cin;
  int t = i / g.Cin;
  const int s = t % g.S; t /= g.S;
  const int r = t % g.R;
  const int kk = t / g.R;
  const long M = (long)g.N * g.Ho * g.Wo;
  const long end = ((long)blockIdx.y + 1) * chunk < M ? ((long)blockIdx.y + 1) * chunk : M;
  const int per = (chunk + H - 1) / H;
  const long m0 = (long)blockIdx.y * chunk + run * per;
  const long m1 = m0 + per < end ? m0 + per : end;
  // Q positions per round, all loads issued before the first product (one position at a time is a
  // chain of memory latencies behind 64-bit divisions: 29 us for a 3->16 gradient of 8192 positions, 64 to a sum;
  // with its reduction eight at a time 14.6, sixteen and two threads to a sum 11.5); a position outside the image or the range reads element 0 and multiplies zero.  The
  // position's coordinates advance by one, as the positions do.
  int wo, ho, n;
  {
    if (M <= 0x7fffffffL) {
      const unsigned q = (unsigned)m0 / (unsigned)g.Wo;
      wo = (int)((unsigned)m0 - q * (unsigned)g.Wo);
      n = (int)(q / (unsigned)g.Ho);
      ho = (int)(q - (unsigned)n * (unsigned)g.Ho);
    } else {
      wo = (int)(m0 % g.Wo);
      const long q = m0 / g.Wo;
      ho = (int)(q % g.Ho);
      n = (int)(q / g.Ho);
    }
  }
  float acc = 0.f;
  for (long m = m0; m < m1; m += Q) {
    float dv[Q], xv[Q];
#pragma unroll
    for (int k = 0; k < Q; ++k) {
      const int hi = ho * g.stride + r - g.pad, wi = wo * g.stride + s - g.pad;
      const bool ok = m + k < m1 && hi >= 0 && hi < g.H && wi >= 0 && wi < g.W;
      const float d = Elem<T>::ld(dy + (ok ? (size_t)(m + k) * g.Cout + kk : (size_t)0));
      xv[k] = Elem<T>::ld(x + (ok ? (((size_t)n * g.H + hi) * g.W + wi) * g.Cin + c : (size_t)0));
      dv[k] = d;
      if (!ok) { dv[k] = 0.f; xv[k] = 0.f; }
      if (++wo == g.Wo) { wo = 0; if (++ho == g.Ho) { ho = 0; ++n; } }
    }
#pragma unroll
    for (int k = 0; k < Q; ++k) acc = fmaf(dv[k], xv[k], acc);
  }
  if (H > 1) {
    if (run == 1) other[col] = acc;
    __syncthreads();
    if (run > 0) return;
    acc += other[col];
  }
  if (mine < nw) part[(size_t)blockIdx.y * nw + i] = acc;
}

// out[i] = sum_p part[p][i], deterministic.  GROUPS thread groups share the P partials of a float4 column (group g takes p = g, g+GROUPS, ...);
// their sums are combined through LDS in group order.  More groups = more, shorter-lived threads:
// 16 for many partials (a 64x576 gradient split 108 ways is 16 MB to read), 4 otherwise.
struct SgdArgs {
  float* w;
  float* v;
  bf16_t* wlp;
  float lr, mu, wd;
};

__device__ __forceinline__ float sgd_apply(float wi, float vi, float gi, const SgdArgs& sg, float* vn) {
  const float gp = fmaf(sg.wd, wi, gi);
  *vn = fmaf(sg.mu, vi, gp);
  return fmaf(-sg.lr, *vn, wi);
}

// workgroup `block` of the reduction of one tensor; mem: 256 float4 of LDS
template <int GROUPS, bool SGD>
__device__ __forceinline__ void reduce_block(const float* __restrict__ part, float* __restrict__ out, int n, int P,
                                             const SgdArgs& sg, int block, float4* mem) {
  constexpr int COLS = 256 / GROUPS;
  float4(*red)[COLS] = reinterpret_cast<float4(*)[COLS]>(mem);
  const int col = threadIdx.x % COLS, grp = threadIdx.x / COLS;
  const int i4 = block * COLS + col;   // float4 column
  const int n4 = n >> 2;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  // weight and momentum of the fused update are fetched under the partial sums
  float4 wv = make_float4(0.f, 0.f, 0.f, 0.f), vv = wv;
  if (SGD && grp == 0 && i4 < n4) {
    wv = *reinterpret_cast<const float4*>(sg.w + (size_t)i4 * 4);
    vv = *reinterpret_cast<const float4*>(sg.v + (size_t)i4 * 4);
  }
  if (i4 < n4) {
    // up to eight partials per round, all loads issued before the first add: the sum is a chain of
    // memory latencies otherwise (a partial past the end is not loaded and adds zero).  Same order
    // of additions as a plain loop.
    const float* base = part + (size_t)i4 * 4;
    const int rounds = (P + GROUPS - 1) / GROUPS;
    for (int k0 = 0; k0 < rounds; k0 += 8) {
      float4 v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int p = grp + (k0 + k) * GROUPS;
        v[k] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (p < P) v[k] = *reinterpret_cast<const float4*>(base + (size_t)p * n);
      }
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (k0 + k < rounds) { acc.x += v[k].x; acc.y += v[k].y; acc.z += v[k].z; acc.w += v[k].w; }
    }
  }
  red[grp][col] = acc;
  __syncthreads();
  if (grp == 0 && i4 < n4) {
    float4 s = red[0][col];
#pragma unroll
    for (int k = 1; k < GROUPS; ++k) { s.x += red[k][col].x; s.y += red[k][col].y; s.z += red[k][col].z; s.w += red[k][col].w; }
    *reinterpret_cast<float4*>(out + (size_t)i4 * 4) = s;
    if (SGD) {   // the parameter update on the gradient just summed (same arithmetic as the SGD kernel)
      const size_t i = (size_t)i4 * 4;
      float4 vn, wn;
      wn.x = sgd_apply(wv.x, vv.x, s.x, sg, &vn.x);
      wn.y = sgd_apply(wv.y, vv.y, s.y, sg, &vn.y);
      wn.z = sgd_apply(wv.z, vv.z, s.z, sg, &vn.z);
      wn.w = sgd_apply(wv.w, vv.w, s.w, sg, &vn.w);
      *reinterpret_cast<float4*>(sg.v + i) = vn;
      *reinterpret_cast<float4*>(sg.w + i) = wn;
      if (sg.wlp) {
        uint2 pk;
        pk.x = (unsigned)f32_to_bf16(wn.x) | ((unsigned)f32_to_bf16(wn.y) << 16);
        pk.y = (unsigned)f32_to_bf16(wn.z) | ((unsigned)f32_to_bf16(wn.w) << 16);
        *reinterpret_cast<uint2*>(sg.wlp + i) = pk;
      }
    }
  }
  // scalar tail (n not a multiple of 4)
  if (block == 0 && threadIdx.x < (n & 3)) {
    const int i = (n4 << 2) + threadIdx.x;
    float a = 0.f;
    for (int p = 0; p < P; ++p) a += part[(size_t)p * n + i];
    out[i] = a;
    if (SGD) {
      float vn;
      const float wn = sgd_apply(sg.w[i], sg.v[i], a, sg, &vn);
      sg.v[i] = vn;
      sg.w[i] = wn;
      if (sg.wlp) sg.wlp[i] = f32_to_bf16(wn);
    }
  }
}

template <int GROUPS, bool SGD>
__global__ void __launch_bounds__(256) reduce_partials_kernel(const float* __restrict__ part,
                                                              float* __restrict__ out, int n, int P, SgdArgs sg) {
  __shared__ float4 mem[256];
  reduce_block<GROUPS, SGD>(part, out, n, P, sg, blockIdx.x, mem);
}

// The reductions and updates of several tensors in one launch (each alone is 4 to 9 us, most of it the launch and
// one chain of memory latencies).
constexpr int kManyPartials = 32;      // from here on sixteen threads share a column, four below
__global__ void __launch_bounds__(256) reduce_group_kernel(ReduceGroup g) {
  __shared__ float4 mem[256];
  int k = 0;
  while (k + 1 < g.count && (int)blockIdx.x >= g.it[k + 1].block0) ++k;
  const ReduceItem& t = g.it[k];
  const SgdArgs sg{t.w, t.v, t.wlp, g.lr, g.mu, g.wd};
  const int block = blockIdx.x - t.block0;
  if (t.P >= kManyPartials) reduce_block<16, true>(t.part, t.out, t.n, t.P, sg, block, mem);
  else reduce_block<4, true>(t.part, t.out, t.n, t.P, sg, block, mem);
}

void wgrad_split(const ConvGeom& g, int* chunk, int* P) {
  const long M = (long)g.N * g.Ho * g.Wo;
  const long nw = (long)g.Cout * g.R * g.S * g.Cin;
  const long out_blocks = (nw + 255) / 256;
  long want = (2048 + out_blocks - 1) / out_blocks;
  const long maxP = (M + 63) / 64;
  if (want > maxP) want = maxP;
  if (want > 4096) want = 4096;
  if (want < 1) want = 1;
  long ch = (M + want - 1) / want;
  *chunk = (int)ch;
  *P = (int)((M + ch - 1) / ch);
}

}  // namespace

size_t conv_direct_wgrad_ws(const ConvGeom& g) {
  int chunk, P;
  wgrad_split(g, &chunk, &P);
  return (size_t)P * g.Cout * g.R * g.S * g.Cin * sizeof(float);
}

int conv_direct_fwd(const ConvGeom& g, int dtype, const void* x, const void* w, void* y, hipStream_t st) {
  const size_t total = (size_t)g.N * g.Ho * g.Wo * g.Cout;
  const unsigned blocks = (unsigned)((total + 255) / 256);
  // groups that a filter row of three channels fills, or one of 8, 16, .. (sixteen at a time: the same within 4 %)
  const bool nine = g.S * g.Cin % 9 == 0;
  auto run = [&](auto kernel, auto t) {
    using T = decltype(t);
    kernel<<<blocks, 256, 0, st>>>(g, (const T*)x, (const T*)w, (T*)y);
  };
  if (dtype == CNNK_BF16) nine ? run(direct_fwd_kernel<bf16_t, 9>, bf16_t{}) : run(direct_fwd_kernel<bf16_t, 8>, bf16_t{});
  else nine ? run(direct_fwd_kernel<float, 9>, float{}) : run(direct_fwd_kernel<float, 8>, float{});
  return launch_status();
}

int conv_direct_dgrad(const ConvGeom& g, int dtype, const void* dy, const void* w, void* dx, int accumulate,
                      hipStream_t st) {
  const size_t total = (size_t)g.N * g.H * g.W * g.Cin;
  const unsigned blocks = (unsigned)((total + 255) / 256);
  if (dtype == CNNK_BF16)
    direct_dgrad_kernel<bf16_t><<<blocks, 256, 0, st>>>(g, (const bf16_t*)dy, (const bf16_t*)w, (bf16_t*)dx, accumulate);
  else
    direct_dgrad_kernel<float><<<blocks, 256, 0, st>>>(g, (const float*)dy, (const float*)w, (float*)dx, accumulate);
  return launch_status();
}

int conv_direct_wgrad(const ConvGeom& g, int dtype, const void* x, const void* dy, float* dw, void* ws,
                      hipStream_t st) {
  int chunk, P;
  wgrad_split(g, &chunk, &P);
  const int nw = g.Cout * g.R * g.S * g.Cin;
  float* part = (float*)ws;
  // From 17 to 64 positions a sum is three to eight rounds of eight: two threads share it.  (Twice the partial sums instead took twice the
  // scratch, and their reduction what the shorter sums gave: 512 images of 9 x 9, 5 -> 7 strided, one thread 39 us, twice the sums 60, two threads 34.
  // Longer sums, one / two threads: 64 x 16 x 16 positions, 16 -> 32 channels 76 / 84.)
  const bool pairs = chunk > 16 && chunk <= 64;
  auto run = [&](auto kernel, int cols, auto t) {
    using T = decltype(t);
    kernel<<<dim3((nw + cols - 1) / cols, P), 256, 0, st>>>(g, (const T*)x, (const T*)dy, part, chunk);
  };
  if (dtype == CNNK_BF16) pairs ? run(direct_wgrad_kernel<bf16_t, 2, 16>, 128, bf16_t{}) : run(direct_wgrad_kernel<bf16_t, 1, 8>, 256, bf16_t{});
  else pairs ? run(direct_wgrad_kernel<float, 2, 16>, 128, float{}) : run(direct_wgrad_kernel<float, 1, 8>, 256, float{});
  if (launch_status() != CNNK_OK) return CNNK_ERR_HIP;
  return reduce_partials(part, dw, nw, P, st);
}

thread_local SgdFuse* t_cnnk_sgd_fuse = nullptr;

static unsigned reduce_blocks_for(int n, int P) { return (unsigned)(P >= kManyPartials ? (n / 4 + 15) / 16 + 1 : (n / 4 + 63) / 64 + 1); }

int reduce_group(ReduceGroup& g, hipStream_t st) {
  if (g.count == 0) return CNNK_OK;
  int blocks = 0;
  for (int k = 0; k < g.count; ++k) {
    g.it[k].block0 = blocks;
    blocks += (int)reduce_blocks_for(g.it[k].n, g.it[k].P);
  }
  reduce_group_kernel<<<blocks, 256, 0, st>>>(g);
  g.count = 0;
  return launch_status();
}

int reduce_partials(const float* part, float* out, int n, int P, hipStream_t st) {
  const unsigned g16 = reduce_blocks_for(n, kManyPartials), g4 = reduce_blocks_for(n, 0);
  SgdFuse* f = t_cnnk_sgd_fuse;
  if (f && !f->done && ((((size_t)f->w | (size_t)f->v | (size_t)out) & 15) == 0) && (((size_t)f->wlp & 7) == 0)) {
    if (f->group && f->group->count < kReduceGroup) {
      f->group->it[f->group->count++] = ReduceItem{part, out, f->w, f->v, static_cast<bf16_t*>(f->wlp), n, P, 0};
      f->done = true;
      return CNNK_OK;
    }
    if (f->wait && hipStreamWaitEvent(st, f->wait, 0) != hipSuccess) return CNNK_ERR_HIP;
    const SgdArgs sg{f->w, f->v, static_cast<bf16_t*>(f->wlp), f->lr, f->mu, f->wd};
    if (P >= kManyPartials) reduce_partials_kernel<16, true><<<g16, 256, 0, st>>>(part, out, n, P, sg);
    else reduce_partials_kernel<4, true><<<g4, 256, 0, st>>>(part, out, n, P, sg);
    f->done = true;
    return launch_status();
  }
  const SgdArgs none{nullptr, nullptr, nullptr, 0.f, 0.f, 0.f};
  if (P >= kManyPartials) reduce_partials_kernel<16, false><<<g16, 256, 0, st>>>(part, out, n, P, none);
  else reduce_partials_kernel<4, false><<<g4, 256, 0, st>>>(part, out, n, P, none);
  return launch_status();
}
