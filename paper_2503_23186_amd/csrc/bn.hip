// Batch norm (+ residual) (+ ReLU), forward and backward, for NHWC tensors viewed as [m][C].
// Bandwidth-bound: every thread moves 16-byte (bf16) or 32-byte (fp32) vectors of 8 channels,
// per-channel reductions are per-thread partial sums -> LDS -> per-workgroup partials -> a small
// finalising kernel that sums the partials in double precision (fixed order, no atomics).
#include "common.h"
#include <type_traits>
#include "conv.h"

namespace {

constexpr int kT = 256;
constexpr int kMaxBlocks = 2048;

struct RowMap {
  int lanes;   // threads per row = C/8
  int rows;    // rows per workgroup pass = 256 / lanes
};

inline int reduce_blocks(size_t m, int C) {
  const int rows = kT / (C / 8);
  // at least 8 rows per thread (ResNet-18 b256 step: 2.215 ms with 4, 2.195 with 8, 2.27 with 16)
  size_t nb = (m + (size_t)rows * 8 - 1) / ((size_t)rows * 8);
  // a tensor that leaves CUs idle that way: one round of four rows per thread (the launch is then a
  // chain of memory latencies, and a shorter one)
  if (nb < 256) nb = (m + (size_t)rows * 4 - 1) / ((size_t)rows * 4);
  if (nb > kMaxBlocks) nb = kMaxBlocks;
  // every workgroup ends with 2*C scattered 4-byte writes of its partial sums: with many channels
  // fewer, longer-lived workgroups are cheaper (C = 1024: 256 instead of 2048; ResNet-50
  // b256 step 9.57 -> 9.08 ms, 128 or 512 are worse or equal)
  size_t cap = (size_t)262144 / (size_t)C;
  if (cap < 256) cap = 256;
  if (nb > cap) nb = cap;
  if (nb < 1) nb = 1;
  return (int)nb;
}

// Sum the two per-thread vectors of 8 channels over the threads that share a channel octet and
// write them to part[v][c][block] (row block fastest, so the finaliser reads rows).  Up to 32 channels wide `groups` threads share a sum, each
// a run of the rows (one thread each, the 128 rows of 16 channels were a chain of 128 reads: 8 x 32 x 32 7.5 -> 5.2 us).
template <class W>
__device__ __forceinline__ void block_reduce_store(float (*acc)[8], const W& w, int C, float* __restrict__ part) {
  __shared__ float red[2][kT * 8];
  __shared__ float sub[kT];
  const int tid = threadIdx.x, width = w.lanes * 8, sums = 2 * width;
  if (w.rl < w.rows) {
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
      for (int e = 0; e < 8; ++e) red[v][tid * 8 + e] = acc[v][e];
  }
  __syncthreads();
  if (sums <= kT / 4) {
    const int groups = kT / sums, per = (w.rows + groups - 1) / groups, i = tid % sums, g = tid / sums;
    float s = 0.f;
    if (g < groups) {
      const float* q = i < width ? &red[0][i] : &red[1][i - width];
      for (int r = g * per; r < min((g + 1) * per, w.rows); ++r) s += q[r * width];
    }
    sub[tid] = s;
    __syncthreads();
    if (tid < sums) {
      for (int k = 1; k < groups; ++k) s += sub[k * sums + tid];
      part[((size_t)(i >= width) * C + w.slab0 + (i >= width ? i - width : i)) * w.blocks + w.block] = s;
    }
    return;
  }
  for (int i = tid; i < sums; i += kT) {
    const int v = i >= width, c = i - v * width;
    float s = 0.f;
    for (int r = 0; r < w.rows; ++r) s += red[v][r * width + c];
    part[((size_t)v * C + w.slab0 + c) * w.blocks + w.block] = s;
  }
}

// Finalising reduction of the nb per-workgroup partials part[v][c][0..nb) in double: one wavefront per channel (four channels
// per workgroup), the lanes stride over the partials and add up across the wavefront (wave_sum, the total in every
// lane).  Fixed order, no LDS, no barrier.
constexpr int kFinCh = kT / 64;   // channels per finalising workgroup
inline unsigned fin_blocks(int C) { return (unsigned)((C + kFinCh - 1) / kFinCh); }

__device__ __forceinline__ void finalize_sums(const float* __restrict__ part, int nb, int C, int c,
                                              double* s1_out, double* s2_out) {
  const int lane = threadIdx.x & 63;
  double s1 = 0.0, s2 = 0.0;
  const float* p1 = part + ((size_t)0 * C + c) * nb;
  const float* p2 = part + ((size_t)1 * C + c) * nb;
  // up to eight partials per round, all loads issued before the first add (an index past the end
  // is not loaded and adds zero); same order of additions as a plain loop
  const int rounds = (nb + 63) / 64;
  for (int k0 = 0; k0 < rounds; k0 += 8) {
    float v1[8], v2[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int b = lane + (k0 + k) * 64;
      v1[k] = v2[k] = 0.f;
      if (b < nb) {
        v1[k] = p1[b];
        v2[k] = p2[b];
      }
    }
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (k0 + k < rounds) {
        s1 += (double)v1[k];
        s2 += (double)v2[k];
      }
  }
  *s1_out = wave_sum(s1);
  *s2_out = wave_sum(s2);
}

// Row walk of the reductions and of the element-wise kernels: a thread owns one octet of
// channels for the whole launch, keeps that octet's coefficients in registers, and walks rows
// first, first + step, ..., four rows in flight.  No per-vector index arithmetic beyond one multiply-add, no
// per-vector coefficient loads.
//
// Without SLAB a workgroup takes whole rows; with it, 64 of the channels (a 128-byte line of bf16 per row) of 32 rows at a time, the
// slabs of a row block being consecutive workgroups.  A slab's workgroup needs the sums of its own channels only, and a tensor of C channels has C / 64
// times fewer partial sums per channel, so few that every consumer can add them up for itself (slab_sums).
constexpr int kSlab = 64;
template <bool SLAB> struct RowWalk {
  int lanes, rows, rl;     // octets and rows of a workgroup's pass, this thread's row in it (none from `rows` on)
  int c, slab0;            // its first channel; the workgroup's
  int block, blocks;       // row block of the workgroup, of how many
  __device__ __forceinline__ RowWalk(int C) {
    const int slabs = SLAB ? C / kSlab : 1;
    block = SLAB ? uniform_div(blockIdx.x, slabs) : blockIdx.x;
    blocks = SLAB ? uniform_div(gridDim.x, slabs) : gridDim.x;
    slab0 = SLAB ? ((int)blockIdx.x - block * slabs) * kSlab : 0;
    lanes = SLAB ? kSlab / 8 : C / 8;
    rows = kT / lanes;
    rl = threadIdx.x / lanes;
    c = slab0 + (threadIdx.x - rl * lanes) * 8;
  }
  template <typename F> __device__ __forceinline__ void rows4(size_t m, int C, F body) const {
    if (rl >= rows) return;
    const size_t step = (size_t)blocks * rows;
    size_t r = (size_t)block * rows + rl;
    for (; r + 3 * step < m; r += 4 * step) {
      const size_t i0 = r * C + c, d = step * C;
      body(i0, i0 + d, i0 + 2 * d, i0 + 3 * d, std::integral_constant<int, 4>{});
    }
    for (; r < m; r += step) {
      const size_t i0 = r * C + c;
      body(i0, i0, i0, i0, std::integral_constant<int, 1>{});
    }
  }
};

// The sums of a workgroup's slab out of the partials part[v][c][0..nb): four threads to a channel, up to 32 loads in flight each,
// added in double in a fixed order.  sum[v][channel of the slab], behind a barrier.
__device__ __forceinline__ void slab_sums(const float* __restrict__ part, int nb, int C, int slab0, float (*sum)[kSlab]) {
  const int q = threadIdx.x & 3, ch = threadIdx.x >> 2;
  const float* p[2] = {part + (size_t)(slab0 + ch) * nb, part + (size_t)(C + slab0 + ch) * nb};
  double s[2] = {0.0, 0.0};
  if ((nb & 3) == 0) {
    for (int k0 = q * 4; k0 < nb; k0 += 64) {
      float4 v[2][4];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int k = 0; k < 4; ++k) v[t][k] = *reinterpret_cast<const float4*>(p[t] + (k0 + 16 * k < nb ? k0 + 16 * k : 0));
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (k0 + 16 * k < nb) s[t] += ((double)v[t][k].x + (double)v[t][k].y) + ((double)v[t][k].z + (double)v[t][k].w);
    }
  } else {
    for (int k0 = q; k0 < nb; k0 += 32) {
      float v[2][8];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int k = 0; k < 8; ++k) v[t][k] = p[t][k0 + 4 * k < nb ? k0 + 4 * k : 0];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if (k0 + 4 * k < nb) s[t] += (double)v[t][k];
    }
  }
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    s[t] += __shfl_xor(s[t], 1, 64);
    s[t] += __shfl_xor(s[t], 2, 64);
    if (q == 0) sum[t][ch] = (float)s[t];
  }
  __syncthreads();
}

// Partial sums of (x - shift) and (x - shift)^2 with shift = x[0][c] (keeps fp32 sums benign).
template <typename T>
__global__ void __launch_bounds__(kT) stats_partial_kernel(const T* __restrict__ x, size_t m, int C,
                                                           float* __restrict__ part) {
  const RowWalk<false> w(C);
  float acc[2][8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[0][e] = acc[1][e] = 0.f;
  if (w.rl < w.rows) {
    float sh[8];
    load8(x + w.c, sh);
    // four rows per round, all loads issued before the first use (a plain row loop is compiled to
    // one load in flight per thread)
    w.rows4(m, C, [&](size_t i0, size_t i1, size_t i2, size_t i3, auto NN) {
      constexpr int n = decltype(NN)::value;
      const size_t idx[4] = {i0, i1, i2, i3};
      float v[4][8];
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (k < n) load8(x + idx[k], v[k]);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (k >= n) break;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float d = v[k][e] - sh[e];
          acc[0][e] += d;
          acc[1][e] = fmaf(d, d, acc[1][e]);
        }
      }
    });
  }
  block_reduce_store(acc, w, C, part);
}

// y = a + b, and the partial sums of stats_partial_kernel over y as stored: the sum's own pass over it is saved (WRN-28-10 b128, twelve sums
// of 84 to 21 MB: 10 + 10.5 us a sum in two launches).  Where it is the slower one: add_stats_pays.
template <typename T>
__global__ void __launch_bounds__(kT) add_stats_kernel(const T* __restrict__ a, const T* __restrict__ b, T* __restrict__ y, size_t m, int C,
                                                       float* __restrict__ part) {
  const RowWalk<false> w(C);
  float acc[2][8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[0][e] = acc[1][e] = 0.f;
  if (w.rl < w.rows) {
    float sh[8], sb[8];
    load8(a + w.c, sh);
    load8(b + w.c, sb);
#pragma unroll
    for (int e = 0; e < 8; ++e) {      // row 0 of y
      sh[e] += sb[e];
      if (sizeof(T) == 2) sh[e] = bf16_to_f32(f32_to_bf16_hw(sh[e]));
    }
    w.rows4(m, C, [&](size_t i0, size_t i1, size_t i2, size_t i3, auto NN) {
      constexpr int n = decltype(NN)::value;
      const size_t idx[4] = {i0, i1, i2, i3};
      float v[4][8], u[4][8];
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (k < n) {
          load8(a + idx[k], v[k]);
          load8(b + idx[k], u[k]);
        }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (k >= n) break;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[k][e] += u[k][e];
        store8_back(y + idx[k], v[k]);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float d = v[k][e] - sh[e];
          acc[0][e] += d;
          acc[1][e] = fmaf(d, d, acc[1][e]);
        }
      }
    });
  }
  block_reduce_store(acc, w, C, part);
}

// mode 0: write save_mean / save_invstd (+ running stats); mode 1: write plain sum, sum of squares.
template <typename T>
__global__ void __launch_bounds__(kT) stats_finalize_kernel(const float* __restrict__ part, int nb,
                                                            const T* __restrict__ x, size_t m, int C, int mode,
                                                            float eps, float momentum, float* __restrict__ o0,
                                                            float* __restrict__ o1, float* __restrict__ rmean,
                                                            float* __restrict__ rvar) {
  const int c = blockIdx.x * kFinCh + (threadIdx.x >> 6);
  if (c >= C) return;
  double s1, s2;
  finalize_sums(part, nb, C, c, &s1, &s2);
  if ((threadIdx.x & 63) != 0) return;
  const double sh = (double)Elem<T>::ld(x + c);
  const double dm = (double)m;
  if (mode == 1) {
    o0[c] = (float)(s1 + dm * sh);
    o1[c] = (float)(s2 + 2.0 * sh * s1 + dm * sh * sh);
    return;
  }
  const double mean_s = s1 / dm;
  double var = s2 / dm - mean_s * mean_s;
  if (var < 0.0) var = 0.0;
  o0[c] = (float)(sh + mean_s);
  o1[c] = (float)(1.0 / sqrt(var + (double)eps));
  if (rmean) {
    const double unb = m > 1 ? var * dm / (dm - 1.0) : var;
    rmean[c] = (float)((1.0 - momentum) * rmean[c] + momentum * (sh + mean_s));
    rvar[c] = (float)((1.0 - momentum) * rvar[c] + momentum * unb);
  }
}

__global__ void __launch_bounds__(kT) sums_finalize_kernel(const float* __restrict__ part, int nb, int C,
                                                           float* __restrict__ ch_sum, float* __restrict__ ch_sumsq) {
  const int c = blockIdx.x * kFinCh + (threadIdx.x >> 6);
  if (c >= C) return;
  double s1, s2;
  finalize_sums(part, nb, C, c, &s1, &s2);
  if ((threadIdx.x & 63) != 0) return;
  ch_sum[c] = (float)s1;
  ch_sumsq[c] = (float)s2;
}

// The same with a whole workgroup per channel, for many partials (a wavefront alone would walk
// them in nb/64 dependent rounds): threads stride the partials, butterfly per wavefront, the four
// wavefront sums added in order.
constexpr int kWideFinalize = 1024;   // partials per channel from which the wide kernels are used
__device__ __forceinline__ void finalize_sums_wide(const float* __restrict__ part, int nb, int C, int c,
                                                   double* s1_out, double* s2_out) {
  __shared__ double comb[2][kT / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float* p1 = part + ((size_t)0 * C + c) * nb;
  const float* p2 = part + ((size_t)1 * C + c) * nb;
  double s1 = 0.0, s2 = 0.0;
  const int rounds = (nb + kT - 1) / kT;       // up to eight partials per round, as above
  for (int k0 = 0; k0 < rounds; k0 += 8) {
    float v1[8], v2[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int b = tid + (k0 + k) * kT;
      v1[k] = v2[k] = 0.f;
      if (b < nb) {
        v1[k] = p1[b];
        v2[k] = p2[b];
      }
    }
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (k0 + k < rounds) {
        s1 += (double)v1[k];
        s2 += (double)v2[k];
      }
  }
  s1 = wave_sum(s1);
  s2 = wave_sum(s2);
  if (lane == 0) { comb[0][wave] = s1; comb[1][wave] = s2; }
  __syncthreads();
  double t1 = comb[0][0], t2 = comb[1][0];
#pragma unroll
  for (int w_ = 1; w_ < kT / 64; ++w_) { t1 += comb[0][w_]; t2 += comb[1][w_]; }
  *s1_out = t1;
  *s2_out = t2;
}

__global__ void __launch_bounds__(kT) sums_finalize_wide_kernel(const float* __restrict__ part, int nb, int C,
                                                                float* __restrict__ ch_sum,
                                                                float* __restrict__ ch_sumsq) {
  double s1, s2;
  finalize_sums_wide(part, nb, C, blockIdx.x, &s1, &s2);
  if (threadIdx.x != 0) return;
  ch_sum[blockIdx.x] = (float)s1;
  ch_sumsq[blockIdx.x] = (float)s2;
}

// sc = gamma * invstd, bi = beta - mean * sc: the one place this is written, so that the forward
// kernels and the mask recomputation of the backward kernels round identically.
__device__ __forceinline__ void bn_scale_bias(float g, float b, float mu, float is, float* sc, float* bi) {
  *sc = g * is;
  *bi = fmaf(-mu, *sc, b);
}

template <typename T, class W>
__device__ __forceinline__ void bn_apply_rows(const W& w, const T* __restrict__ x, const T* __restrict__ res, T* __restrict__ y,
                                              size_t m, int C, int relu, const float* sc, const float* bi,
                                              unsigned char* __restrict__ mask = nullptr) {
  w.rows4(m, C, [&](size_t i0, size_t i1, size_t i2, size_t i3, auto NN) {
    constexpr int n = decltype(NN)::value;
    const size_t idx[4] = {i0, i1, i2, i3};
    float v[4][8], r[4][8];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (k < n) load8(x + idx[k], v[k]);
    if (res) {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (k < n) load8(res + idx[k], r[k]);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (k >= n) break;
#pragma unroll
      for (int e = 0; e < 8; ++e) v[k][e] = fmaf(v[k][e], sc[e], bi[e]);
      if (res) {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[k][e] += r[k][e];
      }
      if (relu) {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[k][e] = v[k][e] > 0.f ? v[k][e] : 0.f;
        if (mask) {
          unsigned bits = 0;
#pragma unroll
          for (int e = 0; e < 8; ++e) bits |= v[k][e] > 0.f ? 1u << e : 0u;
          mask[idx[k] / 8] = (unsigned char)bits;
        }
      }
      store8(y + idx[k], v[k]);
    }
  });
}

// y = gamma * (x - mean) * invstd + beta (+ residual) (ReLU), as x * sc + bi with sc = gamma * invstd,
// bi = beta - mean * sc (the same two roundings whichever kernel produced the statistics).
template <typename T>
__global__ void __launch_bounds__(kT) bn_apply_kernel(const T* __restrict__ x, const T* __restrict__ res,
                                                      const float* __restrict__ gamma,
                                                      const float* __restrict__ beta,
                                                      const float* __restrict__ mean,
                                                      const float* __restrict__ invstd, T* __restrict__ y,
                                                      size_t m, int C, int relu, unsigned char* __restrict__ mask) {
  const RowWalk<false> w(C);
  float g[8], b[8], mu[8], is[8], sc[8], bi[8];
  load8(gamma + w.c, g);
  load8(beta + w.c, b);
  load8(mean + w.c, mu);
  load8(invstd + w.c, is);
#pragma unroll
  for (int e = 0; e < 8; ++e) bn_scale_bias(g[e], b[e], mu[e], is[e], &sc[e], &bi[e]);
  bn_apply_rows<T>(w, x, res, y, m, C, relu, sc, bi, mask);
}

// Inference mode: the running statistics stand in for the batch's; nothing is reduced or updated.
template <typename T>
__global__ void __launch_bounds__(kT) bn_infer_kernel(const T* __restrict__ x, const T* __restrict__ res,
                                                      const float* __restrict__ gamma,
                                                      const float* __restrict__ beta,
                                                      const float* __restrict__ rmean,
                                                      const float* __restrict__ rvar, float eps,
                                                      T* __restrict__ y, size_t m, int C, int relu) {
  const RowWalk<false> w(C);
  float g[8], b[8], mu[8], var[8], sc[8], bi[8];
  load8(gamma + w.c, g);
  load8(beta + w.c, b);
  load8(rmean + w.c, mu);
  load8(rvar + w.c, var);
#pragma unroll
  for (int e = 0; e < 8; ++e) bn_scale_bias(g[e], b[e], mu[e], 1.f / sqrtf(var[e] + eps), &sc[e], &bi[e]);
  bn_apply_rows<T>(w, x, res, y, m, C, relu, sc, bi);
}

// Normalise (+ residual) (+ ReLU) with the statistics taken directly from per-channel sums
// (sum x, sum x^2 over m positions, e.g. from the convolution that produced x): every thread
// derives mean / invstd of its 8 channels itself, so no separate statistics kernel runs.
// The first row block also writes save_mean / save_invstd and updates the running statistics.
// SLAB: the sums come as nb partials per channel (ch_sum: part[2][C][nb]) and are added up here.
template <typename T, bool SLAB>
__global__ void __launch_bounds__(kT) bn_apply_sums_kernel(const T* __restrict__ x, const T* __restrict__ res,
                                                           const float* __restrict__ gamma,
                                                           const float* __restrict__ beta,
                                                           const float* __restrict__ ch_sum,
                                                           const float* __restrict__ ch_sumsq, int nb, float inv_m,
                                                           float unbias, float eps, float momentum,
                                                           float* __restrict__ save_mean,
                                                           float* __restrict__ save_invstd,
                                                           float* __restrict__ rmean, float* __restrict__ rvar,
                                                           T* __restrict__ y, size_t m, int C, int relu,
                                                           unsigned char* __restrict__ mask) {
  __shared__ __align__(16) float sums[2][kSlab];
  const RowWalk<SLAB> w(C);
  if (SLAB) slab_sums(ch_sum, nb, C, w.slab0, sums);
  const float* p1 = SLAB ? sums[0] : ch_sum;
  const float* p2 = SLAB ? sums[1] : ch_sumsq;
  if (w.block == 0) {
    for (int k = threadIdx.x; k < (SLAB ? kSlab : C); k += kT) {
      const int c = w.slab0 + k;
      const float mu = p1[k] * inv_m;
      const float var = fmaxf(fmaf(p2[k], inv_m, -mu * mu), 0.f);
      save_mean[c] = mu;
      save_invstd[c] = rsqrtf(var + eps);
      if (rmean) {
        rmean[c] = (1.f - momentum) * rmean[c] + momentum * mu;
        rvar[c] = (1.f - momentum) * rvar[c] + momentum * var * unbias;
      }
    }
  }
  float s1[8], s2[8], g[8], b[8], sc[8], bi[8];
  load8(p1 + (w.c - w.slab0), s1);
  load8(p2 + (w.c - w.slab0), s2);
  load8(gamma + w.c, g);
  load8(beta + w.c, b);
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float mu = s1[e] * inv_m;
    const float var = fmaxf(fmaf(s2[e], inv_m, -mu * mu), 0.f);
    const float is = rsqrtf(var + eps);
    bn_scale_bias(g[e], b[e], mu, is, &sc[e], &bi[e]);
  }
  bn_apply_rows<T>(w, x, res, y, m, C, relu, sc, bi, mask);
}

// Partial sums of dz and dz*xhat.  MODE 0: no ReLU; 1: mask [y > 0]; 2: mask [x*sc + bi > 0]
// recomputed with the forward's arithmetic (y is not read); 4: `y` is the mask that the forward pass kept, one bit
// per element.  The element-wise kernel also knows MODE 3: dz was written by this kernel into dres (the residual
// gradient is dz itself), read it there.
template <typename T, int MODE, bool SLAB>
__global__ void __launch_bounds__(kT) bwd_partial_kernel(const T* __restrict__ dy, const T* __restrict__ x,
                                                         const void* __restrict__ y_or_mask,
                                                         const float* __restrict__ gamma,
                                                         const float* __restrict__ beta,
                                                         const float* __restrict__ mean,
                                                         const float* __restrict__ invstd, size_t m, int C,
                                                         float* __restrict__ part, T* __restrict__ dz_out) {
  const T* __restrict__ y = (const T*)y_or_mask;
  const unsigned char* __restrict__ mask = (const unsigned char*)y_or_mask;
  const RowWalk<SLAB> w(C);
  float acc[2][8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[0][e] = acc[1][e] = 0.f;
  if (w.rl < w.rows) {
    float mu[8], is[8], sc[8], bi[8];
    load8(mean + w.c, mu);
    load8(invstd + w.c, is);
    if (MODE == 2) {
      float ga[8], be[8];
      load8(gamma + w.c, ga);
      load8(beta + w.c, be);
#pragma unroll
      for (int e = 0; e < 8; ++e) bn_scale_bias(ga[e], be[e], mu[e], is[e], &sc[e], &bi[e]);
    }
    // four rows per round, all loads issued before the first use (a plain row loop is compiled to
    // one load in flight per thread)
    w.rows4(m, C, [&](size_t i0, size_t i1, size_t i2, size_t i3, auto NN) {
      constexpr int n = decltype(NN)::value;
      const size_t idx[4] = {i0, i1, i2, i3};
      float g[4][8], xv[4][8], yv[4][8];
      unsigned mb[4];
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (k < n) {
          load8(dy + idx[k], g[k]);
          load8(x + idx[k], xv[k]);
          if (MODE == 1) load8(y + idx[k], yv[k]);
          if (MODE == 4) mb[k] = mask[idx[k] / 8];
        }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (k >= n) break;
        if (MODE == 1) {
#pragma unroll
          for (int e = 0; e < 8; ++e) g[k][e] = yv[k][e] > 0.f ? g[k][e] : 0.f;
        }
        if (MODE == 2) {
#pragma unroll
          for (int e = 0; e < 8; ++e) g[k][e] = fmaf(xv[k][e], sc[e], bi[e]) > 0.f ? g[k][e] : 0.f;
        }
        if (MODE == 4) {
#pragma unroll
          for (int e = 0; e < 8; ++e) g[k][e] = (mb[k] >> e) & 1u ? g[k][e] : 0.f;
        }
        // the masked gradient is exact in the storage type (dy or 0): written here, it spares the
        // element-wise pass the reads of dy and y
        if (dz_out) store8(dz_out + idx[k], g[k]);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          acc[0][e] += g[k][e];
          acc[1][e] = fmaf(g[k][e], xv[k][e] - mu[e], acc[1][e]);   // times invstd once, below
        }
      }
    });
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[1][e] *= is[e];
  }
  block_reduce_store(acc, w, C, part);
}

__global__ void __launch_bounds__(kT) bwd_finalize_kernel(const float* __restrict__ part, int nb, int C,
                                                          float* __restrict__ dgamma, float* __restrict__ dbeta) {
  const int c = blockIdx.x * kFinCh + (threadIdx.x >> 6);
  if (c >= C) return;
  double s1, s2;
  finalize_sums(part, nb, C, c, &s1, &s2);
  if ((threadIdx.x & 63) != 0) return;
  dbeta[c] = (float)s1;
  dgamma[c] = (float)s2;
}

__global__ void __launch_bounds__(kT) bwd_finalize_wide_kernel(const float* __restrict__ part, int nb, int C,
                                                               float* __restrict__ dgamma, float* __restrict__ dbeta) {
  double s1, s2;
  finalize_sums_wide(part, nb, C, blockIdx.x, &s1, &s2);
  if (threadIdx.x != 0) return;
  dbeta[blockIdx.x] = (float)s1;
  dgamma[blockIdx.x] = (float)s2;
}

// SLAB: the sums come as nb partials per channel (part[2][C][nb]) and are added up here; the first row block writes
// dgamma and dbeta.  Otherwise it reads them.
template <typename T, int MODE, bool SLAB>
__global__ void __launch_bounds__(kT) bwd_apply_kernel(const T* __restrict__ dy, const T* __restrict__ x,
                                                       const void* __restrict__ y_or_mask, const float* __restrict__ gamma,
                                                       const float* __restrict__ beta,
                                                       const float* __restrict__ mean,
                                                       const float* __restrict__ invstd,
                                                       const float* __restrict__ part, int nb,
                                                       float* __restrict__ dgamma,
                                                       float* __restrict__ dbeta, T* __restrict__ dx,
                                                       T* __restrict__ dres, size_t m, int C, float inv_m,
                                                       int flags) {
  __shared__ __align__(16) float sums[2][kSlab];
  const T* __restrict__ y = (const T*)y_or_mask;
  const unsigned char* __restrict__ mask = (const unsigned char*)y_or_mask;
  const RowWalk<SLAB> w(C);
  if (SLAB) {
    slab_sums(part, nb, C, w.slab0, sums);
    if (w.block == 0 && threadIdx.x < kSlab) {
      dbeta[w.slab0 + threadIdx.x] = sums[0][threadIdx.x];
      dgamma[w.slab0 + threadIdx.x] = sums[1][threadIdx.x];
    }
  }
  // dx = a * (dz - (dbeta + xhat * dgamma) / m), xhat = (x - mu) * is, a = gamma * is
  float a[8], mu[8], is[8], dgm[8], dbm[8], sc[8], bi[8];
  {
    float ga[8], dg[8], db[8];
    load8(gamma + w.c, ga);
    load8(mean + w.c, mu);
    load8(invstd + w.c, is);
    load8(SLAB ? &sums[1][w.c - w.slab0] : dgamma + w.c, dg);
    load8(SLAB ? &sums[0][w.c - w.slab0] : dbeta + w.c, db);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      a[e] = ga[e] * is[e];
      dgm[e] = dg[e] * inv_m * is[e];   // xhat * dgamma / m = (x - mu) * (invstd * dgamma / m)
      dbm[e] = db[e] * inv_m;
    }
    if (MODE == 2) {
      float be[8];
      load8(beta + w.c, be);
#pragma unroll
      for (int e = 0; e < 8; ++e) bn_scale_bias(ga[e], be[e], mu[e], is[e], &sc[e], &bi[e]);
    }
  }
  w.rows4(m, C, [&](size_t i0, size_t i1, size_t i2, size_t i3, auto NN) {
    constexpr int n = decltype(NN)::value;
    const size_t idx[4] = {i0, i1, i2, i3};
    float g[4][8], xv[4][8], yv[4][8];
    unsigned mb[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (k < n) {
        load8((MODE == 3 ? dres : dy) + idx[k], g[k]);
        load8(x + idx[k], xv[k]);
        if (MODE == 1) load8(y + idx[k], yv[k]);
        if (MODE == 4) mb[k] = mask[idx[k] / 8];
      }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (k >= n) break;
      float out[8];
      if (MODE == 1) {
#pragma unroll
        for (int e = 0; e < 8; ++e) g[k][e] = yv[k][e] > 0.f ? g[k][e] : 0.f;
      }
      if (MODE == 2) {
#pragma unroll
        for (int e = 0; e < 8; ++e) g[k][e] = fmaf(xv[k][e], sc[e], bi[e]) > 0.f ? g[k][e] : 0.f;
      }
      if (MODE == 4) {
#pragma unroll
        for (int e = 0; e < 8; ++e) g[k][e] = (mb[k] >> e) & 1u ? g[k][e] : 0.f;
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        out[e] = a[e] * (g[k][e] - fmaf(xv[k][e] - mu[e], dgm[e], dbm[e]));
      }
      if (flags & 1) {
        float old[8];
        load8(dx + idx[k], old);
#pragma unroll
        for (int e = 0; e < 8; ++e) out[e] += old[e];
      }
      store8(dx + idx[k], out);
      if (dres && MODE != 3) {
        if (flags & 2) {
          float old[8];
          load8(dres + idx[k], old);
#pragma unroll
          for (int e = 0; e < 8; ++e) g[k][e] += old[e];
        }
        store8(dres + idx[k], g[k]);
      }
    }
  });
}

// Grid of the element-wise kernels: every thread gets about eight rows (four where eight leave CUs idle), capped.
inline unsigned row_blocks(size_t m, int C) {
  const int rows = kT / (C / 8);
  size_t b = (m + (size_t)rows * 8 - 1) / ((size_t)rows * 8);
  if (b < 256) b = (m + (size_t)rows * 4 - 1) / ((size_t)rows * 4);
  if (b > 4096) b = 4096;
  return (unsigned)(b < 1 ? 1 : b);
}

// Whether a batch norm's last pass adds up nb partials per channel itself instead of reading what a finalising launch left (4 to 5 us, two
// of them to a batch norm's forward and backward, and as much enqueueing).  Every workgroup reads the 512 nb bytes of its slab's
// partials first, so there is a limit.  us per step with none, up to 16, 64, 128, 256 partials (tuning key 19): ResNet-18 b32
// 1095, 1040, 1013, 1005, 1003; b77 1389, 1369, 1339, 1343, 1325; b256 2055, 2056, 2022, 2018, 2008; ResNet-50 b16 2603, 2323, 2270, 2261, 2262;
// b256 7751, 7698, 7571, 7566, 7652; VGG-style b128 467, 465, 459, 457, 457; WRN-28-10 b128 6504, 6548, 6478, 6465, 6481.  Fewer partials by more
// rows to a thread in the first backward pass: slower wherever that leaves fewer than 256 workgroups (ResNet-50 b256 7566, at most 128 row blocks 7623).
inline bool slab_pays(int C, int nb) { return C % kSlab == 0 && nb <= (g_cnnk_tune[19] ? g_cnnk_tune[19] : 128); }
// rows per thread and workgroups of a pass in slabs, as reduce_blocks and row_blocks have them without
inline int slab_blocks(size_t m, int C) {
  const size_t slabs = C / kSlab, rows = kT / (kSlab / 8);
  size_t nb = (m + rows * 8 - 1) / (rows * 8);
  if (nb * slabs < 256) nb = (m + rows * 4 - 1) / (rows * 4);
  const size_t cap = kMaxBlocks / slabs;
  return (int)(nb > cap ? cap : nb);
}

int validate_bn(const cnnk_bn_desc* d) {
  if (!d) return CNNK_ERR_NULL;
  if (d->N <= 0 || d->H <= 0 || d->W <= 0 || d->C <= 0) return CNNK_ERR_SHAPE;
  if (d->dtype != CNNK_F32 && d->dtype != CNNK_BF16) return CNNK_ERR_UNSUPPORTED;
  if (d->C % 8 != 0 || d->C > 2048) return CNNK_ERR_UNSUPPORTED;
  return CNNK_OK;
}

}  // namespace

thread_local PartSums* t_cnnk_part_sums = nullptr;

// Rows from which slabs are slower whatever the partials: with 1024 channels and more, passes over whole rows move large tensors
// faster than passes over 128 bytes of every row.  Backward in bf16, us in slabs / over whole rows and with the launch, without and with a residual: 1024
// channels 16384 rows 37.6 / 41.8, 50.6 / 52.7; 32768 67.6 / 66.8, 101 / 94; 65536 152 / 136, 212 / 184; 1536 channels 16384 rows 54.5 / 59.6, 77 / 80; 32768
// 116 / 105, 171 / 140; 2048 channels 16384 rows 64 / 70, 98 / 101; 24576 106 / 105, 158 / 143; 32768 147 / 136, 211 / 188.  960 channels, 32768 rows 62.9 /
// 64.1, 89 / 103 (more rows have more than 128 partials).
bool bn_slabs_pay_for(size_t m, int C) { return C < 1024 || m <= 16384; }

int channel_sums_finalize(const float* part, int nb, int C, float* ch_sum, float* ch_sumsq, hipStream_t st) {
  if (t_cnnk_part_sums && slab_pays(C, nb)) {
    t_cnnk_part_sums->part = part;
    t_cnnk_part_sums->nb = nb;
    return CNNK_OK;
  }
  if (nb >= kWideFinalize) sums_finalize_wide_kernel<<<C, kT, 0, st>>>(part, nb, C, ch_sum, ch_sumsq);
  else sums_finalize_kernel<<<fin_blocks(C), kT, 0, st>>>(part, nb, C, ch_sum, ch_sumsq);
  return launch_status();
}

size_t channel_stats_ws(size_t m, int C) { return (size_t)reduce_blocks(m, C) * 2 * C * sizeof(float); }

int channel_stats(int dtype, const void* x, size_t m, int C, float* ch_sum, float* ch_sumsq, void* ws,
                  hipStream_t st) {
  const int nb = reduce_blocks(m, C);
  float* part = (float*)ws;
  if (dtype == CNNK_BF16) {
    stats_partial_kernel<bf16_t><<<nb, kT, 0, st>>>((const bf16_t*)x, m, C, part);
    stats_finalize_kernel<bf16_t><<<fin_blocks(C), kT, 0, st>>>(part, nb, (const bf16_t*)x, m, C, 1, 0.f, 0.f,
                                                                    ch_sum, ch_sumsq, nullptr, nullptr);
  } else {
    stats_partial_kernel<float><<<nb, kT, 0, st>>>((const float*)x, m, C, part);
    stats_finalize_kernel<float><<<fin_blocks(C), kT, 0, st>>>(part, nb, (const float*)x, m, C, 1, 0.f, 0.f,
                                                                   ch_sum, ch_sumsq, nullptr, nullptr);
  }
  return launch_status();
}

// Few workgroups walk a tensor of many channels (reduce_blocks), too few to add large bf16 ones at the memory rate.  us, in one launch / the sum and the batch
// norm's first pass: bf16, 384 channels 131072 rows 61.2 / 68.2; 512 channels 32768 rows 25.2 / 29.6, 65536 50.7 / 47.3; 640 channels 65536 rows 67.1 /
// 57.8; 768 channels 16384 rows 21.4 / 23.7, 32768 49.3 / 40.8; 1024 channels 16384 rows 30.6 / 29.6, 32768 71.0 / 49.4; 2048 channels 8192 rows 29.3 / 32.3,
// 16384 75.4 / 53.4.  fp32: 512 channels 65536 rows 83.0 / 90.7, 1024 channels 32768 rows 82.9 / 89.9.
bool add_stats_pays(int dtype, size_t m, int C) { return dtype != CNNK_BF16 || C < 512 || m * C <= (size_t)1 << 24; }

int add_stats(int dtype, const void* a, const void* b, void* y, size_t m, int C, PartSums* out, void* ws, hipStream_t st) {
  const int nb = reduce_blocks(m, C);
  float* part = (float*)ws;
  if (dtype == CNNK_BF16) add_stats_kernel<bf16_t><<<nb, kT, 0, st>>>((const bf16_t*)a, (const bf16_t*)b, (bf16_t*)y, m, C, part);
  else add_stats_kernel<float><<<nb, kT, 0, st>>>((const float*)a, (const float*)b, (float*)y, m, C, part);
  *out = PartSums{part, nb, true};
  return launch_status();
}

extern "C" size_t cnnk_bn_workspace_bytes(const cnnk_bn_desc* d) {
  if (validate_bn(d) != CNNK_OK) return 0;
  return align_up(channel_stats_ws((size_t)d->N * d->H * d->W, d->C), 256);
}

int bn_relu_fwd(const cnnk_bn_desc* d, const void* x, const void* residual, const float* gamma, const float* beta, void* y,
                unsigned char* mask, float* save_mean, float* save_invstd, float* running_mean, float* running_var,
                const float* ch_sum, const float* ch_sumsq, const PartSums* partials, void* ws, size_t ws_bytes, void* stream) {
  int rc = validate_bn(d);
  if (rc != CNNK_OK) return rc;
  if (!x || !gamma || !beta || !y || !save_mean || !save_invstd) return CNNK_ERR_NULL;
  if ((running_mean == nullptr) != (running_var == nullptr)) return CNNK_ERR_NULL;
  if ((ch_sum == nullptr) != (ch_sumsq == nullptr)) return CNNK_ERR_NULL;
  const size_t m = (size_t)d->N * d->H * d->W;
  const int C = d->C;
  hipStream_t st = (hipStream_t)stream;
  if (!ch_sum) {
    if (!ws || ws_bytes < channel_stats_ws(m, C)) return CNNK_ERR_WORKSPACE;
    const bool given = partials && partials->shifted;
    const int nb = given ? partials->nb : reduce_blocks(m, C);
    const float* part = given ? partials->part : (const float*)ws;
    if (d->dtype == CNNK_BF16) {
      if (!given) stats_partial_kernel<bf16_t><<<nb, kT, 0, st>>>((const bf16_t*)x, m, C, (float*)ws);
      stats_finalize_kernel<bf16_t><<<fin_blocks(C), kT, 0, st>>>(part, nb, (const bf16_t*)x, m, C, 0, d->eps,
                                                                      d->momentum, save_mean, save_invstd,
                                                                      running_mean, running_var);
    } else {
      if (!given) stats_partial_kernel<float><<<nb, kT, 0, st>>>((const float*)x, m, C, (float*)ws);
      stats_finalize_kernel<float><<<fin_blocks(C), kT, 0, st>>>(part, nb, (const float*)x, m, C, 0, d->eps,
                                                                     d->momentum, save_mean, save_invstd,
                                                                     running_mean, running_var);
    }
  } else {
    // statistics handed in as sums, or as few partial sums: one fused kernel (statistics + normalise)
    const float inv_m = (float)(1.0 / (double)m);
    const float unbias = m > 1 ? (float)((double)m / ((double)m - 1.0)) : 1.f;
    const int nb = partials ? partials->nb : 0;
    const float* sum = nb ? partials->part : ch_sum;
#define CNNK_BN_SUMS(T, SLAB)                                                                                                     \
  bn_apply_sums_kernel<T, SLAB><<<SLAB ? slab_blocks(m, C) * (C / kSlab) : row_blocks(m, C), kT, 0, st>>>(                        \
      (const T*)x, (const T*)residual, gamma, beta, sum, ch_sumsq, nb, inv_m, unbias, d->eps, d->momentum, save_mean,            \
      save_invstd, running_mean, running_var, (T*)y, m, C, d->relu, mask)
    if (d->dtype == CNNK_BF16) {
      if (nb) CNNK_BN_SUMS(bf16_t, true); else CNNK_BN_SUMS(bf16_t, false);
    } else {
      if (nb) CNNK_BN_SUMS(float, true); else CNNK_BN_SUMS(float, false);
    }
#undef CNNK_BN_SUMS
    return launch_status();
  }
  if (launch_status() != CNNK_OK) return CNNK_ERR_HIP;
  if (d->dtype == CNNK_BF16)
    bn_apply_kernel<bf16_t><<<row_blocks(m, C), kT, 0, st>>>((const bf16_t*)x, (const bf16_t*)residual, gamma, beta,
                                                          save_mean, save_invstd, (bf16_t*)y, m, C, d->relu, mask);
  else
    bn_apply_kernel<float><<<row_blocks(m, C), kT, 0, st>>>((const float*)x, (const float*)residual, gamma, beta,
                                                         save_mean, save_invstd, (float*)y, m, C, d->relu, mask);
  return launch_status();
}

extern "C" int cnnk_bn_relu_fwd(const cnnk_bn_desc* d, const void* x, const void* residual, const float* gamma,
                                const float* beta, void* y, float* save_mean, float* save_invstd,
                                float* running_mean, float* running_var, const float* ch_sum,
                                const float* ch_sumsq, void* ws, size_t ws_bytes, void* stream) {
  return bn_relu_fwd(d, x, residual, gamma, beta, y, nullptr, save_mean, save_invstd, running_mean, running_var, ch_sum,
                     ch_sumsq, nullptr, ws, ws_bytes, stream);
}

extern "C" int cnnk_bn_relu_infer(const cnnk_bn_desc* d, const void* x, const void* residual, const float* gamma,
                                  const float* beta, const float* running_mean, const float* running_var,
                                  void* y, void* stream) {
  int rc = validate_bn(d);
  if (rc != CNNK_OK) return rc;
  if (!x || !gamma || !beta || !running_mean || !running_var || !y) return CNNK_ERR_NULL;
  const size_t m = (size_t)d->N * d->H * d->W;
  const int C = d->C;
  hipStream_t st = (hipStream_t)stream;
  if (d->dtype == CNNK_BF16)
    bn_infer_kernel<bf16_t><<<row_blocks(m, C), kT, 0, st>>>((const bf16_t*)x, (const bf16_t*)residual, gamma, beta,
                                                          running_mean, running_var, d->eps, (bf16_t*)y, m, C,
                                                          d->relu);
  else
    bn_infer_kernel<float><<<row_blocks(m, C), kT, 0, st>>>((const float*)x, (const float*)residual, gamma, beta,
                                                         running_mean, running_var, d->eps, (float*)y, m, C,
                                                         d->relu);
  return launch_status();
}

template <typename T, int MODE>
static int bn_bwd_launch(const cnnk_bn_desc* d, const void* dy, const void* x, const void* y, const float* gamma,
                         const float* beta, const float* save_mean, const float* save_invstd, void* dx,
                         void* dresidual, int flags, float* dgamma, float* dbeta, float* part, hipStream_t st) {
  const size_t m = (size_t)d->N * d->H * d->W;
  const int C = d->C;
  const float inv_m = (float)(1.0 / (double)m);
  // a residual gradient that is written, not accumulated, is written by the first pass already
  const bool dz_first = (MODE == 1 || MODE == 4) && dresidual && !(flags & 2);
  constexpr int APPLY = MODE == 1 || MODE == 4 ? 3 : MODE;      // the last pass behind dz_first
  T* const dz = dz_first ? (T*)dresidual : nullptr;
  const int nbs = C % kSlab == 0 ? slab_blocks(m, C) : 0;
  if (nbs > 0 && bn_slabs_pay_for(m, C) && slab_pays(C, nbs) && (size_t)nbs * 2 * C * sizeof(float) <= channel_stats_ws(m, C)) {
    const unsigned grid = (unsigned)nbs * (C / kSlab);
    bwd_partial_kernel<T, MODE, true><<<grid, kT, 0, st>>>((const T*)dy, (const T*)x, y, gamma, beta, save_mean, save_invstd, m, C, part, dz);
    if (dz_first)
      bwd_apply_kernel<T, APPLY, true><<<grid, kT, 0, st>>>((const T*)dy, (const T*)x, y, gamma, beta, save_mean, save_invstd, part, nbs,
                                                            dgamma, dbeta, (T*)dx, (T*)dresidual, m, C, inv_m, flags);
    else
      bwd_apply_kernel<T, MODE, true><<<grid, kT, 0, st>>>((const T*)dy, (const T*)x, y, gamma, beta, save_mean, save_invstd, part, nbs,
                                                           dgamma, dbeta, (T*)dx, (T*)dresidual, m, C, inv_m, flags);
    return launch_status();
  }
  const int nb = reduce_blocks(m, C);
  bwd_partial_kernel<T, MODE, false><<<nb, kT, 0, st>>>((const T*)dy, (const T*)x, y, gamma, beta, save_mean, save_invstd, m, C, part, dz);
  if (nb >= kWideFinalize) bwd_finalize_wide_kernel<<<C, kT, 0, st>>>(part, nb, C, dgamma, dbeta);
  else bwd_finalize_kernel<<<fin_blocks(C), kT, 0, st>>>(part, nb, C, dgamma, dbeta);
  if (dz_first)
    bwd_apply_kernel<T, APPLY, false><<<row_blocks(m, C), kT, 0, st>>>((const T*)dy, (const T*)x, y, gamma, beta, save_mean, save_invstd,
                                                                       nullptr, 0, dgamma, dbeta, (T*)dx, (T*)dresidual, m, C, inv_m, flags);
  else
    bwd_apply_kernel<T, MODE, false><<<row_blocks(m, C), kT, 0, st>>>((const T*)dy, (const T*)x, y, gamma, beta, save_mean, save_invstd,
                                                                      nullptr, 0, dgamma, dbeta, (T*)dx, (T*)dresidual, m, C, inv_m, flags);
  return launch_status();
}

int bn_relu_bwd(const cnnk_bn_desc* d, const void* dy, const void* x, const void* y, const unsigned char* mask, const float* gamma,
                const float* beta, const float* save_mean, const float* save_invstd, void* dx, void* dresidual, int flags,
                float* dgamma, float* dbeta, void* ws, size_t ws_bytes, void* stream) {
  int rc = validate_bn(d);
  if (rc != CNNK_OK) return rc;
  if (!dy || !x || !gamma || !save_mean || !save_invstd || !dx || !dgamma || !dbeta) return CNNK_ERR_NULL;
  // ReLU mask: from y, or recomputed from x when y is withheld (no residual branch, beta given)
  if (d->relu && !mask && !y && (!beta || dresidual)) return CNNK_ERR_NULL;
  const int mode = !d->relu ? 0 : (mask ? 4 : y ? 1 : 2);
  const size_t m = (size_t)d->N * d->H * d->W;
  if (!ws || ws_bytes < channel_stats_ws(m, d->C)) return CNNK_ERR_WORKSPACE;
  hipStream_t st = (hipStream_t)stream;
  float* part = (float*)ws;
#define CNNK_BN_BWD(T, MODE) \
  return bn_bwd_launch<T, MODE>(d, dy, x, MODE == 4 ? (const void*)mask : y, gamma, beta, save_mean, save_invstd, dx, dresidual, flags, dgamma, \
                                dbeta, part, st)
  if (d->dtype == CNNK_BF16) {
    if (mode == 0) CNNK_BN_BWD(bf16_t, 0);
    if (mode == 1) CNNK_BN_BWD(bf16_t, 1);
    if (mode == 4) CNNK_BN_BWD(bf16_t, 4);
    CNNK_BN_BWD(bf16_t, 2);
  }
  if (mode == 0) CNNK_BN_BWD(float, 0);
  if (mode == 1) CNNK_BN_BWD(float, 1);
  if (mode == 4) CNNK_BN_BWD(float, 4);
  CNNK_BN_BWD(float, 2);
#undef CNNK_BN_BWD
}

extern "C" int cnnk_bn_relu_bwd(const cnnk_bn_desc* d, const void* dy, const void* x, const void* y,
                                const float* gamma, const float* beta, const float* save_mean,
                                const float* save_invstd, void* dx, void* dresidual, int flags, float* dgamma,
                                float* dbeta, void* ws, size_t ws_bytes, void* stream) {
  return bn_relu_bwd(d, dy, x, y, nullptr, gamma, beta, save_mean, save_invstd, dx, dresidual, flags, dgamma, dbeta, ws,
                     ws_bytes, stream);
}
