// Pooling, element-wise sums and gradient routing: bandwidth-bound kernels moving vectors of 8
// channels per thread (NHWC, C a multiple of 8).
#include "common.h"
#include "compensated.h"

namespace {
constexpr int kT = 256;

inline unsigned ew_blocks(size_t n) {
  size_t b = (n + kT - 1) / kT;
  if (b > 16384) b = 16384;
  return (unsigned)(b < 1 ? 1 : b);
}

template <typename T>
__global__ void __launch_bounds__(kT) maxpool_fwd_kernel(const T* __restrict__ x, T* __restrict__ y,
                                                         unsigned char* __restrict__ am, int N, int H, int W, int C) {
  const int Ho = H / 2, Wo = W / 2, C8 = C / 8;
  const size_t total = (size_t)N * Ho * Wo * C8;
  for (size_t i = (size_t)blockIdx.x * kT + threadIdx.x; i < total; i += (size_t)gridDim.x * kT) {
    const int c8 = (int)(i % C8);
    size_t p = i / C8;
    const int wo = (int)(p % Wo); p /= Wo;
    const int ho = (int)(p % Ho);
    const int n = (int)(p / Ho);
    float best[8];
    unsigned char code[8];
    const T* base = x + (((size_t)n * H + 2 * ho) * W + 2 * wo) * C + c8 * 8;
    load8(base, best);
#pragma unroll
    for (int e = 0; e < 8; ++e) code[e] = 0;
#pragma unroll
    for (int k = 1; k < 4; ++k) {
      float v[8];
      load8(base + ((size_t)(k >> 1) * W + (k & 1)) * C, v);
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (v[e] > best[e]) { best[e] = v[e]; code[e] = (unsigned char)k; }
    }
    store8(y + i * 8, best);
    uint2 pk;
    pk.x = code[0] | (code[1] << 8) | (code[2] << 16) | (code[3] << 24);
    pk.y = code[4] | (code[5] << 8) | (code[6] << 16) | (code[7] << 24);
    *reinterpret_cast<uint2*>(am + i * 8) = pk;
  }
}

template <typename T>
__global__ void __launch_bounds__(kT) maxpool_bwd_kernel(const T* __restrict__ dy,
                                                         const unsigned char* __restrict__ am, T* __restrict__ dx,
                                                         int N, int H, int W, int C, int accumulate) {
  const int Ho = H / 2, Wo = W / 2, C8 = C / 8;
  const size_t total = (size_t)N * Ho * Wo * C8;
  for (size_t i = (size_t)blockIdx.x * kT + threadIdx.x; i < total; i += (size_t)gridDim.x * kT) {
    const int c8 = (int)(i % C8);
    size_t p = i / C8;
    const int wo = (int)(p % Wo); p /= Wo;
    const int ho = (int)(p % Ho);
    const int n = (int)(p / Ho);
    float g[8];
    load8(dy + i * 8, g);
    const uint2 pk = *reinterpret_cast<const uint2*>(am + i * 8);
    T* base = dx + (((size_t)n * H + 2 * ho) * W + 2 * wo) * C + c8 * 8;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      float v[8];
      T* dst = base + ((size_t)(k >> 1) * W + (k & 1)) * C;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const unsigned code = ((e < 4 ? pk.x : pk.y) >> ((e & 3) * 8)) & 0xffu;
        v[e] = code == (unsigned)k ? g[e] : 0.f;
      }
      if (accumulate) {
        float o[8];
        load8(dst, o);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += o[e];
      }
      store8(dst, v);
    }
  }
}

// Global average pool, many octets: a thread each, eight positions' loads in flight, their sum a tree and these sums'
// sum compensated (the threads of the kernel below have shorter chains to begin with; rms error of a mean of 56 x 56
// standard normal values plus 0.5 2.1e-8, below 5.7e-8).  From 1 MiB for one position of all images on (65536 octets of
// bf16, 32768 of fp32) they fill the device.  This kernel and the one below, us: 256 images of 2048 channels at 8 x 8 10.9
// and 12.1 (fp32 20.4 and 22.6), at 7 x 7 9.3 and 9.8, fp32 512 of 512 at 7 x 7 9.4 and 9.8; bf16 512 of 512 at 7 x 7,
// half a MiB, with a plain sum 5.5 and 4.7.  Below 16 positions both take a launch's 4 us, and the tree saves no rounding.
constexpr size_t kGapManyBytes = 1 << 20;
constexpr int kGapManyPositions = 16;
template <typename T>
__global__ void __launch_bounds__(kT) gap_fwd_many_kernel(const T* __restrict__ x, T* __restrict__ y, size_t total, int HW, int C) {
  const int C8 = C / 8;
  const size_t i = (size_t)blockIdx.x * kT + threadIdx.x;
  if (i >= total) return;
  const int c8 = (int)(i % C8);
  const size_t n = i / C8;
  float acc[8], low[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = low[e] = 0.f;
  auto add = [&](const float (&v)[8][8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e)
      compensated_add(((v[0][e] + v[1][e]) + (v[2][e] + v[3][e])) + ((v[4][e] + v[5][e]) + (v[6][e] + v[7][e])), acc[e], low[e]);
  };
  const T* at = x + n * HW * C + c8 * 8;
  int p = 0;
  for (; p + 8 <= HW; p += 8, at += 8 * (size_t)C) {
    float v[8][8];
#pragma unroll
    for (int k = 0; k < 8; ++k) load8(at + (size_t)k * C, v[k]);
    add(v);
  }
  if (p < HW) {     // the first one's place for those past the end, as zeros
    float v[8][8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const bool in = p + k < HW;
      load8(at + (size_t)(in ? k : 0) * C, v[k]);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[k][e] = in ? v[k][e] : 0.f;
    }
    add(v);
  }
  const float inv = 1.f / (float)HW;
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] *= inv;
  store8(y + i * 8, acc);
}

// Fewer octets.  One workgroup per image and group of L channel octets: L threads side by side read
// a position's channels, 256 / L positions at a time, and the per-thread sums (four loads in flight) are
// combined through LDS in position order.  Bound by the latency of a thread's chain of loads: with a
// thread per octet that walks all positions, 8 images of 16 channels at 32 x 32 took 73 us on 16 threads;
// here 4.6 us.
template <typename T>
__global__ void __launch_bounds__(kT) gap_fwd_kernel(const T* __restrict__ x, T* __restrict__ y, int HW, int C, int L) {
  __shared__ float red[kT * 8];
  const int o = threadIdx.x % L, p0 = threadIdx.x / L, P = kT / L;
  const int c8 = blockIdx.y * L + o;
  const size_t n = blockIdx.x;
  float acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.f;
  if (c8 * 8 < C) {
    const T* base = x + n * HW * C + c8 * 8;
    for (int p = p0; p < HW; p += 4 * P) {
      float v[4][8];
#pragma unroll
      for (int k = 0; k < 4; ++k) load8(base + (size_t)(p + k * P < HW ? p + k * P : p) * C, v[k]);
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (p + k * P < HW)
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[e] += v[k][e];
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) red[e * kT + threadIdx.x] = acc[e];   // [e][position slot][octet]
  for (int s = P / 2; s > 0; s >>= 1) {
    __syncthreads();
    if (p0 < s)
#pragma unroll
      for (int e = 0; e < 8; ++e) red[e * kT + threadIdx.x] += red[e * kT + threadIdx.x + s * L];
  }
  if (p0 == 0 && c8 * 8 < C) {
    const float inv = 1.f / (float)HW;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = red[e * kT + o] * inv;
    store8(y + n * C + c8 * 8, acc);
  }
}

template <typename T>
__global__ void __launch_bounds__(kT) gap_bwd_kernel(const T* __restrict__ dy, T* __restrict__ dx, int N, int HW,
                                                     int C, int accumulate) {
  const int C8 = C / 8;
  const size_t total = (size_t)N * HW * C8;
  const float inv = 1.f / (float)HW;
  for (size_t i = (size_t)blockIdx.x * kT + threadIdx.x; i < total; i += (size_t)gridDim.x * kT) {
    const int c8 = (int)(i % C8);
    const size_t n = i / ((size_t)C8 * HW);
    float g[8];
    load8(dy + n * C + c8 * 8, g);
#pragma unroll
    for (int e = 0; e < 8; ++e) g[e] *= inv;
    if (accumulate) {
      float o[8];
      load8(dx + i * 8, o);
#pragma unroll
      for (int e = 0; e < 8; ++e) g[e] += o[e];
    }
    store8(dx + i * 8, g);
  }
}

// mode 0: y = a + b; mode 1: y = a; mode 2: y += a      (scalar tail handled by the same loop)
template <typename T>
__global__ void __launch_bounds__(kT) ew_kernel(const T* __restrict__ a, const T* __restrict__ b, T* __restrict__ y,
                                                size_t n, int mode) {
  const size_t n8 = n / 8;
  for (size_t i = (size_t)blockIdx.x * kT + threadIdx.x; i < n8; i += (size_t)gridDim.x * kT) {
    float u[8], v[8];
    load8(a + i * 8, u);
    if (mode == 0) load8(b + i * 8, v);
    if (mode == 2) load8(y + i * 8, v);
    if (mode != 1) {
#pragma unroll
      for (int e = 0; e < 8; ++e) u[e] += v[e];
    }
    store8(y + i * 8, u);
  }
  if (blockIdx.x == 0 && threadIdx.x < (n & 7)) {
    const size_t i = n8 * 8 + threadIdx.x;
    float u = Elem<T>::ld(a + i);
    if (mode == 0) u += Elem<T>::ld(b + i);
    if (mode == 2) u += Elem<T>::ld(y + i);
    Elem<T>::st(y + i, u);
  }
}

// the gradient of a sum to both summands (WRN-28-10 b128, twelve sums: 2 x 9.7 us a sum in two launches)
template <typename T>
__global__ void __launch_bounds__(kT) route2_kernel(const T* __restrict__ a, T* __restrict__ y0, int acc0, T* __restrict__ y1, int acc1, size_t n) {
  const size_t n8 = n / 8;
  for (size_t i = (size_t)blockIdx.x * kT + threadIdx.x; i < n8; i += (size_t)gridDim.x * kT) {
    float u[8], v0[8], v1[8];
    load8(a + i * 8, u);
    if (acc0) load8(y0 + i * 8, v0);
    if (acc1) load8(y1 + i * 8, v1);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      v0[e] = acc0 ? u[e] + v0[e] : u[e];
      v1[e] = acc1 ? u[e] + v1[e] : u[e];
    }
    store8(y0 + i * 8, v0);
    store8(y1 + i * 8, v1);
  }
  if (blockIdx.x == 0 && threadIdx.x < (n & 7)) {
    const size_t i = n8 * 8 + threadIdx.x;
    const float u = Elem<T>::ld(a + i);
    Elem<T>::st(y0 + i, acc0 ? u + Elem<T>::ld(y0 + i) : u);
    Elem<T>::st(y1 + i, acc1 ? u + Elem<T>::ld(y1 + i) : u);
  }
}

int validate_pool(const cnnk_pool_desc* d) {
  if (!d) return CNNK_ERR_NULL;
  if (d->N <= 0 || d->H <= 0 || d->W <= 0 || d->C <= 0) return CNNK_ERR_SHAPE;
  if (d->dtype != CNNK_F32 && d->dtype != CNNK_BF16) return CNNK_ERR_UNSUPPORTED;
  if (d->mode != CNNK_POOL_MAX2 && d->mode != CNNK_POOL_GAP) return CNNK_ERR_UNSUPPORTED;
  if (d->C % 8 != 0) return CNNK_ERR_UNSUPPORTED;
  if (d->mode == CNNK_POOL_MAX2 && ((d->H & 1) || (d->W & 1))) return CNNK_ERR_SHAPE;
  return CNNK_OK;
}
}  // namespace

extern "C" int cnnk_pool_fwd(const cnnk_pool_desc* d, const void* x, void* y, unsigned char* argmax, void* stream) {
  int rc = validate_pool(d);
  if (rc != CNNK_OK) return rc;
  if (!x || !y || (d->mode == CNNK_POOL_MAX2 && !argmax)) return CNNK_ERR_NULL;
  hipStream_t st = (hipStream_t)stream;
  if (d->mode == CNNK_POOL_MAX2) {
    const size_t total = (size_t)d->N * (d->H / 2) * (d->W / 2) * (d->C / 8);
    if (d->dtype == CNNK_BF16)
      maxpool_fwd_kernel<bf16_t><<<ew_blocks(total), kT, 0, st>>>((const bf16_t*)x, (bf16_t*)y, argmax, d->N, d->H, d->W, d->C);
    else
      maxpool_fwd_kernel<float><<<ew_blocks(total), kT, 0, st>>>((const float*)x, (float*)y, argmax, d->N, d->H, d->W, d->C);
  } else {
    const size_t octets = (size_t)d->N * (d->C / 8);
    if (d->H * d->W >= kGapManyPositions && octets * 8 * (d->dtype == CNNK_BF16 ? 2 : 4) >= kGapManyBytes) {
      const unsigned nb = (unsigned)((octets + kT - 1) / kT);
      if (d->dtype == CNNK_BF16)
        gap_fwd_many_kernel<bf16_t><<<nb, kT, 0, st>>>((const bf16_t*)x, (bf16_t*)y, octets, d->H * d->W, d->C);
      else
        gap_fwd_many_kernel<float><<<nb, kT, 0, st>>>((const float*)x, (float*)y, octets, d->H * d->W, d->C);
      return launch_status();
    }
    // octets per workgroup: a power of two, enough of them for 64-byte reads, and no more threads across
    // the positions than there are positions
    const int HW = d->H * d->W;
    int L = 4;
    while (L < 32 && L * 8 < d->C && (L * HW < kT || d->N * ((d->C / 8 + L - 1) / L) > 1024)) L *= 2;
    const dim3 grid((unsigned)d->N, (unsigned)((d->C / 8 + L - 1) / L));
    if (d->dtype == CNNK_BF16)
      gap_fwd_kernel<bf16_t><<<grid, kT, 0, st>>>((const bf16_t*)x, (bf16_t*)y, HW, d->C, L);
    else
      gap_fwd_kernel<float><<<grid, kT, 0, st>>>((const float*)x, (float*)y, HW, d->C, L);
  }
  return launch_status();
}

extern "C" int cnnk_pool_bwd(const cnnk_pool_desc* d, const void* dy, const unsigned char* argmax, void* dx,
                             int accumulate, void* stream) {
  int rc = validate_pool(d);
  if (rc != CNNK_OK) return rc;
  if (!dy || !dx || (d->mode == CNNK_POOL_MAX2 && !argmax)) return CNNK_ERR_NULL;
  hipStream_t st = (hipStream_t)stream;
  if (d->mode == CNNK_POOL_MAX2) {
    const size_t total = (size_t)d->N * (d->H / 2) * (d->W / 2) * (d->C / 8);
    if (d->dtype == CNNK_BF16)
      maxpool_bwd_kernel<bf16_t><<<ew_blocks(total), kT, 0, st>>>((const bf16_t*)dy, argmax, (bf16_t*)dx, d->N, d->H, d->W, d->C, accumulate);
    else
      maxpool_bwd_kernel<float><<<ew_blocks(total), kT, 0, st>>>((const float*)dy, argmax, (float*)dx, d->N, d->H, d->W, d->C, accumulate);
  } else {
    const size_t total = (size_t)d->N * d->H * d->W * (d->C / 8);
    if (d->dtype == CNNK_BF16)
      gap_bwd_kernel<bf16_t><<<ew_blocks(total), kT, 0, st>>>((const bf16_t*)dy, (bf16_t*)dx, d->N, d->H * d->W, d->C, accumulate);
    else
      gap_bwd_kernel<float><<<ew_blocks(total), kT, 0, st>>>((const float*)dy, (float*)dx, d->N, d->H * d->W, d->C, accumulate);
  }
  return launch_status();
}

static int launch_ew(size_t n, int dtype, const void* a, const void* b, void* y, int mode, hipStream_t st) {
  if (dtype != CNNK_F32 && dtype != CNNK_BF16) return CNNK_ERR_UNSUPPORTED;
  if (n == 0) return CNNK_OK;
  if (dtype == CNNK_BF16)
    ew_kernel<bf16_t><<<ew_blocks(n / 8 + 1), kT, 0, st>>>((const bf16_t*)a, (const bf16_t*)b, (bf16_t*)y, n, mode);
  else
    ew_kernel<float><<<ew_blocks(n / 8 + 1), kT, 0, st>>>((const float*)a, (const float*)b, (float*)y, n, mode);
  return launch_status();
}

extern "C" int cnnk_add(size_t n, int dtype, const void* a, const void* b, void* y, void* stream) {
  if (n && (!a || !b || !y)) return CNNK_ERR_NULL;
  return launch_ew(n, dtype, a, b, y, 0, (hipStream_t)stream);
}

extern "C" int cnnk_grad_route(size_t n, int dtype, const void* src, void* dst, int accumulate, void* stream) {
  if (n && (!src || !dst)) return CNNK_ERR_NULL;
  return launch_ew(n, dtype, src, nullptr, dst, accumulate ? 2 : 1, (hipStream_t)stream);
}

int grad_route2(size_t n, int dtype, const void* src, void* d0, int acc0, void* d1, int acc1, hipStream_t st) {
  if (n && (!src || !d0 || !d1)) return CNNK_ERR_NULL;
  if (n == 0) return CNNK_OK;
  if (dtype == CNNK_BF16) route2_kernel<bf16_t><<<ew_blocks(n / 8 + 1), kT, 0, st>>>((const bf16_t*)src, (bf16_t*)d0, acc0, (bf16_t*)d1, acc1, n);
  else route2_kernel<float><<<ew_blocks(n / 8 + 1), kT, 0, st>>>((const float*)src, (float*)d0, acc0, (float*)d1, acc1, n);
  return launch_status();
}
