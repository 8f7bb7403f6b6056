// Shared device/host helpers for the cnnk HIP kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>
#include "../../include/cnnk.h"
#include "fastdiv.h"

typedef unsigned short bf16_t;  // raw bfloat16 bits

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf16_to_f32(bf16_t v) { return __uint_as_float(((unsigned)v) << 16); }

// Round to nearest, ties to even; NaN stays NaN.
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
  unsigned u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (bf16_t)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (bf16_t)(u >> 16);
}

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef int i32x4_t __attribute__((ext_vector_type(4)));

// Hardware conversion (v_cvt_pk_bf16_f32: round to nearest even, NaN stays NaN).
__device__ __forceinline__ unsigned pack_bf16x2(float lo, float hi) {
  f32x2_t v = {lo, hi};
  return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2_t));
}
__device__ __forceinline__ bf16_t f32_to_bf16_hw(float f) { return (bf16_t)(pack_bf16x2(f, 0.f) & 0xffffu); }

// Raw buffer view of a tensor: loads whose byte offset is >= `bytes` return zeros, which is how
// the convolution kernels zero-pad without branches (invalid elements get offset kOobOffset).
constexpr unsigned kOobOffset = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ uint4 buffer_load16(__amdgpu_buffer_rsrc_t r, unsigned voffset, unsigned soffset) {
  return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)voffset, (int)soffset, 0));
}

template <typename T> struct Elem;
template <> struct Elem<float> {
  static __device__ __forceinline__ float ld(const float* p) { return *p; }
  static __device__ __forceinline__ void st(float* p, float v) { *p = v; }
};
template <> struct Elem<bf16_t> {
  static __device__ __forceinline__ float ld(const bf16_t* p) { return bf16_to_f32(*p); }
  static __device__ __forceinline__ void st(bf16_t* p, float v) { *p = f32_to_bf16(v); }
};

// 8 consecutive elements <-> 8 floats (16-byte access for bf16, 2x16 for float).
__device__ __forceinline__ void load8(const bf16_t* p, float* f) {
  uint4 v = *reinterpret_cast<const uint4*>(p);
  unsigned w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f[2 * i] = __uint_as_float(w[i] << 16);
    f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
  }
}
__device__ __forceinline__ void unpack8(uint4 v, float* f) {   // 8 bf16 held in registers
  unsigned w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f[2 * i] = __uint_as_float(w[i] << 16);
    f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
  }
}
__device__ __forceinline__ void load8(const float* p, float* f) {
  float4 a = *reinterpret_cast<const float4*>(p);
  float4 b = *reinterpret_cast<const float4*>(p + 4);
  f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w;
  f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
}
__device__ __forceinline__ void store8(bf16_t* p, const float* f) {
  uint4 v;
  v.x = pack_bf16x2(f[0], f[1]);
  v.y = pack_bf16x2(f[2], f[3]);
  v.z = pack_bf16x2(f[4], f[5]);
  v.w = pack_bf16x2(f[6], f[7]);
  *reinterpret_cast<uint4*>(p) = v;
}
__device__ __forceinline__ void store8(float* p, const float* f) {
  *reinterpret_cast<float4*>(p) = make_float4(f[0], f[1], f[2], f[3]);
  *reinterpret_cast<float4*>(p + 4) = make_float4(f[4], f[5], f[6], f[7]);
}

// store8 that leaves in f what was stored
__device__ __forceinline__ void store8_back(bf16_t* p, float* f) {
  const uint4 v = {pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]), pack_bf16x2(f[6], f[7])};
  *reinterpret_cast<uint4*>(p) = v;
  unpack8(v, f);
}
__device__ __forceinline__ void store8_back(float* p, float* f) { store8(p, f); }

// eight bf16 plus eight bf16, rounded again
__device__ __forceinline__ uint4 add_bf16x8(uint4 a, uint4 b) {
  float x[8], y[8];
  unpack8(a, x);
  unpack8(b, y);
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] += y[e];
  return uint4{pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(x[4], x[5]), pack_bf16x2(x[6], x[7])};
}
// v of the lane N before this one in its sixteen, around the end (an operand modifier, no pass through LDS)
template <int N> __device__ __forceinline__ float row_rotated(float v) {
  return __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), 0x120 + N, 0xf, 0xf, true));
}

// f over the 64 lanes of a wavefront, the result in every lane: rotations within rows of sixteen as operand modifiers, then rows and halves that
// trade places (v_permlane*_swap).  Through LDS (ds_bpermute) each of the six steps was a round trip, which is what
// the short kernels are made of: the classifier head of eight samples of 16 features, with the rest of its changes, 10.5 -> 6.8 us, layer norm of
// 788 rows of 768 4.6 -> 4.3.
// f has to be commutative; all lanes then see the same roundings.
template <int N> __device__ __forceinline__ int row_rotated(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x120 + N, 0xf, 0xf, true); }
template <int N> __device__ __forceinline__ double row_rotated(double v) {
  const uint2 u = __builtin_bit_cast(uint2, v);
  return __builtin_bit_cast(double, make_uint2((unsigned)row_rotated<N>((int)u.x), (unsigned)row_rotated<N>((int)u.y)));
}
template <class F> __device__ __forceinline__ float across_rows(float v, F f) {
  const unsigned u = __float_as_uint(v);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const unsigned w = __float_as_uint(f(__uint_as_float(r[0]), __uint_as_float(r[1])));
  const auto h = __builtin_amdgcn_permlane32_swap(w, w, false, false);
  return f(__uint_as_float(h[0]), __uint_as_float(h[1]));
}
template <class F> __device__ __forceinline__ int across_rows(int v, F f) {
  const auto r = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
  const int w = f((int)r[0], (int)r[1]);
  const auto h = __builtin_amdgcn_permlane32_swap((unsigned)w, (unsigned)w, false, false);
  return f((int)h[0], (int)h[1]);
}
template <class F> __device__ __forceinline__ double across_rows(double v, F f) {
  uint2 u = __builtin_bit_cast(uint2, v);
  const auto x = __builtin_amdgcn_permlane16_swap(u.x, u.x, false, false), y = __builtin_amdgcn_permlane16_swap(u.y, u.y, false, false);
  u = __builtin_bit_cast(uint2, f(__builtin_bit_cast(double, make_uint2(x[0], y[0])), __builtin_bit_cast(double, make_uint2(x[1], y[1]))));
  const auto z = __builtin_amdgcn_permlane32_swap(u.x, u.x, false, false), w = __builtin_amdgcn_permlane32_swap(u.y, u.y, false, false);
  return f(__builtin_bit_cast(double, make_uint2(z[0], w[0])), __builtin_bit_cast(double, make_uint2(z[1], w[1])));
}
template <class T, class F> __device__ __forceinline__ T wave_all(T v, F f) {
  v = f(v, row_rotated<8>(v));
  v = f(v, row_rotated<4>(v));
  v = f(v, row_rotated<2>(v));
  v = f(v, row_rotated<1>(v));
  return across_rows(v, f);
}
template <class T> __device__ __forceinline__ T wave_sum(T v) {
  return wave_all(v, [](T a, T b) { return a + b; });
}
__device__ __forceinline__ float wave_max(float v) {
  return wave_all(v, [](float a, float b) { return fmaxf(a, b); });
}
__device__ __forceinline__ int wave_min(int v) {
  return wave_all(v, [](int a, int b) { return a < b ? a : b; });
}

// n / d of wavefront-uniform 0 <= n < 2^20, d >= 1, without the compiler's integer division (about 150 clocks in front of a
// kernel's first load).  Exact: (n + 1/2) / d is at least 1 / (2 d) from a whole number, which the two roundings (below
// 2^-22 of the quotient) do not reach; with d = 1 exact up to 2^23.
__device__ __forceinline__ int uniform_div(int n, int d) {
  return __builtin_amdgcn_readfirstlane((int)(((float)n + 0.5f) * __builtin_amdgcn_rcpf((float)d)));
}

static inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
static inline int conv_out(int H, int pad, int R, int stride) { return (H + 2 * pad - R) / stride + 1; }
static inline size_t elem_size(int dtype) { return dtype == CNNK_BF16 ? 2 : 4; }

static inline int launch_status() { return hipGetLastError() == hipSuccess ? CNNK_OK : CNNK_ERR_HIP; }

int cnnk_validate_conv(const cnnk_conv_desc* d);
