// Division of non-negative integers by a runtime constant without the ~30-instruction hardware-less integer
// division: q = (x * magic) >> (31 + l) with l = ceil(log2 d) and magic = floor(2^(31 + l) / d) + 1, which fits 32
// bits because d > 2^(l - 1).  Exact for every 0 <= x < 2^31: with e = magic * d - 2^(31 + l) <= d <= 2^l, the
// product exceeds x / d by x * e / (d * 2^(31 + l)) < 1 / d.  (A fixed shift by 32 needs x * d < 2^32, which pixel
// indices of large images exceed: the quotient is then one too large next to a row's end.)
#pragma once

struct FastDiv {
  unsigned d, magic, shift;
  __host__ __device__ void init(unsigned dd) {
    unsigned l = 0;
    while (l < 31 && (1u << l) < dd) ++l;
    d = dd;
    magic = dd > 1 ? (unsigned)((1ull << (31 + l)) / dd) + 1u : 0u;
    shift = l > 0 ? l - 1 : 0;
  }
  __host__ __device__ __forceinline__ int div(int x) const {
    return d > 1 ? (int)((unsigned)(((unsigned long long)(unsigned)x * magic) >> 32) >> shift) : x;
  }
  __host__ __device__ __forceinline__ void divmod(int x, int* q, int* r) const { *q = div(x); *r = x - *q * (int)d; }
};
