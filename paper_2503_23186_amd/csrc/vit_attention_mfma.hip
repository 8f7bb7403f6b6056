// Self-attention on the matrix cores for bf16 storage, head size 64 and sequences of at most 256
// tokens (a ViT-B/16 image: 197): forward and backward of softmax(q k^T / 8) v, one (image, head) or a part of one
// per workgroup, 32-token blocks by wavefronts (v_mfma_f32_32x32x16_bf16, fp32 accumulation).
//
// The two matrices that a workgroup walks over (K and V; for dk and dv: Q and dO) sit in LDS, in their natural
// [token][feature] layout: two planes of 32 features with 64-byte rows whose 16-byte chunks are
// XOR-swizzled by row bits 2-3.  Products that reduce over features read fragments with 16-byte loads
// (a token per lane); products that reduce over tokens read the same bytes with the transposing
// load ds_read_b64_tr_b16 (a feature per lane, four consecutive tokens per read).  Both patterns touch
// every LDS bank once per pass.
//
// Score tiles are computed transposed (rows = keys, columns = queries) where the softmax runs over
// keys, so that a query's row statistics are per-lane scalars, and the accumulator of a score tile is
// at once the B operand of the product that follows it: register i of lane l holds key
// (i/4)*8 + (l/32)*4 + i%4 of the tile, so registers 8j..8j+7 are the lane's eight reduction slots of
// 16-key step j, and the A operand is read with the same key-to-slot assignment (rows h*4..h*4+3 and
// 8+h*4..8+h*4+3 of the step for lane half h) instead of the usual 8 consecutive ones.
// Probabilities are not stored: the forward pass writes log-sum-exp per query and the backward pass
// recomputes exp(s - lse).  The backward pass walks twice, by query block for dq and
// by key block for dk and dv (which recomputes the score tiles in the other orientation), in workgroups of their own or one after the
// other, so every sum has one owner and a fixed order: no atomics, bit-reproducible.
#include "common.h"
#include "../../include/cnnk_vit.h"

namespace {
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef short s16x8_t __attribute__((ext_vector_type(8)));
constexpr int kDH = 64;
constexpr int ROW_B = 64;       // bytes of one token's 32 features of a plane

__device__ __forceinline__ int chunk_off(int row, int c16) { return row * ROW_B + ((c16 ^ ((row >> 2) & 3)) << 4); }

// 16-byte fragment read: token `row`, features d0 .. d0+7 (d0 a multiple of 8)
__device__ __forceinline__ bf16x8_t frag_read(const unsigned char* t, int plane_b, int row, int d0) {
  const unsigned char* p = t + (d0 >> 5) * plane_b + chunk_off(row, (d0 & 31) >> 3);
  return *reinterpret_cast<const bf16x8_t*>(p);
}
// Transposing fragment read for a product that reduces over tokens: the lane gets feature
// mt*32 + lane%32 of tokens rbase + h*4 + 0..3 and rbase + 8 + h*4 + 0..3 (h = lane / 32).
__device__ __forceinline__ bf16x8_t frag_read_tr(const unsigned char* t, int plane_b, int mt, int rbase, int lane) {
  const int g = lane >> 4, i16 = lane & 15;
  const int ch0 = (g & 1) * 16 + (i16 & 3) * 4;               // first of the 4 features this lane's address names
  const int row = rbase + (g >> 1) * 4 + (i16 >> 2);
  const unsigned char* base = t + mt * plane_b + (ch0 & 7) * 2;
  const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (s16x4_t __attribute__((address_space(3)))*)(base + chunk_off(row, ch0 >> 3)));
  const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (s16x4_t __attribute__((address_space(3)))*)(base + chunk_off(row + 8, ch0 >> 3)));
  const s16x8_t v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  return __builtin_bit_cast(bf16x8_t, v);
}
__device__ __forceinline__ bf16x8_t pack_frag(const f32x16_t& a, int j) {
  uint4 v;
  v.x = pack_bf16x2(a[8 * j + 0], a[8 * j + 1]);
  v.y = pack_bf16x2(a[8 * j + 2], a[8 * j + 3]);
  v.z = pack_bf16x2(a[8 * j + 4], a[8 * j + 5]);
  v.w = pack_bf16x2(a[8 * j + 6], a[8 * j + 7]);
  return __builtin_bit_cast(bf16x8_t, v);
}
__device__ __forceinline__ f32x16_t zero16() {
  f32x16_t z;
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = 0.f;
  return z;
}
// Rows [0, Tp) of a head's 64 features (global rows `ld` elements apart) into the two LDS planes; rows
// >= T are zero.  A workgroup has at least 64 threads per 64 rows, so a thread moves at most NP = 8 16-byte
// pieces of a matrix (4 where there are 64 threads per 32 rows): fetch() issues the loads, put() stores them - a caller fetches all its
// matrices before it puts the first, so that a thread has all its loads in flight at once (as a loop of
// load-then-store the sixteen loads of the backward pass ran one after the other, a third of the launch).
template <int NP> struct Pieces {
  uint4 v[NP];
  __device__ __forceinline__ void fetch(const bf16_t* src, size_t ld, int T) {
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const int i = threadIdx.x + k * blockDim.x, r = i >> 3, c8 = i & 7;
      v[k] = make_uint4(0u, 0u, 0u, 0u);
      if (r < T) v[k] = *reinterpret_cast<const uint4*>(src + (size_t)r * ld + c8 * 8);
    }
  }
  __device__ __forceinline__ void put(unsigned char* dst, int plane_b, int Tp) const {
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const int i = threadIdx.x + k * blockDim.x, r = i >> 3, c8 = i & 7;
      if (NP == 4 || r < Tp) *reinterpret_cast<uint4*>(dst + (c8 >> 2) * plane_b + chunk_off(r, c8 & 3)) = v[k];
    }
  }
};
// the four fragments of the wavefront's own tokens, straight from memory (zeros past T)
__device__ __forceinline__ void own_frags(const bf16_t* src, size_t ld, int token, int T, int h, bf16x8_t* f) {
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (token < T) v = *reinterpret_cast<const uint4*>(src + (size_t)token * ld + ks * 16 + h * 8);
    f[ks] = __builtin_bit_cast(bf16x8_t, v);
  }
}
__device__ __forceinline__ float dot8(uint4 a, uint4 b) {
  float x[8], y[8], s = 0.f;
  unpack8(a, x);
  unpack8(b, y);
#pragma unroll
  for (int e = 0; e < 8; ++e) s = fmaf(x[e], y[e], s);
  return s;
}
// What a workgroup of a launch over `heads` (image, head) pairs works on: which pair (false: none) and which of `parts` parts of it.  The parts of a
// pair run on one XCD (every 8th workgroup shares its L2), one behind the other.
__device__ __forceinline__ bool head_part(int heads, int parts, int* head, int* part) {
  const int l = blockIdx.x >> 3, g = l / parts;
  *part = l - g * parts;
  *head = g * 8 + (blockIdx.x & 7);
  return *head < heads;
}
// a 32 x 32 tile of X Y^T over the 64 features: rows = tokens arow0.. of the LDS matrix `a`, columns =
// the wave's own tokens, whose four fragments are in `b`
__device__ __forceinline__ f32x16_t tile_nt(const unsigned char* a, int plane_b, int arow0, const bf16x8_t* b, int lane) {
  f32x16_t acc = zero16();
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_read(a, plane_b, arow0 + (lane & 31), ks * 16 + (lane >> 5) * 8), b[ks], acc, 0, 0, 0);
  return acc;
}
// The accumulator of a [64 features] x [32 own tokens] product: a lane holds four consecutive features of every eight, its
// partner in the other half the other four.  They trade, so that a lane stores eight.
__device__ __forceinline__ void store_cols(bf16_t* dst_row, const f32x16_t* acc, int h, bool inside) {
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int i8 = 0; i8 < 2; ++i8) {
      const f32x16_t& a = acc[mt];
      unsigned w[4];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const unsigned lo = pack_bf16x2(a[8 * i8 + 2 * k], a[8 * i8 + 2 * k + 1]), hi = pack_bf16x2(a[8 * i8 + 4 + 2 * k], a[8 * i8 + 5 + 2 * k]);
        const auto t = __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
        w[k] = t[0];
        w[2 + k] = t[1];
      }
      if (inside) *reinterpret_cast<uint4*>(dst_row + mt * 32 + i8 * 16 + h * 8) = uint4{w[0], w[1], w[2], w[3]};
    }
}

// Forward, one walk over the keys (online softmax: M. Milakov, N. Gimelshein, 2018; the lazily raised reference is FlashAttention-4's
// conditional rescaling).  The sums are kept relative to a reference m of the raw scores, common to a query's two lanes: the running
// maximum, but raised (and what was summed rescaled) only when a score passes it by more than `kSlack` / c in the exponent, so that
// after the first tile this hardly happens; probabilities stay below 2^kSlack, and the division by their sum comes last.  (Two walks, the
// second with the first's sum, computed every score and exponential twice: 197 tokens, 12 heads, batch 64 30.5 -> 26.0 us, batch 8 11.0 -> 8.3,
// batch 4 10.8 -> 7.9.)
constexpr float kSlack = 8.f;
template <int NP>
__global__ void __launch_bounds__(512, 4) attn_mfma_fwd_kernel(const bf16_t* __restrict__ qkv, bf16_t* __restrict__ o,
                                                               float* __restrict__ lse, int T, int heads, int pairs, int parts) {
  extern __shared__ __align__(16) unsigned char smem[];
  int pair, part;
  if (!head_part(pairs, parts, &pair, &part)) return;
  const int NT = (T + 31) >> 5, Tp = NT * 32, plane_b = Tp * ROW_B;
  unsigned char* Ks = smem;
  unsigned char* Vs = smem + 2 * plane_b;
  const int b = pair / heads, head = pair - b * heads, d = heads * kDH;
  const bf16_t* base = qkv + (size_t)b * T * 3 * d + head * kDH;
  Pieces<NP> pk, pv;
  pk.fetch(base + d, 3 * (size_t)d, T);
  pv.fetch(base + 2 * d, 3 * (size_t)d, T);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n = lane & 31, h = lane >> 5;
  const int blk = part * (blockDim.x >> 6) + wave, q = blk * 32 + n;
  bf16x8_t bq[4];
  own_frags(base, 3 * (size_t)d, q, T, h, bq);
  pk.put(Ks, plane_b, Tp);
  pv.put(Vs, plane_b, Tp);
  __syncthreads();
  if (blk >= NT) return;
  // exp(s / 8 - x) = exp2(s c - x c) with c = log2 e / 8: the scale rides in the multiply-add in front of
  // the exponential.  Keys past T exist only in the last tile, so only that tile masks.
  const float c2 = 0.125f * 1.44269504088896341f;
  float m = -INFINITY, l = 0.f;      // l: of this lane's half of the keys
  f32x16_t oacc[2] = {zero16(), zero16()};
  for (int kt = 0; kt < NT; ++kt) {
    f32x16_t s = tile_nt(Ks, plane_b, kt * 32, bq, lane);
    if (kt == NT - 1) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (kt * 32 + (i >> 2) * 8 + h * 4 + (i & 3) >= T) s[i] = -INFINITY;
    }
    float tm = s[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) tm = fmaxf(tm, s[i]);
    const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(tm), __float_as_uint(tm), false, false);
    tm = fmaxf(__uint_as_float(halves[0]), __uint_as_float(halves[1]));
    if (__any(tm > m + kSlack / c2)) {
      const float mn = fmaxf(m, tm);
      const float f = m == mn ? 1.f : __builtin_amdgcn_exp2f((m - mn) * c2);      // also where both are -inf
      l *= f;
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[mt][i] *= f;
      m = mn;
    }
    const float mc = m > -INFINITY ? m * c2 : 0.f;
    float add[2] = {0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      s[i] = __builtin_amdgcn_exp2f(fmaf(s[i], c2, -mc));
      add[i & 1] += s[i];
    }
    l += add[0] + add[1];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const bf16x8_t pb = pack_frag(s, j);
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
        oacc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_read_tr(Vs, plane_b, mt, kt * 32 + 16 * j, lane), pb, oacc[mt], 0, 0, 0);
    }
  }
  l += __shfl_xor(l, 32, 64);
  const float L2 = fmaf(m, c2, __builtin_amdgcn_logf(l));      // log2 of the sum of exp(s / 8)
  // Undivided sums are up to 2^kSlack T times the result.  Where one left the range of fp32 (values of V above 5e33), walk again with
  // probabilities that are divided first, whose sums are no larger than the largest value.  (The test: 197 tokens, 768 heads 28.4 -> 28.7 us.)
  float part4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int i = 0; i < 16; ++i) part4[i & 3] = fmaf(oacc[mt][i], 0.f, part4[i & 3]);      // not a number if one is infinite or none
  const float left = (part4[0] + part4[1]) + (part4[2] + part4[3]);
  float inv = 1.f / l;
  if (__builtin_expect(__any(left != 0.f), 0)) {
    inv = 1.f;
    oacc[0] = oacc[1] = zero16();
    for (int kt = 0; kt < NT; ++kt) {
      f32x16_t s = tile_nt(Ks, plane_b, kt * 32, bq, lane);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        s[i] = __builtin_amdgcn_exp2f(fmaf(s[i], c2, -L2));
        if (kt * 32 + (i >> 2) * 8 + h * 4 + (i & 3) >= T) s[i] = 0.f;
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const bf16x8_t pb = pack_frag(s, j);
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
          oacc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_read_tr(Vs, plane_b, mt, kt * 32 + 16 * j, lane), pb, oacc[mt], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int i = 0; i < 16; ++i) oacc[mt][i] *= inv;
  store_cols(o + ((size_t)b * T + q) * d + head * kDH, oacc, h, q < T);
  if (q < T && h == 0) lse[((size_t)b * heads + head) * T + q] = L2 * 0.69314718055994531f;
}

// The backward pass's walks.  X, Y: K and V of all keys for dq, Q and dO of all queries for dk and dv, in LDS; x, y: the lane's own row
// of the others.
// Tokens past T are rows of zeros in all four matrices.  A query past T has L = D = 0: its probabilities are exp(0 - 0) = 1
// and multiply its zero rows of dO and Q in dv and dk, so the walk over the queries masks nothing.  A key past T meets real
// queries: its score is 0, and where a query's log-sum-exp lies below -88 its exponential is infinite, times its zero row
// of K not a number.  The walk over the keys masks the last tile.  (The lane's own token past T ends in a column that is not stored.)
constexpr float kScale = 0.125f, kLog2e = 1.44269504088896341f, kC2 = 0.125f * 1.44269504088896341f;
// dq^T = k^T ds^T, of the lane's query: exp(s / 8 - L) = exp2(s c - L2) with c = log2 e / 8, and ds = p (dp - D) / 8 = p (dp / 8 - Dsc)
__device__ __forceinline__ void walk_keys(const unsigned char* Xs, const unsigned char* Ys, int plane_b, int NT, int T, const bf16x8_t* x, const bf16x8_t* y,
                                          float L2, float Dsc, int lane, f32x16_t (&dq)[2]) {
  const int h = lane >> 5;
  dq[0] = dq[1] = zero16();
  for (int kt = 0; kt < NT; ++kt) {
    const f32x16_t s = tile_nt(Xs, plane_b, kt * 32, x, lane);     // [key][query]
    f32x16_t dp = tile_nt(Ys, plane_b, kt * 32, y, lane);
#pragma unroll
    for (int i = 0; i < 16; ++i) dp[i] = __builtin_amdgcn_exp2f(fmaf(s[i], kC2, -L2)) * fmaf(dp[i], kScale, -Dsc);
    if (kt == NT - 1) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (kt * 32 + (i >> 2) * 8 + h * 4 + (i & 3) >= T) dp[i] = 0.f;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const bf16x8_t dsb = pack_frag(dp, j);
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
        dq[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_read_tr(Xs, plane_b, mt, kt * 32 + 16 * j, lane), dsb, dq[mt], 0, 0, 0);
    }
  }
}
// dv^T = do^T p, dk^T = q^T ds, of the lane's key; Ls, Ds: L2 and Dsc of every query
__device__ __forceinline__ void walk_queries(const unsigned char* Xs, const unsigned char* Ys, const float* Ls, const float* Ds, int plane_b, int NT,
                                             const bf16x8_t* x, const bf16x8_t* y, int lane, f32x16_t (&dk)[2], f32x16_t (&dv)[2]) {
  const int h = lane >> 5;
  dk[0] = dk[1] = zero16();
  dv[0] = dv[1] = zero16();
  for (int qt = 0; qt < NT; ++qt) {
    f32x16_t p = tile_nt(Xs, plane_b, qt * 32, x, lane);           // [query][key]
    f32x16_t dp = tile_nt(Ys, plane_b, qt * 32, y, lane);
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      const int r0 = qt * 32 + i4 * 8 + h * 4;
      const float4 L4 = *reinterpret_cast<const float4*>(Ls + r0);
      const float4 D4 = *reinterpret_cast<const float4*>(Ds + r0);
      const float Lr[4] = {L4.x, L4.y, L4.z, L4.w}, Dr[4] = {D4.x, D4.y, D4.z, D4.w};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int i = i4 * 4 + k;
        const float pp = __builtin_amdgcn_exp2f(fmaf(p[i], kC2, -Lr[k]));
        p[i] = pp;
        dp[i] = pp * fmaf(dp[i], kScale, -Dr[k]);
      }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const bf16x8_t pb = pack_frag(p, j), dsb = pack_frag(dp, j);
#pragma unroll
      for (int mt = 0; mt < 2; ++mt) {
        dv[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_read_tr(Ys, plane_b, mt, qt * 32 + 16 * j, lane), pb, dv[mt], 0, 0, 0);
        dk[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_read_tr(Xs, plane_b, mt, qt * 32 + 16 * j, lane), dsb, dk[mt], 0, 0, 0);
      }
    }
  }
}
template <int CTRL> __device__ __forceinline__ float lane_moved(float v) {
  return __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), CTRL, 0xf, 0xf, true));
}
// Dsc of the tokens whose pieces of dO and O a thread holds, from the eight lanes of a token; Ls of all tokens
template <int NP>
__device__ __forceinline__ void put_sums(const Pieces<NP>& g, const Pieces<NP>& o, const float* lrow, int T, int Tp, float* Ls, float* Ds) {
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    float D = dot8(o.v[k], g.v[k]);
    D += lane_moved<0xb1>(D);       // from the neighbour, from the other pair of four, from the other four of eight
    D += lane_moved<0x4e>(D);
    D += lane_moved<0x141>(D);
    const int i = threadIdx.x + k * blockDim.x, r = i >> 3;
    if ((i & 7) == 0 && r < Tp) Ds[r] = D * kScale;
  }
  for (int t = threadIdx.x; t < Tp; t += blockDim.x) Ls[t] = t < T ? lrow[t] * kLog2e : 0.f;
}

// Backward, a workgroup to a pair: all four matrices in LDS, a wavefront to a 32-token block, dq first.  Where the pairs that
// a CU holds keep it busy this loads everything once; where they do not the kernel below is faster (attn_mfma_bwd has the line).
__global__ void __launch_bounds__(512) attn_mfma_bwd_whole_kernel(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ o,
                                                                  const bf16_t* __restrict__ d_o, const float* __restrict__ lse,
                                                                  bf16_t* __restrict__ dqkv, int T, int heads) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int NT = blockDim.x >> 6, Tp = NT * 32, plane_b = Tp * ROW_B;
  unsigned char* Qs = smem;
  unsigned char* Ks = smem + 2 * plane_b;
  unsigned char* Vs = smem + 4 * plane_b;
  unsigned char* Gs = smem + 6 * plane_b;
  float* Ls = reinterpret_cast<float*>(smem + 8 * plane_b);
  float* Ds = Ls + Tp;
  const int pair = blockIdx.x, b = pair / heads, head = pair - b * heads, d = heads * kDH;
  const size_t ld = 3 * (size_t)d;
  const bf16_t* base = qkv + (size_t)b * T * ld + head * kDH;
  bf16_t* dbase = dqkv + (size_t)b * T * ld + head * kDH;
  {
    Pieces<4> pq, pk, pv, pg, po;
    pq.fetch(base, ld, T);
    pk.fetch(base + d, ld, T);
    pv.fetch(base + 2 * d, ld, T);
    pg.fetch(d_o + (size_t)b * T * d + head * kDH, d, T);
    po.fetch(o + (size_t)b * T * d + head * kDH, d, T);
    pq.put(Qs, plane_b, Tp);
    pk.put(Ks, plane_b, Tp);
    pv.put(Vs, plane_b, Tp);
    pg.put(Gs, plane_b, Tp);
    put_sums(pg, po, lse + (size_t)pair * T, T, Tp, Ls, Ds);
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, own = (threadIdx.x >> 6) * 32 + (lane & 31), h = lane >> 5;      // this lane's query, then its key
  bf16x8_t x[4], y[4];
  {
    f32x16_t dq[2];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      x[ks] = frag_read(Qs, plane_b, own, ks * 16 + h * 8);
      y[ks] = frag_read(Gs, plane_b, own, ks * 16 + h * 8);
    }
    walk_keys(Ks, Vs, plane_b, NT, T, x, y, Ls[own], Ds[own], lane, dq);
    store_cols(dbase + (size_t)own * ld, dq, h, own < T);
  }
  f32x16_t dk[2], dv[2];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    x[ks] = frag_read(Ks, plane_b, own, ks * 16 + h * 8);
    y[ks] = frag_read(Vs, plane_b, own, ks * 16 + h * 8);
  }
  walk_queries(Qs, Gs, Ls, Ds, plane_b, NT, x, y, lane, dk, dv);
  store_cols(dbase + (size_t)own * ld + d, dk, h, own < T);
  store_cols(dbase + (size_t)own * ld + 2 * d, dv, h, own < T);
}

// Backward, a pair in parts: a workgroup of at most four wavefronts forms dq (part even) or dk and dv (odd) of some 32-token blocks of a pair.  It has two of the
// four matrices in LDS and its wavefronts' own rows of the others in registers, so that two workgroups share a CU and one
// loads while the other computes: with all four in LDS there is room for one.  197 tokens, 12 heads: batch 8 21.0 -> 16.3 us, batch 64 72 and
// 68: there the operand reads from LDS (768 clocks a tile pair of dk and dv, shared by four SIMDs), the vector ALU (800) and the matrix products (512)
// of two wavefronts a SIMD follow one another more than they overlap.
template <int NP>
__global__ void __launch_bounds__(256, 2) attn_mfma_bwd_kernel(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ o,
                                                               const bf16_t* __restrict__ d_o, const float* __restrict__ lse,
                                                               bf16_t* __restrict__ dqkv, int T, int heads, int pairs, int parts) {
  extern __shared__ __align__(16) unsigned char smem[];
  int pair, part;
  if (!head_part(pairs, parts, &pair, &part)) return;
  const int NT = (T + 31) >> 5, Tp = NT * 32, plane_b = Tp * ROW_B, waves = blockDim.x >> 6;
  unsigned char* Xs = smem;                      // K or Q
  unsigned char* Ys = smem + 2 * plane_b;        // V or dO
  const int b = pair / heads, head = pair - b * heads, d = heads * kDH;
  const size_t ld = 3 * (size_t)d;
  const bf16_t* base = qkv + (size_t)b * T * ld + head * kDH;
  const bf16_t* gbase = d_o + (size_t)b * T * d + head * kDH;
  const bf16_t* obase = o + (size_t)b * T * d + head * kDH;
  const float* lrow = lse + (size_t)pair * T;
  bf16_t* dbase = dqkv + (size_t)b * T * ld + head * kDH;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), n = lane & 31, h = lane >> 5;
  const int group = part >> 1, groups = parts >> 1;      // this workgroup's blocks: every groups * waves-th
  if ((part & 1) == 0) {
    // ---- by query block ----
    Pieces<NP> px, py;
    px.fetch(base + d, ld, T);
    py.fetch(base + 2 * d, ld, T);
    px.put(Xs, plane_b, Tp);
    py.put(Ys, plane_b, Tp);
    bool staged = false;
    for (int blk = group * waves + wave; blk < NT || !staged; blk += groups * waves) {
      const int own = blk * 32 + n;            // this lane's query
      bf16x8_t bq[4], bg[4], bo[4];
      own_frags(base, ld, own, T, h, bq);
      own_frags(gbase, d, own, T, h, bg);
      own_frags(obase, d, own, T, h, bo);
      const float L2 = own < T ? lrow[own] * kLog2e : 0.f;
      float D = 0.f;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) D += dot8(__builtin_bit_cast(uint4, bo[ks]), __builtin_bit_cast(uint4, bg[ks]));
      D += __shfl_xor(D, 32, 64);
      if (!staged) __syncthreads();
      staged = true;
      if (blk >= NT) break;
      f32x16_t dq[2];
      walk_keys(Xs, Ys, plane_b, NT, T, bq, bg, L2, D * kScale, lane, dq);
      store_cols(dbase + (size_t)own * ld, dq, h, own < T);
    }
  } else {
    // ---- by key block ----
    float* Ls = reinterpret_cast<float*>(smem + 4 * plane_b);
    float* Ds = Ls + Tp;
    {
      Pieces<NP> px, py, po;
      px.fetch(base, ld, T);
      py.fetch(gbase, d, T);
      po.fetch(obase, d, T);
      px.put(Xs, plane_b, Tp);
      py.put(Ys, plane_b, Tp);
      put_sums(py, po, lrow, T, Tp, Ls, Ds);
    }
    bool staged = false;
    for (int blk = group * waves + wave; blk < NT || !staged; blk += groups * waves) {
      const int own = blk * 32 + n;            // this lane's key
      bf16x8_t bk[4], bv[4];
      own_frags(base + d, ld, own, T, h, bk);
      own_frags(base + 2 * d, ld, own, T, h, bv);
      if (!staged) __syncthreads();
      staged = true;
      if (blk >= NT) break;
      f32x16_t dk[2], dv[2];
      walk_queries(Xs, Ys, Ls, Ds, plane_b, NT, bk, bv, lane, dk, dv);
      store_cols(dbase + (size_t)own * ld + d, dk, h, own < T);
      store_cols(dbase + (size_t)own * ld + 2 * d, dv, h, own < T);
    }
  }
}

template <typename Kern> int raise_lds(Kern kern, bool* raised, int bytes) {
  if (*raised) return CNNK_OK;
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, bytes) != hipSuccess) return CNNK_ERR_HIP;
  *raised = true;
  return CNNK_OK;
}
template <int NP>
int fwd_launch(const cnnk_attn_desc* d, const void* qkv, void* o, float* lse, int waves, int parts, hipStream_t st) {
  static bool raised = false;
  const int NT = (d->T + 31) / 32, pairs = d->B * d->heads;
  const int rc = raise_lds(attn_mfma_fwd_kernel<NP>, &raised, 4 * 8 * 32 * ROW_B);
  if (rc != CNNK_OK) return rc;
  attn_mfma_fwd_kernel<NP><<<(pairs + 7) / 8 * 8 * parts, 64 * waves, (size_t)4 * NT * 32 * ROW_B, st>>>((const bf16_t*)qkv, (bf16_t*)o, lse, d->T, d->heads, pairs, parts);
  return launch_status();
}
template <int NP>
int bwd_launch(const cnnk_attn_desc* d, const void* qkv, const void* o, const void* d_o, const float* lse, void* dqkv, int waves, int parts, hipStream_t st) {
  static bool raised = false;
  const int NT = (d->T + 31) / 32, pairs = d->B * d->heads;
  const int rc = raise_lds(attn_mfma_bwd_kernel<NP>, &raised, 4 * 8 * 32 * ROW_B + 2 * 8 * 32 * 4);
  if (rc != CNNK_OK) return rc;
  attn_mfma_bwd_kernel<NP><<<(pairs + 7) / 8 * 8 * parts, 64 * waves, (size_t)4 * NT * 32 * ROW_B + (size_t)2 * NT * 32 * sizeof(float), st>>>(
      (const bf16_t*)qkv, (const bf16_t*)o, (const bf16_t*)d_o, lse, (bf16_t*)dqkv, d->T, d->heads, pairs, parts);
  return launch_status();
}
int bwd_whole_launch(const cnnk_attn_desc* d, const void* qkv, const void* o, const void* d_o, const float* lse, void* dqkv, hipStream_t st) {
  static bool raised = false;
  const int NT = (d->T + 31) / 32;
  const int rc = raise_lds(attn_mfma_bwd_whole_kernel, &raised, 8 * 8 * 32 * ROW_B + 2 * 8 * 32 * 4);
  if (rc != CNNK_OK) return rc;
  attn_mfma_bwd_whole_kernel<<<d->B * d->heads, 64 * NT, (size_t)8 * NT * 32 * ROW_B + (size_t)2 * NT * 32 * sizeof(float), st>>>(
      (const bf16_t*)qkv, (const bf16_t*)o, (const bf16_t*)d_o, lse, (bf16_t*)dqkv, d->T, d->heads);
  return launch_status();
}
}  // namespace

bool attn_mfma_supported(const cnnk_attn_desc* d) {
  return d->dtype == CNNK_BF16 && d->dh == kDH && d->T <= 256;
}

int attn_mfma_fwd(const cnnk_attn_desc* d, const void* qkv, void* o, float* lse, hipStream_t st) {
  const int NT = (d->T + 31) / 32, half = (NT + 1) / 2;
  // Long sequences in two halves of their queries where that still gives a CU one workgroup at most (197 tokens: 96 pairs 8.3 us,
  // whole 9.1; 192 pairs 11.5, whole 10.6).
  if (NT > 4 && d->B * d->heads <= 128) return fwd_launch<8>(d, qkv, o, lse, half, 2, st);
  return fwd_launch<4>(d, qkv, o, lse, NT, 1, st);
}

// Which backward kernel.  In parts a pair's work overlaps better within a CU, as a whole it is loaded once and a CU holds nearly as many pairs in
// less LDS than twice the parts take.  Up to 128 tokens: as a whole where the parts need so many more rounds that they are slower, a round of whole
// pairs taking about 1.6 rounds of parts.  A CU holds 9, 4, 3, 2 whole pairs of one to four blocks (LDS) and the parts of 4, 2, 1, 1
// (registers: eight wavefronts).  us, whole / parts / all four matrices in LDS in every case, as before the parts: 32 tokens 768 pairs 11.3 / 11.6 / 11.8, 1536 16.6 /
// 20.7 / 18.5; 64 tokens 512 pairs 14.9 / 14.0 / 15.2, 576 15.9 / 17.7 / 17.0; 65 tokens 256 pairs 11.7 / 10.3 / 11.8, 576 19.6 / 21.9 / 19.4, 1536 37.5 /
// 46.2 / 42.4; 128 tokens 512 pairs 25.2 / 27.3 / 26.9, 576 33.9 / 31.5 / 36.4.
// Longer sequences: four parts where they all fit the device at once, then as a whole while that is one round, or a second one that is
// nearly full, otherwise two parts of two blocks to a wavefront.  us, whole / two / four parts: 197 tokens 96 pairs 20.8 / 17.6 / 16.3, 160 22.6 / 24.4 / 24.4, 256
// 26.7 / 28.0 / 31.3, 288 42.8 / 37.1 / 36.3, 512 49.1 / 49.8 / 56.4, 768 71.7 / 68.4 / 76.6.
int attn_mfma_bwd(const cnnk_attn_desc* d, const void* qkv, const void* o, const void* d_o, const float* lse, void* dqkv,
                  hipStream_t st) {
  const int NT = (d->T + 31) / 32, half = (NT + 1) / 2, pairs = d->B * d->heads;
  bool whole;
  if (NT <= 4) {
    constexpr int kHeld[4] = {9, 4, 3, 2}, kHeldInParts[4] = {4, 2, 1, 1};
    const long rounds = (pairs + 256L * kHeld[NT - 1] - 1) / (256 * kHeld[NT - 1]), parts = (pairs + 256L * kHeldInParts[NT - 1] - 1) / (256 * kHeldInParts[NT - 1]);
    whole = 8 * rounds < 5 * parts;
  } else {
    whole = (pairs > 128 && pairs <= 256) || (pairs > 448 && pairs <= 512);
  }
  if (whole) return bwd_whole_launch(d, qkv, o, d_o, lse, dqkv, st);
  if (NT <= 4) return bwd_launch<4>(d, qkv, o, d_o, lse, dqkv, NT, 2, st);
  return bwd_launch<8>(d, qkv, o, d_o, lse, dqkv, half, pairs <= 128 ? 4 : 2, st);
}
