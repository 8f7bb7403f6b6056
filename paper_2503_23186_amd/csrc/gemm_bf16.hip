// Dense bf16 matrix products of the Vision Transformer step's linear layers on the gfx950 matrix
// cores (v_mfma_f32_32x32x16_bf16, fp32 accumulation): y = x W^T (+ bias, + GELU), dx = dy W,
// dW = dy^T x.  One kernel, three operand orientations.
//
// Large problems (all shapes: kTiles): workgroup tile 256 x 128 (or 192 x 128), four wavefronts of 128 x 64 (0.75 KB of LDS operand reads per
// MFMA), LDS stage buffers filled straight from memory (buffer_load ... lds; out-of-range rows deposit
// zeros), one barrier per stage, two workgroups per CU.  Two configurations: 32 reduction elements per
// stage in 64-byte LDS rows with three stage buffers (loads two stages ahead), or - for the long
// reductions of an operand whose reduction index is the contiguous one - 64 elements per stage in
// 128-byte rows with two buffers (see Cfg below for why).  An operand whose reduction index is its
// contiguous one ("natural": x and W of the forward product, dy of the data gradient) lies in LDS as
// [row][reduction elements of the stage] and is read with 16-byte loads; an operand whose reduction
// index is its row index (W of the data gradient, both operands of the weight gradient) lies as planes
// of [reduction rows][32 or 64 columns] and is read with the transposing load ds_read_b64_tr_b16, so no
// operand is ever transposed in memory.  The 16-byte chunks of a row are XOR-swizzled so that both kinds
// of read touch every bank once per pass (swz_of).  Because the hardware fixes where a direct load's
// bytes land (lane i at base + 16 i), the layout is produced by which global bytes each lane asks for.
// Epilogue per wavefront through a private LDS strip (accumulator quads in, transposing reads out):
// 16-byte stores of 8 consecutive columns; bias and GELU are applied to the fp32 accumulator first, so
// an output is rounded once.  The weight gradient splits the row range over blockIdx.z and writes
// fp32 partials that a second kernel adds in a fixed order.
#include "common.h"
#include "gelu.h"
#include "gemm.h"
#include "mfma_tile.h"

extern int g_cnnk_tune[];

namespace {
template <bool ATR, bool BTR, int TM, int TN, int BK, int RB, int NST, int KG>
using Cfg = Tile<ATR, BTR, TM, TN, 2, BK, RB, NST, KG>;

struct Args {
  const bf16_t* A;
  const bf16_t* B;
  bf16_t* C;          // bf16 output [M][N] (EPI 0, 1)
  bf16_t* C2;         // EPI 1: gelu(C); EPI 4: C * gelu'(res)
  float* part;        // EPI 2: fp32 output, or partials zstride elements apart; EPI 4: [WM * mtiles][N] column sums of C2 before it is rounded
  float* rsum;        // EPI 2, nullable: [M] sums of A over the reduction (likewise zstride apart)
  size_t zstride;
  const float* bias;  // [N] or null
  const bf16_t* res;  // EPI 3: [M][N] added to the rounded output (a residual connection); EPI 4: gelu's argument
  int M, N, K;        // output rows, output columns, reduction length
  int lda, ldb, ldc;
  int k_per_split;    // reduction elements per blockIdx.z (a multiple of BK)
  int mtiles, ntiles;
  unsigned a_bytes, b_bytes, c_bytes;
  int fold;           // EPI 2, tiles that have the registers: stages between two folds of the accumulators
};

// the operands of a dense product
template <class C> struct DenseLoader {
  i32x4_t a_rs, b_rs;
  // byte offset of this lane's 16 bytes in stage 0, and their reduction index (the first element of a natural
  // operand's, the row of a transposed one's); those of stage t are in range while kk0 + t * BK < kend
  unsigned voff[C::NLOAD];
  int kk0[C::NLOAD];
  unsigned vinc_a, vinc_b;
  int kend, t;
  __device__ __forceinline__ void init(const Args& a, int m0, int n0, int kbeg, int kend_, int wave, int lane) {
    a_rs = make_desc(a.A, a.a_bytes);
    b_rs = make_desc(a.B, a.b_bytes);
    kend = kend_;
    vinc_a = C::ATR ? (unsigned)(C::BK * a.lda * 2) : C::BK * 2;
    vinc_b = C::BTR ? (unsigned)(C::BK * a.ldb * 2) : C::BK * 2;
#pragma unroll
    for (int j = 0; j < C::NLOAD; ++j) {
      const bool isA = j < C::NLOAD_A;
      const int ld = isA ? a.lda : a.ldb, o0 = isA ? m0 : n0, olim = isA ? a.M : a.N;
      const LoadSlot s = load_slot<C>(j, wave, lane);
      if (!(isA ? C::ATR : C::BTR)) {
        const int row = o0 + s.row;
        kk0[j] = row < olim ? kbeg + 8 * s.chunk : (1 << 30);
        voff[j] = (unsigned)((row * ld + kbeg + 8 * s.chunk) * 2);
      } else {
        const int col = o0 + s.plane * C::PC + 8 * s.chunk;
        kk0[j] = col < olim ? kbeg + s.row : (1 << 30);
        voff[j] = (unsigned)(((kbeg + s.row) * ld + col) * 2);
      }
    }
  }
  __device__ __forceinline__ void begin(int stage) { t = stage; }
  __device__ __forceinline__ unsigned offset(int j) const {
    return kk0[j] + t * C::BK < kend ? voff[j] + (unsigned)t * (j < C::NLOAD_A ? vinc_a : vinc_b) : kOobOffset;
  }
};

// Rows between two folds of a weight gradient's accumulators, near 3.4 sqrt(rows), where the errors of the two chains
// balance (a chain's grows with the root of its steps; 1568 rows 8.7e-8 with 128 and 9.3e-8 with 256, 12608 rows the
// same with 256 and 512, 27648 rows 2.0e-7 and 1.75e-7).
__host__ __device__ __forceinline__ int fold_rows(int rows) { return rows <= 2048 ? 128 : rows <= 10240 ? 256 : 512; }

// Writes a tile out.  prefetch() fetches what its first rows need besides the accumulators.
template <class C, int EPI> struct GemmEpilogue {
  static constexpr int TM = C::TM, TN = C::TN;
  static constexpr int STORES = TM * TN * 2 * (EPI == 1 || EPI == 4 ? 2 : 1);
  uint4 rv[2][TN][2];
  float bv[TN];
  // Loads and stores are buffer operations: a position outside the output reads zeros and
  // stores nothing, without a branch, so the number in flight is known and a wait is for what it needs.
  static __device__ __forceinline__ unsigned place(const Args& a, int m0, int n0, int i, int j, int rb, int lane, int wave) {
    const int wm = wave / C::WN, wn = wave % C::WN, g = lane >> 4, i16 = lane & 15;
    const int row = m0 + wm * (TM * 32) + i * 32 + rb * 16 + i16, col = n0 + wn * (TN * 32) + j * 32 + g * 8;
    return row < a.M && col < a.N ? (unsigned)(row * a.ldc + col) * 2u : kOobOffset;
  }
  // the residual (or gelu's argument) of a 32-row block is fetched while the block before it is worked on
  __device__ __forceinline__ void fetch(const Args& a, int m0, int n0, int i, int lane, int wave) {
    const __amdgpu_buffer_rsrc_t r_rs = make_rsrc(a.res, a.c_bytes);
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) rv[i & 1][j][rb] = buffer_load16(r_rs, place(a, m0, n0, i, j, rb, lane, wave), 0);
  }
  __device__ __forceinline__ void prefetch(const Args& a, int mt, int nt, int lane, int wave) {
    const int m0 = mt * C::BM, n0 = nt * C::BN, wn = wave % C::WN;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int colv = n0 + wn * (TN * 32) + j * 32 + (lane & 31);
      bv[j] = (a.bias && colv < a.N) ? a.bias[colv] : 0.f;
    }
    if (EPI == 3 || EPI == 4) fetch(a, m0, n0, 0, lane, wave);
  }
  // S0: LDS for a strip per wavefront
  __device__ __forceinline__ void write(const Args& a, int mt, int nt, f32x16_t (&acc)[TM][TN], int lane, int wave, unsigned char* S0) {
    const int wm = wave / C::WN, wn = wave % C::WN, g = lane >> 4, i16 = lane & 15;
    const int m0 = mt * C::BM, n0 = nt * C::BN;
    unsigned char* S = S0 + wave * (32 * SP);
    const __amdgpu_buffer_rsrc_t c_rs = make_rsrc(a.C, a.c_bytes);
    const __amdgpu_buffer_rsrc_t c2_rs = EPI == 1 || EPI == 4 ? make_rsrc(a.C2, a.c_bytes) : c_rs;
    float cs[TN][8];      // EPI 4: this lane's rows' share of the column sums
    if (EPI == 4) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 8; ++e) cs[j][e] = 0.f;
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      if ((EPI == 3 || EPI == 4) && i + 1 < TM) fetch(a, m0, n0, i + 1, lane, wave);
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        float v[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = acc[i][j][r] + bv[j];
        uint4 o[2];
        strip_transpose(S, lane, v, o);
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) {
          if (EPI == 3) o[rb] = add_bf16x8(o[rb], rv[i & 1][j][rb]);     // + residual: the sum of two stored values, rounded again
          buffer_store16(c_rs, o[rb], place(a, m0, n0, i, j, rb, lane, wave));
          if (EPI == 4) {     // the gradient of the activation's argument, from the gradient as stored
            float x[8], r[8];
            unpack8(o[rb], x);
            unpack8(rv[i & 1][j][rb], r);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              x[e] *= gelu_grad_f(r[e]);
              cs[j][e] += x[e];            // a row past the end adds zero
            }
            buffer_store16(c2_rs, uint4{pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(x[4], x[5]), pack_bf16x2(x[6], x[7])}, place(a, m0, n0, i, j, rb, lane, wave));
          }
        }
        if (EPI == 1) {
          // the activation of the value as stored
#pragma unroll
          for (int r = 0; r < 16; ++r) v[r] = gelu_f(bf16_to_f32(f32_to_bf16_hw(v[r])));
          strip_transpose(S, lane, v, o);
#pragma unroll
          for (int rb = 0; rb < 2; ++rb) buffer_store16(c2_rs, o[rb], place(a, m0, n0, i, j, rb, lane, wave));
        }
      }
    }
    if (EPI == 4) {
      // the bias gradient of the layer below sums the products before they are rounded: one partial row per row of
      // wavefronts, its sixteen lanes of a column added first
#pragma unroll
      for (int j = 0; j < TN; ++j) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          cs[j][e] += row_rotated<8>(cs[j][e]);
          cs[j][e] += row_rotated<4>(cs[j][e]);
          cs[j][e] += row_rotated<2>(cs[j][e]);
          cs[j][e] += row_rotated<1>(cs[j][e]);
        }
        const int col = n0 + wn * (TN * 32) + j * 32 + g * 8;
        if (i16 == 0 && col < a.N) {
          float* q = a.part + (size_t)(mt * C::WM + wm) * a.N + col;
          *reinterpret_cast<float4*>(q) = make_float4(cs[j][0], cs[j][1], cs[j][2], cs[j][3]);
          *reinterpret_cast<float4*>(q + 4) = make_float4(cs[j][4], cs[j][5], cs[j][6], cs[j][7]);
        }
      }
    }
  }
};

// One workgroup's tile (mt, nt) over the reduction range of split z: a weight gradient, two groups of wavefronts, or one tile to a workgroup.
template <class C, int EPI>
__device__ __forceinline__ void gemm_tile(const Args& a, int mt, int nt, int z) {
  constexpr int TM = C::TM, TN = C::TN, BK = C::BK, KG = C::KG;
  extern __shared__ __align__(16) unsigned char smem[];   // stage buffers, and the epilogue's room where it has its own
  const int lane = threadIdx.x & 63;
  const int kg = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8);   // reduction group
  const int tid = threadIdx.x & 255;                                                     // within the group
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / C::WN, wn = wave % C::WN, h = lane >> 5;
  const int m0 = mt * C::BM, n0 = nt * C::BN;
  int kbeg = z * a.k_per_split;
  int kend = kbeg + a.k_per_split;
  if (kend > a.K) kend = a.K;
  int nst = kend > kbeg ? (kend - kbeg + BK - 1) / BK : 0;
  if (KG > 1) {      // this group's part of the range; every group runs the same number of stages (the last ones load zeros past kend)
    nst = (nst + KG - 1) / KG;
    kbeg += kg * nst * BK;
    kend = min(kend, kbeg + nst * BK);
  }
  DenseLoader<C> ld;
  ld.init(a, m0, n0, kbeg, kend, wave, lane);
  // sums of A over the reduction (a bias gradient), by the wavefronts that hold the first column of tiles:
  // the operand is in their registers, and the vector ALU has room beside the MFMAs
  constexpr bool ROWS = EPI == 2 && KG == 1;
  const bool row_sums = ROWS && a.rsum != nullptr && nt == 0 && wn == 0;
  constexpr bool FOLD = EPI == 2 && TM * TN <= 6;
  tile_stream<C, 0, ROWS, FOLD>(ld, 1, nst, kg, wave, lane, smem, row_sums, a.fold, [](int) {}, [](int) {},
                                [&](int, f32x16_t (&acc)[TM][TN], float (&rs)[TM], unsigned char* strip) __attribute__((always_inline)) {
    if (KG > 1) tile_join_groups<C>(acc, kg, tid, smem);
    if (kg > 0) return;
    if constexpr (EPI == 2) {
      float* out = a.part + (size_t)z * a.zstride;
      if (row_sums) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          const float t = rs[i] + __shfl_xor(rs[i], 32, 64);     // the two halves of every reduction step
          const int row = m0 + wm * (TM * 32) + i * 32 + lane;
          if (lane < 32 && row < a.M) a.rsum[(size_t)z * a.zstride + row] = t;
        }
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const int col = n0 + wn * (TN * 32) + j * 32 + (lane & 31);
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int row = m0 + wm * (TM * 32) + i * 32 + (r >> 2) * 8 + h * 4 + (r & 3);
            if (row < a.M && col < a.N) out[(size_t)row * a.ldc + col] = acc[i][j][r];
          }
        }
    } else {
      GemmEpilogue<C, EPI> ep;
      ep.prefetch(a, mt, nt, lane, wave);
      ep.write(a, mt, nt, acc, lane, wave, KG > 1 ? smem + C::HAND_B : strip);      // HAND_B: behind the accumulators just taken over
    }
  });
}

// Tile number l of the XCD that this workgroup runs on (workgroups that share its L2 are every 8th), false past the last.
// An XCD owns a contiguous range of the row-major tile list, i.e. a band of tile rows, and walks it column by
// column: the workgroups in flight on it then share the band's rows of A, which stay in its L2,
// while B streams through once per XCD.
__device__ __forceinline__ bool band_tile(const Args& a, int l, int* mt_out, int* nt_out) {
  const int ntot = a.mtiles * a.ntiles, chunk = (ntot + 7) >> 3;
  const int c0 = (blockIdx.x & 7) * chunk, c1 = min(c0 + chunk, ntot);
  if (c0 + l >= c1) return false;
  const int r0 = uniform_div(c0, a.ntiles), s0 = c0 - r0 * a.ntiles, r1 = uniform_div(c1 - 1, a.ntiles), e1 = (c1 - 1) - r1 * a.ntiles + 1;
  if (r0 == r1) {
    *mt_out = r0;
    *nt_out = s0 + l;
    return true;
  }
  // Column nt has the whole rows between, the band's first row from column s0 on, its last row up to column e1: three
  // ranges of columns of equal height.  (Counted column by column, 48 columns took 1 us.)
  const int whole = r1 - r0 - 1, lo = min(s0, e1), hi = max(s0, e1);
  int h = whole + 1, first = 0, col = 0;                  // columns below lo: no first row, but the last
  if (l >= lo * h) {
    l -= lo * h;
    col = lo;
    h = whole + (s0 < e1 ? 2 : 0);
    first = s0 < e1 ? 1 : 0;
    if (l >= (hi - lo) * h) {
      l -= (hi - lo) * h;
      col = hi;
      h = whole + 1;
      first = 1;
    }
  }
  const int q = uniform_div(l, h);
  *nt_out = col + q;
  *mt_out = r0 + (l - q * h) + (1 - first);
  return true;
}

template <bool ATR, bool BTR, int EPI, int TM, int TN, int BK, int RB, int NSTAGE, int KG, bool WALK>
__global__ void __launch_bounds__(256 * KG, (Cfg<ATR, BTR, TM, TN, BK, RB, NSTAGE, KG>::WPE)) gemm_kernel(Args a) {
  using C = Cfg<ATR, BTR, TM, TN, BK, RB, NSTAGE, KG>;
  int mt, nt;
  const int l = blockIdx.x >> 3, step = gridDim.x >> 3;
  if (!band_tile(a, l, &mt, &nt)) return;
  if constexpr (!WALK) {
    gemm_tile<C, EPI>(a, mt, nt, blockIdx.z);
  } else {
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int ntot = a.mtiles * a.ntiles, chunk = (ntot + 7) >> 3, mine = min(chunk, ntot - (int)(blockIdx.x & 7) * chunk);
    DenseLoader<C> ld;
    GemmEpilogue<C, EPI> ep;
    // the tile whose products are formed; the loads may already be at the next one
    int cmt = 0, cnt = 0;
    tile_stream<C, GemmEpilogue<C, EPI>::STORES, false, false>(
        ld, (mine - l + step - 1) / step, (a.K + BK - 1) / BK, 0, wave, lane, smem, false, 0,
        [&](int k) __attribute__((always_inline)) {
          if (k > 0) band_tile(a, l + k * step, &mt, &nt);
          ld.init(a, mt * C::BM, nt * C::BN, 0, a.K, wave, lane);
        },
        [&](int k) __attribute__((always_inline)) {
          band_tile(a, l + k * step, &cmt, &cnt);
          ep.prefetch(a, cmt, cnt, lane, wave);
        },
        [&](int, f32x16_t (&acc)[TM][TN], float (&)[TM], unsigned char* strip) __attribute__((always_inline)) { ep.write(a, cmt, cnt, acc, lane, wave, strip); });
  }
}

// Several weight gradients in one launch.  Alone, one of ViT-B/16's has 18 to 72 tiles of 256 x 128 for 256
// CUs and had to be split three to ten ways over its rows, each split a partial to write and to add up; the
// tiles of a block together fill the device unsplit.  Tiles of 192 x 128 at most: a wavefront then has registers for
// the second set of accumulators that an unsplit sum over all rows needs to be as exact as a split one (ViT-B/16 at
// batch 64, step 11.32 ms; 128 x 128 tiles 11.62; 256 x 128 without the second set 11.21).
constexpr int kGroupMax = 32;
struct GroupProblem {
  const bf16_t* dy;
  const bf16_t* x;
  float* dw;
  float* db;
  int rows, K, N, ntiles, tile0;
};
struct GroupArgs {
  int count, tiles, splits;
  GroupProblem p[kGroupMax];
  float* part;                 // splits > 1: [splits][elements of all problems]
  size_t zstride;              // elements of all problems
  size_t off[kGroupMax];       // splits > 1: where problem i starts in a partial (dw, then db)
};
template <int TM, int TN, int BK, int RB, int NSTAGE>
__global__ void __launch_bounds__(256, (Cfg<true, true, TM, TN, BK, RB, NSTAGE, 1>::WPE)) wgrad_group_kernel(GroupArgs ga) {
  // an XCD (every 8th workgroup) owns a contiguous range of the tile list
  const int chunk = (ga.tiles + 7) >> 3, l = blockIdx.x >> 3;
  const int tile = (blockIdx.x & 7) * chunk + l;
  if (l >= chunk || tile >= ga.tiles) return;
  int i = 0;
  while (i + 1 < ga.count && tile >= ga.p[i + 1].tile0) ++i;
  const GroupProblem& p = ga.p[i];
  Args a{};
  a.A = p.dy; a.B = p.x;
  a.M = p.N; a.N = p.K; a.K = p.rows; a.lda = p.N; a.ldb = p.K; a.ldc = p.K;
  a.a_bytes = (unsigned)p.rows * (unsigned)p.N * 2u; a.b_bytes = (unsigned)p.rows * (unsigned)p.K * 2u;
  const int stages = ((p.rows + BK - 1) / BK + ga.splits - 1) / ga.splits;
  a.k_per_split = stages * BK;
  a.fold = fold_rows(p.rows) / BK;
  if (ga.splits > 1) {
    a.part = ga.part + ga.off[i];
    a.rsum = p.db ? a.part + (size_t)p.N * p.K : nullptr;
    a.zstride = ga.zstride;
  } else {
    a.part = p.dw;
    a.rsum = p.db;
  }
  const int q = tile - p.tile0, mt = q / p.ntiles;
  gemm_tile<Cfg<true, true, TM, TN, BK, RB, NSTAGE, 1>, 2>(a, mt, q - mt * p.ntiles, blockIdx.z);
}
// sums of the partials of a group, in split order
__global__ void __launch_bounds__(256) sum_group_kernel(GroupArgs ga) {
  for (size_t e = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4; e < ga.zstride; e += (size_t)gridDim.x * 1024) {
    float4 s = *reinterpret_cast<const float4*>(ga.part + e);
    for (int z = 1; z < ga.splits; ++z) {
      const float4 v = *reinterpret_cast<const float4*>(ga.part + (size_t)z * ga.zstride + e);
      s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
    int i = 0;
    while (i + 1 < ga.count && e >= ga.off[i + 1]) ++i;
    const size_t k = e - ga.off[i], nw = (size_t)ga.p[i].N * ga.p[i].K;      // both multiples of 8
    if (k < nw) *reinterpret_cast<float4*>(ga.p[i].dw + k) = s;
    else if (ga.p[i].db) *reinterpret_cast<float4*>(ga.p[i].db + (k - nw)) = s;
  }
}

// out[i] = sum over splits (ascending) of part[z][i]; n a multiple of 4
__global__ void __launch_bounds__(256) sum_partials_kernel(const float* __restrict__ part, int splits, size_t n,
                                                           float* __restrict__ out) {
  for (size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4; i < n; i += (size_t)gridDim.x * 1024) {
    float4 s = *reinterpret_cast<const float4*>(part + i);
    for (int z = 1; z < splits; ++z) {
      const float4 p = *reinterpret_cast<const float4*>(part + (size_t)z * n + i);
      s.x += p.x; s.y += p.y; s.z += p.z; s.w += p.w;
    }
    *reinterpret_cast<float4*>(out + i) = s;
  }
}

template <typename Kern>
int launch(Kern kern, bool* raised, int threads, int smem_bytes, int per_xcd, const Args& a, int splits, hipStream_t st) {
  if (!*raised) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, smem_bytes) != hipSuccess)
      return CNNK_ERR_HIP;
    *raised = true;
  }
  hipLaunchKernelGGL(kern, dim3(8 * per_xcd, 1, splits), dim3(threads), smem_bytes, st, a);
  return launch_status();
}
template <bool ATR, bool BTR, int EPI, int TM, int TN, int BK, int RB, int NST, int KG>
int launch_cfg(Args& a, int splits, hipStream_t st) {
  static bool raised[2] = {false, false};
  using C = Cfg<ATR, BTR, TM, TN, BK, RB, NST, KG>;
  constexpr bool WALKS = EPI != 2 && C::WALKS;
  a.mtiles = (a.M + C::BM - 1) / C::BM;
  a.ntiles = (a.N + C::BN - 1) / C::BN;
  // As many workgroups as the device holds at a time, each walking several tiles where there are more (tuning key 18).  12608 x
  // 768 -> 3072 83 -> 77 us, -> 2304 63 -> 58, against one to a tile.  Otherwise the kernel that has one tile only (2 KB of
  // instructions and about twenty registers less): 788 x 384 -> 384 in 64 x 128 tiles 5.7 -> 5.15 us, 6240 x 3072 -> 768 in 128 x 128 tiles 49.0 -> 46.7.
  const int tiles = (a.mtiles * a.ntiles + 7) / 8, most = !WALKS || g_cnnk_tune[18] < 0 ? tiles : g_cnnk_tune[18] > 0 ? g_cnnk_tune[18] : 32 * C::RESIDENT;
  if constexpr (WALKS)
    if (tiles > most) return launch(gemm_kernel<ATR, BTR, EPI, TM, TN, BK, RB, NST, KG, true>, &raised[1], C::THREADS, C::SMEM, most, a, splits, st);
  return launch(gemm_kernel<ATR, BTR, EPI, TM, TN, BK, RB, NST, KG, false>, &raised[0], C::THREADS, C::SMEM, tiles, a, splits, st);
}
// The tile shapes and what a launch of each costs.  With few tiles the device is bound by the latency of the operand
// loads and by how many CUs have a tile at all, so small problems want small tiles, 128-byte operand rows and two
// groups of wavefronts on one tile (KG = 2: twice the loads in flight per CU); large ones 256 x 128 or 192 x 128 tiles,
// with 64-byte rows and three stage buffers or with 128-byte rows and two (L192_WIDE: one load request per line).
// Estimated time (us) of a launch in rounds of resident workgroups; a round with c of them on a CU takes
//   c * tile + stages * max(alone, c * stage),      stages of 64 reduction elements (per group)
// and the launch `start` besides.  Constants fitted to a sweep of all shapes over 64 to 25216 rows and eighteen pairs
// of widths from 128 to 4096, forward, with GELU, with a residual, data gradient (1152 points), of kernels that had one tile
// to a workgroup and read operands and issued loads in another order.  With the present kernels, on operands that the L2s do not hold,
// 197 to 12608 rows and ten pairs of widths, forward and data gradient (120 points): what is chosen takes 2.3 % more than the fastest
// shape in the mean and 18 % at worst (3152 x 2304 -> 768 27.6 us in 64 x 64 tiles, 23.5 in 64 x 128).  The choice of 256 or 192 rows
// that was there before them / this one, us, both with the kernels of that time: 788 x 3072 -> 768 42.4 / 13.6, 788 x 768 -> 2304 17.2 / 9.9, 197 x
// 768 -> 768 15.2 / 6.2, 1576 x 768 -> 768 15.7 / 8.1, 6240 x 384 -> 384 10.6 / 6.9, 12608 x 768 -> 2304 61.0 / 55.0.
enum { T64 = 0, T64G2, T64x128, T64x128G2, T128, T_SMALL, L256 = T_SMALL, L192, L192_WIDE, T_SHAPES };
struct TileCost {
  int rows, cols, kgroups, resident;      // workgroup tile, groups of wavefronts, workgroups per CU
  float start, tile, stage, alone;        // us
};
constexpr TileCost kTiles[T_SHAPES] = {{64, 64, 1, 3, 1.84f, 1.00f, 0.237f, 0.367f},  {64, 64, 2, 1, 0.597f, 2.89f, 0.231f, 0.461f},
                                       {64, 128, 1, 2, 1.66f, 1.78f, 0.228f, 0.702f}, {64, 128, 2, 1, 0.288f, 4.27f, 0.671f, 0.576f},
                                       {128, 128, 1, 2, 1.93f, 3.33f, 0.302f, 0.859f},
                                       {256, 128, 1, 2, 2.59f, 4.57f, 0.861f, 1.62f},
                                       {192, 128, 1, 2, 2.27f, 5.27f, 0.708f, 1.09f}, {192, 128, 1, 2, 2.13f, 4.62f, 0.346f, 0.912f}};
inline int ceil_div(int a, int b) { return (a + b - 1) / b; }
float tile_time(const TileCost& t, int out_rows, int out_cols, int k) {
  const int tiles = ceil_div(out_rows, t.rows) * ceil_div(out_cols, t.cols), slots = 256 * t.resident;
  const float stages = (float)k / 64 / t.kgroups;
  auto round = [&](int c) { return c * t.tile + stages * (c * t.stage > t.alone ? c * t.stage : t.alone); };
  return t.start + tiles / slots * round(t.resident) + (tiles % slots ? round(ceil_div(tiles % slots, 256)) : 0.f);
}
// The same for the weight gradient (both operands through the transposing load; T128 has no such kernel), unsplit, up
// to 5000 rows: fixed and stage in us of a sweep over 197 to 3152 rows.  Beyond, the split launch and its sum are faster
// (fastest in 67 of 72 at 8192 rows and more; 4 of 36 at 4096 and 4728, where this estimate decides): 12608 x 2048 -> 512
// 51.7 us, 70.3 unsplit.
struct WgradCost { float fixed, stage; };
constexpr WgradCost kWgrad[T128] = {{4.1f, 0.23f}, {4.2f, 0.41f}, {4.1f, 0.345f}, {4.4f, 0.635f}};
constexpr int kWgradUnsplitRows = 5000;
// the fastest of the small shapes for a weight gradient, or -1 if `best` (us) is less
int pick_wgrad(int out_rows, int out_cols, int rows, float best) {
  int pick = -1;
  for (int c = 0; c < T128 && rows <= kWgradUnsplitRows; ++c) {
    const TileCost& t = kTiles[c];
    const int tiles = ceil_div(out_rows, t.rows) * ceil_div(out_cols, t.cols), stages = ceil_div(rows, 64);
    const float us = t.kgroups > 1 ? ceil_div(tiles, 256) * (kWgrad[c].fixed + ceil_div(stages, t.kgroups) * kWgrad[c].stage)
                                   : ceil_div(tiles, 256 * t.resident) * kWgrad[c].fixed + (float)ceil_div(tiles, 256) * stages * kWgrad[c].stage;
    if (us < best) { best = us; pick = c; }
  }
  return pick;
}
template <bool ATR, bool BTR, int EPI>
int launch_small(Args& a, int shape, hipStream_t st) {
  switch (shape) {
    case T64: return launch_cfg<ATR, BTR, EPI, 1, 1, 64, 128, 3, 1>(a, 1, st);
    case T64G2: return launch_cfg<ATR, BTR, EPI, 1, 1, 64, 128, 3, 2>(a, 1, st);
    case T64x128: return launch_cfg<ATR, BTR, EPI, 1, 2, 64, 128, 3, 1>(a, 1, st);
    case T64x128G2: return launch_cfg<ATR, BTR, EPI, 1, 2, 64, 128, 3, 2>(a, 1, st);
    case T128:
      if constexpr (!(ATR && BTR)) return launch_cfg<ATR, BTR, EPI, 2, 2, 64, 128, 2, 1>(a, 1, st);
      return CNNK_ERR_UNSUPPORTED;
    default: return CNNK_ERR_UNSUPPORTED;
  }
}
// The shape of a launch of an orientation with a natural operand.  The tuning table forces one (15 = 1 / 2: the large
// ones with 64- / 128-byte rows, 16 + n: small shape n; -1: no such shape).  With a reduction below 2048 the large ones
// only where every CU gets a tile: launches that follow one another in a step find cold operands, and a CU without a
// tile has nothing to hide that behind (1576 x 768 -> 3072 with GELU, 216 tiles of 192 rows, in a step: 24.0 us, 22.3
// with 128 x 128 tiles; launched alone 21.8 and 20.8).
int nat_shape(int M, int N, int K) {
  const int force = g_cnnk_tune[15];
  if (force >= 16) return force - 16 < T_SMALL ? force - 16 : -1;
  int first = T64, last = L192_WIDE;
  if (force == 1) { first = L256; last = L192; }
  if (force == 2) first = L192_WIDE;
  int best = first;
  float best_us = 1e30f;
  for (int c = first; c <= last; ++c) {
    if (force == 0 && c >= T_SMALL && K < 2048 && ceil_div(M, kTiles[c].rows) * ceil_div(N, 128) < 256) continue;
    const float us = tile_time(kTiles[c], M, N, K);
    if (us < best_us) { best_us = us; best = c; }
  }
  return best;
}
template <bool BTR, int EPI>
int launch_nat(Args& a, hipStream_t st) {
  const int shape = nat_shape(a.M, a.N, a.K);
  switch (shape) {
    case L192_WIDE: return launch_cfg<false, BTR, EPI, 3, 2, 64, 128, 2, 1>(a, 1, st);
    case L192: return launch_cfg<false, BTR, EPI, 3, 2, 32, 64, 3, 1>(a, 1, st);
    case L256: return launch_cfg<false, BTR, EPI, 4, 2, 32, 64, 3, 1>(a, 1, st);
    default: return launch_small<false, BTR, EPI>(a, shape, st);
  }
}

bool fits32(long long rows, long long cols) { return rows * cols * 2 < 2147483647LL; }
int wgrad_splits(int rows, int tiles) {
  int s = (192 + tiles - 1) / tiles;           // workgroups of a launch: it runs beside the main stream's kernels (128-192 measured best)
  const int max_s = rows / (8 * 32);           // at least 8 stages each
  if (s > max_s) s = max_s;
  return s < 1 ? 1 : s;
}
}  // namespace

bool gemm_bf16_supported(long long rows, int K, int N) {
  return rows > 0 && K > 0 && N > 0 && K % 8 == 0 && N % 8 == 0 && fits32(rows, K) && fits32(rows, N) && fits32(N, K);
}

int gemm_bf16_fwd(long long rows, int K, int N, const bf16_t* x, const bf16_t* w, const float* bias, const bf16_t* res, bool gelu,
                  bf16_t* u, bf16_t* y, hipStream_t st) {
  Args a{};
  a.A = x; a.B = w; a.bias = bias; a.res = res;
  a.C = gelu ? u : y; a.C2 = gelu ? y : nullptr;
  a.M = (int)rows; a.N = N; a.K = K; a.lda = K; a.ldb = K; a.ldc = N; a.k_per_split = K;
  a.a_bytes = (unsigned)(rows * K * 2); a.b_bytes = (unsigned)((long long)N * K * 2); a.c_bytes = (unsigned)(rows * N * 2);
  if (res) return launch_nat<false, 3>(a, st);
  return gelu ? launch_nat<false, 1>(a, st) : launch_nat<false, 0>(a, st);
}

int gemm_bf16_dgrad(long long rows, int K, int N, const bf16_t* dy, const bf16_t* w, bf16_t* dx, hipStream_t st) {
  Args a{};
  a.A = dy; a.B = w; a.C = dx;
  a.M = (int)rows; a.N = K; a.K = N; a.lda = N; a.ldb = K; a.ldc = K; a.k_per_split = N;
  a.a_bytes = (unsigned)(rows * N * 2); a.b_bytes = (unsigned)((long long)N * K * 2); a.c_bytes = (unsigned)(rows * K * 2);
  return launch_nat<true, 0>(a, st);
}

int gemm_bf16_dgrad_gelu_parts(long long rows, int K, int N) {
  const int shape = nat_shape((int)rows, K, N);
  return 2 * ceil_div((int)rows, shape < 0 ? 64 : kTiles[shape].rows);
}

int gemm_bf16_dgrad_gelu(long long rows, int K, int N, const bf16_t* dy, const bf16_t* w, const bf16_t* u, bf16_t* dg, bf16_t* du,
                         float* sums, hipStream_t st) {
  Args a{};
  a.A = dy; a.B = w; a.C = dg; a.C2 = du; a.res = u; a.part = sums;
  a.M = (int)rows; a.N = K; a.K = N; a.lda = N; a.ldb = K; a.ldc = K; a.k_per_split = N;
  a.a_bytes = (unsigned)(rows * N * 2); a.b_bytes = (unsigned)((long long)N * K * 2); a.c_bytes = (unsigned)(rows * K * 2);
  return launch_nat<true, 4>(a, st);
}

size_t gemm_bf16_wgrad_ws(long long rows, int K, int N) {
  const int tiles = ((N + 255) / 256) * ((K + 127) / 128);
  const int s = wgrad_splits((int)rows, tiles);
  return s > 1 ? (size_t)s * N * K * sizeof(float) : 0;
}

int gemm_bf16_wgrad(long long rows, int K, int N, const bf16_t* x, const bf16_t* dy, float* dw, void* ws, hipStream_t st) {
  Args a{};
  a.A = dy; a.B = x;
  a.M = N; a.N = K; a.K = (int)rows; a.lda = N; a.ldb = K; a.ldc = K;
  a.mtiles = (N + 255) / 256; a.ntiles = (K + 127) / 128;
  const int splits = wgrad_splits((int)rows, a.mtiles * a.ntiles);
  const int stages = (((int)rows + 31) / 32 + splits - 1) / splits;
  a.k_per_split = stages * 32;
  a.part = splits > 1 ? (float*)ws : dw;
  a.zstride = (size_t)N * K;
  a.a_bytes = (unsigned)(rows * N * 2); a.b_bytes = (unsigned)(rows * K * 2);
  const int force = g_cnnk_tune[15];
  if (force == 0 || force >= 16) {
    // the split launch and its sum, in the units of kWgrad
    const float us = 12.f + 0.6f * stages + 0.2f * splits;
    const int small = force >= 16 ? force - 16 : pick_wgrad(N, K, (int)rows, us);
    if (small >= 0 && small != T128) {
      a.part = dw;
      a.k_per_split = (int)rows;
      a.fold = fold_rows((int)rows) / 64;
      return launch_small<true, true, 2>(a, small, st);
    }
  }
  // 64-column planes (128-byte rows) measured 5-10 % slower here than 32-column ones; kept selectable
  const int rc = force == 2 ? launch_cfg<true, true, 2, 4, 2, 32, 128, 3, 1>(a, splits, st) : launch_cfg<true, true, 2, 4, 2, 32, 64, 3, 1>(a, splits, st);
  if (rc != CNNK_OK || splits == 1) return rc;
  const size_t n = (size_t)N * K;
  size_t blocks = (n / 4 + 255) / 256;
  if (blocks > 2048) blocks = 2048;
  sum_partials_kernel<<<(unsigned)blocks, 256, 0, st>>>((const float*)ws, splits, n, dw);
  return launch_status();
}

// ---- groups of weight gradients --------------------------------------------------------------------------
namespace {
int group_tiles(const GemmWgrad* p, int n, int bm) {
  int t = 0;
  for (int i = 0; i < n; ++i) t += ceil_div(p[i].N, bm) * ceil_div(p[i].K, 128);
  return t;
}
// 192 x 128 tiles where they give every CU one, 64 x 128 tiles otherwise.  Either adds up the same products in the same
// order.
bool group_large(const GemmWgrad* p, int n) { return group_tiles(p, n, 192) >= 256; }
size_t group_elems(const GemmWgrad* p, int n) {
  size_t e = 0;
  for (int i = 0; i < n; ++i) e += (size_t)p[i].N * p[i].K + p[i].N;
  return e;
}
}  // namespace

int gemm_bf16_wgrad_group_max() { return kGroupMax; }
int gemm_bf16_wgrad_tiles(int K, int N) { return ceil_div(N, 192) * ceil_div(K, 128); }

// Unsplit with the large tiles; with the small ones the row range is split until the device holds two workgroups per CU
// (but never below eight stages of 64 rows each).
int gemm_bf16_wgrad_group_splits(const GemmWgrad* p, int n) {
  if (group_large(p, n)) return 1;
  long long rows = p[0].rows;
  for (int i = 1; i < n; ++i) rows = p[i].rows < rows ? p[i].rows : rows;
  int splits = 512 / group_tiles(p, n, 64);
  if (splits > (int)(rows / 512)) splits = (int)(rows / 512);
  return splits < 1 ? 1 : splits;
}

size_t gemm_bf16_wgrad_group_ws(const GemmWgrad* p, int n, int splits) {
  return splits > 1 ? (size_t)splits * group_elems(p, n) * sizeof(float) : 0;
}

int gemm_bf16_wgrad_group(const GemmWgrad* p, int n, int splits, void* ws, hipStream_t st) {
  if (n < 1 || n > kGroupMax || splits < 1) return CNNK_ERR_SHAPE;
  const bool large = group_large(p, n);
  GroupArgs a{};
  a.count = n; a.splits = splits; a.part = (float*)ws; a.zstride = group_elems(p, n);
  size_t off = 0;
  for (int i = 0; i < n; ++i) {
    const int nt = ceil_div(p[i].K, 128);
    a.p[i] = GroupProblem{p[i].dy, p[i].x, p[i].dw, p[i].db, (int)p[i].rows, p[i].K, p[i].N, nt, a.tiles};
    a.off[i] = off;
    a.tiles += ceil_div(p[i].N, large ? 192 : 64) * nt;
    off += (size_t)p[i].N * p[i].K + p[i].N;
  }
  const dim3 grid(8 * ((a.tiles + 7) / 8), 1, splits);
  auto go = [&](auto kern, int smem, bool* raised) -> int {
    if (!*raised) {
      if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, smem) != hipSuccess)
        return CNNK_ERR_HIP;
      *raised = true;
    }
    hipLaunchKernelGGL(kern, grid, dim3(256), smem, st, a);
    return launch_status();
  };
  static bool raised_l = false, raised_s = false;
  const int rc = large ? go(wgrad_group_kernel<3, 2, 32, 64, 3>, Cfg<true, true, 3, 2, 32, 64, 3, 1>::SMEM, &raised_l)
                       : go(wgrad_group_kernel<1, 2, 64, 128, 3>, Cfg<true, true, 1, 2, 64, 128, 3, 1>::SMEM, &raised_s);
  if (rc != CNNK_OK || splits == 1) return rc;
  size_t blocks = (a.zstride / 4 + 255) / 256;
  if (blocks > 2048) blocks = 2048;
  sum_group_kernel<<<(unsigned)blocks, 256, 0, st>>>(a);
  return launch_status();
}
