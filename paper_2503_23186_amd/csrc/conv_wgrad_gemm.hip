// Weight gradient of the convolutions that the patch kernels do not take (1x1, strided, padded thin inputs) on the
// tile loop of the dense products (mfma_tile.h): GEMM rows are output channels, columns (filter tap, input channel),
// the reduction runs over output pixels.  Both operands have the reduction index as their slow one, so pixel rows
// of dy and x go from memory straight into LDS and are transposed by the LDS read; a 16-byte piece of x belongs to
// one tap, and its lane asks for the pixel that the tap shifts the output pixel to, or for the out-of-range offset,
// which deposits zeros.  The pixel range is split, each split leaves a partial sum that the caller adds up.
// What bounds it: the 1x1 layers of large images the memory rate (64 -> 256 channels, 32 x 32, batch 256: 168 MB in 35
// us), the others the operand path into LDS.  Against the kernel it replaced, which moved both operands through
// registers to transpose them, us with the sum of the partials: that layer 51 -> 35, 512 -> 256 at 16 x 16 54 -> 35,
// 1024 -> 256 at 8 x 8 33 -> 27, 512 -> 512 3x3 strided at 8 x 8 54 -> 41 (batch 256), 320 -> 640 3x3 strided at
// 16 x 16, batch 128, 70 -> 56.
#include "common.h"
#include "conv.h"
#include "mfma_tile.h"

namespace {

struct WgArgs {
  const bf16_t* x;
  const bf16_t* dy;
  float* part;                 // [splits][Cout][Q]
  int M, Cout, Q, Cin;         // output pixels; Q = R * S * Cin
  int H, W, Ho, Wo, S, stride, pad;
  int chunk;                   // output pixels per split
  int ntiles, tiles, items;    // column tiles; tiles; tiles * splits
  unsigned x_bytes, dy_bytes;
  FastDiv dW, dH;              // by Wo, Ho
};

// LIN: 1x1 with stride 1, where output pixel m is input pixel m
template <class C, bool LIN> struct WgLoader {
  static constexpr int NA = C::NLOAD_A, NB = C::NLOAD - C::NLOAD_A;
  i32x4_t a_rs, b_rs;
  const WgArgs* a;
  int m, m_end;                                  // first pixel of the stage being loaded; end of the split
  int arow[NA], brow[NB], dr[NB], dc[NB];        // pixel within the stage (2^30: no such column); tap's shift
  unsigned acol[NA], bcol[NB];                   // byte offset within the pixel's channels
  int m_begin;
  __device__ __forceinline__ void init(const WgArgs& args, int k0, int q0, int mb, int me, int wave, int lane) {
    a = &args;
    a_rs = make_desc(args.dy, args.dy_bytes);
    b_rs = make_desc(args.x, args.x_bytes);
    m_begin = mb;
    m_end = me;
#pragma unroll
    for (int j = 0; j < NA; ++j) {
      const LoadSlot s = load_slot<C>(j, wave, lane);
      const int k = k0 + s.plane * C::PC + 8 * s.chunk;
      arow[j] = k < args.Cout ? s.row : 1 << 30;
      acol[j] = (unsigned)k * 2u;
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const LoadSlot s = load_slot<C>(NA + j, wave, lane);
      const int q = q0 + s.plane * C::PC + 8 * s.chunk;
      const int t = LIN ? 0 : q / args.Cin;
      brow[j] = q < args.Q ? s.row : 1 << 30;
      bcol[j] = (unsigned)(q - t * args.Cin) * 2u;
      if (!LIN) {
        dr[j] = t / args.S - args.pad;
        dc[j] = t % args.S - args.pad;
      }
    }
  }
  __device__ __forceinline__ void begin(int t) { m = m_begin + t * C::BK; }
  __device__ __forceinline__ unsigned offset(int j) const {
    if (j < NA) {
      const int p = m + arow[j];
      return p < m_end ? (unsigned)(p * a->Cout) * 2u + acol[j] : kOobOffset;
    }
    j -= NA;
    const int p = m + brow[j];
    if (LIN) return p < m_end ? (unsigned)(p * a->Cin) * 2u + bcol[j] : kOobOffset;
    int q, wo, n, ho;
    a->dW.divmod(p < m_end ? p : 0, &q, &wo);
    a->dH.divmod(q, &n, &ho);
    const int hi = ho * a->stride + dr[j], wi = wo * a->stride + dc[j];
    const bool ok = p < m_end && (unsigned)hi < (unsigned)a->H && (unsigned)wi < (unsigned)a->W;
    return ok ? (unsigned)(((n * a->H + hi) * a->W + wi) * a->Cin) * 2u + bcol[j] : kOobOffset;
  }
};

template <class C, bool LIN>
__global__ void __launch_bounds__(C::THREADS, C::WPE) wgrad_gemm_kernel(WgArgs a) {
  constexpr int TM = C::TM, TN = C::TN;
  extern __shared__ __align__(16) unsigned char smem[];   // stage buffers (no epilogue needs LDS here)
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int wm = wave / C::WN, wn = wave % C::WN, h = lane >> 5;
  // an XCD (every 8th workgroup) owns a contiguous range of the list (split, tile): the tiles of one split read the
  // same pixels, which its L2 then holds
  const int per = (a.items + 7) >> 3, l = blockIdx.x >> 3, item = (blockIdx.x & 7) * per + l;
  if (l >= per || item >= a.items) return;
  const int z = uniform_div(item, a.tiles), tile = item - z * a.tiles, mt = uniform_div(tile, a.ntiles), nt = tile - mt * a.ntiles;
  const int k0 = mt * C::BM, q0 = nt * C::BN, m_begin = z * a.chunk, m_end = min(m_begin + a.chunk, a.M);
  WgLoader<C, LIN> ld;
  ld.init(a, k0, q0, m_begin, m_end, wave, lane);
  tile_stream<C, 0, false, false>(ld, 1, (m_end - m_begin + C::BK - 1) / C::BK, 0, wave, lane, smem, false, 0, [](int) {}, [](int) {},
                                  [&](int, f32x16_t (&acc)[TM][TN], float (&)[TM], unsigned char*) __attribute__((always_inline)) {
    float* out = a.part + (size_t)z * a.Cout * a.Q;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int col = q0 + wn * (TN * 32) + j * 32 + (lane & 31);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = k0 + wm * (TM * 32) + i * 32 + (r >> 2) * 8 + h * 4 + (r & 3);
          if (row < a.Cout && col < a.Q) out[(size_t)row * a.Q + col] = acc[i][j][r];
        }
      }
  });
}

struct Plan { int bm, bn, chunk, splits; };
// Tiles as large as the gradient allows (operands are read once per tile) and 1.5 workgroups per CU of the budget, each
// with at least 256 pixels (ResNet-50 b256 step with 112 / 168 / 224 workgroups in all: 7.85 / 7.78 / 7.81 ms).  Where so
// few pixels leave half of them out, smaller tiles (256 -> 512 3x3 strided at 8 x 8, batch 32: 256 rows 20.4 us, 64 rows 16.0).
// The workspace is asked for with the whole device as the budget; a tile that shrinks there has the largest split there is.
Plan plan(const ConvGeom& g, int cus) {
  const int Q = g.R * g.S * g.Cin;
  const long M = (long)g.N * g.Ho * g.Wo, maxs = (M + 255) / 256;
  const long target = g_cnnk_tune[3] > 0 ? g_cnnk_tune[3] : 3L * cus / 2;
  Plan p;
  p.bm = g.Cout > 128 ? 256 : g.Cout > 64 ? 128 : 64;
  p.bn = Q > 64 ? 128 : 64;
  long tiles;
  for (;; p.bm /= 2) {
    tiles = (long)((g.Cout + p.bm - 1) / p.bm) * ((Q + p.bn - 1) / p.bn);
    if (p.bm == 64 || 2 * tiles * maxs >= target) break;
  }
  long want = (target + tiles - 1) / tiles;
  if (want > maxs) want = maxs;
  const long ch = ((M + want - 1) / want + 63) / 64 * 64;
  p.chunk = (int)ch;
  p.splits = (int)((M + ch - 1) / ch);
  return p;
}

template <class C, bool LIN>
int launch(const WgArgs& a, hipStream_t st) {
  static bool raised = false;
  auto kern = wgrad_gemm_kernel<C, LIN>;
  if (!raised) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, C::SMEM) != hipSuccess)
      return CNNK_ERR_HIP;
    raised = true;
  }
  hipLaunchKernelGGL(kern, dim3(8 * ((a.items + 7) / 8)), dim3(C::THREADS), C::SMEM, st, a);
  return launch_status();
}
template <bool LIN>
int dispatch(const WgArgs& a, int bm, int bn, hipStream_t st) {
  if (bm == 256 && bn == 128) return launch<Tile<true, true, 4, 2, 2, 32, 64, 3, 1>, LIN>(a, st);
  if (bm == 256) return launch<Tile<true, true, 4, 1, 2, 32, 64, 3, 1>, LIN>(a, st);
  if (bm == 128 && bn == 128) return launch<Tile<true, true, 2, 2, 2, 32, 64, 3, 1>, LIN>(a, st);
  if (bm == 128) return launch<Tile<true, true, 2, 1, 2, 64, 128, 3, 1>, LIN>(a, st);
  if (bn == 128) return launch<Tile<true, true, 1, 2, 2, 64, 128, 3, 1>, LIN>(a, st);
  return launch<Tile<true, true, 1, 1, 2, 64, 128, 3, 1>, LIN>(a, st);
}
}  // namespace

size_t conv_wgrad_gemm_ws(const ConvGeom& g) {
  const Plan p = plan(g, 256);
  return p.splits > 1 ? (size_t)p.splits * g.Cout * g.R * g.S * g.Cin * sizeof(float) : 0;
}

int conv_wgrad_gemm(const ConvGeom& g, const bf16_t* x, const bf16_t* dy, float* dw, void* ws, const float** part, int* P,
                    hipStream_t st) {
  const Plan p = plan(g, t_cnnk_wgrad_cus);
  WgArgs a{};
  a.x = x; a.dy = dy;
  a.part = p.splits > 1 ? reinterpret_cast<float*>(ws) : dw;
  a.M = g.N * g.Ho * g.Wo; a.Cout = g.Cout; a.Cin = g.Cin; a.Q = g.R * g.S * g.Cin;
  a.H = g.H; a.W = g.W; a.Ho = g.Ho; a.Wo = g.Wo; a.S = g.S; a.stride = g.stride; a.pad = g.pad;
  a.chunk = p.chunk;
  a.ntiles = (a.Q + p.bn - 1) / p.bn;
  a.tiles = a.ntiles * ((g.Cout + p.bm - 1) / p.bm);
  a.items = a.tiles * p.splits;
  a.x_bytes = (unsigned)((long)g.N * g.H * g.W * g.Cin * 2);
  a.dy_bytes = (unsigned)((long)a.M * g.Cout * 2);
  a.dW.init((unsigned)g.Wo);
  a.dH.init((unsigned)g.Ho);
  *part = a.part;
  *P = p.splits;
  const bool lin = g.R == 1 && g.stride == 1 && g.pad == 0;
  return lin ? dispatch<true>(a, p.bm, p.bn, st) : dispatch<false>(a, p.bm, p.bn, st);
}
