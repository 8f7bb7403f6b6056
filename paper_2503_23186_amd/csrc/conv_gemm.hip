// Convolutions as implicit GEMM on the shared tile loop (mfma_tile.h): forward and data gradient of 1x1 and
// 3x3 filters, stride 1 and 2, bf16 with fp32 accumulation.  GEMM rows are output pixels, columns output
// channels, the reduction runs over (filter tap, source channel) in stages of one tap and 64 (or 32) channels.
// A stage's pixel rows go from memory straight into LDS: a lane asks for 16 bytes of the pixel that the tap
// shifts its output pixel to, or, where that pixel is padding, for the out-of-range offset, which deposits
// zeros - a nine-bit mask per lane and row, computed once, says which taps are inside the image.  The forward
// pass reads the weights [Cout][tap][Cin] as a natural operand; the data gradient reads the same array through
// the transposing LDS load (its reduction index, the output channel, is the slow one), so no transposed copy of
// the weights is needed.  A strided data gradient is one class of launch indices per output parity, which
// visits only the taps that reach it.
// What bounds it: the 1x1 layers of large images are at the memory rate (64 -> 256 channels, 32 x 32, batch 256: 168 MB
// in 36 us), the rest at L2 and launch latency.  Against the gathered kernel, us (data gradients with the transposition
// that they no longer need): 512 -> 256 at 16 x 16, batch 256: 33 -> 27, its data gradient 40 -> 31; 1024 -> 2048
// strided at 8 x 8: 25 -> 22 and 46 -> 32; 256 -> 512 3x3 strided at 8 x 8, batch 32: 20 -> 15 and 27 -> 13.
#include "common.h"
#include "conv.h"
#include "mfma_tile.h"

namespace {

constexpr int kMaxTaps = 9;

struct Taps {
  int nclass;
  int begin[5];                               // taps of class c: begin[c] .. begin[c + 1]
  int dh[kMaxTaps], dw[kMaxTaps];             // source shift
  int widx[kMaxTaps];                         // index into the weight array
  int Hm[4], Wm[4], oh[4], ow[4];             // class c: output sub-grid and its first pixel
  FastDiv dH[4], dW[4];
};

struct ConvGemmArgs {
  const bf16_t* src;
  const bf16_t* wt;
  bf16_t* dst;
  int Nimg, Hs, Ws, Cs;                       // source
  int Hd, Wd, Cd;                             // destination
  int T;                                      // taps in the weight array
  int ss, os;                                 // source step per sub-grid index; destination step
  int accumulate;
  int mtiles, ntiles;
  unsigned src_bytes, wt_bytes, dst_bytes;
  float* stats;                               // STATS kernels: [2][Cd][mtiles] column sums and sums of squares
  ConvTail tail;                              // TAIL kernels
  Taps tt;
};
enum { PLAIN = 0, STATS, TAIL };

template <class C> struct ConvLoader {
  static constexpr int NA = C::NLOAD_A, NB = C::NLOAD - C::NLOAD_A;
  i32x4_t a_rs, b_rs;
  unsigned aoff[NA], amask[NA], boff[NB];
  const ConvGemmArgs* a;
  int tap, tap_end, chunk, nchunk;            // of the next stage to load
  unsigned a_add, b_add, bit;                 // of the stage whose loads are being issued
  __device__ __forceinline__ void init(const ConvGemmArgs& args, int cls, int M, int m0, int n0, int stage0, int wave, int lane) {
    a = &args;
    a_rs = make_desc(args.src, args.src_bytes);
    b_rs = make_desc(args.wt, args.wt_bytes);
    const int t0 = args.tt.begin[cls], t1 = args.tt.begin[cls + 1];
    nchunk = args.Cs / C::BK;
    tap = t0 + uniform_div(stage0, nchunk);
    chunk = stage0 - (tap - t0) * nchunk;
    tap_end = t1;
#pragma unroll
    for (int j = 0; j < NA; ++j) {
      const LoadSlot s = load_slot<C>(j, wave, lane);
      const int m = m0 + s.row;
      int q, jj, n, ii;
      args.tt.dW[cls].divmod(m < M ? m : 0, &q, &jj);
      args.tt.dH[cls].divmod(q, &n, &ii);
      const int hh = ii * args.ss, ww = jj * args.ss;
      aoff[j] = (unsigned)(((n * args.Hs + hh) * args.Ws + ww) * args.Cs + 8 * s.chunk) * 2u;
      amask[j] = 0;
      if (m < M)
        for (int t = t0; t < t1; ++t)
          amask[j] |= ((unsigned)(hh + args.tt.dh[t]) < (unsigned)args.Hs && (unsigned)(ww + args.tt.dw[t]) < (unsigned)args.Ws) ? 1u << t : 0u;
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const LoadSlot s = load_slot<C>(NA + j, wave, lane);
      if (!C::BTR) {
        const int n = n0 + s.row;
        boff[j] = n < args.Cd ? (unsigned)(n * args.T * args.Cs + 8 * s.chunk) * 2u : kOobOffset;
      } else {
        const int n = n0 + s.plane * C::PC + 8 * s.chunk;
        boff[j] = n < args.Cd ? (unsigned)(s.row * args.T * args.Cd + n) * 2u : kOobOffset;
      }
    }
  }
  __device__ __forceinline__ void begin(int) {
    // past the last stage: bit 31 of no mask is set, and the weights are at the out-of-range offset
    const bool live = tap < tap_end;
    const int t = live ? tap : 0;
    const int c0 = chunk * C::BK;
    bit = live ? (unsigned)t : 31u;
    a_add = (unsigned)(((a->tt.dh[t] * a->Ws + a->tt.dw[t]) * a->Cs + c0) * 2);
    b_add = live ? (unsigned)((C::BTR ? c0 * a->T * a->Cd + a->tt.widx[t] * a->Cd : a->tt.widx[t] * a->Cs + c0) * 2) : kOobOffset;
    if (++chunk == nchunk) { chunk = 0; ++tap; }
  }
  __device__ __forceinline__ unsigned offset(int j) const {
    if (j < NA) return (amask[j] >> bit) & 1u ? aoff[j] + a_add : kOobOffset;
    return b_add == kOobOffset ? kOobOffset : boff[j - NA] + b_add;     // boff out of range stays so: offsets are below 2^31
  }
};

// Writes tile (mt, nt) of class cls out.  smem: EPI_B bytes of LDS that are free to use (the strips, then the sums); called by every
// wavefront that holds accumulators (group 0).
template <class C, int EP>
__device__ __forceinline__ void conv_gemm_epilogue(const ConvGemmArgs& a, int cls, int M, int mt, int nt, f32x16_t (&acc)[C::TM][C::TN], int tid,
                                                   unsigned char* smem) {
  constexpr int TM = C::TM, TN = C::TN;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / C::WN, wn = wave % C::WN, g = lane >> 4, i16 = lane & 15;
  const int m0 = mt * C::BM, n0 = nt * C::BN;
  if constexpr (EP == STATS) {
    // column sums and sums of squares of the fp32 accumulators over the tile's rows (rows past M are zeros):
    // per wavefront, then the wavefronts that share the columns in order, one partial per pixel tile
    float* red = reinterpret_cast<float*>(smem + C::NW * 32 * SP);     // [2][WM][BN]
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      float s1 = 0.f, s2 = 0.f;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float v = acc[i][j][r];
          s1 += v;
          s2 = fmaf(v, v, s2);
        }
      s1 += __shfl_xor(s1, 32, 64);
      s2 += __shfl_xor(s2, 32, 64);
      if (lane < 32) {
        const int c = wn * TN * 32 + j * 32 + lane;
        red[wm * C::BN + c] = s1;
        red[(C::WM + wm) * C::BN + c] = s2;
      }
    }
    workgroup_barrier();
    if (tid < 2 * C::BN) {
      const int v = tid / C::BN, c = tid % C::BN;
      float t = red[v * C::WM * C::BN + c];
#pragma unroll
      for (int w = 1; w < C::WM; ++w) t += red[(v * C::WM + w) * C::BN + c];
      if (n0 + c < a.Cd) a.stats[((size_t)v * a.Cd + n0 + c) * a.mtiles + mt] = t;
    }
  }
  unsigned char* S = smem + wave * (32 * SP);
  const __amdgpu_buffer_rsrc_t d_rs = make_rsrc(a.dst, a.dst_bytes);
  const bool add = EP == TAIL ? a.tail.res != nullptr : a.accumulate != 0;
  const __amdgpu_buffer_rsrc_t r_rs = make_rsrc(EP == TAIL ? a.tail.res : a.dst, a.dst_bytes);
  // byte offset of this lane's 16 bytes: rows i16 / 16 + i16 of block i, columns g * 8 .. of block j
  unsigned row_off[TM][2];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
      const int m = m0 + wm * (TM * 32) + i * 32 + rb * 16 + i16;
      int at = m;
      if (a.os != 1) {
        int q, jj, n, ii;
        a.tt.dW[cls].divmod(m < M ? m : 0, &q, &jj);
        a.tt.dH[cls].divmod(q, &n, &ii);
        at = (n * a.Hd + ii * a.os + a.tt.oh[cls]) * a.Wd + jj * a.os + a.tt.ow[cls];
      }
      row_off[i][rb] = m < M ? (unsigned)(at * a.Cd) * 2u : kOobOffset;
    }
  auto place = [&](int i, int j, int rb) __attribute__((always_inline)) -> unsigned {
    const int col = n0 + wn * (TN * 32) + j * 32 + g * 8;
    return col < a.Cd && row_off[i][rb] != kOobOffset ? row_off[i][rb] + (unsigned)col * 2u : kOobOffset;
  };
  // what is added to a 32-row block (the residual, or the gradient so far) is fetched while the block before it is
  // worked on
  uint4 rv[2][TN][2];
  auto fetch = [&](int i) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) rv[i & 1][j][rb] = buffer_load16(r_rs, place(i, j, rb), 0);
  };
  float sc[TN], bi[TN];
  if constexpr (EP == TAIL) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int col = n0 + wn * (TN * 32) + j * 32 + (lane & 31);
      tail_coef(a.tail, col, col < a.Cd, &sc[j], &bi[j]);
    }
  }
  if (add) fetch(0);
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    if (add && i + 1 < TM) fetch(i + 1);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      f32x16_t t = acc[i][j];
      if constexpr (EP == TAIL) t = tail_acc(t, sc[j], bi[j], a.tail.relu && !a.tail.res);
      float v[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) v[r] = t[r];
      uint4 o[2];
      strip_transpose(S, lane, v, o);
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) {
        if (add) o[rb] = EP == TAIL ? tail_residual(a.tail, o[rb], rv[i & 1][j][rb]) : add_bf16x8(rv[i & 1][j][rb], o[rb]);
        buffer_store16(d_rs, o[rb], place(i, j, rb));
      }
    }
  }
}

template <class C, int EP, bool WALK>
__global__ void __launch_bounds__(C::THREADS, C::WPE) conv_gemm_kernel(ConvGemmArgs a) {
  constexpr int TM = C::TM, TN = C::TN, KG = C::KG;
  extern __shared__ __align__(16) unsigned char smem[];   // stage buffers, and the epilogue's room where it has its own
  const int lane = threadIdx.x & 63;
  const int kg = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8);
  const int tid = threadIdx.x & 255;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // an XCD (every 8th workgroup) owns a contiguous range of the tile list, channel tiles of a pixel tile side by
  // side: they read the same pixels, which its L2 then holds.  Its workgroups take every step-th tile of the range.
  const int cls = blockIdx.z;
  const int M = a.Nimg * a.tt.Hm[cls] * a.tt.Wm[cls];
  const int tiles = ((M + C::BM - 1) / C::BM) * a.ntiles, chunk = (tiles + 7) >> 3, step = (int)gridDim.x >> 3;
  const int first = (blockIdx.x & 7) * chunk, l = blockIdx.x >> 3, mine = min(chunk, tiles - first);
  if (l >= mine) return;
  const int total = (a.tt.begin[cls + 1] - a.tt.begin[cls]) * (a.Cs / C::BK);
  // An output parity that no tap reaches: nothing to add, or zeros.  Three of four of a 1x1 stride-2 layer, bound by the
  // stores; through the epilogue below / from here, us: 64 images 56 x 56, 64 <- 128 channels 11.2 / 9.6, 32 of 56 x 56,
  // 256 <- 512 21.8 / 19.6.
  if (total == 0) {
    if (a.accumulate) return;
    const __amdgpu_buffer_rsrc_t z_rs = make_rsrc(a.dst, a.dst_bytes);
    for (int tile = first + l; tile < first + mine; tile += step) {
      const int mt = tile / a.ntiles, m0 = mt * C::BM, n0 = (tile - mt * a.ntiles) * C::BN;
      for (int k = threadIdx.x; k < C::BM * (C::BN / 8); k += C::THREADS) {
        const int m = m0 + k / (C::BN / 8), col = n0 + k % (C::BN / 8) * 8;
        int q, jj, n, ii;
        a.tt.dW[cls].divmod(m < M ? m : 0, &q, &jj);
        a.tt.dH[cls].divmod(q, &n, &ii);
        const int at = (n * a.Hd + ii * a.os + a.tt.oh[cls]) * a.Wd + jj * a.os + a.tt.ow[cls];
        buffer_store16(z_rs, make_uint4(0u, 0u, 0u, 0u), m < M && col < a.Cd ? (unsigned)(at * a.Cd + col) * 2u : kOobOffset);
      }
    }
    return;
  }
  ConvLoader<C> ld;
  if constexpr (!WALK) {
    // one tile to a workgroup (the grid has one for each), its stages split over the groups, if there are several; the
    // last group's stages past the end load zeros
    const int tile = first + l, mt = uniform_div(tile, a.ntiles), nt = tile - mt * a.ntiles, nst = (total + KG - 1) / KG;
    ld.init(a, cls, M, mt * C::BM, nt * C::BN, kg * nst, wave, lane);
    tile_stream<C, 0, false, false>(ld, 1, nst, kg, wave, lane, smem, false, 0, [](int) {}, [](int) {},
                                    [&](int, f32x16_t (&acc)[TM][TN], float (&)[TM], unsigned char* strip) __attribute__((always_inline)) {
      if (KG > 1) tile_join_groups<C>(acc, kg, tid, smem);
      if (kg == 0) conv_gemm_epilogue<C, EP>(a, cls, M, mt, nt, acc, tid, KG > 1 ? smem + C::HAND_B : strip);
      else if (EP == STATS) workgroup_barrier();        // the epilogue's barrier is the workgroup's
    });
  } else {
    auto next = [&](int k) __attribute__((always_inline)) {
      const int tile = first + l + k * step, mt = uniform_div(tile, a.ntiles), nt = tile - mt * a.ntiles;
      ld.init(a, cls, M, mt * C::BM, nt * C::BN, 0, wave, lane);
    };
    tile_stream<C, TM * TN * 2, false, false>(ld, (mine - l + step - 1) / step, total, 0, wave, lane, smem, false, 0, next, [](int) {},
                                [&](int k, f32x16_t (&acc)[TM][TN], float (&)[TM], unsigned char* strip) __attribute__((always_inline)) {
                                  const int tile = first + l + k * step, mt = uniform_div(tile, a.ntiles);
                                  conv_gemm_epilogue<C, EP>(a, cls, M, mt, tile - mt * a.ntiles, acc, tid, strip);
                                });
  }
}

// ---- host side -------------------------------------------------------------------------------------------
template <class C, int EP, bool WALK>
int launch_grid(const ConvGemmArgs& a, int per_xcd, hipStream_t st) {
  static bool raised = false;
  auto kern = conv_gemm_kernel<C, EP, WALK>;
  if (!raised) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, C::SMEM) != hipSuccess)
      return CNNK_ERR_HIP;
    raised = true;
  }
  hipLaunchKernelGGL(kern, dim3(8 * per_xcd, 1, a.tt.nclass), dim3(C::THREADS), C::SMEM, st, a);
  return launch_status();
}
template <class C, int EP>
int launch(ConvGemmArgs& a, long maxM, hipStream_t st) {
  a.mtiles = (int)((maxM + C::BM - 1) / C::BM);
  a.ntiles = (a.Cd + C::BN - 1) / C::BN;
  // as many workgroups as the device holds at a time, each walking several tiles where there are more (tuning key 18);
  // otherwise the kernel that has one tile only, whose start is 0.2 to 0.5 us shorter
  const int per_xcd = (a.mtiles * a.ntiles + 7) / 8, most = !C::WALKS || g_cnnk_tune[18] < 0 ? per_xcd : g_cnnk_tune[18] > 0 ? g_cnnk_tune[18] : 32 * C::RESIDENT;
  if constexpr (C::WALKS)
    if (per_xcd > most) return launch_grid<C, EP, true>(a, most, st);
  return launch_grid<C, EP, false>(a, per_xcd, st);
}

// Tile shapes and the time (us) of a launch, fitted to a sweep over 1x1 and strided 3x3 layers of 64 to 2048
// channels on 4 x 4 to 32 x 32 images at batch 16 to 256, forward and data gradient, on operands that the L2s do not
// hold (866 points, with the 64 x 64 tile as it is now, one to a workgroup: mean loss against the fastest shape 2.1 %, largest 30 %;
// 256 -> 256 3x3 strided at 16 x 16, batch 200, 30 us, 1024 -> 2048 strided data gradient 25):
//   one workgroup per CU at a time (two groups of wavefronts):  fixed + rounds * (tile + stages per group * stage)
//   several:  fixed + tile * tiles / 256 + max(tiles per CU * stages * stage, rounds of resident ones * stages * alone)
// `stage` is the time of a stage while other workgroups keep the CU busy, `alone` its latency; a stage is 64 channels
// of one tap.  Small tiles win while the grid is below the device, the deep ones on the long reductions of few
// pixels, 256 rows where memory bounds (fewest weight reads per pixel).
struct Shape { int bm, bn, kgroups, resident; float fixed, tile, stage, alone; };
constexpr int kShapes = 8;
constexpr Shape kShape[kShapes] = {{64, 64, 1, 3, 2.99f, 0.664f, 0.09f, 0.517f}, {64, 64, 2, 1, 2.21f, 2.45f, 0.53f, 0.f},
                                   {64, 128, 1, 2, 3.79f, 1.12f, 0.32f, 0.439f}, {64, 128, 2, 1, 2.46f, 2.73f, 0.691f, 0.f},
                                   {128, 128, 1, 2, 5.3f, 1.30f, 0.60f, 0.71f}, {128, 64, 1, 2, 4.2f, 0.962f, 0.35f, 0.56f},
                                   {256, 64, 1, 2, 5.5f, 2.00f, 0.60f, 1.13f}, {256, 128, 1, 2, 6.5f, 1.90f, 1.18f, 1.30f}};
inline long ceil_div(long a, long b) { return (a + b - 1) / b; }

template <bool BTR, int EP>
int dispatch(ConvGemmArgs& a, long maxM, int shape, hipStream_t st) {
  if (a.Cs % 64 == 0) {
    switch (shape) {
      case 0: return launch<Tile<false, BTR, 1, 1, 2, 64, 128, 3, 1>, EP>(a, maxM, st);
      case 1: return launch<Tile<false, BTR, 1, 1, 2, 64, 128, 3, 2>, EP>(a, maxM, st);
      case 2: return launch<Tile<false, BTR, 1, 2, 2, 64, 128, 3, 1>, EP>(a, maxM, st);
      case 3: return launch<Tile<false, BTR, 1, 2, 2, 64, 128, 3, 2>, EP>(a, maxM, st);
      case 4: return launch<Tile<false, BTR, 2, 2, 2, 64, 128, 2, 1>, EP>(a, maxM, st);
      case 5: return launch<Tile<false, BTR, 1, 2, 1, 64, 128, 3, 1>, EP>(a, maxM, st);
      case 6: return launch<Tile<false, BTR, 2, 2, 1, 64, 128, 2, 1>, EP>(a, maxM, st);
      case 7: return launch<Tile<false, BTR, 4, 2, 2, 32, 64, 3, 1>, EP>(a, maxM, st);
    }
  } else {
    switch (shape) {
      case 0: return launch<Tile<false, BTR, 1, 1, 2, 32, 64, 3, 1>, EP>(a, maxM, st);
      case 2: return launch<Tile<false, BTR, 1, 2, 2, 32, 64, 3, 1>, EP>(a, maxM, st);
      case 4: return launch<Tile<false, BTR, 2, 2, 2, 32, 64, 3, 1>, EP>(a, maxM, st);
      case 5: return launch<Tile<false, BTR, 1, 2, 1, 32, 64, 3, 1>, EP>(a, maxM, st);
      case 6: return launch<Tile<false, BTR, 2, 2, 1, 32, 64, 3, 1>, EP>(a, maxM, st);
      case 7: return launch<Tile<false, BTR, 4, 2, 2, 32, 64, 3, 1>, EP>(a, maxM, st);
    }
  }
  return CNNK_ERR_UNSUPPORTED;
}

void init_divs(Taps* t) {
  for (int c = 0; c < t->nclass; ++c) {
    t->dW[c].init((unsigned)t->Wm[c]);
    t->dH[c].init((unsigned)t->Hm[c]);
  }
}
}  // namespace

// 1x1 filters, and 3x3 filters with stride 2.  (3x3 with stride 1 reads every pixel nine times, which the patch
// kernel's resident input saves: 128 channels at 16 x 16, batch 256: 23 us against 27 us here.)  A reduction of one
// stage into few channels is left to the gathered kernel.  The line was drawn when only that one walked several tiles and had the next
// tile's loads in flight while it wrote; with both walking, us gathered / here on operands that the L2s do not hold, batch 256: plain forward 64 -> 64 at 16
// x 16 8.1 / 8.7, at 32 x 32 19.2 / 19.6, at 56 x 56 53.5 / 43.7, 64 -> 128 at 32 x 32 30.2 / 32.5, at 16 x 16 12.2 / 10.9; with channel sums (and the
// launch that adds them up) 12.2 / 12.2, 29.7 / 23.2, 87.1 / 52.5, 37.0 / 37.4, 16.0 / 14.5; batch 8 at 32 x 32, 64 -> 64 5.0 / 4.3.  Over 32, 64 ->
// 32 to 128 channels, 1 to 256 images of 8 x 8 to 56 x 56 the kernel here takes 0.86 of the gathered one's time, 0.73 to 1.08 plain and 0.59 to 1.01
// with sums.  Its own tuning keys ask for the gathered kernel, too.
bool conv_gemm_supported(const ConvGeom& g, int pass) {
  if (g_cnnk_tune[16] < 0 || !conv_mfma_supported(g, pass)) return false;
  const int Cs = pass == CNNK_PASS_FWD ? g.Cin : g.Cout, Cd = pass == CNNK_PASS_FWD ? g.Cout : g.Cin;
  if (Cs % 32 != 0) return false;
  if (g_cnnk_tune[16] > 0) return true;
  if (g_cnnk_tune[0] > 0 || g_cnnk_tune[1] > 0 || g_cnnk_tune[2] > 0 || g_cnnk_tune[14] > 0) return false;
  if (g.R == 1) return Cs > 64 || Cd > 128;
  return g.stride == 2;
}

namespace {
int pick(const ConvGeom& g, int pass) {
  const bool fwd = pass == CNNK_PASS_FWD;
  const int Cs = fwd ? g.Cin : g.Cout, Cd = fwd ? g.Cout : g.Cin;
  const bool deep = Cs % 64 == 0;        // 64 channels per stage, else 32 (and no split over two groups)
  const int f = g_cnnk_tune[16] - 1;
  if (f >= 0) return !deep && (f == 1 || f == 3) ? f - 1 : f;
  // classes of output pixels: rows, taps
  long rows[4];
  int taps[4], n = 0;
  if (fwd || g.stride == 1) {
    rows[n] = (long)g.N * (fwd ? (long)g.Ho * g.Wo : (long)g.H * g.W);
    taps[n++] = g.R * g.S;
  } else {
    for (int eh = 0; eh < 2; ++eh)
      for (int ew = 0; ew < 2; ++ew) {
        rows[n] = (long)g.N * ((g.H - eh + 1) / 2) * ((g.W - ew + 1) / 2);
        auto reach = [&](int e, int R) { int k = 0; for (int r = 0; r < R; ++r) k += (e + g.pad - r) % 2 == 0; return k; };
        taps[n++] = reach(eh, g.R) * reach(ew, g.S);
      }
  }
  int best = 0;
  float best_us = 1e30f;
  for (int c = 0; c < kShapes; ++c) {
    const Shape& t = kShape[c];
    if (!deep && t.kgroups > 1) continue;
    long tiles = 0;
    float stages = 0, longest = 0;       // over all tiles; of the longest tile
    for (int k = 0; k < n; ++k) {
      const long tk = ceil_div(rows[k], t.bm) * ceil_div(Cd, t.bn);
      const float sk = taps[k] * Cs / 64.f;
      tiles += tk;
      stages += tk * sk;
      if (sk > longest) longest = sk;
    }
    const float per = stages / tiles;
    const long cu = ceil_div(tiles, 256), rounds = ceil_div(tiles, 256L * t.resident);
    auto at_least = [](float a, float b) { return a > b ? a : b; };
    const float us = t.kgroups > 1
                         ? t.fixed + cu * t.tile + cu * (cu == 1 ? longest : per) * t.stage / t.kgroups
                         : t.fixed + t.tile * tiles / 256 + at_least(at_least(cu * per, longest) * t.stage, at_least(rounds * per, longest) * t.alone);
    if (us < best_us) { best_us = us; best = c; }
  }
  return best;
}
}  // namespace

int conv_gemm_stat_rows(const ConvGeom& g) {
  const int bm = kShape[pick(g, CNNK_PASS_FWD)].bm;
  return (int)(((long)g.N * g.Ho * g.Wo + bm - 1) / bm);
}

int conv_gemm_fwd(const ConvGeom& g, const bf16_t* x, const bf16_t* w, bf16_t* y, float* stats, hipStream_t st, const ConvTail* tail) {
  ConvGemmArgs a{};
  a.src = x; a.wt = w; a.dst = y; a.stats = stats;
  a.Nimg = g.N; a.Hs = g.H; a.Ws = g.W; a.Cs = g.Cin; a.Hd = g.Ho; a.Wd = g.Wo; a.Cd = g.Cout;
  a.T = g.R * g.S; a.ss = g.stride; a.os = 1;
  a.src_bytes = (unsigned)((long)g.N * g.H * g.W * g.Cin * 2);
  a.wt_bytes = (unsigned)((long)g.Cout * a.T * g.Cin * 2);
  a.dst_bytes = (unsigned)((long)g.N * g.Ho * g.Wo * g.Cout * 2);
  a.tt.nclass = 1;
  a.tt.begin[1] = a.T;
  for (int t = 0; t < a.T; ++t) { a.tt.dh[t] = t / g.S - g.pad; a.tt.dw[t] = t % g.S - g.pad; a.tt.widx[t] = t; }
  a.tt.Hm[0] = g.Ho; a.tt.Wm[0] = g.Wo;
  init_divs(&a.tt);
  const long M = (long)g.N * g.Ho * g.Wo;
  const int shape = pick(g, CNNK_PASS_FWD);
  if (tail) {
    a.tail = *tail;
    return dispatch<false, TAIL>(a, M, shape, st);
  }
  return stats ? dispatch<false, STATS>(a, M, shape, st) : dispatch<false, PLAIN>(a, M, shape, st);
}

int conv_gemm_dgrad(const ConvGeom& g, const bf16_t* dy, const bf16_t* w, bf16_t* dx, int accumulate, hipStream_t st) {
  ConvGemmArgs a{};
  a.src = dy; a.wt = w; a.dst = dx; a.accumulate = accumulate;
  a.Nimg = g.N; a.Hs = g.Ho; a.Ws = g.Wo; a.Cs = g.Cout; a.Hd = g.H; a.Wd = g.W; a.Cd = g.Cin;
  a.T = g.R * g.S; a.ss = 1; a.os = g.stride;
  a.src_bytes = (unsigned)((long)g.N * g.Ho * g.Wo * g.Cout * 2);
  a.wt_bytes = (unsigned)((long)g.Cout * a.T * g.Cin * 2);
  a.dst_bytes = (unsigned)((long)g.N * g.H * g.W * g.Cin * 2);
  long maxM = 0;
  int ntap = 0;
  for (int eh = 0; eh < g.stride; ++eh)
    for (int ew = 0; ew < g.stride; ++ew) {
      const int c = a.tt.nclass++;
      a.tt.begin[c] = ntap;
      for (int t = 0; t < a.T; ++t) {
        const int th = eh + g.pad - t / g.S, tw = ew + g.pad - t % g.S;      // dy row = th / stride where that is whole
        if (((th % g.stride) + g.stride) % g.stride != 0 || ((tw % g.stride) + g.stride) % g.stride != 0) continue;
        a.tt.dh[ntap] = th / g.stride; a.tt.dw[ntap] = tw / g.stride; a.tt.widx[ntap] = t;
        ++ntap;
      }
      a.tt.Hm[c] = (g.H - eh + g.stride - 1) / g.stride;
      a.tt.Wm[c] = (g.W - ew + g.stride - 1) / g.stride;
      a.tt.oh[c] = eh; a.tt.ow[c] = ew;
      const long m = (long)g.N * a.tt.Hm[c] * a.tt.Wm[c];
      if (m > maxM) maxM = m;
    }
  a.tt.begin[a.tt.nclass] = ntap;
  init_divs(&a.tt);
  return dispatch<true, PLAIN>(a, maxM, pick(g, CNNK_PASS_DGRAD), st);
}
