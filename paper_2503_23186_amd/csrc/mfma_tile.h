// The main loop shared by the dense products (gemm_bf16.hip) and the implicit-GEMM convolutions
// (conv_gemm.hip): one workgroup's output tile on v_mfma_f32_32x32x16_bf16, operands filled straight into LDS
// stage buffers (buffer_load ... lds; out-of-range offsets deposit zeros), one barrier per stage.  Where the
// bytes of a stage come from is the loader's business; how they lie in LDS, and so how they are read, is here.
//
// An operand whose reduction index is its contiguous one ("natural") lies in LDS as [row][reduction elements
// of the stage] and is read with 16-byte loads; an operand whose reduction index is its row index lies as
// planes of [reduction rows][32 or 64 columns] and is read with the transposing load ds_read_b64_tr_b16, so no
// operand is ever transposed in memory.  The 16-byte chunks of a row are XOR-swizzled so that both kinds of
// read touch every bank once per pass (swz_of).  Because the hardware fixes where a direct load's bytes land
// (lane i at base + 16 i), the layout is produced by which global bytes each lane asks for.
#pragma once
#include "common.h"
#include "compensated.h"

typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef short s16x8_t __attribute__((ext_vector_type(8)));

constexpr int SP = 72;                         // epilogue strip pitch (bytes per column)

// TM, TN: 32-row and 32-column blocks of a wavefront's tile; WN: wavefronts along the columns (4 / WN along the rows).
// RB: bytes of an LDS row = bytes of an operand row that one group of lanes fetches.  The path from L2
// into LDS moves a fixed number of requests per clock whatever their size up to a 128-byte line
// (measured: 16 TB/s with 64-byte row segments, 32 TB/s with 128-byte ones), and with 64-byte rows that
// path, not the matrix pipe, bounds the large tiles.  128-byte rows of an operand whose reduction index is
// the contiguous one mean 64 reduction elements per stage; an operand read through the transposing load
// takes 128-byte rows by widening its planes to 64 columns, at any stage depth.
//
// KG: groups of four wavefronts in a workgroup.  They share the output tile and split the reduction range,
// each with stage buffers of its own, and their accumulators are added through LDS at the end.
template <bool ATR_, bool BTR_, int TM_, int TN_, int WN_, int BK_, int RB_, int NST_, int KG_> struct Tile {
  static constexpr bool ATR = ATR_, BTR = BTR_;          // operand read through the transposing load
  static constexpr int TM = TM_, TN = TN_, WN = WN_, WM = 4 / WN, BK = BK_, RB = RB_, KG = KG_;
  static constexpr int NW = 4, THREADS = 64 * NW * KG;
  static constexpr int NST = NST_;                       // stage buffers; loads run NST - 1 stages ahead
  static constexpr int BM = 32 * TM * WM, BN = 32 * TN * WN, A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE_B = A_BYTES + B_BYTES;
  static constexpr int NLOAD = STAGE_B / 1024 / NW;      // direct loads per wavefront and stage
  static constexpr int NLOAD_A = A_BYTES / 1024 / NW;    // the first of them fill the first operand
  static constexpr int LPR = RB / 16, RPL = 1024 / RB;   // lanes per LDS row, rows per direct load
  static constexpr int PC = RB / 2, PLANE_B = BK * RB;   // a transposed operand: planes of BK reduction rows x PC columns
  static constexpr int KS = BK / 16;                     // MFMA reduction steps per stage
  static constexpr int SMEM = KG * NST * STAGE_B;
  static constexpr int HAND_B = (KG - 1) * TM * TN * 16 * 256 * 4;   // accumulators of the groups past the first
  // wavefronts per SIMD the register allocation leaves room for: two workgroups per CU where their LDS fits
  static constexpr int WPE = KG * (2 * SMEM <= 160 * 1024 ? 2 : 1);
  static_assert(A_BYTES % (1024 * NW) == 0 && B_BYTES % (1024 * NW) == 0, "every load of a wavefront belongs to one operand");
  static_assert(SMEM <= 160 * 1024 && HAND_B + NW * 32 * SP <= SMEM, "LDS");
  static_assert((ATR || BK * 2 == RB) && (BTR || BK * 2 == RB), "a natural operand's LDS row is its BK reduction elements");
  static_assert((BM % PC == 0 || !ATR) && (BN % PC == 0 || !BTR), "whole planes");
  static_assert(NST == 2 || NLOAD < 16, "the wait below encodes the load count in four bits");
};

__device__ __forceinline__ i32x4_t make_desc(const void* p, unsigned bytes) {
  const unsigned long long a = reinterpret_cast<unsigned long long>(p);
  return i32x4_t{(int)(unsigned)a, (int)((unsigned)(a >> 32) & 0xffffu), (int)bytes, 0x00020000};
}
// lane i of the wavefront moves 16 bytes from byte offset voff of the buffer to LDS address
// lds_addr + 16 i (zeros when voff is out of range).  Assembly, so that the compiler does not make
// every later LDS read wait for all outstanding direct loads; the waits are explicit below.
__device__ __forceinline__ void load16_to_lds(i32x4_t desc, unsigned lds_addr, unsigned voff) {
  unsigned keep;
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tbuffer_load_dwordx4 %2, %3, 0 offen lds\n\ts_mov_b32 m0, %0"
               : "=&s"(keep)
               : "s"(lds_addr), "v"(voff), "s"(desc)
               : "memory");
}
// What the index of a 16-byte chunk is XORed with to give its position in the LDS row.  64-byte rows
// read with 16-byte loads: row bits 2-3; read with the transposing load: nothing, four consecutive
// rows are the 64 banks whatever the order inside a row.
// 128-byte rows read with 16-byte loads (sixteen rows of one chunk per pass): with row bits 1-3, so that
// the eight rows of either parity - a row's parity picks the half of the banks - sit on eight different
// chunk positions.  128-byte rows read with the transposing load (four rows x 64 bytes per pass): the
// two 64-byte halves swap on every second pair of rows, which puts the four rows on four bank quarters.
template <int RB, bool TR> __device__ __forceinline__ int swz_of(int row) {
  if (RB == 64) return TR ? 0 : (row >> 2) & 3;
  return TR ? ((row >> 1) & 1) << 2 : (row >> 1) & 7;
}

// Which operand row and chunk (natural), or reduction row, plane and chunk (transposed), this lane supplies in
// load j of its wavefront.
struct LoadSlot {
  int row, plane, chunk;     // natural: row of the tile; transposed: reduction row of the stage
};
template <class C> __device__ __forceinline__ LoadSlot load_slot(int j, int wave, int lane) {
  const bool isA = j < C::NLOAD_A;
  const int qq = j * C::NW + wave - (isA ? 0 : C::A_BYTES / 1024), p = lane % C::LPR;
  LoadSlot s;
  if (!(isA ? C::ATR : C::BTR)) {
    s.row = qq * C::RPL + lane / C::LPR;
    s.plane = 0;
    s.chunk = p ^ swz_of<C::RB, false>(s.row);
  } else {
    s.plane = qq / (C::BK / C::RPL);
    s.row = (qq % (C::BK / C::RPL)) * C::RPL + lane / C::LPR;
    s.chunk = p ^ swz_of<C::RB, true>(s.row);
  }
  return s;
}

// sum of the eight bf16 elements of an operand fragment
__device__ __forceinline__ float sum8(bf16x8_t f) {
  float v[8];
  unpack8(__builtin_bit_cast(uint4, f), v);
  return ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
}

// acc = sum over the loader's nst stages.  LD: a_rs, b_rs (buffer descriptors), begin(t) in front of the loads of
// stage t (stages in order), offset(j) of this lane's 16 bytes in load j.  ROWS: where row_sums is set, rs[i] also
// receives this lane's share of the first operand's sums over the reduction (rows i * 32 + lane % 32; the two
// halves of the wavefront hold the two halves of every reduction step), as a compensated sum.  FOLD: the accumulators
// are set aside and begun anew every `fold` stages, and what was set aside is added in a chain of its own: two chains
// of about the square root of the steps instead of one of all of them, for reductions of thousands of steps (relative
// error of a product of 12608 rows 1.7e-7 instead of 7.1e-7).  The workgroup's LDS holds the stage
// buffers and nothing else (LDS address 0).  Every wavefront of the workgroup runs the same number of stages.  On
// return all direct loads have landed.
template <class C, bool ROWS, bool FOLD, class LD>
__device__ __forceinline__ void tile_main_loop(LD& ld, int nst, int kg, int wave, int lane, unsigned char* smem,
                                               f32x16_t (&acc)[C::TM][C::TN], bool row_sums, float (&rs)[C::TM], int fold = 0) {
  constexpr int TM = C::TM, TN = C::TN, RB = C::RB, STAGE_B = C::STAGE_B, NST = C::NST, KS = C::KS, A_BYTES = C::A_BYTES, NLOAD = C::NLOAD;
  const int wm = wave / C::WN, wn = wave % C::WN, h = lane >> 5, g = lane >> 4, i16 = lane & 15;
  const int sbase = kg * NST * STAGE_B;    // LDS address of the group's stage buffers
  auto issue = [&](int t, int sb) __attribute__((always_inline)) {
    ld.begin(t);
#pragma unroll
    for (int j = 0; j < NLOAD; ++j)
      load16_to_lds(j < C::NLOAD_A ? ld.a_rs : ld.b_rs, (unsigned)(sbase + sb + (j * C::NW + wave) * 1024), ld.offset(j));
  };
  // ---- fragment addresses (stage-relative) ----
  // natural: 16 bytes = reduction elements ks * 16 + h * 8 .. + 8 of row lane % 32 of a 32-row block;
  // blocks lie 32 rows apart and the swizzle repeats every 16 rows.  The chunk index ks * 2 + h meets
  // the swizzle in an XOR, so step ks is the address of step 0 XOR ks * 32.
  // transposed: a pair of transposing reads, reduction rows ks * 16 + h * 8 + (lane % 16) / 4 and + 4,
  // of 32-column block sub of the wavefront's tile.
  int a_n0 = 0, b_n0 = 0;            // natural: address of step 0, block 0
  int a_t0 = 0, b_t0 = 0;            // transposed: address of step 0 within a 32-column block at column 0
  int a_sub[TM], b_sub[TN];          // transposed: where block sub lies (plane, and half of a 128-byte row)
  auto nat0 = [&](int row) { return row * RB + ((h ^ swz_of<RB, false>(row)) << 4); };
  auto tr0 = [&]() {
    const int ch0 = (g & 1) * 16 + (i16 & 3) * 4, row = h * 8 + (i16 >> 2);
    return row * RB + ((ch0 >> 3) << 4) + (ch0 & 7) * 2;        // 128-byte rows: which half of the row is in a_sub / b_sub
  };
  auto tr_sub = [&](int cb) {        // cb: 32-column block of the operand's tile
    if (RB == 64) return cb * C::PLANE_B;
    const int sw = swz_of<128, true>(i16 >> 2) >> 2;            // the same for every row this lane reads
    return (cb >> 1) * C::PLANE_B + (((cb & 1) ^ sw) << 6);
  };
  if (!C::ATR) a_n0 = nat0(wm * (TM * 32) + (lane & 31)); else a_t0 = tr0();
  if (!C::BTR) b_n0 = A_BYTES + nat0(wn * (TN * 32) + (lane & 31)); else b_t0 = A_BYTES + tr0();
#pragma unroll
  for (int i = 0; i < TM; ++i) a_sub[i] = C::ATR ? tr_sub(wm * TM + i) : i * 32 * RB;
#pragma unroll
  for (int j = 0; j < TN; ++j) b_sub[j] = C::BTR ? tr_sub(wn * TN + j) : j * 32 * RB;
  auto read_frag = [&](const unsigned char* sb, bool tr, int n0a, int t0a, int subo, int ks) __attribute__((always_inline)) -> bf16x8_t {
    if (!tr) return *reinterpret_cast<const bf16x8_t*>(sb + (n0a ^ (ks << 5)) + subo);
    const unsigned char* q = sb + t0a + ks * 16 * RB + subo;
    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4_t __attribute__((address_space(3)))*)q);
    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4_t __attribute__((address_space(3)))*)(q + 4 * RB));
    const s16x8_t v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8_t, v);
  };
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
#pragma unroll
  for (int i = 0; i < TM; ++i) rs[i] = 0.f;
  f32x16_t aside[FOLD ? TM : 1][FOLD ? TN : 1];
  float lost[TM];          // of rs: what the last addition rounded off
#pragma unroll
  for (int i = 0; i < TM; ++i) lost[i] = 0.f;
  int left = fold;
  if (FOLD) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) aside[i][j][r] = 0.f;
  }

#pragma unroll
  for (int d = 0; d < NST - 1; ++d)
    if (d < nst) issue(d, d * STAGE_B);
  int cur = 0;
  for (int t = 0; t < nst; ++t) {
    // this wave's loads of stage t have landed; those of the stages issued after it may stay in flight
    if (NST == 3 && t + 1 < nst) __builtin_amdgcn_s_waitcnt(0x0f70 | NLOAD);
    else __builtin_amdgcn_s_waitcnt(0x0f70);
    __builtin_amdgcn_s_barrier();
    if (t + NST - 1 < nst) {
      int fill = cur + (NST - 1) * STAGE_B;
      if (fill >= NST * STAGE_B) fill -= NST * STAGE_B;
      issue(t + NST - 1, fill);
    }
    const unsigned char* sb = smem + sbase + cur;
    bf16x8_t af[2][TM], bfr[2][TN];
#pragma unroll
    for (int kp = 0; kp < KS; kp += 2) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
        for (int i = 0; i < TM; ++i) af[ks][i] = read_frag(sb, C::ATR, a_n0, a_t0, a_sub[i], kp + ks);
#pragma unroll
        for (int j = 0; j < TN; ++j) bfr[ks][j] = read_frag(sb, C::BTR, b_n0, b_t0, b_sub[j], kp + ks);
      }
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[ks][i], bfr[ks][j], acc[i][j], 0, 0, 0);
      if (ROWS && row_sums) {
#pragma unroll
        for (int i = 0; i < TM; ++i) compensated_add(sum8(af[0][i]) + sum8(af[1][i]), rs[i], lost[i]);
      }
    }
    cur += STAGE_B;
    if (cur == NST * STAGE_B) cur = 0;
    if (FOLD && --left == 0) {
      left = fold;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            aside[i][j][r] += acc[i][j][r];
            acc[i][j][r] = 0.f;
          }
    }
  }
  if (FOLD) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] += aside[i][j][r];
  }
}

// Behind the main loop: the groups past the first hand their accumulators to the first through LDS, in group
// order.  All wavefronts call it; afterwards group 0 holds the sums and every stage buffer is free past HAND_B.
template <class C>
__device__ __forceinline__ void tile_join_groups(f32x16_t (&acc)[C::TM][C::TN], int kg, int tid, unsigned char* smem) {
  __syncthreads();     // every wave is done reading the stage buffers
  if constexpr (C::KG > 1) {
    float* R = reinterpret_cast<float*>(smem);
    if (kg > 0) {
#pragma unroll
      for (int i = 0; i < C::TM; ++i)
#pragma unroll
        for (int j = 0; j < C::TN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) R[(((kg - 1) * C::TM * C::TN + i * C::TN + j) * 16 + r) * 256 + tid] = acc[i][j][r];
    }
    __syncthreads();
    if (kg == 0) {
#pragma unroll
      for (int k = 0; k < C::KG - 1; ++k)
#pragma unroll
        for (int i = 0; i < C::TM; ++i)
#pragma unroll
          for (int j = 0; j < C::TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] += R[((k * C::TM * C::TN + i * C::TN + j) * 16 + r) * 256 + tid];
    }
  }
}

// 32 x 32 fp32 values (accumulator layout) as bf16 through a wavefront's private LDS strip (32 * SP bytes): lane
// (g, i16) gets the eight columns g * 8 .. of rows i16 (out[0]) and 16 + i16 (out[1]).
__device__ __forceinline__ void strip_transpose(unsigned char* S, int lane, const float* v, uint4* out) {
  const int g = lane >> 4, i16 = lane & 15;
  const int wr_off = (lane & 31) * SP + (lane >> 5) * 8, rd_off = (g * 8 + (i16 >> 2)) * SP + (i16 & 3) * 8;
#pragma unroll
  for (int q = 0; q < 4; ++q)
    *reinterpret_cast<uint2*>(S + wr_off + q * 16) = make_uint2(pack_bf16x2(v[q * 4], v[q * 4 + 1]), pack_bf16x2(v[q * 4 + 2], v[q * 4 + 3]));
  // the reads go through another type than the writes: tell the compiler that they touch the same memory (the
  // hardware keeps a wave's LDS operations in order)
  asm volatile("" ::: "memory");
#pragma unroll
  for (int rb = 0; rb < 2; ++rb) {
    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4_t __attribute__((address_space(3)))*)(S + rd_off + rb * 32));
    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4_t __attribute__((address_space(3)))*)(S + rd_off + 4 * SP + rb * 32));
    const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
    out[rb] = uint4{l2.x, l2.y, h2.x, h2.y};
  }
  asm volatile("" ::: "memory");
}

__device__ __forceinline__ void buffer_store16(__amdgpu_buffer_rsrc_t r, uint4 v, unsigned off) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(i32x4_t, v), r, (int)off, 0, 0);
}
// eight bf16 plus eight bf16, rounded again
__device__ __forceinline__ uint4 add_bf16x8(uint4 a, uint4 b) {
  float x[8], y[8];
  unpack8(a, x);
  unpack8(b, y);
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] += y[e];
  return uint4{pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(x[4], x[5]), pack_bf16x2(x[6], x[7])};
}
