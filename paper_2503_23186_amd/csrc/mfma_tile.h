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
#include <type_traits>
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
template <bool ATR_, bool BTR_, int TM_, int TN_, int WN_, int BK_, int RB_, int NST_, int KG_, int NW_ = 4> struct Tile {
  static constexpr bool ATR = ATR_, BTR = BTR_;          // operand read through the transposing load
  static constexpr int TM = TM_, TN = TN_, NW = NW_, WN = WN_, WM = NW / WN, BK = BK_, RB = RB_, KG = KG_;
  static constexpr int THREADS = 64 * NW * KG;          // NW: wavefronts of a group
  static constexpr int NST = NST_;                       // stage buffers; loads run NST - 1 stages ahead
  static constexpr int BM = 32 * TM * WM, BN = 32 * TN * WN, A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE_B = A_BYTES + B_BYTES;
  static constexpr int NLOAD = STAGE_B / 1024 / NW;      // direct loads per wavefront and stage
  static constexpr int NLOAD_A = A_BYTES / 1024 / NW;    // the first of them fill the first operand
  static constexpr int LPR = RB / 16, RPL = 1024 / RB;   // lanes per LDS row, rows per direct load
  static constexpr int PC = RB / 2, PLANE_B = BK * RB;   // a transposed operand: planes of BK reduction rows x PC columns
  static constexpr int KS = BK / 16;                     // MFMA reduction steps per stage
  // Whether workgroups walk several tiles.  Not with a single block to a wavefront, where a walk's registers and instructions cost
  // more than the start of a tile: 12608 x 768 -> 768 in 64 x 64 tiles 33.0 us, one to a workgroup 32.1; 200 images of 16 x 16, 128 ->
  // 256 3x3 strided 31.4 and 26.5.
  static constexpr bool WALKS = KG == 1 && TM * TN > 1;
  // LDS of the epilogue: a strip per wavefront, and two sums per column and row of wavefronts.  In a walk it takes room of its
  // own where that costs no workgroup, otherwise the stage buffer that is done with; behind a single tile the first ones.
  static constexpr int EPI_B = NW * 32 * SP + 2 * WM * BN * 4;
  static constexpr bool EPI_OWN = WALKS && 160 * 1024 / (NST * STAGE_B + EPI_B) == 160 * 1024 / (NST * STAGE_B);
  static constexpr int SMEM = KG * NST * STAGE_B + (EPI_OWN ? EPI_B : 0);
  static constexpr int HAND_B = (KG - 1) * TM * TN * 16 * 256 * 4;   // accumulators of the groups past the first
  // wavefronts per SIMD the register allocation leaves room for: two workgroups per CU where their LDS fits (and where
  // it does not, no more registers either: past 256 the accumulators would move between the two register files)
  static constexpr int WPE = KG == 1 ? (NW == 8 && 2 * SMEM <= 160 * 1024 ? 4 : 2) : KG * (2 * SMEM <= 160 * 1024 ? 2 : 1);
  // workgroups that a CU holds by their LDS (at most four: what the registers of the tiles that walk leave)
  static constexpr int RESIDENT = 160 * 1024 / SMEM < 4 ? 160 * 1024 / SMEM : 4;
  static_assert(A_BYTES % (1024 * NW) == 0 && B_BYTES % (1024 * NW) == 0, "every load of a wavefront belongs to one operand");
  static_assert(SMEM <= 160 * 1024 && HAND_B + EPI_B <= SMEM && (!WALKS || EPI_OWN || STAGE_B >= EPI_B), "LDS");
  static_assert((ATR || BK * 2 == RB) && (BTR || BK * 2 == RB), "a natural operand's LDS row is its BK reduction elements");
  static_assert((BM % PC == 0 || !ATR) && (BN % PC == 0 || !BTR), "whole planes");
  static_assert(NLOAD * (NST - 2) < 64, "the waits encode the number of loads in flight in six bits");
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

// barrier of the workgroup's LDS accesses: loads into LDS and stores to memory that are in flight stay so
__device__ __forceinline__ void workgroup_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// sum of the eight bf16 elements of an operand fragment
__device__ __forceinline__ float sum8(bf16x8_t f) {
  float v[8];
  unpack8(__builtin_bit_cast(uint4, f), v);
  return ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
}

// Where a lane reads its MFMA operands in a stage buffer (stage-relative addresses).
// natural: 16 bytes = reduction elements ks * 16 + h * 8 .. + 8 of row lane % 32 of a 32-row block; blocks lie 32 rows
// apart and the swizzle repeats every 16 rows.  The chunk index ks * 2 + h meets the swizzle in an XOR, so step ks is
// the address of step 0 XOR ks * 32.
// transposed: a pair of transposing reads, reduction rows ks * 16 + h * 8 + (lane % 16) / 4 and + 4, of 32-column block
// sub of the wavefront's tile.
template <class C> struct FragReader {
  static constexpr int TM = C::TM, TN = C::TN, RB = C::RB;
  int a0, b0;                // address of step 0: of block 0 (natural), or within a 32-column block at column 0 (transposed)
  int a_sub[TM], b_sub[TN];  // where block sub lies (transposed: plane, and half of a 128-byte row)
  __device__ __forceinline__ void init(int wm, int wn, int lane) {
    const int h = lane >> 5, g = lane >> 4, i16 = lane & 15;
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
    a0 = C::ATR ? tr0() : nat0(wm * (TM * 32) + (lane & 31));
    b0 = C::A_BYTES + (C::BTR ? tr0() : nat0(wn * (TN * 32) + (lane & 31)));
#pragma unroll
    for (int i = 0; i < TM; ++i) a_sub[i] = C::ATR ? tr_sub(wm * TM + i) : i * 32 * RB;
#pragma unroll
    for (int j = 0; j < TN; ++j) b_sub[j] = C::BTR ? tr_sub(wn * TN + j) : j * 32 * RB;
  }
  static __device__ __forceinline__ bf16x8_t read(const unsigned char* sb, bool tr, int at0, int sub, int ks) {
    if (!tr) return *reinterpret_cast<const bf16x8_t*>(sb + (at0 ^ (ks << 5)) + sub);
    const unsigned char* q = sb + at0 + ks * 16 * RB + sub;
    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4_t __attribute__((address_space(3)))*)q);
    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4_t __attribute__((address_space(3)))*)(q + 4 * RB));
    const s16x8_t v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8_t, v);
  }
  __device__ __forceinline__ bf16x8_t a(const unsigned char* sb, int i, int ks) const { return read(sb, C::ATR, a0, a_sub[i], ks); }
  __device__ __forceinline__ bf16x8_t b(const unsigned char* sb, int j, int ks) const { return read(sb, C::BTR, b0, b_sub[j], ks); }
};
template <class C> __device__ __forceinline__ void zero_acc(f32x16_t (&acc)[C::TM][C::TN]) {
#pragma unroll
  for (int i = 0; i < C::TM; ++i)
#pragma unroll
    for (int j = 0; j < C::TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
}
// s_waitcnt vmcnt(N): at most N of the wavefront's memory operations are still in flight
template <int N> __device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "six bits");
  __builtin_amdgcn_s_waitcnt(0x0f70 | (N & 15) | ((N >> 4) << 14));
}
// The products of one or several tiles, as one stream of stages: the direct loads run NST - 1 stages ahead of the products,
// also across the border of two tiles, so that the start of a tile (addresses, first loads) and the stores of the
// tile before it lie under products.
//
// Inside a wavefront everything is in order, so what is not interleaved adds up: issuing the direct loads of a stage
// (a CU takes 64 bytes a clock: 512 clocks for 128 x 128 x 64), then reading the operands (latency), then the
// products took 0.69 us a stage of 128 x 128 x 64 whose products take 0.22, with the loads three stages ahead and nothing else
// on the CU.
// So the operands of a reduction step are read under the products of the step before it, and with more than two buffers the
// direct loads are issued one by one between products and the operands of a stage's first step are read under the last products
// of the stage before (CROSS).  Not with two buffers, and not with a single block to a wavefront, where that takes two thirds of a
// stage off the time the loads have: 788 x 768 -> 3072 with GELU in a step, weights out of memory, 17.0 us, CROSS 21.1.
// With two buffers the loads have one stage's time, and all are issued in front of it: 128 x 128 tiles, one to a workgroup, 6240 x
// 3072 -> 768 49.0 us, between the products of half the stage 52.1; walking, 12608 x 768 -> 3072 82.5 and 86.4.
//
// LD: a_rs, b_rs (buffer descriptors); begin(t) in front of the loads of stage t of its tile (stages in order; past the last one
// every offset is out of range), offset(j) of this lane's 16 bytes in load j; next(k) points it at the workgroup's k-th tile (k ascending, each once).
// prefetch(k), in front of the last stage's products, may start loads that tile k's epilogue needs.  epilogue(k, acc, rs,
// strip) takes tile k's accumulators; strip: EPI_B bytes of LDS that are the caller's until it returns.  E: memory
// operations of one epilogue that can still be in flight behind it (its stores; a count that is too small waits longer
// than needed, never too short).
// ROWS: where row_sums is set, rs[i] also receives this lane's share of the first operand's sums over the reduction (rows i *
// 32 + lane % 32; the two halves of the wavefront hold the two halves of every reduction step), as a compensated sum.  FOLD:
// the accumulators are set aside and begun anew every `fold` stages, and what was set aside is added in a chain of its
// own: two chains of about the square root of the steps instead of one of all of them, for reductions of thousands of steps
// (relative error of a product of 12608 rows 1.7e-7 instead of 7.1e-7).  The workgroup's LDS holds the stage buffers (of
// group kg: kg * NST ..) and, behind them, the epilogue's room where it has its own (LDS address 0); ntiles is 1 where C::WALKS is not set.  Every
// wavefront of the workgroup runs the same number of stages.  On return all direct loads have landed.
template <class C, int E, bool ROWS, bool FOLD, class LD, class NEXT, class PRE, class EPI>
__device__ __forceinline__ void tile_stream(LD& ld, int ntiles, int nst, int kg, int wave, int lane, unsigned char* smem, bool row_sums, int fold,
                                            NEXT next, PRE prefetch, EPI epilogue) {
  constexpr int TM = C::TM, TN = C::TN, STAGE_B = C::STAGE_B, NST = C::NST, KS = C::KS, NLOAD = C::NLOAD, MM = TM * TN;
  constexpr bool CROSS = NST > 2 && MM > 1;              // the operands of a stage's first step are read under the stage before
  constexpr int LK = CROSS ? KS - 1 : 1;                 // reduction steps that the loads of a stage are spread over
  constexpr int PER = (NLOAD + LK - 1) / LK;             // direct loads in each of them
  static_assert(KS % 2 == 0 && LK >= 1, "two operand sets take turns");
  const int total = ntiles * nst;
  const int sbase = kg * NST * STAGE_B;    // LDS address of the group's stage buffers
  int p_tile = 0, p_st = 0;                // next stage to load
  auto load = [&](int sb, int j) __attribute__((always_inline)) {
    load16_to_lds(j < C::NLOAD_A ? ld.a_rs : ld.b_rs, (unsigned)(sbase + sb + (j * C::NW + wave) * 1024), ld.offset(j));
  };
  auto loaded = [&]() __attribute__((always_inline)) {
    if (++p_st == nst) {
      p_st = 0;
      if (++p_tile < ntiles) next(p_tile);
    }
  };
  FragReader<C> fr;
  fr.init(wave / C::WN, wave % C::WN, lane);
  f32x16_t acc[TM][TN], aside[FOLD ? TM : 1][FOLD ? TN : 1];
  bf16x8_t af[2][TM], bfr[2][TN];
  float rs[TM], lost[TM];                  // lost, of rs: what the last addition rounded off
  auto read = [&](int set, int buf, int ks) __attribute__((always_inline)) {
    const unsigned char* sb = smem + sbase + buf;
#pragma unroll
    for (int i = 0; i < TM; ++i) af[set][i] = fr.a(sb, i, ks);
#pragma unroll
    for (int j = 0; j < TN; ++j) bfr[set][j] = fr.b(sb, j, ks);
  };
  int cur = 0, s = 0, since = NST;         // buffer and index of the stage; stages since the last epilogue
  // This wave's loads of the stage that is read next have landed.  What was issued after them may be in flight: the loads
  // of NST - 2 stages, and the stores of an epilogue that came after them; near the end nothing is issued any more.
  auto wait_stage = [&](bool more) __attribute__((always_inline)) {
    constexpr int most = NLOAD * (NST - 2) + E < 64 ? NLOAD * (NST - 2) + E : 63;
    if (!more) wait_vm<0>();
    else if (since < (CROSS ? NST - 2 : NST - 1)) wait_vm<most>();
    else wait_vm<NLOAD * (NST - 2)>();
  };
  // One stage, with or without the loads of a later one: straight-line code either way, in which the accumulators stay
  // where they are (behind a branch they would be copied at its end).
  auto stage = [&](int k, bool last, auto more_c) __attribute__((always_inline)) {
    constexpr bool more = decltype(more_c)::value;
    int fill = cur + (NST - 1) * STAGE_B, nxt = cur + STAGE_B;
    if (fill >= NST * STAGE_B) fill -= NST * STAGE_B;
    if (nxt == NST * STAGE_B) nxt = 0;
    if (!CROSS) {
      wait_stage(more);
      __builtin_amdgcn_s_barrier();
    }
    if (last) prefetch(k);
    if (more) ld.begin(p_st);
    if (!CROSS) {
      if (more && MM > 1) {                // two buffers: the loads have one stage's time, all of it
#pragma unroll
        for (int c = 0; c < NLOAD; ++c) load(fill, c);
      }
      read(0, cur, 0);
    }
    float pair[ROWS ? TM : 1];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (ks + 1 < KS) {
        read((ks + 1) & 1, cur, ks + 1);
      } else if (CROSS) {
        // every wave is done reading this stage's buffer (its next loads are issued behind this barrier), and its loads
        // of the next stage have landed
        wait_stage(more);
        workgroup_barrier();
        read(0, nxt, 0);
      }
      if (more && ks == 0 && MM == 1) {    // under the latency of the first operands
#pragma unroll
        for (int c = 0; c < NLOAD; ++c) load(fill, c);
      }
      __builtin_amdgcn_sched_barrier(0);
      const int set = ks & 1;
      int j = ks * PER;                    // a constant once unrolled
#pragma unroll
      for (int m = 0; m < MM; ++m) {
        acc[m / TN][m % TN] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[set][m / TN], bfr[set][m % TN], acc[m / TN][m % TN], 0, 0, 0);
        if (more && ks < LK && CROSS) {
#pragma unroll
          for (int c = PER * m / MM; c < PER * (m + 1) / MM; ++c, ++j)
            if (j < NLOAD) {
              __builtin_amdgcn_sched_barrier(0);
              load(fill, j);
              __builtin_amdgcn_sched_barrier(0);
            }
        }
      }
      if constexpr (ROWS) {
        if (row_sums) {
#pragma unroll
          for (int i = 0; i < TM; ++i) {
            const float t = sum8(af[set][i]);
            if (ks & 1) compensated_add(pair[i] + t, rs[i], lost[i]); else pair[i] = t;
          }
        }
      }
      if (more && ks == LK - 1) loaded();
    }
    cur = nxt;
    ++s;
    ++since;
  };
  next(0);
#pragma unroll
  for (int d = 0; d < NST - 1; ++d)
    if (d < total) {
      ld.begin(p_st);
#pragma unroll
      for (int j = 0; j < NLOAD; ++j) load(d * STAGE_B, j);
      loaded();
    }
  if (CROSS) {
    if (total >= NST - 1) wait_vm<NLOAD * (NST - 2)>(); else wait_vm<0>();
    __builtin_amdgcn_s_barrier();
    read(0, 0, 0);
  }
  for (int k = 0; k < ntiles; ++k) {
    zero_acc<C>(acc);
    if constexpr (FOLD) zero_acc<C>(aside);
#pragma unroll
    for (int i = 0; i < TM; ++i) rs[i] = lost[i] = 0.f;
    int left = fold;
    auto fold_in = [&]() __attribute__((always_inline)) {
      if constexpr (FOLD) {
        if (--left == 0) {
          left = fold;
#pragma unroll
          for (int m = 0; m < MM; ++m)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              aside[m / TN][m % TN][r] += acc[m / TN][m % TN][r];
              acc[m / TN][m % TN][r] = 0.f;
            }
        }
      }
    };
    const int loading = min(nst, max(0, total - (NST - 1) - s));     // stages of this tile with a later one to load
    int t = 0;
    for (; t < loading; ++t) {
      stage(k, t + 1 == nst, std::true_type{});
      fold_in();
    }
    for (; t < nst; ++t) {
      stage(k, t + 1 == nst, std::false_type{});
      fold_in();
    }
    if constexpr (FOLD) {
#pragma unroll
      for (int m = 0; m < MM; ++m)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[m / TN][m % TN][r] += aside[m / TN][m % TN][r];
    }
    // The epilogue's room, where it is the buffer of the tile's last stage: every wave is done reading that (CROSS: behind
    // that stage's barrier), and it is filled again only behind a barrier that all waves reach after their epilogue.  Where there is
    // one tile only, every buffer is free by then.
    if (!CROSS && !C::EPI_OWN) workgroup_barrier();
    epilogue(k, acc, rs, smem + (C::EPI_OWN ? C::KG * NST * STAGE_B : !C::WALKS ? 0 : cur == 0 ? (NST - 1) * STAGE_B : cur - STAGE_B));
    if (CROSS && !C::EPI_OWN) workgroup_barrier();
    since = 0;
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
