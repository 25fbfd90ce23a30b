// Tile machinery shared by the MFMA kernels of libmtpc: tile geometry, the
// direct-to-LDS operand ring, the workgroup GEMM  D = A_slab x B_tile^T  with both
// operands K-contiguous, and the column-wise log-sum-exp of a finished tile.
#pragma once

#include "mtpc_internal.h"

#include <type_traits>

namespace mtpc {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) int i32x4_t;

constexpr int NSLOT = 16;         // positions sampled per pass of the draw loop

// PH: one more block of 16 position columns per wave (kernels on the 16x16 MFMA blocks only), for tiles
// whose width is not a multiple of 32 columns per wave.
// VH: so many 16-row blocks fewer than WV * VB * 2 in all (the same kernels, two waves along the vocabulary):
// the first wave of a column keeps 2 VB - VH / 2 of them, the second one less when VH is odd.  Wave groups 0-3
// and 4-7 are then the two halves of the rows, so that every SIMD has one wave of each half and the rows that
// are not there cost no SIMD any time.
template <int WV, int WB, int VB, int PB, int SB, int NS, int PH = 0, int VH = 0>
struct Tile {
  static constexpr int NW = WV * WB;
  static constexpr int NT = NW * 64;
  static constexpr int TV = WV * VB * 32 - VH * 16;
  static constexpr int WROWS = VB * 32 - VH / 2 * 16;  // rows of a wave (the last one may have 16 fewer)
  static __device__ __forceinline__ int wv(int wave) { return VH ? wave >> 2 : wave % WV; }
  static __device__ __forceinline__ int wb(int wave) { return VH ? wave & 3 : wave / WV; }
  static constexpr int WP = PB * 32 + PH * 16;         // position columns of a wave
  static constexpr int TP = WB * WP;
  static constexpr int ROWS = TV + TP;
  static constexpr int CPR = SB / 16;                  // 16-byte chunks per row per stage
  static constexpr int RPL = 64 / CPR;                 // rows covered by one 1 KiB wave-load
  static constexpr int NWL = ROWS / RPL;               // wave-loads per stage
  static constexpr int LPW = (NWL + NW - 1) / NW;      // wave-loads per wave per stage (some waves: LPW-1)
  // A last load that one wave alone would issue is dealt in quarters of 16 lanes over the four waves of its group:
  // a branch that tells the waves of a group apart would sit in the K loop (with it, and the registers it cost, the
  // 272-row tile of fp32 terms took 5.3 ms where the 320-row one takes 3.6).
  static constexpr bool QUARTERS = NW == 8 && (NWL % NW == 1 || NWL % NW == 5);
  static constexpr int PER = (NWL % NW == 0 || (QUARTERS && NWL % NW == 5)) ? LPW : LPW - 1;   // loads every wave surely issues
  static constexpr int KS = SB / 32;                   // MFMA k-substeps (2 chunks each) per stage
  static constexpr int STAGE = ROWS * SB;
  static constexpr int VPL = (TV + 63) / 64;           // values per lane in the draw scan
  static constexpr int RED_OFF = NS * STAGE;           // float2 red[WV][TP]
  static constexpr int MISC_OFF = RED_OFF + WV * TP * 8;   // int cnt, list[TP], slot[TP]
  static constexpr int SMEM = MISC_OFF + 16 + TP * 8;
  static_assert(VH == 0 || (WV == 2 && WB == 4), "two halves of the rows, one per wave group");
  static_assert(SB == 64 || SB == 128, "stage bytes");
  static_assert(NS >= 2 && ROWS % RPL == 0, "ring geometry");
  static_assert(NSLOT * VPL * 64 * 4 <= NS * STAGE, "draw buffer must fit in the stage buffers");
  static_assert(SMEM <= 160 * 1024, "LDS budget of one CU");
};

// How the accumulators of a wave are laid out.  The tile geometry counts in blocks of 32 rows
// (VB) x 32 positions (PB) per wave; the MFMA that fills them is either 32x32 (one block each,
// 16 registers: lane (l % 32, l / 32) holds position column l % 32 and rows 8q + 4 (l / 32) + t,
// register 4q + t) or 16x16 (M16: four blocks per 32 x 32, 4 registers each: lane (l % 16, l / 16)
// holds column l % 16 and rows 4 (l / 16) + t).  bf16 kernels with two waves per SIMD take the
// 16x16x32 instruction: with real operands the chip is power limited, and the same products cost
// less through it (register operands only: 1.93 against 1.76 PFLOP/s on the same board).
template <bool M16>
struct Frag {
  static constexpr int BR = M16 ? 16 : 32;             // rows and columns of a block
  static constexpr int NI = M16 ? 4 : 16;              // accumulator registers of a block
  static constexpr int SUB = 32 / BR;                  // blocks per 32 rows (or columns)
  using blk_t = typename std::conditional<M16, f32x4_t, f32x16_t>::type;
  static __device__ __forceinline__ int lcol(int lane) { return lane & (BR - 1); }   // column inside a block
  static __device__ __forceinline__ int lgrp(int lane) { return lane / BR; }         // this lane's rows start at 4 * lgrp
  static __device__ __forceinline__ constexpr int roff(int i) { return M16 ? i : 8 * (i >> 2) + (i & 3); }
  // combine the values the lanes that share a column hold
  template <class F>
  static __device__ __forceinline__ float across(float x, F f) {
    x = f(x, __shfl_xor(x, 32));
    if constexpr (M16) x = f(x, __shfl_xor(x, 16));
    return x;
  }
};

// bf16 tiles of 8 waves (two per SIMD, ping-pong schedule) multiply through 16x16x32 MFMAs
template <int WV, int WB, int SB, int NS, bool BF16>
constexpr bool use_m16() { return BF16 && WV * WB == 8 && SB == 64 && NS >= 3; }

template <bool BF16>
__device__ __forceinline__ void mma_step(f32x4_t& acc, const i32x4_t& a, const i32x4_t& b) {
  static_assert(BF16, "the 16x16 blocks are used by the bf16 kernels only");
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b),
                                                acc, 0, 0, 0);
}

// the same product of fp16 terms (tile_gemm_run_split)
__device__ __forceinline__ void mma_step_f16(f32x4_t& acc, const i32x4_t& a, const i32x4_t& b) {
  acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), acc, 0, 0, 0);
}

template <bool BF16>
__device__ __forceinline__ void mma_step(f32x16_t& acc, const i32x4_t& a, const i32x4_t& b) {
  if constexpr (BF16) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                  __builtin_bit_cast(bf16x8_t, b), acc, 0, 0, 0);
  } else {
    f32x4_t af = __builtin_bit_cast(f32x4_t, a), bf = __builtin_bit_cast(f32x4_t, b);
#pragma unroll
    for (int t = 0; t < 4; ++t)
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(af[t], bf[t], acc, 0, 0, 0);
  }
}

// Map the hardware workgroup id to a (slab, position tile) pair.  Workgroup ids
// are dealt round-robin to the 8 XCDs, each with its own L2: give every XCD a
// contiguous range of logical ids, and walk logical ids through groups of 4
// slabs x all position tiles so that concurrently running workgroups of an XCD
// share a few W slabs and a few h tiles.
__device__ __forceinline__ void tile_of_block(int w, int nbt, int nslab, int& slab, int& bt) {
  const int total = nbt * nslab;
  const int per = total >> 3;
  int lid = (w < per * 8) ? (w & 7) * per + (w >> 3) : w;
  constexpr int GS = 4;
  const int gsz = GS * nbt;
  const int g = lid / gsz, rem = lid - g * gsz;
  const int gs = min(GS, nslab - g * GS);
  bt = rem / gs;
  slab = g * GS + (rem - bt * gs);
}

// s_waitcnt that waits only for the vector-memory counter to drop to n
#define MTPC_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(0x0F70 | ((n) & 15) | (((n) >> 4) << 14))

// One 16-byte-per-lane load from global memory straight into LDS: lane L's data
// lands at lds_base + 16*L.  A BUFFER load (resource descriptor + 32-bit lane
// offset + scalar offset) is used on purpose: its address is formed in the
// texture-address unit, whereas global/flat loads form theirs on the vector ALU
// and are starved for as long as another wave keeps the matrix pipe busy
// (measured on MI355X: buffer loads keep their full rate beside back-to-back
// MFMAs, global loads make no progress).  Issued as inline assembly so that the
// compiler's wait-count insertion does not serialise the ring (it cannot tell
// which stage a later LDS read touches); completion is tracked by hand with
// vmcnt + barrier.  Nothing else in these kernels uses M0.
// NT: the non-temporal hint, for bytes that are read once (a weight matrix streamed through a
// decode-sized call): they then do not push the small operands of the neighbouring kernels (sum-unit
// weights, the table, the verifier's rows) out of the caches.
template <bool NT = false>
__device__ __forceinline__ void load_to_lds(unsigned voff, i32x4_t srd, unsigned soff, unsigned lds_base) {
  if constexpr (NT)
    asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen nt lds"
                 :: "v"(voff), "s"(srd), "s"(soff), "s"(lds_base) : "memory");
  else
    asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds"
                 :: "v"(voff), "s"(srd), "s"(soff), "s"(lds_base) : "memory");
}

// The same for the lanes of `mask` only (wave-uniform): lane L's data still lands at lds_base + 16*L.  All
// lanes must be active.
__device__ __forceinline__ void load_to_lds_masked(unsigned voff, i32x4_t srd, unsigned soff, unsigned lds_base,
                                                   unsigned long long mask) {
  asm volatile("s_mov_b32 m0, %3\n\ts_mov_b64 exec, %4\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds\n\ts_mov_b64 exec, -1"
               :: "v"(voff), "s"(srd), "s"(soff), "s"(lds_base), "s"(mask) : "memory");
}

// Raw buffer resource over [base, base + bytes): reads beyond it return zero.
__device__ __forceinline__ i32x4_t make_srd(const void* base, unsigned bytes) {
  const unsigned long long a = (unsigned long long)base;
  // the descriptor must live in scalar registers: base and size are wave-uniform by
  // construction, readfirstlane makes that visible to the register allocator
  i32x4_t r;
  r[0] = __builtin_amdgcn_readfirstlane((int)(unsigned)(a & 0xffffffffull));
  r[1] = __builtin_amdgcn_readfirstlane((int)(unsigned)((a >> 32) & 0xffffull));   // stride 0, no swizzle
  r[2] = __builtin_amdgcn_readfirstlane((int)bytes);
  r[3] = 0x00020000;                                 // 32-bit data format, raw addressing
  return r;
}

// XOR swizzle of the 16-byte chunks of an LDS row, a function of the row's low
// four bits chosen so that 16 (and any aligned 8) consecutive rows of one logical
// chunk fall into distinct 16-byte bank groups.
template <int CPR>
__device__ __forceinline__ int swz(int row) {
  if constexpr (CPR == 4)
    return ((row >> 2) & 1) | ((((row >> 3) ^ (row >> 1)) & 1) << 1);
  else
    return ((row >> 1) & 3) | (((row ^ (row >> 3)) & 1) << 2);
}

// The swizzle for the fragment reads of the 16x16 blocks (64-byte rows): lane (l % 16, l / 16)
// reads chunk l / 16 of row l % 16.  A ds_read_b128 is served in four cycles of 16 lanes,
// and the lanes that share a cycle are not consecutive: {0-3, 12-15, 20-23, 24-27} and
// {4-7, 8-11, 16-19, 28-31} (the same again for lanes 32-63; inferred from the conflict
// counter, which reads 0 for the swizzle above with the 32x32 pattern and exactly one extra
// pass per read when that swizzle is used with this pattern).  Rows 4 apart share their
// banks, so with f = swizzle of rows k, 4+k, 8+k, 12+k the chunks f(k), f(12+k), 1^f(4+k),
// 1^f(8+k) must differ: f = (0, 3, 2, 1).
__device__ __forceinline__ int swz16(int row) { return (0 - (row >> 2)) & 3; }
// The same for 128-byte rows: two neighbours fill the 64 banks, so rows 2 apart share theirs, and of the eight even (or odd) rows of a
// cycle's 16 lanes four read chunk c and the others c ^ 1: f(row) = row / 2 makes f(0, 2, 12, 14) and 1 ^ f(4, 6, 8, 10), and the other
// cycle's f(4, 6, 8, 10) and 1 ^ f(0, 2, 12, 14), eight different chunks each.
template <int CPR>
__device__ __forceinline__ int swz16(int row) {
  if constexpr (CPR == 4) return swz16(row);
  else return (row >> 1) & 7;
}

// LDS image of an operand given along its rows (KRows): per 64 columns a block of 32 rows of 128 bytes, whose 32-byte pieces (16 columns) are XOR-swizzled so
// that the eight pieces that half a wave reads at once - four neighbouring rows, and the four eight rows on - lie in
// different banks.
__device__ __forceinline__ int swz_krow(int row) { return ((row >> 1) & 1) | (((row >> 3) & 1) << 1); }
// Fragment of 16 columns and 32 rows from there, transposed on the way into registers: the 16 lanes of a group hand in four
// rows of 32 bytes, eight bytes each, and every lane gets its column's four.  p: this lane's eight bytes of rows 8 (l / 16) ...
__device__ __forceinline__ i32x4_t read_krows(const char* p) {
  typedef __attribute__((ext_vector_type(4))) short s16x4_t;
  typedef __attribute__((ext_vector_type(2))) int i32x2_t;
  typedef __attribute__((address_space(3))) s16x4_t* lds_t;
  const i32x2_t lo = __builtin_bit_cast(i32x2_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t)p));
  const i32x2_t hi = __builtin_bit_cast(i32x2_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t)(p + 512)));
  return i32x4_t{lo[0], lo[1], hi[0], hi[1]};
}

// Ring buffers of the plane stages of tile_gemm_run_split.  Two terms: both of them alternate between two.  Three: the first
// ones do, the others have one each.
constexpr int SPLIT_SLOT_HI = 0, SPLIT_SLOT_LO = 2;
constexpr int SPLIT3_SLOT_A0 = 0, SPLIT3_SLOT_C = 2, SPLIT3_SLOT_B = 3;

// Where the operands of one tile come from, and the direct-to-LDS loads that bring them in: open()
// describes the tile and issues the first NS-1 stages of its ring, tile_gemm_run() multiplies.  Apart,
// so that a workgroup that walks several tiles can open the next one (the ring is free once the run
// has returned) before it turns to the epilogue of the one it has just multiplied.
// SPLIT: the operands are fp32 matrices as planes of two fp16 (2) or three bf16 (3) terms (see tile_gemm_run_split).
// KR: operands given along their rows (KRows, open_rows): 2 the one of the tile's columns, 3 both; tiles of 256 x 256.
// ROT: K may start anywhere (open's `first`).
template <int WV, int WB, int VB, int PB, int SB, int NS, bool BF16, bool GATHER = false, bool M16 = false,
          bool WPACK = false, bool STREAMW = false, int PH = 0, int SPLIT = 0, int VH = 0, int KR = 0, bool ROT = false>
struct TileFeed {
  using TL = Tile<WV, WB, VB, PB, SB, NS, PH, VH>;
  static constexpr int ESZ = BF16 ? 2 : 4;
  static constexpr int CPR = TL::CPR;
  i32x4_t srdW, srdH;
  unsigned voff[TL::LPW];                            // lane offsets of this wave's loads, constant over K
  unsigned lds0;
  unsigned kofs;                                     // byte offset along K of the next stage to issue
  unsigned kofsW;                                    // the same for the stage-major W (WPACK)
  unsigned kofsH;                                    // ... and for h, stage-major or not
  unsigned hstep, wstep;
  int wave, hrows;
  // KR: the rows of srdH that are left, in stages, and where it goes on from there
  i32x4_t srdT;
  int hleft;                                         // (ROT: stages that are left before K starts over)
  unsigned hterm;                                    // three terms: the distance of two of them (hleft: how many are issued)

  __device__ __forceinline__ void issue_one(int q, int buf) {   // q-th wave-load of this wave for one stage
    __builtin_assume(wave >= 0 && wave < TL::NW);    // (which loads are W's and which exist is then known per q, mostly)
    int wl = wave + q * TL::NW;
    if constexpr (TL::QUARTERS) {
      static_assert(!STREAMW, "tiles of one wave column");
      if (q == TL::LPW - 1) {
        const bool share = (wave >> 2) == (TL::NWL % TL::NW == 5 ? 1 : 0);       // the group of the last load
        if (share) {
          load_to_lds_masked(voff[q], srdH, kofsH, lds0 + buf * TL::STAGE + (TL::NWL - 1) * 1024, 0xffffull << ((wave & 3) * 16));
          return;
        }
      }
    }
    if (q < TL::PER || wl < TL::NWL) {
      // a wave-load never straddles the W / h boundary (TV is a multiple of RPL)
      const bool isW = wl * TL::RPL < TL::TV;
      if (STREAMW && isW)
        load_to_lds<true>(voff[q], srdW, WPACK ? kofsW : kofs, lds0 + buf * TL::STAGE + wl * 1024);
      else
        load_to_lds(voff[q], isW ? srdW : srdH, isW ? (WPACK || KR == 3 ? kofsW : kofs) : kofsH, lds0 + buf * TL::STAGE + wl * 1024);
    }
  }
  __device__ __forceinline__ void advance() {
    if constexpr (KR == 0 && !WPACK) kofs += SB;
    if constexpr (WPACK || KR == 3) kofsW += wstep;
    kofsH += hstep;
    if constexpr (ROT) {
      static_assert(KR == 0 && SPLIT == 0, "whole values along K");
      const bool over = --hleft == 0;
      if constexpr (WPACK) kofsW = over ? 0u : kofsW;
      else kofs = over ? 0u : kofs;
      kofsH = over ? 0u : kofsH;
    }
    // (kofs: from the first term of 32 rows to that of the next, constant here)
    if constexpr (KR != 0 && SPLIT == 2) hstep = kofs - hstep;
    if constexpr (KR != 0 && SPLIT == 3) {
      hleft = hleft == 2 ? 0 : hleft + 1;
      hstep = hleft == 2 ? kofs - 2 * hterm : hterm;
    }
    if constexpr (KR != 0 && SPLIT == 0) {
      const bool over = --hleft == 0;
#pragma unroll
      for (int i = 0; i < 3; ++i) srdH[i] = over ? srdT[i] : srdH[i];
      kofsH = over ? 0u : kofsH;
    }
  }
  __device__ __forceinline__ void issue(int buf) {
#pragma unroll
    for (int q = 0; q < TL::LPW; ++q) issue_one(q, buf);
    advance();
  }

  // lane offset of the q-th load of an operand given along its rows: eight rows of 64 columns from column 32 * chunk0 on
  // (given for two terms)
  __device__ __forceinline__ unsigned row_offset(int wl, const KRows& m, int chunk0, int chunks) {
    const int lane = threadIdx.x & 63;
    const int row = (wl & 3) * 8 + (lane >> 3), c = (lane & 7) ^ (swz_krow(row) << 1);
    const int chunk = min(chunk0 + 2 * (wl >> 2) + (c >> 2), chunks - 1);       // (columns that are not there: any)
    return (unsigned)chunk * (SPLIT == 3 ? 3 * m.term : m.chunk) + (unsigned)row * m.row + (c & 3) * 16;
  }
  // KR: columns a0 .. of `ak` (of acols; KR = 3) or rows of the stage-major planes at Ap [SPLIT K/32][arows][64] (KR = 2), columns
  // b0 .. of `bk` (of bcols), rows k0 .. k0 + klen - 1.  a0, b0, k0 and klen are multiples of 32.
  __device__ __forceinline__ void open_rows(const void* Ap, int arows, const KRows& ak, int acols, int a0, const KRows& bk, int bcols, int b0,
                                            int k0, int klen, char* smem) {
    static_assert(KR == 2 || KR == 3, "");
    static_assert(TL::TV == 256 && TL::TP == 256 && SB == 64 && TL::LPW == 4, "16 loads of each operand per stage, two and two per wave");
    const int lane = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if constexpr (KR == 3) {
      srdW = make_srd(ak.base, ak.bytes);
      kofsW = (unsigned)__builtin_amdgcn_readfirstlane((int)((unsigned)k0 * ak.row));
      wstep = (unsigned)__builtin_amdgcn_readfirstlane((int)(32u * ak.row));
    } else {
      srdW = make_srd((const char*)Ap + (long long)(k0 / 32) * SPLIT * arows * 64, (unsigned)((long long)klen * 2 * SPLIT * arows));
      kofsW = 0;
      wstep = (unsigned)__builtin_amdgcn_readfirstlane(arows * 64);
    }
    const bool main = k0 < bk.kmain;                   // workgroup-uniform
    srdT = make_srd(bk.tail, bk.tail_bytes);
    srdH = main ? make_srd(bk.base, SPLIT == 3 ? bk.bytes / 2 * 3 : bk.bytes) : srdT;
    hleft = SPLIT == 0 && main ? (bk.kmain - k0) / 32 : 0;
    hterm = (unsigned)__builtin_amdgcn_readfirstlane((int)bk.term);
    kofsH = (unsigned)__builtin_amdgcn_readfirstlane((int)((unsigned)(main ? k0 : k0 - bk.kmain) * bk.row));
    hstep = (unsigned)__builtin_amdgcn_readfirstlane((int)(SPLIT != 0 ? bk.term : 32u * bk.row));
    kofs = (unsigned)__builtin_amdgcn_readfirstlane((int)(32u * bk.row));
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int wl = wave + q * TL::NW;                // loads 0-15 of a stage: the tile's rows, 16-31: its columns
      if constexpr (KR == 3) voff[q] = row_offset(wl, ak, a0 / 32, (acols + 31) / 32);
      else {
        const int row = wl * TL::RPL + lane / CPR, ch = (lane % CPR) ^ swz16(row);
        voff[q] = (unsigned)min(a0 + row, arows - 1) * SB + ch * 16;
      }
      voff[q + 2] = row_offset(wl, bk, b0 / 32, (bcols + 31) / 32);
    }
    lds0 = (unsigned)(size_t)smem;
    if constexpr (SPLIT == 3) {
      issue(SPLIT3_SLOT_A0);
      issue(SPLIT3_SLOT_B);
    } else if constexpr (SPLIT == 2) {
      issue(SPLIT_SLOT_HI);
      issue(SPLIT_SLOT_LO);
      if (klen > 32) issue(SPLIT_SLOT_HI + 1);
    } else {
      for (int s = 0; s < NS - 1; ++s)
        if (s < klen / 32) issue(s);
    }
  }

  // Arguments as for tile_gemm.  The ring must be free (no wave still reads it).
  // first (ROT): the stage that the product starts with; it goes through all of K from there, over its end to its beginning.
  __device__ __forceinline__ void open(const void* Wp, long long ld_w, const void* hp, long long ld_h,
                                       int B, int d, int v, int slab, int b0, char* smem,
                                       const int* rows = nullptr, int nrows = 0, int rdiv = 1,
                                       const void* hs = nullptr, int wrows_total = 0, int wrow0 = 0, int first = 0) {
    const int tid = threadIdx.x, lane = tid & 63;
    wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Two resources: this slab of W (v rows of d, row stride ld_w) and this tile of h (rows b0..).
    // Lane offsets are relative to them and constant over K; the K advance is the
    // instruction's scalar offset.  Rows beyond v / B are clamped (in bounds; their
    // results are masked or never written).
    hrows = GATHER ? nrows : min(B - b0, TL::TP);
    const int hbase = GATHER ? 0 : b0;
    const int hspan = GATHER ? B : hrows;
    const bool wall = WPACK && wrows_total > 0;        // workgroup-uniform
    srdW = wall  ? make_srd(Wp, (unsigned)((long long)wrows_total * d * ESZ))
           : WPACK ? make_srd((const char*)Wp + (long long)slab * v * d * ESZ, (unsigned)((long long)v * d * ESZ))
                   : make_srd((const char*)Wp + (long long)slab * v * ld_w * ESZ,
                              (unsigned)((long long)(v - 1) * ld_w * ESZ + (long long)d * ESZ));
    const bool hpk = !GATHER && hs != nullptr;         // workgroup-uniform
    srdH = hpk ? make_srd(hs, (unsigned)((long long)B * d * ESZ))
               : make_srd((const char*)hp + (long long)hbase * ld_h * ESZ,
                          (unsigned)((long long)(hspan - 1) * ld_h * ESZ + (long long)d * ESZ));
    // wave-load q of this wave covers LDS rows RPL*wl .. RPL*wl+RPL-1 of every stage
#pragma unroll
    for (int q = 0; q < TL::LPW; ++q) {
      const int wl = min(wave + q * TL::NW, TL::NWL - 1);
      const int row = wl * TL::RPL + lane / CPR;
      const int ch = (lane % CPR) ^ (M16 ? swz16<CPR>(row) : swz<CPR>(row));
      if (row < TL::TV) voff[q] = (unsigned)((wall ? wrow0 : 0) + min(row, v - 1)) * (WPACK ? (unsigned)SB : (unsigned)(ld_w * ESZ)) + ch * 16;
      else {
        int hr = min(row - TL::TV, hrows - 1);
        if constexpr (GATHER) hr = min(max(rows[hr] / rdiv, 0), B - 1);
        voff[q] = hpk ? (unsigned)(b0 + hr) * SB + ch * 16 : (unsigned)hr * (unsigned)(ld_h * ESZ) + ch * 16;
      }
    }
    lds0 = (unsigned)(size_t)smem;
    // (steps along K of the stage-major operands; uniform over the workgroup, which the register allocator
    // has to be told where they come out of a select)
    hstep = (unsigned)__builtin_amdgcn_readfirstlane((int)(hpk ? (unsigned)B * SB : (unsigned)SB));
    wstep = (unsigned)__builtin_amdgcn_readfirstlane((int)((unsigned)(wall ? wrows_total : v) * SB));
    first = ROT ? __builtin_amdgcn_readfirstlane(first) : 0;
    kofs = (unsigned)first * SB;
    kofsW = (unsigned)first * wstep;
    kofsH = (unsigned)first * hstep;
    if constexpr (ROT) hleft = d * ESZ / SB - first;
    if constexpr (SPLIT == 3) {
      issue(SPLIT3_SLOT_A0);
      issue(SPLIT3_SLOT_B);
    } else if constexpr (SPLIT == 2) {
      issue(SPLIT_SLOT_HI);
      issue(SPLIT_SLOT_LO);
      if (d > 64) issue(SPLIT_SLOT_HI + 1);
    } else {
      const int KI = d * ESZ / SB;
      for (int s = 0; s < NS - 1; ++s)
        if (s < KI) issue(s);
    }
  }
};

// The stage that a slab's product starts with where every workgroup streams a slab of its own (starts_differ): one further than the
// slab before it, slab mod stages by the reciprocal of `stages`, 2^32 / stages rounded up.  stages = 0: the beginning.
__device__ __forceinline__ int first_stage(unsigned slab, unsigned stages, unsigned reciprocal) {
  return stages == 0 ? 0 : (int)(slab - __umulhi(slab, reciprocal) * stages);
}

// The product of a tile whose feed is open: on return every wave holds its VB x PB accumulator blocks and
// all waves have passed a barrier (the ring is free).
template <int WV, int WB, int VB, int PB, int SB, int NS, bool BF16, bool GATHER, bool M16, bool WPACK, bool STREAMW, int PH, int VH, int KR, bool ROT>
__device__ __forceinline__ void tile_gemm_run(TileFeed<WV, WB, VB, PB, SB, NS, BF16, GATHER, M16, WPACK, STREAMW, PH, 0, VH, KR, ROT>& feed,
                                              int d, char* smem,
                                              typename Frag<M16>::blk_t (&acc)[PB * Frag<M16>::SUB + PH][VB * Frag<M16>::SUB - VH / 2]) {
  using TL = Tile<WV, WB, VB, PB, SB, NS, PH, VH>;
  static_assert((PH == 0 && VH == 0) || M16, "half blocks: 16x16 MFMA blocks only");
  using FR = Frag<M16>;
  static_assert(!M16 || (BF16 && NS >= 3 && TL::NW == 8 && SB == 64),
                "16x16 blocks: bf16, two waves per SIMD, one MFMA k-step per 64-byte stage");
  constexpr int ESZ = BF16 ? 2 : 4;
  constexpr int CPR = TL::CPR, KS = TL::KS;
  const int tid = threadIdx.x, lane = tid & 63, wave = feed.wave;
  const int wv = TL::wv(wave), wb = TL::wb(wave);
  const int l31 = lane & 31, lhalf = lane >> 5;
  const int hrows = feed.hrows;
  auto issue_one = [&](int q, int buf) { feed.issue_one(q, buf); };
  auto advance = [&]() { feed.advance(); };
  auto issue = [&](int buf) { feed.issue(buf); };

#pragma unroll
  for (int pb = 0; pb < PB * FR::SUB + PH; ++pb)
#pragma unroll
    for (int vb = 0; vb < VB * FR::SUB - VH / 2; ++vb)
#pragma unroll
      for (int i = 0; i < FR::NI; ++i) acc[pb][vb][i] = 0.f;

  const int KI = d * ESZ / SB;
  const int sw = swz<CPR>(l31);
  const int a_off = (wv * VB * 32 + l31) * SB + ((lhalf ^ sw) << 4);
  const int b_off = (TL::TV + wb * TL::WP + l31) * SB + ((lhalf ^ sw) << 4);

  // logical chunk 2*ks + lhalf of a row sits at byte offset base ^ (32*ks)
  // One k-substep: the PB*VB MFMAs on fragment set `cs`, and interleaved with them
  // in a fixed order (pinned by scheduling barriers) the LDS reads that fetch
  // fragment set `ns` (k-substep nks of the stage at nsrc; nullptr: none) and this
  // substep's share of the direct-to-LDS loads for ring buffer `buf` (< 0: none).
  // Memory instructions issued back to back keep the wave away from the matrix
  // pipe; one behind each MFMA disappears in that MFMA's shadow.  Reads are issued
  // in the order the next substep consumes them.
  i32x4_t fa[2][VB], fb[2][PB];
  bool act[PB];                                      // wave-uniform: position block holds rows
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) act[pb] = !GATHER || (wb * PB + pb) * 32 < hrows;
  constexpr int NM = PB * VB;                        // MFMAs per substep
  constexpr int NR = VB + PB;                        // fragment reads per substep
  constexpr int LPS = (TL::LPW + KS - 1) / KS;       // direct-to-LDS loads per substep
  constexpr int NOPS = NR + LPS;
  auto read_frag = [&](const char* s, int ks, int set, int r) {
    if (r == 0) fb[set][0] = *(const i32x4_t*)(s + (b_off ^ (ks * 32)));
    else if (r <= VB) fa[set][r - 1] = *(const i32x4_t*)(s + ((a_off + (r - 1) * 32 * SB) ^ (ks * 32)));
    else fb[set][r - VB] = *(const i32x4_t*)(s + ((b_off + (r - VB) * 32 * SB) ^ (ks * 32)));
  };
  auto load_frags = [&](const char* s, int ks, int set) {
#pragma unroll
    for (int r = 0; r < NR; ++r) read_frag(s, ks, set, r);
  };
  // (rd: whether there is a next fragment set to read; a flag of its own, known where the loops are
  // unrolled: that a pointer into LDS is not null is not)
  auto substep = [&](int cs, int ks, bool rd, const char* nsrc, int nks, int ns, int buf) {
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      if constexpr (!M16)
        if (!GATHER || act[m / VB]) mma_step<BF16>(acc[m / VB][m % VB], fa[cs][m % VB], fb[cs][m / VB]);
#pragma unroll
      for (int o = 0; o < NOPS; ++o) {
        if ((o * NM) / NOPS != m) continue;          // op o rides behind MFMA o*NM/NOPS
        if (o < NR) {
          if (rd) read_frag(nsrc, nks, ns, o);
        } else {
          const int q = ks * LPS + (o - NR);
          if (buf >= 0 && q < TL::LPW) {
            issue_one(q, buf);
            if (q == TL::LPW - 1) advance();
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  if constexpr (NS >= 3 && TL::NW == 8) {
    // Ping-pong schedule for two waves per SIMD.  When both waves of a SIMD have an
    // MFMA ready the older one always wins, and a wave that alternates MFMAs with
    // memory instructions leaves gaps its partner cannot use; so each wave handles
    // a stage in two clusters separated by workgroup barriers: a memory cluster
    // (all fragment reads of the stage, the direct-to-LDS loads of stage s+NS-1)
    // and a compute cluster (all MFMAs of the stage, back to back, at raised
    // priority).  Waves 0-3 and 4-7 (w and w+4 share a SIMD) run one cluster apart,
    // so each SIMD always has one wave in its compute cluster.  Every wave executes
    // 2*KI + 2 barriers.
    static_assert(KS == 2, "ping-pong is written for two k-substeps per stage");
    const int group = wave >> 2;
    // 16x16 blocks: lane (l15, lq) reads chunk lq of row l15 of every 16-row block, the
    // whole 64-byte stage is one k-step of 2 VB x 2 PB MFMAs
    const int l15 = lane & 15, lq = lane >> 4;
    const int sw16 = swz16(l15);
    const int a16 = (wv * TL::WROWS + l15) * SB + ((lq ^ sw16) << 4);
    constexpr int NVB16 = 2 * VB - VH / 2;     // 16-row blocks of a wave (group 1: one fewer when VH is odd)
    constexpr int NPB16 = 2 * PB + PH;
    const int b16 = (TL::TV + wb * TL::WP + l15) * SB + ((lq ^ sw16) << 4);
    // operands along their rows: this lane's row and eight bytes of the first piece; piece p of a 64-column block is at ^ (32 p)
    static_assert(KR == 0 || (M16 && KR == 3 && TL::WP == 64 && TL::WROWS == 128), "64 columns of one block per wave, 128 rows of two");
    const int krow = 8 * lq + (l15 >> 2), k16 = krow * 128 + (swz_krow(krow) << 5) + (l15 & 3) * 8;
    i32x4_t ga[NVB16], gb[NPB16];
    bool act16[NPB16];
#pragma unroll
    for (int pb = 0; pb < NPB16; ++pb) act16[pb] = !GATHER || wb * TL::WP + pb * 16 < hrows;
    // Operands along their rows take two fragment reads where others take one: the memory cluster is then the longer one, and
    // the loads, too, leave behind every eighth product instead (dh of n r = 1024, d = 3072, B = 4096: 6.29 / 5.79 ms; with
    // one read per fragment, 40 products a cluster, 5.7 / 6.3 ms for the evidence pass).
    constexpr bool LATE = KR == 3;
    static_assert(!LATE || (TL::LPW == NPB16 && NVB16 == 8), "one load per row of eight products");
    // memory cluster of stage `it`: its fragments, and (LOAD) the loads of stage it+NS-1 into the
    // buffer of stage it-1 (last read before the previous barrier)
    auto mem_cluster = [&](int it, auto load, auto nvb) {
      const char* cur = smem + (it % NS) * TL::STAGE;
      if constexpr (KR == 3) {
#pragma unroll
        for (int pb = 0; pb < NPB16; ++pb) gb[pb] = read_krows(cur + (TL::TV * SB + wb * 4096) + (k16 ^ ((pb & 3) << 5)));
#pragma unroll
        for (int vb = 0; vb < NVB16; ++vb) ga[vb] = read_krows(cur + (wv * 2 + (vb >> 2)) * 4096 + (k16 ^ ((vb & 3) << 5)));
      } else if constexpr (M16) {
#pragma unroll
        for (int pb = 0; pb < NPB16; ++pb) gb[pb] = *(const i32x4_t*)(cur + b16 + pb * 16 * SB);
#pragma unroll
        for (int vb = 0; vb < decltype(nvb)::value; ++vb) ga[vb] = *(const i32x4_t*)(cur + a16 + vb * 16 * SB);
      } else {
        load_frags(cur, 0, 0);
        load_frags(cur, 1, 1);
      }
      if constexpr (!LATE && decltype(load)::value) issue((it + NS - 1) % NS);
      __builtin_amdgcn_sched_barrier(0);
    };
    // (a branch between two MFMAs costs about as much as an MFMA: empty position blocks are
    // skipped a whole row of products at a time)
    auto compute_cluster = [&](int it, auto load, auto nvb) {
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(1);
      if constexpr (M16) {
#pragma unroll
        for (int pb = 0; pb < NPB16; ++pb)
          if (!GATHER || act16[pb]) {
#pragma unroll
            for (int vb = 0; vb < decltype(nvb)::value; ++vb) {
              mma_step<BF16>(acc[pb][vb], ga[vb], gb[pb]);
              __builtin_amdgcn_sched_barrier(0);
              if constexpr (LATE && decltype(load)::value)
                if (vb == 3) {
                  issue_one(pb, (it + NS - 1) % NS);
                  if (pb == NPB16 - 1) advance();
                  __builtin_amdgcn_sched_barrier(0);
                }
            }
          }
      } else {
        substep(0, 0, false, nullptr, 0, 0, -1);
        substep(1, 1, false, nullptr, 0, 0, -1);
      }
      __builtin_amdgcn_s_setprio(0);
      __builtin_amdgcn_sched_barrier(0);
    };
    auto barrier = [&]() {
      __builtin_amdgcn_sched_barrier(0);
      __syncthreads();
      __builtin_amdgcn_sched_barrier(0);
    };
    if (KI > NS - 2) MTPC_WAIT_VMCNT((NS - 2) * TL::PER); else MTPC_WAIT_VMCNT(0);
    __syncthreads();                        // stage 0 has landed everywhere
    // One copy of the loop per wave group, and the iterations that still issue loads apart from
    // the last NS-1: no branch but the loop's own between two barriers.  A wave waits for its own
    // loads of stage it+1 (stages up to it+NS-1 are issued, so all but the (NS-2) youngest stages'
    // loads have landed) before the barrier after which the other group reads that stage: group 1
    // at the end of its memory cluster, group 0 after its compute cluster.
    auto run = [&](auto grp) {
      constexpr int G = decltype(grp)::value;
      constexpr std::integral_constant<int, NVB16 - (G == 1 ? VH % 2 : 0)> nvb{};
      const int KM = max(KI - (NS - 1), 0);
      int it = 0;
      for (; it < KM; ++it) {
        mem_cluster(it, std::true_type{}, nvb);
        if constexpr (G == 1) MTPC_WAIT_VMCNT((NS - (LATE ? 3 : 2)) * TL::PER);
        barrier();
        compute_cluster(it, std::true_type{}, nvb);
        if constexpr (G == 0) MTPC_WAIT_VMCNT((NS - 2) * TL::PER);
        barrier();
      }
      for (; it < KI; ++it) {
        mem_cluster(it, std::false_type{}, nvb);
        if constexpr (G == 1) MTPC_WAIT_VMCNT(0);
        barrier();
        compute_cluster(it, std::false_type{}, nvb);
        if constexpr (G == 0) MTPC_WAIT_VMCNT(0);
        barrier();
      }
    };
    if (group == 1) {
      __syncthreads();                      // start one cluster late
      run(std::integral_constant<int, 1>{});
    } else {
      run(std::integral_constant<int, 0>{});
    }
    if (group == 0) __syncthreads();        // pairs with the late start of the other group
  } else if constexpr (NS >= 3) {
    // Plain ring (tiles of fewer than 8 waves: the decode-sized tiles and the narrow ones of the sum units,
    // all bound by the latency of their stream).  At the barrier of iteration `it` stage `it` has landed and
    // nobody reads stage it-1 any more: its buffer takes all loads of stage it+NS-1 at once, so NS-1 stages
    // are in flight while stage `it` is multiplied (its first fragments are read behind that barrier; reading
    // them one stage ahead would need stage it+1 complete here, i.e. one stage less in flight).
    // Waves issue LPW or LPW-1 loads per stage; allowing y*PER loads to stay in flight guarantees, for either
    // kind, that all but the y youngest stages have landed (one count for all waves keeps the loop branch-free).
    const int KM = max(KI - (NS - 1), 0);   // iterations that still issue a stage
    int it = 0;
    for (; it < KM; ++it) {
      MTPC_WAIT_VMCNT((NS - 2) * TL::PER);   // stage `it` landed (stages up to it+NS-2 issued)
      __syncthreads();                       // ... everywhere; stage it-1 is no longer read
      issue((it + NS - 1) % NS);
      const char* cur = smem + (it % NS) * TL::STAGE;
      load_frags(cur, 0, 0);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) substep(ks & 1, ks, ks + 1 < KS, cur, ks + 1, (ks + 1) & 1, -1);
    }
    for (; it < KI; ++it) {
      MTPC_WAIT_VMCNT(0);
      __syncthreads();
      const char* cur = smem + (it % NS) * TL::STAGE;
      load_frags(cur, 0, 0);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) substep(ks & 1, ks, ks + 1 < KS, cur, ks + 1, (ks + 1) & 1, -1);
    }
  } else {
    // two stages: the other buffer is being filled while this one is multiplied
    for (int it = 0; it < KI; ++it) {
      MTPC_WAIT_VMCNT(0);
      __syncthreads();                       // stage `it` landed everywhere; stage it-1 no longer read
      const int pbuf = (it + 1 < KI) ? ((it + 1) & 1) : -1;
      const char* cur = smem + (it & 1) * TL::STAGE;
      load_frags(cur, 0, 0);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        substep(ks & 1, ks, ks + 1 < KS, cur, ks + 1, (ks + 1) & 1, pbuf);
    }
  }
  __syncthreads();     // all waves are done reading the ring
}

// The product of two fp32 operands on the fp16 matrix pipes.  A row of either operand, scaled by a power of two that
// takes its largest value into [2^14, 2^15), is the sum of two fp16 terms x1 + x2 (see split2), 11 bits each, up to half a
// unit of bit 23 or, where that is more, 2^-40 of the row's largest value; and
//   x y = x1 y2 + x1 y1 + x2 y1 + (x2 y2),
// where what is left out is at most 2^-22 |x y| and 2^-25 of it on average, without a sign of its own.  The three products
// cost 3 / 16 of the fp32 instruction's time; products are exact and sums fp32 as there, with one rounding per 32 terms of K
// instead of one per 1 or 2: in a sum of a few hundred terms those roundings, not the terms, are the error that is left.
// The row scales are powers of two that the epilogue takes out again.
// Both operands are stage-major (TileFeed with WPACK and hs) in 64-byte stages that hold 32 columns of ONE
// term: stages 2k and 2k+1 are terms 1 and 2 of columns 32k .. 32k+31.  d: fp32 columns.
// Schedule: the ping-pong clusters of tile_gemm_run, three per 32 columns; a cluster reads only what it does not have
// (28 fragment reads per 120 products where the bf16 kernel needs 42), and the ring takes two stages for three clusters.
// Of its four buffers two alternate for each term; loads are issued three or four clusters before their first use.
// Bound by the power of the products and of the two operand stages behind every three of them: 1.45 PFLOP/s of issued products
// (B = 2048, n r = 256, d = 3072, v = 268: 1.83 ms; three bf16 terms and six products 3.19 ms, the fp32 instruction 7.29 ms;
// registers only, the fp16 product runs at 1.88 PFLOP/s and the bf16 one at 2.02).
// SPLIT = 3, for operands that those terms do not do justice (k_split_rows): three bf16 terms, each the nearest bf16 of what the
// ones before leave (split3), whose sum is the value, whatever its row holds.
//   x y = x1 y1 + x1 y2 + x2 y2 + x2 y1 + x3 y1 + x1 y3 + (x2 y3 + x3 y2 + x3 y3)
// leaves out at most about 2^-24 |x y| (|x2| <= 2^-8, |x3| <= 2^-17 of the leading power of two), what one fp32 multiply-add may
// round off.  Stages 3k .. 3k+2 are the terms of columns 32k .. 32k+31; six clusters per 32 columns, each of which reads
// the operand that changes; loads are issued four or five clusters before their first use.
template <int WV, int WB, int VB, int PB, int SB, int NS, int PH, int SPLIT, int VH, int KR>
__device__ __forceinline__ void tile_gemm_run_split(TileFeed<WV, WB, VB, PB, SB, NS, true, false, true, true, false, PH, SPLIT, VH, KR>& feed,
                                                    int d, char* smem, f32x4_t (&acc)[2 * PB + PH][2 * VB - VH / 2]) {
  using TL = Tile<WV, WB, VB, PB, SB, NS, PH, VH>;
  constexpr int NPB16 = 2 * PB + PH, NVB16 = 2 * VB - VH / 2;
  static_assert(TL::NW == 8 && SB == 64 && NS == 4, "ping-pong of two wave groups over four ring buffers");
  const int lane = threadIdx.x & 63, wave = feed.wave;
  const int wv = TL::wv(wave), wb = TL::wb(wave);
  const int l15 = lane & 15, lq = lane >> 4;
  const int sw16 = swz16(l15);
  const int a16 = (wv * TL::WROWS + l15) * SB + ((lq ^ sw16) << 4);
  const int b16 = (TL::TV + wb * TL::WP + l15) * SB + ((lq ^ sw16) << 4);
#pragma unroll
  for (int pb = 0; pb < NPB16; ++pb)
#pragma unroll
    for (int vb = 0; vb < NVB16; ++vb) acc[pb][vb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  i32x4_t ga[NVB16], gb[NPB16];
  auto read_a = [&](int slot, auto nvb) {
    const char* cur = smem + slot * TL::STAGE;
#pragma unroll
    for (int vb = 0; vb < decltype(nvb)::value; ++vb) ga[vb] = *(const i32x4_t*)(cur + a16 + vb * 16 * SB);
  };
  static_assert(KR == 0 || (KR == 2 && TL::WP == 64), "64 columns of one block per wave");
  const int krow = 8 * lq + (l15 >> 2), k16 = krow * 128 + (swz_krow(krow) << 5) + (l15 & 3) * 8;    // (as in tile_gemm_run)
  auto read_b = [&](int slot) {
    const char* cur = smem + slot * TL::STAGE;
#pragma unroll
    for (int pb = 0; pb < NPB16; ++pb) {
      if constexpr (KR == 2) gb[pb] = read_krows(cur + (TL::TV * SB + wb * 4096) + (k16 ^ ((pb & 3) << 5)));
      else gb[pb] = *(const i32x4_t*)(cur + b16 + pb * 16 * SB);
    }
  };
  auto barrier = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
  };
  auto compute = [&](auto nvb) {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int pb = 0; pb < NPB16; ++pb)
#pragma unroll
      for (int vb = 0; vb < decltype(nvb)::value; ++vb) {
        if constexpr (SPLIT == 3) mma_step<true>(acc[pb][vb], ga[vb], gb[pb]);
        else mma_step_f16(acc[pb][vb], ga[vb], gb[pb]);
        __builtin_amdgcn_sched_barrier(0);
      }
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
  };
  const int KI = d / 32;
  // both terms of the first columns have landed (of three: the first)
  if (SPLIT == 3 || KI > 1) MTPC_WAIT_VMCNT(TL::PER); else MTPC_WAIT_VMCNT(0);
  __syncthreads();
  auto run = [&](auto grp) {
    constexpr int G = decltype(grp)::value;
    constexpr std::integral_constant<int, NVB16 - (G == 1 ? VH % 2 : 0)> nvb{};
    // What follows the reads and loads of a memory cluster.  ALLOW: loads of this wave that may still be on their way when
    // the next cluster reads (negative: that cluster reads no new buffer).  Group 1 waits at the end of its memory
    // cluster, group 0 after its products: either way before the barrier that lets the other group read.
    auto rest = [&](auto allow) {
      constexpr int ALLOW = decltype(allow)::value;
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (G == 1 && ALLOW >= 0) MTPC_WAIT_VMCNT(ALLOW >= 0 ? ALLOW : 0);
      barrier();
      compute(nvb);
      if constexpr (G == 0 && ALLOW >= 0) MTPC_WAIT_VMCNT(ALLOW >= 0 ? ALLOW : 0);
      barrier();
    };
    // The three products of 32 columns, LEFT of them still to come (2: or more).  Loads go where nobody reads any more since
    // the last barrier: the second terms of the columns after these over those of the ones before, the first terms
    // of the columns after next over this pair's, once both operands' are in registers.
    auto columns = [&](int k, auto left) {
      constexpr int LEFT = decltype(left)::value;
      const int hi = SPLIT_SLOT_HI + (k & 1), lo = SPLIT_SLOT_LO + (k & 1);
      read_b(lo); read_a(hi, nvb);          // x1 y2
      if constexpr (LEFT >= 1) feed.issue(lo ^ 1);
      rest(std::integral_constant<int, -1>{});
      read_b(hi);                           // x1 y1
      rest(std::integral_constant<int, -1>{});
      read_a(lo, nvb);                      // x2 y1
      if constexpr (LEFT >= 2) feed.issue(hi);
      rest(std::integral_constant<int, LEFT >= 2 ? TL::PER : LEFT == 1 ? 0 : -1>{});     // the next pair landed
    };
    // The six products of the three-term form; the last ones issue no more.
    auto columns3 = [&](int k, auto lastk) {
      constexpr bool LAST = decltype(lastk)::value;
      const int a = SPLIT3_SLOT_A0 + (k & 1);
      read_a(a, nvb); read_b(a);            // x1 y1.  Third terms and the next first terms go where nobody reads
      feed.issue(SPLIT3_SLOT_C);            // any more since the last barrier
      rest(std::integral_constant<int, TL::PER>{});            // second terms landed
      read_b(SPLIT3_SLOT_B);                // x1 y2
      if constexpr (!LAST) feed.issue(a ^ 1);
      rest(std::integral_constant<int, -1>{});
      read_a(SPLIT3_SLOT_B, nvb);           // x2 y2
      rest(std::integral_constant<int, -1>{});
      read_b(a);                            // x2 y1: the buffer of the second terms is free
      if constexpr (!LAST) feed.issue(SPLIT3_SLOT_B);
      rest(std::integral_constant<int, LAST ? 0 : 2 * TL::PER>{});   // third terms landed
      read_a(SPLIT3_SLOT_C, nvb);           // x3 y1
      rest(std::integral_constant<int, -1>{});
      read_a(a, nvb); read_b(SPLIT3_SLOT_C);      // x1 y3
      rest(std::integral_constant<int, LAST ? -1 : TL::PER>{});      // the next first terms landed
    };
    int k = 0;
    if constexpr (SPLIT == 3) {
      for (; k < KI - 1; ++k) columns3(k, std::false_type{});
      columns3(k, std::true_type{});
    } else {
      for (; k < KI - 2; ++k) columns(k, std::integral_constant<int, 2>{});
      if (k < KI - 1) columns(k++, std::integral_constant<int, 1>{});
      columns(k, std::integral_constant<int, 0>{});
    }
  };
  if (wave >> 2) {
    __syncthreads();                        // start one cluster late
    run(std::integral_constant<int, 1>{});
  } else {
    run(std::integral_constant<int, 0>{});
    __syncthreads();                        // pairs with the late start of the other group
  }
  __syncthreads();                          // all waves are done reading the ring
}

// The scales of the rows of both operands out of the finished accumulators: acc *= 2^(rows + cols).  s_e holds the exponents
// of the tile's TV rows and TP columns (LDS; the caller's barrier lies behind its stores).
template <class TL, int NPB, int NVB>
__device__ __forceinline__ void tile_unscale(f32x4_t (&acc)[NPB][NVB], const int* s_e, int rbase, int cbase) {
  int ec[NPB];
#pragma unroll
  for (int pb = 0; pb < NPB; ++pb) ec[pb] = s_e[TL::TV + cbase + pb * 16];
#pragma unroll
  for (int vb = 0; vb < NVB; ++vb) {
    const int* er = s_e + min(rbase + vb * 16, TL::TV - 4);          // (a block that is not there: any)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int pb = 0; pb < NPB; ++pb) acc[pb][vb][i] = __builtin_amdgcn_ldexpf(acc[pb][vb][i], er[i] + ec[pb]);
  }
}

// D = W_slab x h_tile^T for one workgroup; on return every wave holds its VB x PB
// accumulator blocks and all waves have passed a barrier (the ring is free).
// GATHER: the tile's position rows are not consecutive: row p of the tile is row
// rows[p] / rdiv of h (p < nrows <= TP, nrows >= 1; b0 is ignored and the whole of h,
// which must span less than 4 GiB, is one resource).  32-row position blocks past nrows
// are not multiplied (their accumulators stay zero), so a nearly empty tile is cheap.
// WPACK: Wp is the stage-major copy of W (mtpc_pack_weights): per slab, the SB bytes that a K stage takes
// from each of the v rows lie back to back ([stage][row][SB], ld_w is ignored), so a stage of a
// slab is one contiguous run of v * SB bytes instead of SB bytes from each of v rows d elements apart.
// WPACK with wrows_total > 0: Wp is ONE stage-major matrix of wrows_total rows, [d*esz/SB][wrows_total][SB], of which
// this workgroup takes rows wrow0 .. wrow0 + v - 1 (slab is ignored).
// hs (not with GATHER): the stage-major copy of all of h in stages of SB bytes, [d*esz/SB][B][SB]; the tile's
// rows of a stage are then one contiguous run, read instead of hp.
// STREAMW: every byte of W is read once by the whole launch (one tile of positions): loaded with the
// non-temporal hint.
template <int WV, int WB, int VB, int PB, int SB, int NS, bool BF16, bool GATHER = false, bool M16 = false,
          bool WPACK = false, bool STREAMW = false, int PH = 0, int VH = 0>
__device__ __forceinline__ void tile_gemm(const void* Wp, long long ld_w, const void* hp, long long ld_h,
                                          int B, int d, int v, int slab, int b0, char* smem,
                                          typename Frag<M16>::blk_t (&acc)[PB * Frag<M16>::SUB + PH][VB * Frag<M16>::SUB - VH / 2],
                                          const int* rows = nullptr, int nrows = 0, int rdiv = 1,
                                          const void* hs = nullptr, int wrows_total = 0, int wrow0 = 0) {
  TileFeed<WV, WB, VB, PB, SB, NS, BF16, GATHER, M16, WPACK, STREAMW, PH, 0, VH> feed;
  feed.open(Wp, ld_w, hp, ld_h, B, d, v, slab, b0, smem, rows, nrows, rdiv, hs, wrows_total, wrow0);
  tile_gemm_run(feed, d, smem, acc);
}

// Softmax statistics of every position column of the tile: max and log-sum-exp
// over the v vocabulary rows.  With FR = Frag<M16>, lane (lcol, lgrp) of wave (wv, wb) holds, for
// position column p = wb*PB*32 + pb*FR::BR + lcol, the vocabulary rows
//   row(vb, i) = wv*WROWS + vb*FR::BR + 4*lgrp + FR::roff(i).
// Contains one workgroup barrier; `red` must not be reused before the next one.
template <int WV, int WB, int VB, int PB, int SB, int NS, bool M16 = false, int PH = 0, int VH = 0>
__device__ __forceinline__ void tile_lse(const typename Frag<M16>::blk_t (&acc)[PB * Frag<M16>::SUB + PH][VB * Frag<M16>::SUB - VH / 2],
                                         int v, float2* red, float (&mx)[PB * Frag<M16>::SUB + PH],
                                         float (&lse)[PB * Frag<M16>::SUB + PH]) {
  using TL = Tile<WV, WB, VB, PB, SB, NS, PH, VH>;
  using FR = Frag<M16>;
  constexpr int NPB = PB * FR::SUB + PH, NVB = VB * FR::SUB - VH / 2;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wv = TL::wv(wave), wb = TL::wb(wave);
  const int lcol = FR::lcol(lane), lgrp = FR::lgrp(lane);
  const int rbase = wv * TL::WROWS + 4 * lgrp;
  // exp(l - m) = 2^(l * log2(e) - m * log2(e)): one fused multiply-add and one v_exp per logit.
  // A tile whose v fills all TV rows (v = 320 on the 320-row tiles) needs no row masks.
  constexpr float LOG2E = 1.4426950408889634f;
  const bool full = v == TL::TV && VH % 2 == 0;
#pragma unroll
  for (int pb = 0; pb < NPB; ++pb) {
    float m = neg_inf();
    if (full) {
#pragma unroll
      for (int vb = 0; vb < NVB; ++vb)
#pragma unroll
        for (int i = 0; i < FR::NI; ++i) m = fmaxf(m, acc[pb][vb][i]);
    } else {
#pragma unroll
      for (int vb = 0; vb < NVB; ++vb)
#pragma unroll
        for (int i = 0; i < FR::NI; ++i) {
          const int row = rbase + vb * FR::BR + FR::roff(i);
          if (row < v) m = fmaxf(m, acc[pb][vb][i]);
        }
    }
    m = FR::across(m, [](float x, float y) { return fmaxf(x, y); });
    const float ms = (m == neg_inf()) ? 0.f : m;
    const float ms2 = -ms * LOG2E;
    float s = 0.f;
    if (full) {
#pragma unroll
      for (int vb = 0; vb < NVB; ++vb)
#pragma unroll
        for (int i = 0; i < FR::NI; ++i) s += __builtin_amdgcn_exp2f(fmaf(acc[pb][vb][i], LOG2E, ms2));
    } else {
#pragma unroll
      for (int vb = 0; vb < NVB; ++vb)
#pragma unroll
        for (int i = 0; i < FR::NI; ++i) {
          const int row = rbase + vb * FR::BR + FR::roff(i);
          if (row < v) s += __builtin_amdgcn_exp2f(fmaf(acc[pb][vb][i], LOG2E, ms2));
        }
    }
    s = FR::across(s, [](float x, float y) { return x + y; });
    if (lgrp == 0) red[wv * TL::TP + wb * TL::WP + pb * FR::BR + lcol] = make_float2(m, s);
  }
  __syncthreads();
#pragma unroll
  for (int pb = 0; pb < NPB; ++pb) {
    const int p = wb * TL::WP + pb * FR::BR + lcol;
    float M = neg_inf();
#pragma unroll
    for (int w = 0; w < WV; ++w) M = fmaxf(M, red[w * TL::TP + p].x);
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < WV; ++w) {
      const float2 t = red[w * TL::TP + p];
      if (t.y > 0.f) s += t.y * __expf(t.x - M);
    }
    mx[pb] = M;
    lse[pb] = M + __logf(s);
  }
}

}  // namespace mtpc
