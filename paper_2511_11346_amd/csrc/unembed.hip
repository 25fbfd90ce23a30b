// Fused unembedding kernel of the MtPC head for gfx950 (Sec. 3.3):
//   l[b,i,j,:] = W[i,j] h[b]   (MFMA, fp32 accumulate)
//   LSE over the vocabulary in registers, then either the evidence
//   e[b,i,j] = l[x] - LSE at the target token or an inverse-CDF token draw.
// The (B, n, r, v) logits live only in accumulator registers.
//
// Tiling.  One workgroup computes D = W_slab (v rows) x h_tile^T (TP positions):
// the vocabulary is the MFMA M dimension, positions the N dimension, so that the
// accumulator block of a lane holds 16 (32x32 MFMA) or 4 (16x16) vocabulary rows of ONE
// position and the softmax reduction is almost entirely lane-local.  Wave grid WV (vocab)
// x WB (positions); a wave owns VB x PB blocks of 32x32 (see Frag for the two layouts).
// K is consumed in stages of SB bytes per row (SB = 64 or 128).  Both operand
// tiles go from global memory straight into LDS (buffer_load_dwordx4 ... lds) through
// a ring of NS stages with unpadded, XOR-swizzled rows; fragments are read with
// conflict-free 16-byte LDS loads one half-step ahead of the MFMAs using them.
#include "tile.h"
#include "sumunit.h"

namespace mtpc {

// ---- token draws on a finished tile -------------------------------------------------------
// A wave holds exp(l - max) of one position in vocabulary order, VPL consecutive tokens per
// lane (`vals`), `ls` their sum, `incl` the inclusive scan of ls over lanes, Z the total.
// Inverse CDF (Alg. 1): the smallest k with u * Z < cdf[k]; if rounding leaves u * Z >= Z,
// the last token with positive mass.  Returns the token in the lane for which `writer` is set.
template <int VPL>
__device__ __forceinline__ int wave_draw_token(const float (&vals)[VPL], float ls, float incl, float Z, float u,
                                               int lane, bool& writer) {
  const float tgt = u * Z;
  const unsigned long long cross = __ballot(tgt < incl);
  if (cross != 0ull) {
    const int L = __ffsll((long long)cross) - 1;
    float run = incl - ls;
    int tok = lane * VPL + VPL - 1;
    bool found = false;
#pragma unroll
    for (int q = 0; q < VPL; ++q) {
      run += vals[q];
      if (!found && tgt < run) { tok = lane * VPL + q; found = true; }
    }
    writer = lane == L;
    return tok;
  }
  int last = -1;
#pragma unroll
  for (int q = 0; q < VPL; ++q)
    if (vals[q] > 0.f) last = lane * VPL + q;
  const unsigned long long pos = __ballot(last >= 0);
  writer = lane == 63 - __clzll((long long)pos);
  return last;
}

// the most likely token of the position a wave holds (ties: the smallest id); all lanes get it
template <int VPL>
__device__ __forceinline__ int wave_argmax_token(const float (&vals)[VPL], int lane) {
  float best = -1.f;
  int arg = 0;
#pragma unroll
  for (int q = 0; q < VPL; ++q)
    if (vals[q] > best) { best = vals[q]; arg = lane * VPL + q; }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const float ob = __shfl_xor(best, o);
    const int oa = __shfl_xor(arg, o);
    if (ob > best || (ob == best && oa < arg)) { best = ob; arg = oa; }
  }
  return arg;
}

// Draw stage of a tile whose LSE statistics are known.  The tile-local positions that draw
// are listed in LDS (s_list[0..cnt), written before the preceding barrier).  NSL positions
// at a time: their accumulator columns are dumped as exp(l - max) in vocabulary order into
// the (now free) stage buffers, then one wave per position scans its row and calls
// body(p, vals, ls, incl, Z).
template <class TL, int VB, int PB, int NSL, bool M16, class Body>
__device__ __forceinline__ void tile_draws(const typename Frag<M16>::blk_t (&acc)[PB * Frag<M16>::SUB][VB * Frag<M16>::SUB],
                                           const float (&mx)[PB * Frag<M16>::SUB], int v, char* smem, int cnt, Body body) {
  using FR = Frag<M16>;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wv = wave % (TL::TV / (VB * 32)), wb = wave / (TL::TV / (VB * 32));
  const int lcol = FR::lcol(lane);
  const int rbase = wv * VB * 32 + 4 * FR::lgrp(lane);
  int* s_list = (int*)(smem + TL::MISC_OFF) + 4;
  int* s_slot = s_list + TL::TP;
  float* probs = (float*)smem;
  constexpr int SLOT = TL::VPL * 64 + 1;     // odd stride: the lanes of a wave dump different slots into different banks
  static_assert(NSL * SLOT * 4 <= TL::RED_OFF, "draw buffer must fit in the stage buffers");
  for (int c0 = 0; c0 < cnt; c0 += NSL) {
    const int nsl = min(NSL, cnt - c0);
    for (int p = tid; p < TL::TP; p += TL::NT) s_slot[p] = -1;
    __syncthreads();
    if (tid < nsl) s_slot[s_list[c0 + tid]] = tid;
    __syncthreads();
#pragma unroll
    for (int pb = 0; pb < PB * FR::SUB; ++pb) {
      const int sl = s_slot[wb * PB * 32 + pb * FR::BR + lcol];
      if (sl >= 0) {
#pragma unroll
        for (int vb = 0; vb < VB * FR::SUB; ++vb)
#pragma unroll
          for (int i = 0; i < FR::NI; ++i) {
            const int row = rbase + vb * FR::BR + FR::roff(i);
            probs[sl * SLOT + row] = (row < v) ? expf(acc[pb][vb][i] - mx[pb]) : 0.f;
          }
      }
    }
    __syncthreads();
    for (int k = wave; k < nsl; k += TL::NW) {
      float vals[TL::VPL];
      float ls = 0.f;
#pragma unroll
      for (int q = 0; q < TL::VPL; ++q) {
        vals[q] = probs[k * SLOT + lane * TL::VPL + q];
        ls += vals[q];
      }
      float incl = ls;   // inclusive scan over lanes
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const float t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
      }
      const float Z = __shfl(incl, 63);
      body(s_list[c0 + k], vals, ls, incl, Z);
    }
    __syncthreads();
  }
}

// Draws for every position column of a tile at once, from the accumulators (16x16 blocks): one token per
// column p with need(p), by inverse CDF (Alg. 1: the smallest token k with u Z < cdf[k]; the last token with
// positive mass if rounding leaves u Z >= Z) or, greedy, the most likely token (ties: the smallest id).
// A column's v values lie in 4 lane groups x NVB blocks x WV waves; each lane forms the prefix of its own
// rows (sums over the lane groups by lane permutes, over the blocks in registers, over the waves through
// LDS) and looks for the crossing among its rows; the smallest crossing row of a column wins (LDS minimum).
// Three workgroup barriers per call, all waves busy, nothing dumped to LDS but one sum per column and wave.
// Wide wave tiles (more than three blocks of columns) form the terms of a block a second time after the
// barrier instead of keeping those of all blocks in registers.
// The stage buffers must be free.  uni(p) gives the uniform of column p, out(p, token) takes the result.
template <class TL, int WV, int NVB, int NPB, class Need, class Uni, class Out>
__device__ __forceinline__ void tile_draws_cols(const f32x4_t (&acc)[NPB][NVB], const float (&mx)[NPB], int v,
                                                char* smem, bool greedy, Need need, Uni uni, Out out) {
  constexpr bool KEEP = NPB <= 3;
  constexpr int NK = KEEP ? NPB : 1;
  static_assert(NPB * 16 == TL::WP, "the wave's blocks of 16 position columns");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wv = TL::wv(wave), wb = TL::wb(wave);
  const int lcol = lane & 15, lgrp = lane >> 4;
  const int rbase = wv * TL::WROWS + 4 * lgrp;
  float* wsum = (float*)smem;                                        // [WV][TP] sum of a wave's rows of a column
  int* cand = (int*)(wsum + WV * TL::TP);                            // [TP] smallest crossing row
  int* lastp = cand + TL::TP;                                        // [TP] last row with positive mass
  unsigned long long* best = (unsigned long long*)(lastp + TL::TP);  // [TP] greedy: (value, -row)
  static_assert((WV + 2) * TL::TP * 4 + TL::TP * 8 <= TL::RED_OFF, "fits in the stage buffers");
  for (int p = tid; p < TL::TP; p += TL::NT) {
    cand[p] = 0x7fffffff;
    lastp[p] = -1;
    best[p] = 0ull;
  }
  // the terms of block pb: e = exp(l - max) of this lane's rows, ex = what the lane groups below this one
  // hold of a block of 16 rows, tot = the block's sum; returns the sum of the wave's rows of the column
  auto terms = [&](int pb, float (&e)[NVB][4], float (&ex)[NVB], float (&tot)[NVB]) {
    float colsum = 0.f;
#pragma unroll
    for (int vb = 0; vb < NVB; ++vb) {
#pragma unroll
      for (int t = 0; t < 4; ++t) e[vb][t] = (rbase + vb * 16 + t < v) ? expf(acc[pb][vb][t] - mx[pb]) : 0.f;
      const float s4 = ((e[vb][0] + e[vb][1]) + e[vb][2]) + e[vb][3];
      // inclusive scan over the four lane groups that hold this column (lanes lcol + 16 g)
      const float u1 = __shfl_up(s4, 16);
      const float i1 = lgrp >= 1 ? s4 + u1 : s4;
      const float u2 = __shfl_up(i1, 32);
      const float incl = lgrp >= 2 ? i1 + u2 : i1;
      ex[vb] = incl - s4;
      tot[vb] = __shfl(incl, 48 + lcol);
      colsum += tot[vb];
    }
    return colsum;
  };
  float e[NK][NVB][4], ex[NK][NVB], tot[NK][NVB];
#pragma unroll
  for (int pb = 0; pb < NPB; ++pb) {
    const float colsum = terms(pb, e[KEEP ? pb : 0], ex[KEEP ? pb : 0], tot[KEEP ? pb : 0]);
    if (lgrp == 0) wsum[wv * TL::TP + wb * TL::WP + pb * 16 + lcol] = colsum;
  }
  __syncthreads();
#pragma unroll
  for (int pb = 0; pb < NPB; ++pb) {
    const int col = wb * TL::WP + pb * 16 + lcol;
    constexpr int k0 = 0;
    const int k = KEEP ? pb : k0;
    if constexpr (!KEEP) (void)terms(pb, e[0], ex[0], tot[0]);
    if (greedy) {
      float bv = -1.f;
      int br = 0;
#pragma unroll
      for (int vb = 0; vb < NVB; ++vb)
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if (e[k][vb][t] > bv) { bv = e[k][vb][t]; br = rbase + vb * 16 + t; }
      atomicMax(&best[col], ((unsigned long long)__float_as_uint(bv) << 32) | (unsigned)(0x7fffffff - br));
    } else {
      float below = 0.f, Z = 0.f;
#pragma unroll
      for (int w = 0; w < WV; ++w) {
        const float x = wsum[w * TL::TP + col];
        if (w < wv) below += x;
        Z += x;
      }
      const float tgt = uni(col) * Z;
      float run = below;
      int first = 0x7fffffff, last = -1;
#pragma unroll
      for (int vb = 0; vb < NVB; ++vb) {
        float c = run + ex[k][vb];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          c += e[k][vb][t];
          const int row = rbase + vb * 16 + t;
          if (tgt < c) first = min(first, row);
          if (e[k][vb][t] > 0.f) last = row;
        }
        run += tot[k][vb];
      }
      if (first != 0x7fffffff) atomicMin(&cand[col], first);
      atomicMax(&lastp[col], last);
    }
  }
  __syncthreads();
  if (wv == 0 && lgrp == 0) {
#pragma unroll
    for (int pb = 0; pb < NPB; ++pb) {
      const int col = wb * TL::WP + pb * 16 + lcol;
      if (need(col)) {
        int tok;
        if (greedy) tok = 0x7fffffff - (int)(unsigned)(best[col] & 0xffffffffull);
        else tok = cand[col] != 0x7fffffff ? cand[col] : lastp[col];
        out(col, tok);
      }
    }
  }
  __syncthreads();
}

// Which instantiations of k_unembed walk several tiles per workgroup: the ones whose epilogue leaves the
// ring alone (no draws) on the tiles of training-sized batches.
template <int WB, bool SAMPLE>
constexpr bool unembed_walks_tiles() { return !SAMPLE && WB != 1; }

// SPLIT: fp32 operands as planes of two fp16 terms or three bf16 terms (tile_gemm_run_split); everything but the product, and the
// scales of fp16 terms' rows that come out of the result behind it, is the bf16 kernel's.
// STREAM: one tile of positions, so that every byte of W is read once (loaded with the non-temporal hint).
// PH: 16 more positions per wave (Tile).
// ROT: slabs may start at different stages of K (UnembedArgs::first_stages).
template <int WV, int WB, int VB, int PB, int SB, int NS, bool BF16, bool SAMPLE, bool WPACK = false, int SPLIT = 0, int VH = 0,
          bool STREAM = false, int PH = 0, bool ROT = SPLIT == 0 && !SAMPLE && WB != 1>
__global__ __launch_bounds__(WV * WB * 64)
void k_unembed(const UnembedArgs a) {
  // of the launches over the same fp32 operands one does the work (see launch_split)
  if constexpr (SPLIT != 0 || !BF16)
    if (a.wild != nullptr) {
      const int flag = *a.wild;
      const bool three = a.three != 0 && (flag & SPLIT_WHOLE) == 0;
      if (SPLIT != ((flag & SPLIT_WIDE) == 0 ? 2 : three ? 3 : 0)) return;
    }
  using TL = Tile<WV, WB, VB, PB, SB, NS, PH, VH>;
  constexpr bool M16 = use_m16<WV, WB, SB, NS, BF16>();
  using FR = Frag<M16>;
  constexpr int NPB = PB * FR::SUB + PH, NVB = VB * FR::SUB - VH / 2;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wv = TL::wv(wave), wb = TL::wb(wave);
  const int lcol = FR::lcol(lane), lgrp = FR::lgrp(lane);
  const int nslab = a.n * a.r;
  const int nbt = (a.B + TL::TP - 1) / TL::TP;
  // The evidence kernel of a training-sized batch is launched with one workgroup per CU (unembed_walks_tiles):
  // a workgroup walks the tiles blockIdx.x, blockIdx.x + gridDim.x, ... (the grid is a multiple of the number
  // of XCDs, so all of them lie in this XCD's range of logical tiles) and opens the feed of the next tile
  // before the epilogue of the one it has multiplied: the first stages of the next ring arrive while the
  // softmax statistics are taken, instead of after a workgroup launch with the matrix pipe idle.
  // Every other instantiation has one tile per workgroup and leaves the loop after it.
  constexpr bool WALK = unembed_walks_tiles<WB, SAMPLE>();
  using Feed = TileFeed<WV, WB, VB, PB, SB, NS, BF16, false, M16, WPACK, STREAM, PH, SPLIT, VH, 0, ROT>;
  const void* const hstaged = SPLIT ? a.hq : (WB != 1 && SB == H_STAGE_BYTES) ? a.hs : nullptr;
  const void* const Wfeed = SPLIT ? a.Wq : WPACK ? a.Wp : a.W;
  const int dfeed = SPLIT != 0 ? SPLIT * a.d : a.d;   // 16-bit columns of the planes
  const int* const hexp = SPLIT == 2 ? (const int*)((const char*)a.hq + 4LL * a.B * a.d) : nullptr;      // (plane_exps)
  int* const s_e = (int*)(smem + TL::SMEM);           // SPLIT = 2: exponents of the tile's rows and columns [TV + TP]
  const int ntiles = nbt * nslab;
  int slab, bt;
  tile_of_block(blockIdx.x, nbt, nslab, slab, bt);
  Feed feed;
  const int wrows = SPLIT ? a.Wq_rows : 0;
  // One tile of positions: every workgroup streams a slab of its own, and where W's rows ask for it (starts_differ) from a stage of
  // its own on.  Tiles that share slabs and rows of h in an L2 walk K together, from its beginning (starts that differ: B = 300 .. 1000
  // the same, B = 4096 and 8192 0.4 % slower).  Passes that draw, or fill a table that tokens are drawn from, do as well: with sums in
  // another order one token in 30,000 falls on the other side of its uniform, and a draft of a given seed is to stay what it was (draft
  // and score, B = 61, W's own rows, 320 / 309 us; the gathered draws of n r = 1024, B = 4096 446 / 439; draft, table, scores and
  // verification, n r = 256, d = 2048, B = 256 171 / 152).
  auto first = [&](int sl) { return ROT ? first_stage(sl, a.first_stages, a.first_reciprocal) : 0; };
  feed.open(Wfeed, dfeed, a.h, a.ld_h, a.B, dfeed, a.v, slab, bt * TL::TP, smem, nullptr, 0, 1, hstaged, wrows, slab * a.v,
            first(slab));
  for (int w = blockIdx.x;;) {
  const int b0 = bt * TL::TP;
  const int wi = slab / a.r, wj = slab - wi * a.r;

  // Target tokens of the tile's positions, first XW windows of each: fetched now, while nothing
  // depends on them, parked in LDS after the product (the list / slot area the draws use, idle
  // in this instantiation).  Read in the epilogue they would be one dependent memory round
  // trip per position column and window, with the matrix pipe idle.
  constexpr int XW = 2, XR = (XW * TL::TP + TL::NT - 1) / TL::NT;
  int* s_x = (int*)(smem + TL::MISC_OFF) + 4;        // [XW][TP]
  int xpre[XR];
  int nxw = 0;
  if constexpr (!SAMPLE) if (a.targets != nullptr) {
    nxw = min(a.T + a.T2, XW);
#pragma unroll
    for (int q = 0; q < XR; ++q) {
      const int idx = tid + q * TL::NT, t = idx / TL::TP, p = idx - t * TL::TP;
      const long long b = b0 + p;
      xpre[q] = -1;
      if (t < nxw && b < a.B)
        xpre[q] = t < a.T ? a.targets[(b * a.T + t) * a.n + wi] : a.targets2[(b * a.T2 + (t - a.T)) * a.n + wi];
    }
  }

  // exponents of the tile's operand rows, the same way
  constexpr int XE = (TL::ROWS + TL::NT - 1) / TL::NT;
  int epre[XE];
  if constexpr (SPLIT == 2) {
#pragma unroll
    for (int q = 0; q < XE; ++q) {
      const int idx = min(tid + q * TL::NT, TL::ROWS - 1);
      epre[q] = idx < TL::TV ? a.Wexp[(long long)slab * a.v + min(idx, a.v - 1)] : hexp[min(b0 + idx - TL::TV, a.B - 1)];
    }
  }

  typename FR::blk_t acc[NPB][NVB];
  if constexpr (SPLIT != 0) tile_gemm_run_split(feed, a.d, smem, acc);
  else tile_gemm_run(feed, a.d, smem, acc);
  const int wnext = w + (int)gridDim.x;
  int slab_next = 0, bt_next = 0;
  if constexpr (WALK)
    if (wnext < ntiles) {
      tile_of_block(wnext, nbt, nslab, slab_next, bt_next);
      feed.open(Wfeed, dfeed, a.h, a.ld_h, a.B, dfeed, a.v, slab_next, bt_next * TL::TP, smem, nullptr, 0, 1, hstaged, wrows, slab_next * a.v,
                first(slab_next));
    }

  if constexpr (!SAMPLE) if (a.targets != nullptr) {
#pragma unroll
    for (int q = 0; q < XR; ++q) {
      const int idx = tid + q * TL::NT;
      if (idx < nxw * TL::TP) s_x[idx] = xpre[q];
    }
  }
  // this lane holds, of position column wb*WP + pb*BR + lcol, rows rbase + vb*BR + roff(i)
  const int rbase = wv * TL::WROWS + 4 * lgrp;
  if constexpr (SPLIT == 2) {
#pragma unroll
    for (int q = 0; q < XE; ++q)
      if (tid + q * TL::NT < TL::ROWS) s_e[tid + q * TL::NT] = epre[q];
    __syncthreads();
    tile_unscale<TL>(acc, s_e, rbase, wb * TL::WP + lcol);
  }
  float mx[NPB], lse[NPB];
  tile_lse<WV, WB, VB, PB, SB, NS, M16, PH, VH>(acc, a.v, (float2*)(smem + TL::RED_OFF), mx, lse);   // (one barrier: s_x is visible)

  // evidence at the target tokens (the sampling instantiation never has targets)
  if constexpr (!SAMPLE) if (a.targets != nullptr) {
#pragma unroll
    for (int pb = 0; pb < NPB; ++pb) {
      const int b = b0 + wb * TL::WP + pb * FR::BR + lcol;
      if (b < a.B) {
        const int TT = a.T + a.T2;
        for (int t = 0; t < TT; ++t) {
          const long long rowid = (long long)b * TT + t;
          const int x = t < XW ? s_x[t * TL::TP + (b - b0)]
                        : t < a.T ? a.targets[((long long)b * a.T + t) * a.n + wi]
                                  : a.targets2[((long long)b * a.T2 + (t - a.T)) * a.n + wi];
          float* dst = a.e + (rowid * a.n + wi) * a.r + wj;
          if (x < 0 || x >= a.v) {
            if (wv == 0 && lgrp == 0) *dst = (x == -1) ? 0.f : __builtin_nanf("");
          } else {
            // first the block of the target row, then its register by the bits of the offset
            // (a few dozen selects instead of a compare and a select for every register)
            const int xr = x - rbase;
            if constexpr (M16) {
              // rows rbase + 16 vb + t (t in 0..3)
              if (xr >= 0 && xr < TL::WROWS && (xr & 12) == 0) {
                const int xvb = xr >> 4;
                f32x4_t blk = acc[pb][0];
#pragma unroll
                for (int vb = 1; vb < NVB; ++vb) blk = (xvb == vb) ? acc[pb][vb] : blk;
                const bool t0 = xr & 1, t1 = xr & 2;
                const float c0 = t0 ? blk[1] : blk[0], c1 = t0 ? blk[3] : blk[2];
                *dst = (t1 ? c1 : c0) - lse[pb];
              }
            } else {
              // rows rbase + 32 vb + 8 q + t (q, t in 0..3)
              if (xr >= 0 && xr < VB * 32 && (xr & 4) == 0) {
                const int xvb = xr >> 5;
                f32x16_t blk = acc[pb][0];
#pragma unroll
                for (int vb = 1; vb < VB; ++vb) blk = (xvb == vb) ? acc[pb][vb] : blk;
                const bool t0 = xr & 1, t1 = xr & 2, q0 = xr & 8, q1 = xr & 16;
                const float b0 = t0 ? blk[1] : blk[0], b1 = t0 ? blk[3] : blk[2];
                const float b2 = t0 ? blk[5] : blk[4], b3 = t0 ? blk[7] : blk[6];
                const float b4 = t0 ? blk[9] : blk[8], b5 = t0 ? blk[11] : blk[10];
                const float b6 = t0 ? blk[13] : blk[12], b7 = t0 ? blk[15] : blk[14];
                const float c0 = t1 ? b1 : b0, c1 = t1 ? b3 : b2, c2 = t1 ? b5 : b4, c3 = t1 ? b7 : b6;
                const float lo = q0 ? c1 : c0, hi = q0 ? c3 : c2;
                *dst = (q1 ? hi : lo) - lse[pb];
              }
            }
          }
        }
      }
    }
  }
  if constexpr (!SAMPLE) if (a.phiT != nullptr) {
    // keep the normalised probabilities for the training step (transposed: positions contiguous;
    // the column blocks of a row are stored back to back, together they fill whole lines).
    // phi = 2^((l - lse) log2 e): one fused multiply-add and one v_exp per probability
    constexpr float LOG2E = 1.4426950408889634f;
    const int bl = b0 + wb * TL::WP + lcol;
    float* col = a.phiT + ((long long)slab * a.v + rbase) * a.ld_phi + bl;
    float shift[NPB];
#pragma unroll
    for (int pb = 0; pb < NPB; ++pb) shift[pb] = -lse[pb] * LOG2E;
#pragma unroll
    for (int vb = 0; vb < NVB; ++vb)
#pragma unroll
      for (int i = 0; i < FR::NI; ++i) {
        const int off = vb * FR::BR + FR::roff(i);
        if (rbase + off >= a.v) continue;
#pragma unroll
        for (int pb = 0; pb < NPB; ++pb)
          if (bl + pb * FR::BR < a.B)
            col[off * a.ld_phi + pb * FR::BR] = __builtin_amdgcn_exp2f(fmaf(acc[pb][vb][i], LOG2E, shift[pb]));
      }
  }
  if (a.logphi != nullptr) {
    // table log phi[b][wi][wj][:] for the scoring and verification steps.  Registers
    // 4q..4q+3 of a block hold four consecutive vocabulary rows of one position: one
    // 16-byte store each (the row of a position is 4v bytes long and 16-byte aligned
    // when v is a multiple of 4; otherwise element by element)
    const bool vec = (a.v & 3) == 0;
#pragma unroll
    for (int pb = 0; pb < NPB; ++pb) {
      const int b = b0 + wb * TL::WP + pb * FR::BR + lcol;
      if (b >= a.B) continue;
      float* dst = a.logphi + (((long long)b * a.n + wi) * a.r + wj) * a.v;
#pragma unroll
      for (int vb = 0; vb < NVB; ++vb)
#pragma unroll
        for (int q = 0; q < FR::NI / 4; ++q) {
          const int row = rbase + vb * FR::BR + FR::roff(4 * q);
          if (vec) {
            if (row < a.v)
              *(f32x4_t*)(dst + row) = f32x4_t{acc[pb][vb][4 * q] - lse[pb], acc[pb][vb][4 * q + 1] - lse[pb],
                                               acc[pb][vb][4 * q + 2] - lse[pb], acc[pb][vb][4 * q + 3] - lse[pb]};
          } else {
#pragma unroll
            for (int t = 0; t < 4; ++t)
              if (row + t < a.v) dst[row + t] = acc[pb][vb][4 * q + t] - lse[pb];
          }
        }
    }
  }
  if constexpr (SAMPLE && M16 && WB != 1) {
    // training-sized tiles: the tokens of all columns at once, one pass per draft (only tiles in which some
    // position draws token wi of that draft from component wj)
    if (a.zleaf == nullptr) return;
    const bool one = a.r == 1;                         // (zleaf is 0 throughout, and not written)
    for (int s = 0; s < a.S; ++s) {
      auto need = [&](int p) {
        const long long b = b0 + p;
        return b < a.B && (one || a.zleaf[(b * a.S + s) * a.n + wi] == wj);
      };
      bool any = false;
      for (int p = tid; p < TL::TP; p += TL::NT) any |= need(p);
      if (!__syncthreads_or(any)) continue;
      tile_draws_cols<TL, WV, NVB, NPB>(
          acc, mx, a.v, smem, a.greedy != 0, need,
          [&](int p) { return philox_uniform(a.seed_lo, a.seed_hi, a.offset, (uint32_t)(b0 + p), (uint32_t)s, (uint32_t)wi); },
          [&](int p, int tok) { a.drafts[((long long)(b0 + p) * a.S + s) * a.n + wi] = tok; });
    }
  } else if constexpr (SAMPLE) {
    if (a.zleaf == nullptr) return;
    const bool one = a.r == 1;                         // (zleaf is 0 throughout, and not written)
    // ---- which positions of this tile draw token wi from component wj?
    int* misc = (int*)(smem + TL::MISC_OFF);
    int* s_cnt = misc;
    int* s_list = misc + 4;
    if (tid == 0) *s_cnt = 0;
    __syncthreads();
    for (int p = tid; p < TL::TP; p += TL::NT) {
      const int b = b0 + p;
      bool need = false;
      if (b < a.B)
        for (int s = 0; s < a.S; ++s)
          need |= one || a.zleaf[((long long)b * a.S + s) * a.n + wi] == wj;
      if (need) s_list[atomicAdd(s_cnt, 1)] = p;
    }
    __syncthreads();
    const int cnt = *s_cnt;
    tile_draws<TL, VB, PB, NSLOT, M16>(acc, mx, a.v, smem, cnt, [&](int p, const float (&vals)[TL::VPL], float ls, float incl,
                                                        float Z) {
      const int b = b0 + p;
      for (int s = 0; s < a.S; ++s) {
        const long long di = ((long long)b * a.S + s) * a.n + wi;
        if (!one && a.zleaf[di] != wj) continue;
        int tok;
        bool writer;
        if (a.greedy) {
          tok = wave_argmax_token<TL::VPL>(vals, lane);
          writer = lane == 0;
        } else {
          const float u = philox_uniform(a.seed_lo, a.seed_hi, a.offset, (uint32_t)b, (uint32_t)s, (uint32_t)wi);
          tok = wave_draw_token<TL::VPL>(vals, ls, incl, Z, u, lane, writer);
        }
        if (writer) a.drafts[di] = tok;
      }
    });
  }
  if (!WALK || wnext >= ntiles) break;
  w = wnext;
  slab = slab_next;
  bt = bt_next;
  }
}

// stage geometry of the gathered draw tiles and the positions drawn per pass of their draw loop
constexpr int GATHER_SB = GATHER_STAGE_BYTES, GATHER_NS = 4, GATHER_NSL = 16;
// Token draws of Alg. 1 for training-sized batches: only the input unit a token is drawn
// from is evaluated.  The (b, s, i) triples were bucketed by (i, z) = (token, selected
// unit); a workgroup takes up to TP rows of one bucket, gathers their h rows, multiplies
// them with the one slab W[i][z] and draws every row's token - 1/r of the products a
// pass over all slabs needs.
template <int WV, int WB, int VB, int PB, int SB, int NS, bool BF16, bool WPACK, int PH, int VH>
__global__ __launch_bounds__(WV * WB * 64)
void k_draw_gather(const DrawGatherArgs a) {
  using TL = Tile<WV, WB, VB, PB, SB, NS, PH, VH>;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  // each XCD owns a contiguous range of logical tiles, so that the tiles of a bucket
  // (which share a W slab) run under one L2
  // (the grid is an upper bound; the ranges are cut from the number of tiles there are, so that
  // every XCD gets its share of them)
  const int ngroups = a.n * a.r;
  const int total = a.tile_off[ngroups];
  const int w = blockIdx.x;
  if (w >= total) return;
  const int per = total >> 3;
  const int lid = (w < per * 8) ? (w & 7) * per + (w >> 3) : w;
  const int g = a.tile_bucket[lid];                  // tile_off[g] <= lid < tile_off[g+1]
  const int first = a.row_off[g] + (lid - a.tile_off[g]) * TL::TP;
  const int nrows = min(a.row_off[g + 1] - first, TL::TP);     // >= 1 by construction of tile_off
  const int* rows = a.list + first;
  const int wi = g / a.r;

  constexpr bool M16 = use_m16<WV, WB, SB, NS, BF16>();
  constexpr int NPB = PB * Frag<M16>::SUB + PH, NVB = VB * Frag<M16>::SUB - VH / 2;
  typename Frag<M16>::blk_t acc[NPB][NVB];
  tile_gemm<WV, WB, VB, PB, SB, NS, BF16, true, M16, WPACK, false, PH, VH>(WPACK ? a.Wp : a.W, a.d, a.h, a.ld_h, a.B, a.d, a.v, g, 0, smem,
                                                                       acc, rows, nrows, a.S);
  float mx[NPB], lse[NPB];
  tile_lse<WV, WB, VB, PB, SB, NS, M16, PH, VH>(acc, a.v, (float2*)(smem + TL::RED_OFF), mx, lse);

  if constexpr (M16) {
    const int S = a.S;
    tile_draws_cols<TL, WV, NVB, NPB>(
        acc, mx, a.v, smem, a.greedy != 0, [&](int p) { return p < nrows; },
        [&](int p) {
          const int rid = rows[min(p, nrows - 1)];       // b * S + s
          const int b = rid / S, sd = rid - b * S;
          return philox_uniform(a.seed_lo, a.seed_hi, a.offset, (uint32_t)b, (uint32_t)sd, (uint32_t)wi);
        },
        [&](int p, int tok) { a.drafts[(long long)rows[p] * a.n + wi] = tok; });
  } else {
    int* s_list = (int*)(smem + TL::MISC_OFF) + 4;
    for (int p = tid; p < nrows; p += TL::NT) s_list[p] = p;
    __syncthreads();
    tile_draws<TL, VB, PB, GATHER_NSL, M16>(acc, mx, a.v, smem, nrows, [&](int p, const float (&vals)[TL::VPL], float ls,
                                                                           float incl, float Z) {
      const int rid = rows[p];                         // b * S + s
      const int b = rid / a.S, s = rid - b * a.S;
      int tok;
      bool writer;
      if (a.greedy) {
        tok = wave_argmax_token<TL::VPL>(vals, lane);
        writer = lane == 0;
      } else {
        const float u = philox_uniform(a.seed_lo, a.seed_hi, a.offset, (uint32_t)b, (uint32_t)s, (uint32_t)wi);
        tok = wave_draw_token<TL::VPL>(vals, ls, incl, Z, u, lane, writer);
      }
      if (writer) a.drafts[(long long)rid * a.n + wi] = tok;
    });
  }
}

template <int WV, int WB, int VB, int PB, int PH, bool BF16, int VH = 0, bool WPACK = false>
static hipError_t launch_draw_gather_cfg(const DrawGatherArgs& a, hipStream_t st) {
  using TL = Tile<WV, WB, VB, PB, GATHER_SB, GATHER_NS, PH, VH>;
  static_assert(TL::TP == DRAW_GATHER_TILE || TL::TP == DRAW_GATHER_TILE_WIDE, "the tile heights the bucketing is run with");
  if constexpr (!WPACK)
    if (a.Wp != nullptr) return launch_draw_gather_cfg<WV, WB, VB, PB, PH, BF16, VH, true>(a, st);
  constexpr auto kern = k_draw_gather<WV, WB, VB, PB, GATHER_SB, GATHER_NS, BF16, WPACK, PH, VH>;
  if (hipError_t e = allow_lds<kern>(TL::SMEM); e != hipSuccess) return e;
  const long long rows = (long long)a.B * a.S * a.n;
  const int grid = (int)(rows / TL::TP) + a.n * a.r;             // >= sum over buckets of ceil(rows_g / TP)
  hipLaunchKernelGGL(kern, dim3(grid), dim3(TL::NT), TL::SMEM, st, a);
  return hipGetLastError();
}

template <bool BF16>
static hipError_t launch_draw_gather_dt(const DrawGatherArgs& a, hipStream_t st) {
  if constexpr (BF16)                                // (the wide tile counts its columns in blocks of 16)
    if (a.tile == DRAW_GATHER_TILE_WIDE) {
      if (a.v > 272) return launch_draw_gather_cfg<2, 4, 5, 1, 1, BF16>(a, st);
      if (a.v > 256) return launch_draw_gather_cfg<2, 4, 5, 1, 1, BF16, 3>(a, st);
      if (a.v > 128) return launch_draw_gather_cfg<2, 4, 4, 1, 1, BF16>(a, st);
      return launch_draw_gather_cfg<2, 4, 2, 1, 1, BF16>(a, st);
    }
  if (a.tile != DRAW_GATHER_TILE) return hipErrorInvalidValue;
  if (a.v > 272) return launch_draw_gather_cfg<2, 4, 5, 1, 0, BF16>(a, st);
  if (a.v > 256) return launch_draw_gather_cfg<2, 4, 5, 1, 0, BF16, BF16 ? 3 : 0>(a, st);
  if (a.v > 128) return launch_draw_gather_cfg<2, 4, 4, 1, 0, BF16>(a, st);
  return launch_draw_gather_cfg<2, 4, 2, 1, 0, BF16>(a, st);
}

hipError_t launch_draw_gather(const DrawGatherArgs& a, int dtype, hipStream_t st) {
  return dtype == MTPC_BF16 ? launch_draw_gather_dt<true>(a, st) : launch_draw_gather_dt<false>(a, st);
}

// Sum-unit parameters for many positions (Sec. 3.3): log omega[b,:] = log_softmax(Wsum h[b]), r <= 16 RB units,
// 16 PB positions per workgroup.  The product is small and its chain over d long, so the waves (sixteen, or eight
// where their partial sums and buffers would not fit in LDS) deal its 64-byte steps among themselves (together a contiguous
// piece of every row), each through LDS buffers of its own with U steps in flight and no barrier, and their partial sums are
// added through LDS in a fixed order.
// What limits it is the rate at which a CU takes in operand rows, so every load is 16 whole 64-byte pieces of rows, straight into LDS: as
// fragments in registers four neighbouring lanes ask for four rows, and a load takes four times as long (r = 32, d = 4096 bf16, B = 200:
// 15 -> 11 us with the layers and the copy of h beside it, 25 in three launches; fp32, B = 2048, d = 3072 26 -> 21; as one wave that walks all of d 22 and 57).  Steps that are not there are not loaded.
// The workgroups behind those of the positions see to the call's other parameters.
template <int RB, int PB, bool BF16, int NW, int U>
__global__ __launch_bounds__(NW * 64)
void k_sumunit_mfma(const ParamArgs p) {
  constexpr int ESZ = BF16 ? 2 : 4, NB = RB + PB;
  constexpr int PS = PB * 16 + 1;                    // (odd stride: the lanes of a reduction read different banks)
  constexpr int PART = RB * 16 * PS;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int nsum = (p.B + PB * 16 - 1) / (PB * 16);
  if ((int)blockIdx.x >= nsum) {
    params_beside<NW * 64>(p, (int)blockIdx.x - nsum);
    return;
  }
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int l15 = lane & 15, lq = lane >> 4;
  const int b0 = blockIdx.x * PB * 16, r = p.r;
  const int steps = p.d * ESZ / 64, mine = (steps - wave + NW - 1) / NW;      // (0: fewer steps than waves)
  const int hspan = min(p.B - b0, PB * 16);
  const i32x4_t srdW = make_srd(p.Wsum, (unsigned)((long long)r * p.d * ESZ));
  const i32x4_t srdH = make_srd((const char*)p.h + (long long)b0 * p.ld_h * ESZ, (unsigned)((long long)(hspan - 1) * p.ld_h * ESZ + (long long)p.d * ESZ));
  // this lane's 16 bytes of a block of 16 rows, swizzled for the fragment reads (swz16)
  const int lrow = lane >> 2, lch = ((lane & 3) ^ swz16(lrow)) * 16;
  unsigned voff[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
    voff[i] = i < RB ? (unsigned)min(i * 16 + lrow, r - 1) * (unsigned)(p.d * ESZ) + lch
                     : (unsigned)min((i - RB) * 16 + lrow, hspan - 1) * (unsigned)(p.ld_h * ESZ) + lch;
  char* const ring = smem + wave * (min(U, (steps + NW - 1) / NW) * NB * 1024);      // (of as many steps as a wave has, or U)
  const unsigned lds0 = (unsigned)(size_t)ring;
  auto issue = [&](int j) {
    const unsigned so = (unsigned)(wave + j * NW) * 64, at = lds0 + (unsigned)(j % U) * (NB * 1024);
#pragma unroll
    for (int i = 0; i < NB; ++i) load_to_lds(voff[i], i < RB ? srdW : srdH, so, at + i * 1024);
  };
  f32x4_t acc[PB][RB];
#pragma unroll
  for (int q = 0; q < PB; ++q)
#pragma unroll
    for (int i = 0; i < RB; ++i) acc[q][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  for (int j = 0; j < min(U, mine); ++j) issue(j);
  const int frag = l15 * 64 + ((lq ^ swz16(l15)) << 4);
  for (int j = 0; j < mine; ++j) {
    // step j has landed (a wave's loads arrive in their order; the last U - 1 steps wait for all that are left)
    if (j + U <= mine) MTPC_WAIT_VMCNT((U - 1) * NB); else MTPC_WAIT_VMCNT(0);
    __builtin_amdgcn_sched_barrier(0);
    const char* const cur = ring + (j % U) * (NB * 1024) + frag;
    i32x4_t fw[RB], fh[PB];
#pragma unroll
    for (int i = 0; i < RB; ++i) fw[i] = *(const i32x4_t*)(cur + i * 1024);
#pragma unroll
    for (int q = 0; q < PB; ++q) fh[q] = *(const i32x4_t*)(cur + (RB + q) * 1024);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0xC07F);              // lgkmcnt(0): read, before its buffer takes step j + U
    __builtin_amdgcn_sched_barrier(0);
    if (j + U < mine) issue(j + U);
#pragma unroll
    for (int q = 0; q < PB; ++q)
#pragma unroll
      for (int i = 0; i < RB; ++i) {
        if constexpr (BF16) mma_step<true>(acc[q][i], fw[i], fh[q]);
        else {
          // lane group lq holds columns 4 lq .. 4 lq + 3 of both operands: product t takes one of each
          const f32x4_t x = __builtin_bit_cast(f32x4_t, fw[i]), y = __builtin_bit_cast(f32x4_t, fh[q]);
#pragma unroll
          for (int t = 0; t < 4; ++t) acc[q][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[t], y[t], acc[q][i], 0, 0, 0);
        }
      }
  }
  __syncthreads();                                   // all buffers are read: the partial sums take their place
  float* const part = (float*)smem;                  // [NW][PART]
#pragma unroll
  for (int q = 0; q < PB; ++q)
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int t = 0; t < 4; ++t) part[wave * PART + (i * 16 + 4 * lq + t) * PS + q * 16 + l15] = acc[q][i][t];
  __syncthreads();
  // 32 lanes per position, units j, j + 32, ...
  const int j = threadIdx.x & 31;
  constexpr int Q = (RB + 1) / 2;
  for (int q0 = threadIdx.x >> 5; q0 < PB * 16 && b0 + q0 < p.B; q0 += NW * 2) {
    float x[Q], m = neg_inf();
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int u = j + 32 * q;
      x[q] = neg_inf();
      if (u < r) {
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) sum += part[w * PART + u * PS + q0];
        x[q] = sum;
      }
      m = fmaxf(m, x[q]);
    }
    m = group_max(m, 32);
    const float ms = m == neg_inf() ? 0.f : m;
    float e = 0.f;
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (j + 32 * q < r) e += __expf(x[q] - ms);
    const float lse = m + __logf(group_sum(e, 32));
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (j + 32 * q < r) p.logw[(long long)(b0 + q0) * r + j + 32 * q] = x[q] - lse;
  }
}

template <int RB, int PB, bool BF16, int NW>
static hipError_t launch_sumunit_mfma_nw(const ParamArgs& p, hipStream_t st) {
  constexpr int NB = RB + PB, most = 148 / (NB * NW);          // steps in flight: what fits in LDS, up to eight
  constexpr int U = most < 8 ? most : 8;
  static_assert(U >= 2 && (U - 1) * NB <= 63, "a ring, and a wait that counts its loads");
  constexpr int part = NW * RB * 16 * (PB * 16 + 1) * 4, most_smem = std::max(part, NW * U * NB * 1024);
  static_assert(most_smem <= 160 * 1024, "LDS budget of one CU");
  constexpr auto kern = k_sumunit_mfma<RB, PB, BF16, NW, U>;
  if (hipError_t e = allow_lds<kern>(most_smem); e != hipSuccess) return e;
  const int steps = p.d * (BF16 ? 2 : 4) / 64, smem = std::max(part, NW * std::min(U, (steps + NW - 1) / NW) * NB * 1024);
  const long long grid = (p.B + PB * 16 - 1) / (PB * 16) + param_blocks(p, NW * 64);
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(NW * 64), smem, st, p);
  return hipGetLastError();
}

// (rows of at most 32 steps: four waves have all of them in flight, more would only add partial sums)
template <int RB, int PB, bool BF16>
static hipError_t launch_sumunit_mfma_cfg(const ParamArgs& p, hipStream_t st) {
  if (p.d * (BF16 ? 2 : 4) / 64 <= 32) return launch_sumunit_mfma_nw<RB, PB, BF16, 4>(p, st);
  return launch_sumunit_mfma_nw<RB, PB, BF16, RB * PB <= 2 ? 16 : 8>(p, st);
}

// The same for many units over long rows in bf16: the tile machinery with Wsum as the only "slab" (r <= 128 rows), 32
// positions to a workgroup, every operand row through LDS once per workgroup, K in one chain.
template <int SB>
__global__ __launch_bounds__(128)
void k_sumunit_ring(const void* h, long long ld_h, const void* Wsum, int B, int d, int r, float* logw) {
  using TL = Tile<2, 1, 2, 1, SB, 4>;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int l31 = lane & 31, lhalf = lane >> 5;
  const int b0 = blockIdx.x * TL::TP;
  f32x16_t acc[1][2];
  tile_gemm<2, 1, 2, 1, SB, 4, true>(Wsum, d, h, ld_h, B, d, r, 0, b0, smem, acc);
  float mx[1], lse[1];
  tile_lse<2, 1, 2, 1, SB, 4>(acc, r, (float2*)(smem + TL::RED_OFF), mx, lse);
  const int b = b0 + l31;
  if (b >= B) return;
#pragma unroll
  for (int vb = 0; vb < 2; ++vb)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int row = wv * 64 + 4 * lhalf + vb * 32 + 8 * (i >> 2) + (i & 3);
      if (row < r) logw[(long long)b * r + row] = acc[0][vb][i] - lse[0];
    }
}

// (the other parameters by a launch of their own: this kernel's LDS leaves two of its workgroups to a CU, too few to copy h - r = 128,
// d = 4096, B = 8192, a one-token call 847 us instead of 836 -, and behind it, so that the copy is in the last cache when W's pass begins)
template <int SB>
static hipError_t launch_sumunit_ring(const ParamArgs& p, hipStream_t st) {
  using TL = Tile<2, 1, 2, 1, SB, 4>;
  if (hipError_t e = allow_lds<k_sumunit_ring<SB>>(TL::SMEM); e != hipSuccess) return e;
  hipLaunchKernelGGL(k_sumunit_ring<SB>, dim3((p.B + TL::TP - 1) / TL::TP), dim3(TL::NT), TL::SMEM, st, p.h, p.ld_h, p.Wsum, p.B, p.d, p.r, p.logw);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  ParamArgs rest = p;
  rest.Wsum = nullptr;
  return launch_call_params(rest, MTPC_BF16, st);
}

// 16 positions per workgroup as long as those fill the 256 CUs at most once, else 32: Wsum is then read from the
// L2s half as often.  bf16, more than 64 units, rows of more than 32 steps, and latents to be drawn: the ring above, in whose order the
// weights of a seed's drafts have always been summed.  For scores it is the slower one up to 4000 positions and little faster beyond (one-token
// calls, ring / this, r = 128: d = 4096, B = 500 79 / 73 us, 3000 329 / 326, 8192 850 / 870; d = 2048, B = 129 41 / 34, 2000 128 / 124, 8192 468 / 476;
// v = 320, B = 8000, d = 4096 1905 / 1920).
template <bool BF16>
static hipError_t launch_sumunit_mfma_dt(const ParamArgs& p, hipStream_t st) {
  const bool wide = p.B > 4096;
  const int r = p.r;
  if (BF16 && p.draws && r > 64 && p.d > 1024) return p.d % 64 == 0 ? launch_sumunit_ring<128>(p, st) : launch_sumunit_ring<64>(p, st);
  if (r <= 16) return wide ? launch_sumunit_mfma_cfg<1, 2, BF16>(p, st) : launch_sumunit_mfma_cfg<1, 1, BF16>(p, st);
  if (r <= 32) return wide ? launch_sumunit_mfma_cfg<2, 2, BF16>(p, st) : launch_sumunit_mfma_cfg<2, 1, BF16>(p, st);
  if (r <= 64) return wide ? launch_sumunit_mfma_cfg<4, 2, BF16>(p, st) : launch_sumunit_mfma_cfg<4, 1, BF16>(p, st);
  return launch_sumunit_mfma_cfg<8, 1, BF16>(p, st);
}

hipError_t launch_params_mfma(const ParamArgs& p, int dtype, hipStream_t st) {
  return dtype == MTPC_BF16 ? launch_sumunit_mfma_dt<true>(p, st) : launch_sumunit_mfma_dt<false>(p, st);
}

// Contextual sum layers (Sec. 3.3, sum unit parameters): every sum unit (layer l,
// incoming state k) of every position gets its own weights softmax(R[l][k] h[b] +
// bias[l][k]).  The tile machinery again: a "slab" is one sum unit (r rows of R).
template <int WV, int WB, int VB, int PB, int SB, int NS, bool BF16>
__global__ __launch_bounds__(WV * WB * 64)
void k_ctx_layers(const CtxLayerArgs a) {
  using TL = Tile<WV, WB, VB, PB, SB, NS>;
  constexpr int ESZ = BF16 ? 2 : 4;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wv = wave % WV, wb = wave / WV;
  const int l31 = lane & 31, lhalf = lane >> 5;
  const int nslab = a.L * a.r;
  const int nbt = (a.B + TL::TP - 1) / TL::TP;
  int slab, bt;
  tile_of_block(blockIdx.x, nbt, nslab, slab, bt);
  const int b0 = bt * TL::TP;
  const int l = slab / a.r, k = slab - l * a.r;
  const char* Rlk = (const char*)a.R + ((long long)l * a.R_layer_stride + (long long)k * a.r * a.d) * ESZ;

  f32x16_t acc[PB][VB];
  tile_gemm<WV, WB, VB, PB, SB, NS, BF16>(Rlk, a.d, a.h, a.ld_h, a.B, a.d, a.r, 0, b0, smem, acc);
  const int rbase = wv * VB * 32 + 4 * lhalf;
  if (a.bias != nullptr) {
    const float* bl = a.bias + (long long)l * a.bias_layer_stride + (long long)k * a.r;
#pragma unroll
    for (int vb = 0; vb < VB; ++vb)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int row = rbase + vb * 32 + 8 * (i >> 2) + (i & 3);
        const float bv = row < a.r ? bl[row] : 0.f;
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) acc[pb][vb][i] += bv;
      }
  }
  float mx[PB], lse[PB];
  tile_lse<WV, WB, VB, PB, SB, NS>(acc, a.r, (float2*)(smem + TL::RED_OFF), mx, lse);
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) {
    const int b = b0 + wb * PB * 32 + pb * 32 + l31;
    if (b >= a.B) continue;
    const long long base = ((long long)b * a.L + l) * a.r * a.r;
#pragma unroll
    for (int vb = 0; vb < VB; ++vb)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int row = rbase + vb * 32 + 8 * (i >> 2) + (i & 3);
        if (row < a.r) {
          const float p = __expf(acc[pb][vb][i] - lse[pb]);
          if (a.out_nat) a.out_nat[base + (long long)k * a.r + row] = p;
          if (a.out_tr) a.out_tr[base + (long long)row * a.r + k] = p;
        }
      }
  }
}

// The same for r a power of two in 8..128 and natural layout only: R is taken as one
// dense [L*r*r][d] matrix cut into 256-row slabs, so no matrix-pipe row is wasted on
// padding.  A sum unit is an aligned run of r rows; in the accumulator layout those are
// whole 32-row blocks of one wave (r >= 32) or register groups of a block (r < 32) plus
// the partner lane 32 away, so its softmax needs one cross-lane exchange and no LDS.
template <int R, bool BF16>
__global__ __launch_bounds__(512)
void k_ctx_layers_dense(const CtxLayerArgs a) {
  constexpr int WV = 2, WB = 4, VB = 4, PB = 2, SB = 64, NS = 4;
  using TL = Tile<WV, WB, VB, PB, SB, NS>;
  constexpr int ESZ = BF16 ? 2 : 4;
  constexpr int UB = R >= 32 ? R / 32 : 1;          // blocks per unit
  constexpr int RG = R >= 32 ? 16 : R / 2;          // registers per unit within a block
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wv = wave % WV, wb = wave / WV;
  const int l31 = lane & 31, lhalf = lane >> 5;
  const int Mr = a.L * a.r * a.r;
  const int nslab = (Mr + TL::TV - 1) / TL::TV;
  const int nbt = (a.B + TL::TP - 1) / TL::TP;
  int slab, bt;
  tile_of_block(blockIdx.x, nbt, nslab, slab, bt);
  const int b0 = bt * TL::TP;
  const int rows = min(TL::TV, Mr - slab * TL::TV);
  f32x16_t acc[PB][VB];
  tile_gemm<WV, WB, VB, PB, SB, NS, BF16>((const char*)a.R + (long long)slab * TL::TV * a.d * ESZ, a.d, a.h,
                                          a.ld_h, a.B, a.d, rows, 0, b0, smem, acc);
  const int rbase = wv * VB * 32 + 4 * lhalf;
  if (a.bias != nullptr) {
#pragma unroll
    for (int vb = 0; vb < VB; ++vb)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int row = rbase + vb * 32 + 8 * (i >> 2) + (i & 3);
        const float bv = row < rows ? a.bias[(long long)slab * TL::TV + row] : 0.f;
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) acc[pb][vb][i] += bv;
      }
  }
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) {
    const int b = b0 + wb * PB * 32 + pb * 32 + l31;
#pragma unroll
    for (int vb0 = 0; vb0 < VB; vb0 += UB)
#pragma unroll
      for (int i0 = 0; i0 < 16; i0 += RG) {
        float m = neg_inf();
#pragma unroll
        for (int vb = vb0; vb < vb0 + UB; ++vb)
#pragma unroll
          for (int i = i0; i < i0 + RG; ++i) m = fmaxf(m, acc[pb][vb][i]);
        m = fmaxf(m, __shfl_xor(m, 32));
        float s = 0.f;
#pragma unroll
        for (int vb = vb0; vb < vb0 + UB; ++vb)
#pragma unroll
          for (int i = i0; i < i0 + RG; ++i) {
            acc[pb][vb][i] = __expf(acc[pb][vb][i] - m);
            s += acc[pb][vb][i];
          }
        s += __shfl_xor(s, 32);
        const float inv = 1.f / s;
#pragma unroll
        for (int vb = vb0; vb < vb0 + UB; ++vb)
#pragma unroll
          for (int i = i0; i < i0 + RG; ++i) acc[pb][vb][i] *= inv;
      }
    if (b < a.B) {
      float* dst = a.out_nat + (long long)b * Mr + (long long)slab * TL::TV;
#pragma unroll
      for (int vb = 0; vb < VB; ++vb)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int row = rbase + vb * 32 + 8 * q;
          if (row < rows)
            *(f32x4_t*)(dst + row) = f32x4_t{acc[pb][vb][4 * q], acc[pb][vb][4 * q + 1], acc[pb][vb][4 * q + 2],
                                             acc[pb][vb][4 * q + 3]};
        }
    }
  }
}

template <int R, bool BF16>
static hipError_t launch_ctx_dense(const CtxLayerArgs& a, hipStream_t st) {
  using TL = Tile<2, 4, 4, 2, 64, 4>;
  constexpr auto kern = k_ctx_layers_dense<R, BF16>;
  if (hipError_t e = allow_lds<kern>(TL::SMEM); e != hipSuccess) return e;
  const int Mr = a.L * a.r * a.r;
  const int nbt = (a.B + TL::TP - 1) / TL::TP, nslab = (Mr + TL::TV - 1) / TL::TV;
  hipLaunchKernelGGL(kern, dim3(nbt * nslab), dim3(TL::NT), TL::SMEM, st, a);
  return hipGetLastError();
}

template <bool BF16>
static hipError_t launch_ctx_dense_dt(const CtxLayerArgs& a, hipStream_t st) {
  switch (a.r) {
    case 8: return launch_ctx_dense<8, BF16>(a, st);
    case 16: return launch_ctx_dense<16, BF16>(a, st);
    case 32: return launch_ctx_dense<32, BF16>(a, st);
    case 64: return launch_ctx_dense<64, BF16>(a, st);
    default: return launch_ctx_dense<128, BF16>(a, st);
  }
}

template <int WV, int WB, int VB, int PB, bool BF16>
static hipError_t launch_ctx_cfg(const CtxLayerArgs& a, hipStream_t st) {
  using TL = Tile<WV, WB, VB, PB, 64, 4>;
  constexpr auto kern = k_ctx_layers<WV, WB, VB, PB, 64, 4, BF16>;
  if (hipError_t e = allow_lds<kern>(TL::SMEM); e != hipSuccess) return e;
  const int nbt = (a.B + TL::TP - 1) / TL::TP;
  hipLaunchKernelGGL(kern, dim3(nbt * a.L * a.r), dim3(TL::NT), TL::SMEM, st, a);
  return hipGetLastError();
}

hipError_t launch_ctx_layers(const CtxLayerArgs& a, int dtype, hipStream_t st) {
  const bool bf = dtype == MTPC_BF16;
  const long long rr = (long long)a.r * a.r;
  const bool pow2 = a.r >= 8 && a.r <= 128 && (a.r & (a.r - 1)) == 0;
  const bool dense_R = a.L == 1 || a.R_layer_stride == rr * a.d;
  const bool dense_bias = a.bias == nullptr || a.L == 1 || a.bias_layer_stride == rr;
  if (a.B > 64 && pow2 && dense_R && dense_bias && a.out_nat != nullptr && a.out_tr == nullptr)
    return bf ? launch_ctx_dense_dt<true>(a, st) : launch_ctx_dense_dt<false>(a, st);
  if (a.B > 64) {     // 64- or 128-row unit tiles x 256 positions
    if (a.r > 64) return bf ? launch_ctx_cfg<2, 4, 2, 2, true>(a, st) : launch_ctx_cfg<2, 4, 2, 2, false>(a, st);
    return bf ? launch_ctx_cfg<2, 4, 1, 2, true>(a, st) : launch_ctx_cfg<2, 4, 1, 2, false>(a, st);
  }
  return bf ? launch_ctx_cfg<2, 1, 2, 2, true>(a, st) : launch_ctx_cfg<2, 1, 2, 2, false>(a, st);
}

// Univariate marginals (App. B.1 with every other variable summed out):
//   M[b,i,a] = log sum_j m[b,i,j] phi[b,i,j,a],  m = marginal of the latent that
// indexes leaf i.  One workgroup owns window position i for a tile of positions
// and walks the r slabs, adding exp(l - LSE_j + log m_j) into a second register
// tile, so each slab's logits are again consumed in registers.
template <int WV, int WB, int VB, int PB, int SB, int NS, bool BF16>
__global__ __launch_bounds__(WV * WB * 64)
void k_univariate(const UnivariateArgs a) {
  using TL = Tile<WV, WB, VB, PB, SB, NS>;
  constexpr bool M16 = use_m16<WV, WB, SB, NS, BF16>();
  using FR = Frag<M16>;
  constexpr int NPB = PB * FR::SUB, NVB = VB * FR::SUB;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wv = wave % WV, wb = wave / WV;
  const int lcol = FR::lcol(lane);
  const int nbt = (a.B + TL::TP - 1) / TL::TP;
  const int wi = blockIdx.x / nbt, bt = blockIdx.x - wi * nbt;
  const int b0 = bt * TL::TP;
  const int rbase = wv * VB * 32 + 4 * FR::lgrp(lane);

  typename FR::blk_t run[NPB][NVB];
#pragma unroll
  for (int pb = 0; pb < NPB; ++pb)
#pragma unroll
    for (int vb = 0; vb < NVB; ++vb)
#pragma unroll
      for (int i = 0; i < FR::NI; ++i) run[pb][vb][i] = 0.f;

  for (int j = 0; j < a.r; ++j) {
    typename FR::blk_t acc[NPB][NVB];
    tile_gemm<WV, WB, VB, PB, SB, NS, BF16, false, M16>(a.W, a.d, a.h, a.ld_h, a.B, a.d, a.v, wi * a.r + j, b0, smem, acc);
    float mx[NPB], lse[NPB];
    tile_lse<WV, WB, VB, PB, SB, NS, M16>(acc, a.v, (float2*)(smem + TL::RED_OFF), mx, lse);
#pragma unroll
    for (int pb = 0; pb < NPB; ++pb) {
      const int b = min(b0 + wb * PB * 32 + pb * FR::BR + lcol, a.B - 1);
      const float lm = a.logm[b * a.logm_b + wi * a.logm_i + j];
      // m_j phi_j = 2^((l - lse_j + log m_j) log2 e): one fused multiply-add and one v_exp per logit
      constexpr float LOG2E = 1.4426950408889634f;
      const float shift = (lm - lse[pb]) * LOG2E;
#pragma unroll
      for (int vb = 0; vb < NVB; ++vb)
#pragma unroll
        for (int i = 0; i < FR::NI; ++i) run[pb][vb][i] += __builtin_amdgcn_exp2f(fmaf(acc[pb][vb][i], LOG2E, shift));
    }
    __syncthreads();   // `red` is rewritten by the next slab
  }
#pragma unroll
  for (int pb = 0; pb < NPB; ++pb) {
    const int b = b0 + wb * PB * 32 + pb * FR::BR + lcol;
    if (b >= a.B) continue;
    float* dst = a.out + ((long long)b * a.n + wi) * a.v;
#pragma unroll
    for (int vb = 0; vb < NVB; ++vb)
#pragma unroll
      for (int i = 0; i < FR::NI; ++i) {
        const int row = rbase + vb * FR::BR + FR::roff(i);
        if (row < a.v) dst[row] = __logf(run[pb][vb][i]);
      }
  }
}

template <int WV, int WB, int VB, int PB, int SB, int NS, bool BF16>
static hipError_t launch_uni_cfg(const UnivariateArgs& a, hipStream_t st) {
  using TL = Tile<WV, WB, VB, PB, SB, NS>;
  constexpr auto kern = k_univariate<WV, WB, VB, PB, SB, NS, BF16>;
  if (hipError_t e = allow_lds<kern>(TL::SMEM); e != hipSuccess) return e;
  const int nbt = (a.B + TL::TP - 1) / TL::TP;
  hipLaunchKernelGGL(kern, dim3(nbt * a.n), dim3(TL::NT), TL::SMEM, st, a);
  return hipGetLastError();
}

template <bool BF16>
static hipError_t launch_uni_dt(const UnivariateArgs& a, hipStream_t st) {
  if (a.B > 32) {
    if (a.v > 256) return launch_uni_cfg<2, 4, 5, 1, 64, 4, BF16>(a, st);
    if (a.v > 128) return launch_uni_cfg<2, 4, 4, 1, 64, 4, BF16>(a, st);
    return launch_uni_cfg<2, 4, 2, 1, 64, 4, BF16>(a, st);
  }
  if (a.v > 256) return launch_uni_cfg<5, 1, 2, 1, 64, 4, BF16>(a, st);
  if (a.v > 128) return launch_uni_cfg<4, 1, 2, 1, 64, 4, BF16>(a, st);
  return launch_uni_cfg<2, 1, 2, 1, 64, 4, BF16>(a, st);
}

hipError_t launch_univariate(const UnivariateArgs& a, int dtype, hipStream_t st) {
  return dtype == MTPC_BF16 ? launch_uni_dt<true>(a, st) : launch_uni_dt<false>(a, st);
}

// (of launches with one tile of positions)
static void set_first_stages(UnembedArgs& a, int row_bytes, int SB, int positions) {
  if (a.drawn || !starts_differ(row_bytes, positions)) return;
  a.first_stages = (unsigned)(row_bytes / SB);
  a.first_reciprocal = (unsigned)(((1ull << 32) + a.first_stages - 1) / a.first_stages);     // (exact below 2^32 / stages, far beyond n r)
}

template <int WV, int WB, int VB, int PB, int SB, int NS, bool BF16, bool SAMPLE, bool WPACK = false, int SPLIT = 0, int VH = 0,
          bool STREAM = false, int PH = 0, bool ROT = SPLIT == 0 && !SAMPLE && WB != 1>
static hipError_t launch_cfg(UnembedArgs a, hipStream_t st) {
  using TL = Tile<WV, WB, VB, PB, SB, NS, PH, VH>;
  constexpr auto kern = k_unembed<WV, WB, VB, PB, SB, NS, BF16, SAMPLE, WPACK, SPLIT, VH, STREAM, PH, ROT>;
  constexpr int smem = TL::SMEM + (SPLIT == 2 ? TL::ROWS * 4 : 0);
  static_assert(smem <= 160 * 1024, "LDS budget of one CU");
  if (hipError_t e = allow_lds<kern>(smem); e != hipSuccess) return e;
  const int nbt = (a.B + TL::TP - 1) / TL::TP;
  if constexpr (ROT)
    if (nbt == 1) set_first_stages(a, a.d * (BF16 ? 2 : 4), SB, TL::TP);
  int grid = nbt * a.n * a.r;
  if constexpr (unembed_walks_tiles<WB, SAMPLE>()) {
    // one workgroup per CU (the ring takes most of a CU's LDS, so no two share one), a multiple of the
    // 8 XCDs the workgroup ids are dealt over
    int cus = 0;
    if (hipError_t e = cu_count(&cus); e != hipSuccess) return e;
    if (cus >= 8) grid = std::min(grid, cus / 8 * 8);
  }
  hipLaunchKernelGGL(kern, dim3(grid), dim3(TL::NT), smem, st, a);
  return hipGetLastError();
}

// Tiles of 32 or 64 positions (WV waves over the vocabulary): decode-sized batches, whose one tile of positions
// makes W a stream bound by HBM, and products of few tiles (unembed_positions).  128-byte stages in a 3-stage ring
// when the rows allow it (whole cache lines per row and stage, 90 KB in flight per CU; 1.5-2.5 % faster than
// 64-byte stages in a 4-stage ring).
template <int WV, int PB, bool BF16, bool SAMPLE>
static hipError_t launch_dec(const UnembedArgs& a, int row_bytes, hipStream_t st) {
  static_assert(PACK_STAGE_BYTES == 128, "the stage-major copy of W is cut for the 128-byte stages");
  if (a.B > PB * 32) {
    // (the copy of W in the 64-byte stages that this batch's gathered draws read: a call that scores from W's rows
    // beside them has both in use, 2 x 146 MB at n r = 96, v = 256, d = 2976 where 256 MB are cached: draft and score, B = 126
    // 142 / 93 us)
    if (a.Wp != nullptr && a.Wp_stage == 64) return launch_cfg<WV, 1, 2, PB, 64, 4, BF16, SAMPLE, true>(a, st);
    if constexpr (BF16)                              // (fp32 rows always are of whole 128-byte stages)
      if (row_bytes % 128 != 0) return launch_cfg<WV, 1, 2, PB, 64, 4, BF16, SAMPLE>(a, st);
    return launch_cfg<WV, 1, 2, PB, 128, 3, BF16, SAMPLE>(a, st);
  }
  auto stream = [&](auto rot) {
    constexpr bool ROT = decltype(rot)::value;
    if constexpr (BF16)
      if (row_bytes % 128 != 0) return launch_cfg<WV, 1, 2, PB, 64, 4, BF16, SAMPLE, false, 0, 0, true, 0, ROT>(a, st);
    if (a.Wp != nullptr && a.Wp_stage == 128) return launch_cfg<WV, 1, 2, PB, 128, 3, BF16, SAMPLE, true, 0, 0, true, 0, ROT>(a, st);
    return launch_cfg<WV, 1, 2, PB, 128, 3, BF16, SAMPLE, false, 0, 0, true, 0, ROT>(a, st);
  };
  // (a kernel of its own: what the wrapping round takes of small calls, FF, 24 positions, d = 640, 9.6 / 9.3 us)
  if constexpr (!SAMPLE)
    if (!a.drawn && starts_differ(row_bytes, PB * 32)) return stream(std::true_type{});
  return stream(std::false_type{});
}

// Tiles of 256 (PB = 2), 192 (PB = PH = 1) or 128 positions of the fewest rows that hold the vocabulary (a K stage costs what its rows
// cost: products, loads and fragment reads alike).  The 272-row one exists for 16x16 blocks only: fp32 instructions
// fill 32.  What a narrower tile leaves of LDS goes to a fifth ring buffer.
template <bool BF16, bool SAMPLE, bool WPACK, int SPLIT = 0, int PB = 2, int PH = 0>
static hipError_t launch_train(const UnembedArgs& a, hipStream_t st) {
  constexpr int NS = PB == 1 && PH == 0 ? 5 : 4;
  // A pass that writes the table is bound by its stores where rows of W are short, and those of 16 bytes per lane leave the
  // 272-row tile more slowly (the halves of a column are in different wave groups): v = 268, n r = 960, B = 1182, with 320 / 272
  // rows 939 / 962 us at d = 448, 1178 / 1178 at d = 1024, 880 / 843 at d = 2048 (marginals over all tokens).
  const bool stores = BF16 && SPLIT == 0 && a.logphi != nullptr && a.d < 1024 && a.v < 272 && a.v % 4 == 0;
  if (a.v > 272 || (a.v > 256 && stores)) return launch_cfg<2, 4, 5, PB, 64, NS, BF16, SAMPLE, WPACK, SPLIT, 0, false, PH>(a, st);
  if (a.v > 256) return launch_cfg<2, 4, 5, PB, 64, NS, BF16, SAMPLE, WPACK, SPLIT, BF16 ? 3 : 0, false, PH>(a, st);
  if (a.v > 192) return launch_cfg<2, 4, 4, PB, 64, NS, BF16, SAMPLE, WPACK, SPLIT, 0, false, PH>(a, st);
  if (a.v > 128) return launch_cfg<2, 4, 3, PB, 64, NS, BF16, SAMPLE, WPACK, SPLIT, 0, false, PH>(a, st);
  return launch_cfg<2, 4, 2, PB, 64, NS, BF16, SAMPLE, WPACK, SPLIT, 0, false, PH>(a, st);
}

// Positions per tile of a batch beyond the decode tiles' (launches that walk their tiles, 16x16 blocks): what counts is the
// number of rounds the tiles make over the CUs, times what a round costs.  A round of 192 positions takes 0.77 to 0.87 of
// one of 256 (least at v = 320, most at v = 100), one of 128 between 0.55 and 0.74: a K stage does not shrink with its
// products (two barriers, the same rows of W).  So a narrower tile pays where it saves rounds or makes as many: up to 192 positions
// beyond a multiple of 256, or a last round that is nearly empty.  CP, d = 2048, v = 320, 256 / 192 positions: n r = 512,
// B = 300 281 / 248 us, B = 570 402 / 349; n r = 128, B = 1100 190 / 167; 5 rounds against 6 (n r = 256, B = 1100) 330 / 324 and, at
// v = 100 and d = 4096, 10 against 12 575 / 599: not taken.  n r = 96, B = 570, d = 512, two rounds of any width: 53 / 46 /
// 41 us with 128.  Of 713 sizes (B 140 .. 2000) 385 change: 0.76 to 1.01 of the time, 0.89 in the mean.  Passes that also store
// gain less and lose nowhere: of 60 such sizes (B 143 .. 1500, v 60 .. 320) marginals over all tokens, which write the table, take
// 0.86 to 1.00 of the time with 256 (0.92 in the mean), training steps, which write the probabilities, 0.96 to 1.00; scores 0.77 to 1.01.
// fp32 terms (`terms`; their ring has four buffers, so 128 positions gain nothing there): 0.87 as well up to 272 rows (n r = 256,
// B = 570, d = 2048, v = 268 697 / 583 us), 0.68 to 0.78 of the 320-row tile (854 / 657; 5 rounds against 6, B = 1100, 1202 / 1022).
static hipError_t walk_positions(const UnembedArgs& a, bool terms, int& positions) {
  int cus = 0;
  if (hipError_t e = cu_count(&cus); e != hipSuccess) return e;
  const int width[3] = {256, 192, 128}, cost[3] = {100, terms && a.v > 272 ? 74 : 87, 74};
  long long least = 0;
  for (int k = 0; k < (terms ? 2 : 3); ++k) {
    const long long tiles = (long long)a.n * a.r * ((a.B + width[k] - 1) / width[k]);
    const long long c = (tiles + cus - 1) / cus * cost[k];
    if (k == 0 || c < least) { least = c; positions = width[k]; }
  }
  return hipSuccess;
}

template <bool BF16, bool SAMPLE>
static hipError_t launch_dt(const UnembedArgs& a, hipStream_t st) {
  // Vocabulary tile: 5 blocks of 32 per wave pair covers v <= 320; smaller v take
  // narrower tiles.  Positions: see unembed_positions.
  const int row_bytes = a.d * (BF16 ? 2 : 4);
  int positions = unembed_positions(a.B, a.n, a.r, BF16 ? MTPC_BF16 : MTPC_F32);
  // Tiles of 64 positions draw 16 of them at a time (tile_draws), with two waves where v <= 128; those of 128 draw all at
  // once (tile_draws_cols): 33 / 13 us for 711 positions of n = 12, r = 1, v = 29, d = 64, 46 / 28 us at d = 2048 (256 positions:
  // 21, 43; larger v 27 / 18 to 49 / 46; in fp32 128 positions draw 16 at a time too).
  if (SAMPLE && BF16 && positions == 64 && a.B > 64 && a.v <= 128) positions = 128;
  if (positions >= 128) {
    const bool packed = a.Wp != nullptr && a.Wp_stage == 64;        // the copy of W in the 64-byte stages of these tiles
    if constexpr (BF16 && !SAMPLE) {
      if (positions == 256)
        if (hipError_t e = walk_positions(a, false, positions); e != hipSuccess) return e;
      if (positions == 192) return packed ? launch_train<BF16, SAMPLE, true, 0, 1, 1>(a, st) : launch_train<BF16, SAMPLE, false, 0, 1, 1>(a, st);
    }
    if (positions == 256) return packed ? launch_train<BF16, SAMPLE, true>(a, st) : launch_train<BF16, SAMPLE, false>(a, st);
    return packed ? launch_train<BF16, SAMPLE, true, 0, 1>(a, st) : launch_train<BF16, SAMPLE, false, 0, 1>(a, st);
  }
  if (positions == 64) {
    if (a.v > 256) return launch_dec<5, 2, BF16, SAMPLE>(a, row_bytes, st);
    if (a.v > 128) return launch_dec<4, 2, BF16, SAMPLE>(a, row_bytes, st);
    return launch_dec<2, 2, BF16, SAMPLE>(a, row_bytes, st);
  }
  if (a.v > 256) return launch_dec<5, 1, BF16, SAMPLE>(a, row_bytes, st);
  if (a.v > 128) return launch_dec<4, 1, BF16, SAMPLE>(a, row_bytes, st);
  return launch_dec<2, 1, BF16, SAMPLE>(a, row_bytes, st);
}

// Stage-major copy of a matrix: one thread moves 16 bytes; a workgroup's reads cover 256 / (SB / 16) rows of
// one stage (SB contiguous bytes each), its writes one contiguous run.
__global__ __launch_bounds__(256) void k_pack_rows(const char* __restrict__ src, char* __restrict__ dst, long long slabs, int v,
                                                   int row_bytes, long long row_stride, int stage_bytes) {
  const int cps = stage_bytes / 16;
  const long long per_slab = (long long)v * row_bytes / 16;            // 16-byte chunks of a slab
  const long long t = (long long)blockIdx.x * 256 + threadIdx.x;       // chunk index in the packed order
  if (t >= slabs * per_slab) return;
  const long long slab = t / per_slab, u = t - slab * per_slab;
  const int stage = (int)(u / ((long long)v * cps)), w = (int)(u - (long long)stage * v * cps);
  const int row = w / cps, ch = w - row * cps;
  const i32x4_t x = *(const i32x4_t*)(src + (slab * v + row) * row_stride + (long long)stage * stage_bytes + ch * 16);
  *(i32x4_t*)(dst + t * 16) = x;
}

hipError_t launch_pack_rows(const void* src, void* dst, long long slabs, int v, int row_bytes, long long row_stride,
                            int stage_bytes, hipStream_t st) {
  const long long chunks = slabs * v * (row_bytes / 16);
  hipLaunchKernelGGL(k_pack_rows, dim3((unsigned)((chunks + 255) / 256)), dim3(256), 0, st, (const char*)src, (char*)dst,
                     slabs, v, row_bytes, row_stride, stage_bytes);
  return hipGetLastError();
}

// fp32 rows as planes of two fp16 terms (split2), stage-major: per matrix [2 d/32][v][64 bytes], stage 2k+p holding term p of
// columns 32k..32k+31 times 2^-E, E the exponent of the row (split_exp of its largest finite value), left in exps.
// A workgroup takes eight rows, a thread eight neighbouring columns at a time: four threads read one 128-byte line and write
// 64 contiguous bytes of each plane, eight rows of a stage follow each other.  Rows of up to 4096 columns stay in registers
// between the search for their largest value and the split, so the matrix is read once: 843 MB to as many of planes in 0.34 ms
// (4.9 TB/s); a row at a time per thread quad and three planes took 0.43 ms.
// Raises SPLIT_WHOLE for values beyond SPLIT_LARGE, and SPLIT_WIDE for infinite and NaN ones.  guard: SPLIT_WIDE also when the
// terms may do a row less than justice: a value below SPLIT_SMALL is small beside its row's largest, which matters where much of the row is - one outlier - and not where a
// few values happen to be near 0: more than one in 16 of those that are not 0 (of a row with few of them, any).
// first: raises SPLIT_STOP beside SPLIT_WIDE.  skip: a caller that has no use for the planes of one matrix where another is
// SPLIT_WIDE; nothing is done where the launch before has found that, and little more than the reads where this one does.
// cols: the same counts for every column of the matrix, added up over its rows (for a product whose K runs down the rows).
constexpr int SPLIT_ROWS = 8, SPLIT_KEEP = 8;        // rows of a workgroup, steps of 512 columns kept in registers
// (four waves to a SIMD, so that two workgroups share a CU: with one, the same reads take a quarter longer)
__global__ __launch_bounds__(512, 4) void k_split_rows(const char* __restrict__ src, char* __restrict__ dst, int v, int d,
                                                    long long row_stride, int* __restrict__ exps, int* flag, int guard,
                                                    long long dst_rows, int rows1, const char* __restrict__ src2, int rows2, int first, int skip, int* cols) {
  if (skip && (*flag & SPLIT_STOP) != 0) return;     // (raised by launches before this one only: the same for every wave)
  __shared__ unsigned s_max[8][SPLIT_ROWS];
  __shared__ int s_small[8][SPLIT_ROWS], s_zero[8][SPLIT_ROWS], s_stop;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int rblocks = (v + SPLIT_ROWS - 1) / SPLIT_ROWS;
  const int slab = blockIdx.x / rblocks, rl = (tid >> 2) & (SPLIT_ROWS - 1);
  const int row = (blockIdx.x - slab * rblocks) * SPLIT_ROWS + rl, ch = tid & 3, sub = tid >> 5;
  const bool live = row < v, second = row >= rows1, read = live && (!second || row - rows1 < rows2);
  const char* s = (second ? src2 : src) + ((long long)slab * v + (!read ? 0 : second ? row - rows1 : row)) * row_stride + ch * 32;
  // stages 2k and 2k + 1 of this thread's 16 bytes
  const long long srow = dst_rows > 0 ? dst_rows : v;
  char* const out = dst + ((dst_rows > 0 ? (long long)slab * v : (long long)slab * 2 * (d / 32) * v) + row) * 64 + ch * 16;
  const int stages = d / 32;
  f32x4_t x[SPLIT_KEEP][2];
#pragma unroll
  for (int it = 0; it < SPLIT_KEEP; ++it) {
    const int k = it * 16 + sub;
    x[it][0] = x[it][1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    if (read && k < stages) {
      x[it][0] = __builtin_nontemporal_load((const f32x4_t*)(s + (long long)k * 128));
      x[it][1] = __builtin_nontemporal_load((const f32x4_t*)(s + (long long)k * 128 + 16));
    }
  }
  unsigned m = 0;                                    // largest finite magnitude, as bits
  bool odd = false;                                  // a value that is infinite or NaN
  auto look = [&](const f32x4_t& y) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const unsigned u = __float_as_uint(y[c]) & 0x7fffffffu;
      odd |= u >= 0x7f800000u;
      m = max(m, u < 0x7f800000u ? u : 0u);
    }
  };
#pragma unroll
  for (int it = 0; it < SPLIT_KEEP; ++it) { look(x[it][0]); look(x[it][1]); }
  for (int k = SPLIT_KEEP * 16 + sub; read && k < stages; k += 16) {
    look(*(const f32x4_t*)(s + (long long)k * 128));
    look(*(const f32x4_t*)(s + (long long)k * 128 + 16));
  }
  // the threads of a row: lanes that differ in bits 0, 1 and 5, all eight waves
  auto over = [&](unsigned y, int bit) { return (unsigned)__shfl_xor((int)y, bit); };
  m = max(m, over(m, 1)); m = max(m, over(m, 2)); m = max(m, over(m, 32));
  if ((lane & 35) == 0) s_max[wave][rl] = m;
  if (tid == 0) s_stop = skip ? __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & SPLIT_WIDE : 0;
  __syncthreads();
  if (s_stop != 0) return;
#pragma unroll
  for (int w = 0; w < 8; ++w) m = max(m, s_max[w][rl]);
  const int E = split_exp(__uint_as_float(m));
  int small = 0;                                     // (with those that are 0)
  unsigned hit = 0;                                  // steps with any (the last bit: of those beyond SPLIT_KEEP)
  auto put = [&](const f32x4_t& y0, const f32x4_t& y1, int k, int it) {
    const int before = small;
    if (!live || k >= stages) return;
    struct alignas(16) Oct { unsigned short v[8]; } o[2];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const float y = __builtin_amdgcn_ldexpf(c < 4 ? y0[c & 3] : y1[c & 3], -E);
      small += fabsf(y) < SPLIT_SMALL;
      unsigned short q[2];
      split2(y, q);
      o[0].v[c] = q[0]; o[1].v[c] = q[1];
    }
    hit |= small != before ? 1u << it : 0u;
#pragma unroll
    for (int p = 0; p < 2; ++p)
      *(Oct*)(out + (2LL * k + p) * srow * 64) = o[p];
  };
#pragma unroll
  for (int it = 0; it < SPLIT_KEEP; ++it) put(x[it][0], x[it][1], it * 16 + sub, it);
  const f32x4_t zeros = f32x4_t{0.f, 0.f, 0.f, 0.f};
  for (int k = SPLIT_KEEP * 16 + sub; live && k < stages; k += 16)
    put(read ? *(const f32x4_t*)(s + (long long)k * 128) : zeros, read ? *(const f32x4_t*)(s + (long long)k * 128 + 16) : zeros, k, SPLIT_KEEP);
  int raise = odd ? SPLIT_WIDE | SPLIT_WHOLE : 0;
  if (cols != nullptr) {                             // (reads the few stages with small values or zeros once more)
    // the lanes of a column: those of the eight rows
    const unsigned long long mine = 0x11111111ull << ((lane & 32) + (lane & 3));
    unsigned todo = hit;
    for (int o = 1; o < 64; o <<= 1) todo |= (unsigned)__shfl_xor((int)todo, o);
    while (todo != 0) {
      const int it = __builtin_ctz(todo);
      todo &= todo - 1;
      for (int k = it * 16 + sub; k < (it < SPLIT_KEEP ? min(stages, it * 16 + 16) : stages); k += 16) {
        const f32x4_t y[2] = {read ? *(const f32x4_t*)(s + (long long)k * 128) : zeros, read ? *(const f32x4_t*)(s + (long long)k * 128 + 16) : zeros};
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          const bool none = live && y[c >> 2][c & 3] == 0.f;
          const bool little = live && !none && fabsf(__builtin_amdgcn_ldexpf(y[c >> 2][c & 3], -E)) < SPLIT_SMALL;
          const int nl = __popcll(__ballot(little) & mine), nz = __popcll(__ballot(none) & mine), at = k * 32 + ch * 8 + c;
          if (rl == 0 && nl > 0) atomicAdd(cols + at, nl);
          if (rl == 0 && nz > 0) atomicAdd(cols + d + at, nz);
        }
      }
    }
  }
  if (guard) {
    auto sum = [&](int y) { y += __shfl_xor(y, 1); y += __shfl_xor(y, 2); return y + __shfl_xor(y, 32); };
    small = sum(small);
    if ((lane & 35) == 0) s_small[wave][rl] = small;
    __syncthreads();
    small = 0;
#pragma unroll
    for (int w = 0; w < 8; ++w) small += s_small[w][rl];
    // (up to one in 16 of all, zeros included: no zeros make that more than one in 16 of the others)
    if (__syncthreads_or(live && small > d / 16)) {
      int zero = 0;
      for (int k = sub; live && k < stages; k += 16)
#pragma unroll
        for (int c = 0; c < 8; ++c) zero += !read || *(const float*)(s + (long long)k * 128 + c * 4) == 0.f;
      zero = sum(zero);
      if ((lane & 35) == 0) s_zero[wave][rl] = zero;
      __syncthreads();
      zero = 0;
#pragma unroll
      for (int w = 0; w < 8; ++w) zero += s_zero[w][rl];
      if (ch == 0 && sub == 0 && small - zero > (d - zero) / 16) raise |= SPLIT_WIDE;
    }
  }
  if (live && ch == 0 && sub == 0) {
    exps[(long long)slab * v + row] = E;
    if (__uint_as_float(m) > SPLIT_LARGE) raise |= SPLIT_WHOLE;
  }
  if (live) raise_flag(flag, first && (raise & SPLIT_WIDE) ? raise | SPLIT_STOP : raise);
}

hipError_t launch_split_rows(const void* src, void* dst, long long slabs, int v, int d, long long row_stride, int* exps,
                             int* flag, int guard, hipStream_t st, long long dst_rows, int rows1, const void* src2, int rows2, int first, int skip, int* cols) {
  const long long blocks = slabs * ((v + SPLIT_ROWS - 1) / SPLIT_ROWS);
  hipLaunchKernelGGL(k_split_rows, dim3((unsigned)blocks), dim3(512), 0, st, (const char*)src, (char*)dst, v, d, row_stride, exps,
                     flag, guard, dst_rows, rows1, (const char*)src2, rows2, first, skip, cols);
  return hipGetLastError();
}

// Planes of three bf16 terms: one thread splits 8 columns; four threads read one 128-byte line and write 64 contiguous bytes of
// each plane, neighbouring rows follow (843 MB of W in 0.43 ms, 4.9 TB/s).  Raises SPLIT_WHOLE (a matrix that k_split_rows has skipped
// is seen here first).
__global__ __launch_bounds__(256) void k_split3(const Split3Job j0, const Split3Job j1, int* flag, int whole) {
  const int now = __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if ((now & SPLIT_WIDE) == 0 || (!whole && (now & SPLIT_WHOLE) != 0)) return;
  const bool done = whole && (now & (SPLIT_DONE | SPLIT_UNDONE)) == SPLIT_DONE;       // (not raised by launches with `whole`)
  bool large = false;
  for (int g = 0; g < 2; ++g) {
    const Split3Job& j = g == 0 ? j0 : j1;
    const int row0 = done ? j.done_rows : 0, nrows = j.v - row0;
    const long long per_slab = (long long)nrows * (j.d / 8), total = j.slabs * per_slab;
    const long long srow = j.dst_rows > 0 ? j.dst_rows : j.v;
    for (long long t = (long long)blockIdx.x * 256 + threadIdx.x; t < total; t += (long long)gridDim.x * 256) {
      const long long slab = t / per_slab;
      const int u = (int)(t - slab * per_slab);
      const int k = u / (nrows * 4), w = u - k * nrows * 4, row = row0 + (w >> 2), ch = w & 3;
      const bool second = row >= j.rows1;
      f32x4_t x[2] = {f32x4_t{0.f, 0.f, 0.f, 0.f}, f32x4_t{0.f, 0.f, 0.f, 0.f}};
      if (!second || row - j.rows1 < j.rows2) {
        const char* s = (second ? (const char*)j.src2 + (long long)(row - j.rows1) * j.row_stride : (const char*)j.src + (slab * j.v + row) * j.row_stride) +
                        (long long)k * 128 + ch * 32;
        x[0] = __builtin_nontemporal_load((const f32x4_t*)s);
        x[1] = __builtin_nontemporal_load((const f32x4_t*)(s + 16));
      }
      struct alignas(16) Oct { unsigned short v[8]; } o[3];
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        unsigned short q[3];
        split3(x[c >> 2][c & 3], q);
        large |= !(fabsf(x[c >> 2][c & 3]) <= SPLIT_LARGE);
#pragma unroll
        for (int p = 0; p < 3; ++p) o[p].v[c] = q[p];
      }
      char* const out = (char*)j.dst + ((j.dst_rows > 0 ? slab * j.v : slab * 3 * (j.d / 32) * j.v) + row) * 64 + ch * 16;
#pragma unroll
      for (int p = 0; p < 3; ++p) *(Oct*)(out + (3LL * k + p) * srow * 64) = o[p];
    }
  }
  if (large) raise_flag(flag, whole ? SPLIT_WHOLE : SPLIT_WHOLE | SPLIT_UNDONE);
  if (!whole && threadIdx.x == 0) raise_flag(flag, SPLIT_DONE);
}

hipError_t launch_split3(const Split3Job& j0, const Split3Job& j1, int* flag, int whole, hipStream_t st) {
  const long long chunks = std::max(j0.slabs * j0.v * (j0.d / 8), j1.slabs * j1.v * (j1.d / 8));
  // (at most eight workgroups per CU, which walk: mostly there is nothing to do, and many would take long to say so)
  hipLaunchKernelGGL(k_split3, dim3((unsigned)std::min((chunks + 255) / 256, 2048LL)), dim3(256), 0, st, j0, j1, flag, whole);
  return hipGetLastError();
}

// fp32 operands through their fp16 terms.  Operands that those would not do justice go through three bf16 terms, which cost
// 1.7 times as much (see tile_gemm_run_split), and what those cannot take stays with the fp32 instruction: which of the
// three launches does the work is known on the device only, the others' workgroups leave at once (2 to 3 us each, as the split
// into bf16 terms that is not needed).
static hipError_t launch_split(const UnembedArgs& a0, hipStream_t st) {
  UnembedArgs a = a0;
  const long long slabs = (long long)a.n * a.r;
  if (a.Wexp == nullptr) a.Wexp = plane_exps(a.Wq, slabs * a.v * a.d);
  hipError_t e = launch_split_rows(a.h, a.hq, 1, a.B, a.d, a.ld_h * 4, plane_exps(a.hq, (long long)a.B * a.d), a.wild, 1, st, 0, 0x7fffffff,
                                   nullptr, 0, a.three, 0);
  if (e == hipSuccess) e = launch_split_rows(a.W, a.Wq, slabs, a.v, a.d, a.d * 4LL, a.Wexp, a.wild, 1, st, a.Wq_rows, 0x7fffffff, nullptr, 0, 0, a.three, a.cols);
  if (e == hipSuccess && a.three) {
    const Split3Job jh{a.h, a.hq, 1, a.B, a.d, a.ld_h * 4LL, 0, 0x7fffffff, nullptr, 0, 0};
    const Split3Job jw{a.W, a.Wq, slabs, a.v, a.d, a.d * 4LL, a.Wq_rows, 0x7fffffff, nullptr, 0, 0};
    e = launch_split3(jh, jw, a.wild, 0, st);
  }
  int positions = 256;
  if (e == hipSuccess) e = walk_positions(a, true, positions);
  if (e == hipSuccess)
    e = positions == 192 ? launch_train<true, false, true, 2, 1, 1>(a, st) : launch_train<true, false, true, 2>(a, st);
  if (e == hipSuccess && a.three) e = launch_train<true, false, true, 3>(a, st);
  return e != hipSuccess ? e : launch_dt<false, false>(a, st);
}

// ---- calls of few tiles --------------------------------------------------------------------------------------
// A call whose tiles all run at once is bound by its launches, by the latency of its loads and, in fp32, by the products of the CUs that
// it uses.  So the workgroups behind those of the slabs compute what else the circuit needs, in the same launch: a tile of sum
// units is a slab of r rows whose normalised logits are all kept, and of the layers a wave takes a row.  fp32 takes 16 positions
// to a tile, half of the narrowest tile of k_unembed, on twice the CUs.
// WV waves of 32 vocabulary rows each, 16 NPB positions; plain ring, as in tile_gemm_run.
// (Operands straight into registers cost four times the loads' time: the four lanes that a load serves at once
// are then in four rows, 63 cycles for 1 KB.)
template <bool BF16, int WV, int RB, int NPB, int SB, int NS, bool STREAM>
__global__ __launch_bounds__(WV * 64)
void k_unembed_few(const UnembedArgs a, const ParamArgs p) {
  constexpr int PB = NPB / 2, PH = NPB % 2;
  using TL = Tile<WV, 1, RB / 2, PB, SB, NS, PH>;
  constexpr int ESZ = BF16 ? 2 : 4;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int l15 = lane & 15, lq = lane >> 4;
  const int nbt = (a.B + TL::TP - 1) / TL::TP, ntiles = a.n * a.r * nbt, nsum = p.Wsum != nullptr ? nbt : 0;
  const int w = blockIdx.x;
  if (w >= ntiles + nsum) {
    const long long row = (long long)(w - ntiles - nsum) * WV + wave;
    if (row < (long long)p.nb * p.L * p.r) normalise_layer_row(p.logits, p.layer_stride, p.batch_stride, row, p.L, p.r, p.out_nat, p.out_tr);
    return;
  }
  const bool sum = w >= ntiles;                      // workgroup-uniform
  int slab = 0, bt = w - ntiles;
  if (!sum) tile_of_block(w, nbt, a.n * a.r, slab, bt);
  const int b0 = bt * TL::TP, rows = sum ? p.r : a.v;
  const int wi = slab / a.r, wj = slab - wi * a.r;
  const int KI = a.d * ESZ / SB;
  TileFeed<WV, 1, RB / 2, PB, SB, NS, BF16, false, true, false, STREAM, PH, 0, 0, 0, STREAM> feed;
  // (one tile of positions: slabs from different stages on, and W as a stream, as in k_unembed)
  feed.open(sum ? p.Wsum : a.W, a.d, a.h, a.ld_h, a.B, a.d, rows, slab, b0, smem, nullptr, 0, 1, nullptr, 0, 0,
            STREAM ? first_stage(slab, a.first_stages, a.first_reciprocal) : 0);
  // this lane's target of the first windows: fetched while nothing depends on it
  const int T = sum || a.targets == nullptr ? 0 : a.T, TT = T == 0 ? 0 : T + a.T2;
  auto target = [&](int b, int t) {
    return t < T ? a.targets[((long long)b * T + t) * a.n + wi] : a.targets2[((long long)b * a.T2 + (t - T)) * a.n + wi];
  };
  int x0[NPB];
#pragma unroll
  for (int pb = 0; pb < NPB; ++pb) {
    const int b = b0 + pb * 16 + l15;
    x0[pb] = TT > 0 && b < a.B ? target(b, 0) : -1;
  }
  f32x4_t acc[NPB][RB];
#pragma unroll
  for (int pb = 0; pb < NPB; ++pb)
#pragma unroll
    for (int i = 0; i < RB; ++i) acc[pb][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  // chunk 4 ks + lq of a row lies at ^ (64 ks)
  const int row0 = wave * RB * 16;
  const int sw = swz16<TL::CPR>(l15);
  const int a_off = (row0 + l15) * SB + ((lq ^ sw) << 4), b_off = (TL::TV + l15) * SB + ((lq ^ sw) << 4);
  const bool busy = row0 < rows;                     // wave-uniform
  auto stage = [&](int it) {
    const char* const cur = smem + (it % NS) * TL::STAGE;
    i32x4_t fa[SB / 64][RB], fb[SB / 64][NPB];
#pragma unroll
    for (int ks = 0; ks < SB / 64; ++ks) {
#pragma unroll
      for (int pb = 0; pb < NPB; ++pb) fb[ks][pb] = *(const i32x4_t*)(cur + ((b_off + pb * 16 * SB) ^ (ks * 64)));
#pragma unroll
      for (int i = 0; i < RB; ++i) fa[ks][i] = *(const i32x4_t*)(cur + ((a_off + i * 16 * SB) ^ (ks * 64)));
    }
#pragma unroll
    for (int ks = 0; ks < SB / 64; ++ks) {
      if constexpr (BF16) {
#pragma unroll
        for (int pb = 0; pb < NPB; ++pb)
#pragma unroll
          for (int i = 0; i < RB; ++i) mma_step<true>(acc[pb][i], fa[ks][i], fb[ks][pb]);
      } else {
        // lane group lq holds columns 4 lq .. 4 lq + 3 of both operands: product t takes one of each
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int pb = 0; pb < NPB; ++pb)
#pragma unroll
            for (int i = 0; i < RB; ++i)
              acc[pb][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(f32x4_t, fa[ks][i])[t],
                                                                __builtin_bit_cast(f32x4_t, fb[ks][pb])[t], acc[pb][i], 0, 0, 0);
      }
    }
  };
  const int KM = max(KI - (NS - 1), 0);              // iterations that still issue a stage
  int it = 0;
  for (; it < KM; ++it) {
    MTPC_WAIT_VMCNT((NS - 2) * TL::PER);
    __syncthreads();                                 // stage `it` landed everywhere, nobody reads stage it-1 any more
    feed.issue((it + NS - 1) % NS);
    if (busy) stage(it);
  }
  for (; it < KI; ++it) {
    MTPC_WAIT_VMCNT(0);
    __syncthreads();
    if (busy) stage(it);
  }
  // softmax statistics of the columns: this lane holds rows rbase + 16 i + t of column 16 pb + l15
  const int rbase = row0 + 4 * lq;
  constexpr float LOG2E = 1.4426950408889634f;
  float2* const red = (float2*)(smem + TL::RED_OFF); // [WV][TP]
  float lse[NPB];
#pragma unroll
  for (int pb = 0; pb < NPB; ++pb) {
    float m = neg_inf(), s = 0.f;
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (rbase + i * 16 + t < rows) m = fmaxf(m, acc[pb][i][t]);
    m = Frag<true>::across(m, [](float x, float y) { return fmaxf(x, y); });
    const float ms2 = m == neg_inf() ? 0.f : -m * LOG2E;
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (rbase + i * 16 + t < rows) s += __builtin_amdgcn_exp2f(fmaf(acc[pb][i][t], LOG2E, ms2));
    s = Frag<true>::across(s, [](float x, float y) { return x + y; });
    if (lq == 0) red[wave * TL::TP + pb * 16 + l15] = make_float2(m, s);
  }
  __syncthreads();
#pragma unroll
  for (int pb = 0; pb < NPB; ++pb) {
    float M = neg_inf(), Z = 0.f;
#pragma unroll
    for (int q = 0; q < WV; ++q) M = fmaxf(M, red[q * TL::TP + pb * 16 + l15].x);
#pragma unroll
    for (int q = 0; q < WV; ++q) {
      const float2 y = red[q * TL::TP + pb * 16 + l15];
      if (y.y > 0.f) Z += y.y * __expf(y.x - M);
    }
    lse[pb] = M + __logf(Z);
  }
#pragma unroll
  for (int pb = 0; pb < NPB; ++pb) {
    const int b = b0 + pb * 16 + l15;
    if (b >= a.B) continue;
    if (sum) {
#pragma unroll
      for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if (rbase + i * 16 + t < rows) p.logw[(long long)b * p.r + rbase + i * 16 + t] = acc[pb][i][t] - lse[pb];
      continue;
    }
    for (int t = 0; t < TT; ++t) {
      const int x = t == 0 ? x0[pb] : target(b, t);
      float* const dst = a.e + (((long long)b * TT + t) * a.n + wi) * a.r + wj;
      if (x < 0 || x >= a.v) {
        if (threadIdx.x < 16) *dst = x == -1 ? 0.f : __builtin_nanf("");
      } else {
        const int xr = x - rbase;
        if (xr >= 0 && xr < RB * 16 && (xr & 12) == 0) {
          const bool t0 = xr & 1, t1 = xr & 2;
          float y = 0.f;
#pragma unroll
          for (int i = 0; i < RB; ++i) {
            const float c0 = t0 ? acc[pb][i][1] : acc[pb][i][0], c1 = t0 ? acc[pb][i][3] : acc[pb][i][2];
            y = (xr >> 4) == i ? (t1 ? c1 : c0) : y;
          }
          *dst = y - lse[pb];
        }
      }
    }
    if (a.logphi != nullptr) {
      float* const dst = a.logphi + (((long long)b * a.n + wi) * a.r + wj) * a.v;
#pragma unroll
      for (int i = 0; i < RB; ++i) {
        const int row = rbase + i * 16;
        if ((a.v & 3) == 0) {
          if (row < a.v)
            *(f32x4_t*)(dst + row) = f32x4_t{acc[pb][i][0] - lse[pb], acc[pb][i][1] - lse[pb], acc[pb][i][2] - lse[pb], acc[pb][i][3] - lse[pb]};
        } else {
#pragma unroll
          for (int t = 0; t < 4; ++t)
            if (row + t < a.v) dst[row + t] = acc[pb][i][t] - lse[pb];
        }
      }
    }
  }
}

template <bool BF16, int WV, int RB, int NPB, int SB, int NS, bool STREAM = false>
static hipError_t launch_few_cfg(UnembedArgs a, const ParamArgs& p, hipStream_t st) {
  using TL = Tile<WV, 1, RB / 2, NPB / 2, SB, NS, NPB % 2>;
  const int nbt = (a.B + TL::TP - 1) / TL::TP;
  // Each slab is read once: as a stream, where W is too large for the 256 MB cache to keep much of it from one call to the next (n r =
  // 252, v = 320, B = 1, 165 MB: 37.7 / 33.7 us; 21 MB, n r = 64, B = 30, called again 18.4 / 23.6).
  if constexpr (!STREAM)
    if (nbt == 1 && (long long)a.n * a.r * a.v * a.d * (BF16 ? 2 : 4) > (128LL << 20))
      return launch_few_cfg<BF16, WV, RB, NPB, SB, NS, true>(a, p, st);
  if constexpr (STREAM) set_first_stages(a, a.d * (BF16 ? 2 : 4), SB, TL::TP);
  constexpr auto kern = k_unembed_few<BF16, WV, RB, NPB, SB, NS, STREAM>;
  if (hipError_t e = allow_lds<kern>(TL::SMEM); e != hipSuccess) return e;
  const long long lrows = (long long)p.nb * p.L * p.r;
  const long long grid = ((long long)a.n * a.r + (p.Wsum != nullptr)) * nbt + (lrows + WV - 1) / WV;
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(TL::NT), TL::SMEM, st, a, p);
  return hipGetLastError();
}

// Rows per wave: 32 in fp32, whose products then spread over the SIMDs; 64 in bf16, which reads half as many fragments of h for it.
template <bool BF16, int NPB>
static hipError_t launch_few_rows(const UnembedArgs& a, const ParamArgs& p, hipStream_t st) {
  constexpr int RB = BF16 ? 4 : 2, W = BF16 ? 1 : 2;
  const int need = std::max(a.v, p.Wsum != nullptr ? p.r : 0);
  if constexpr (BF16)                                // (d is a multiple of 32: fp32 rows always are of whole 128-byte stages)
    if (a.d % 64 != 0) return launch_few_cfg<BF16, 5 * W, RB, NPB, 64, 4>(a, p, st);
  if (need > 256) return launch_few_cfg<BF16, 5 * W, RB, NPB, 128, 3>(a, p, st);
  if (need > 128) return launch_few_cfg<BF16, 4 * W, RB, NPB, 128, 4>(a, p, st);
  return launch_few_cfg<BF16, 2 * W, RB, NPB, 128, 4>(a, p, st);
}

hipError_t launch_unembed_few(const UnembedArgs& a, const ParamArgs& p, int dtype, hipStream_t st) {
  const int tile = unembed_few(a.B, a.n, a.r, dtype);
  if (a.zleaf != nullptr || a.phiT != nullptr || a.v > 320 || p.r > 128 || tile == 0) return hipErrorInvalidValue;
  if (dtype == MTPC_F32) return tile == 16 ? launch_few_rows<false, 1>(a, p, st) : launch_few_rows<false, 2>(a, p, st);
  return tile == 16 ? launch_few_rows<true, 1>(a, p, st) : launch_few_rows<true, 2>(a, p, st);
}

hipError_t launch_unembed(const UnembedArgs& a, int dtype, hipStream_t st) {
  const bool sample = a.zleaf != nullptr;
  if (dtype == MTPC_F32 && a.Wq != nullptr) return sample ? hipErrorInvalidValue : launch_split(a, st);
  if (dtype == MTPC_BF16)
    return sample ? launch_dt<true, true>(a, st) : launch_dt<true, false>(a, st);
  return sample ? launch_dt<false, true>(a, st) : launch_dt<false, false>(a, st);
}

}  // namespace mtpc

