// Internal declarations shared by the HIP translation units of libmtpc.
// Not part of the public ABI (see include/mtpc.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "mtpc.h"

namespace mtpc {

// Arguments of the fused unembedding kernel (Sec. 3.3: phi_ij = softmax(W_ij e_t)).
// One workgroup owns ALL v logits of one (i, j) slab for a tile of positions, so
// the softmax over the vocabulary finishes in registers and only O(B n r) values
// are written.
struct UnembedArgs {
  const void* h;        // [B][ld_h]
  long long ld_h;       // elements
  const void* W;        // [n*r][v][d]
  const void* Wp;       // stage-major copy of W (mtpc_pack_weights) or nullptr, in stages of Wp_stage bytes; read
  int Wp_stage;         // instead of W by the tiles whose stages have that size: 128 bytes for B <= 64, else 64
  const void* hs;       // stage-major copy of h in 64-byte stages, [d*esz/64][B][64 bytes] (launch_pack_rows), or
                        // nullptr; read instead of h by the 256-position tiles (B > 64): a stage of a tile is then
                        // one run of 16 KB and the L2 is asked for whole 128-byte lines
  int B, d, v, n, r;
  // evidence: e[(b*T+t)][i][j] = l[x] - LSE for target window t of position b
  const int* targets;   // [B][T][n] or nullptr
  int T;
  const int* targets2;  // [B][T2][n]: a second set of windows per position (rows T..T+T2-1 of a position), or nullptr
  int T2;
  float* e;             // [B*(T+T2)][n][r]
  // sampling: token i of draft (b, s) is drawn from slab (i, zleaf[b][s][i])
  const int* zleaf;     // [B][S][n] or nullptr
  int S;
  int* drafts;          // [B][S][n]
  uint32_t seed_lo, seed_hi, offset;
  int greedy;           // 1: every draw is replaced by the most likely outcome (no random numbers)
  float* logphi;        // [B][n][r][v] normalised logits of every slab, or nullptr
  int drawn;            // tokens are drawn from logphi: sums in the order of the passes that draw
  float* phiT;          // [n*r*v][ld_phi] softmax probabilities, transposed, or nullptr (evidence kernel only)
  long long ld_phi;
  // fp32 operands of 256-position tiles, multiplied as two fp16 terms each (split_pays): scratch that
  // launch_unembed fills with the planes of W, [n*r][2 d/32][v][64 bytes], and of h, [2 d/32][B][64 bytes], the exponents of
  // their rows behind them (plane_exps), and a flag (SPLIT_*) of what the terms do not do justice (k_split_rows).  Or nullptr
  void* Wq;
  void* hq;
  int* wild;
  int* Wexp;            // where the exponents of W's rows go, [n*r*v], or nullptr: behind its planes
  int three;            // operands without SPLIT_WHOLE that are SPLIT_WIDE go through three bf16 terms, in the same scratch
  int* cols;            // counts of the columns of W (launch_split_rows), or nullptr
  int Wq_rows;          // > 0: the planes of W are ONE matrix of so many rows, [2 d/32][Wq_rows][64 bytes], slab after slab
  // the launch's own: stages of K that slabs start at in turn, or 0 (all at its beginning), and their reciprocal (first_stage)
  unsigned first_stages, first_reciprocal;
};

// What a call computes from h and the layer logits alone, before its circuit: log omega (Wsum nullptr: not wanted), the softmax of
// shared layers (L = 0: none), the stage-major copy of h (hs nullptr: none), and ints set to 0 for the launches that follow.  They do not depend
// on each other: one launch.
struct ParamArgs {
  const void* h;
  long long ld_h;
  const void* Wsum;
  int B, d, r;
  float* logw;          // [B][r]: log omega[b][:] = log_softmax(Wsum h[b])
  int draws;            // latents are drawn from log omega: its sums in one order whatever is fastest
  // softmax over the last axis of r x r logits -> linear probabilities.  logits[b*batch_stride + l*layer_stride + k*r + j];
  // out_nat[((b*L + l)*r + k)*r + j] and / or the same transposed, out_tr[((b*L + l)*r + j)*r + k] (either may be nullptr)
  const float* logits;
  long long layer_stride, batch_stride;
  int nb, L;
  float* out_nat;
  float* out_tr;
  void* hs;             // [row_bytes / 64][B][64 bytes]
  int row_bytes;        // of h
  int* clear;
  long long nclear;
};
hipError_t launch_call_params(const ParamArgs& p, int dtype, hipStream_t st);

// Univariate marginals: M[b][i][a] = log sum_j m[b][i][j] phi[b][i][j][a].
struct UnivariateArgs {
  const void* h;
  long long ld_h;
  const void* W;
  int B, d, v, n, r;
  const float* logm;    // log marginal of the latent indexing leaf i: r values at b * logm_b + i * logm_i
  long long logm_b, logm_i;
  float* out;           // [B][n][v]
};

// dWsum[j][c] = sum_b gT[j][b] hT[c][b]; gT [r][ldb], hT [d][ldb] in the dtype of h, ldb a multiple of 32
hipError_t launch_dwsum(const void* gT, const void* hT, long long ldb, int r, int d, int dtype, float* out,
                        hipStream_t st);
// The same from the table of normalised input units log phi[B][n][r][v] (a.h, a.W unused):
// M[b][i][a] = log sum_j exp(logm[b][i][j] + logphi[b][i][j][a]).
hipError_t launch_univariate_table(const UnivariateArgs& a, const float* logphi, hipStream_t st);

// Contextual sum layers: P[b][l][k][:] = softmax(R[l][k] h[b] + bias[l][k][:]) as linear
// probabilities, natural [b][l][k][j] and/or transposed [b][l][j][k] layout.
struct CtxLayerArgs {
  const void* h;
  long long ld_h;
  const void* R;          // [L][r][r][d]
  long long R_layer_stride;   // elements, 0 = shared
  const float* bias;      // [L][r][r] or nullptr
  long long bias_layer_stride;
  int B, d, r, L;         // L = layers to produce
  float* out_nat;         // [B][L][r][r] or nullptr
  float* out_tr;          // [B][L][r][r] transposed or nullptr
};
hipError_t launch_ctx_layers(const CtxLayerArgs& a, int dtype, hipStream_t st);

hipError_t launch_unembed(const UnembedArgs& a, int dtype, hipStream_t st);
// The same evidence (and table) of calls so small that all tiles of 16 or 32 positions run at once, and the sum units and layers of the
// call beside them in one launch (where unembed_few_params says so; else p is empty).  No draws, no probabilities.
hipError_t launch_unembed_few(const UnembedArgs& a, const ParamArgs& p, int dtype, hipStream_t st);
// Whether the tiles of the sum units run at once with those of W.  If not they would come after them, and take as long.
inline bool unembed_few_params(int B, int n, int r, int tile) {
  return ((long long)n * r + 1) * ((B + tile - 1LL) / tile) <= 256;
}
// Positions per tile of such a call, 0: none.  fp32, which is bound by its products, takes 16 wherever that fills no more than the 256
// CUs (B = 64, n = 4, r = 8, d = 256, v = 256 21.3 -> 13.6 us, B = 5, n = 4, r = 20, d = 3072, v = 128 119 -> 49); bf16, as wide a tile as
// that of k_unembed, gains the launches that it saves (B = 64, n = 4, r = 16, d = 256 18.7 -> 11.7, d = 4096 74.7 -> 68.0) and
// the head without sum units has none (B = 500, d = 2048: 24.6 / 26.5).  A stage-major copy of W is not read: calls from the copy through
// k_unembed are slower than these from W's own rows (bf16, n r = 248, v = 320, d = 4096, B = 1 111 / 98 us, n r = 64, B = 64 72 / 67, d = 256 21 / 10; n r =
// 192, v = 256, d = 2048, B = 32 44 / 36; 1.09 to 2.2 times as long at 99 sizes in bf16 and fp32).
inline int unembed_few(int B, int n, int r, int dtype) {
  const long long slabs = (long long)n * r;
  if (dtype == MTPC_F32) return slabs * ((B + 15LL) / 16) <= 256 ? 16 : slabs * ((B + 31LL) / 32) <= 256 ? 32 : 0;
  const int tile = B <= 16 ? 16 : 32;
  return r > 1 && unembed_few_params(B, n, r, tile) ? tile : 0;
}
// Whether slabs that are each streamed by a workgroup of their own (one tile of `positions`) start at different stages of K.  Rows of W
// lie row_bytes apart, and CUs that all walk K from 0 ask the same few memory channels at a time where that is a multiple of a
// large power of two, or next to one.  Log-likelihoods, own rows, the same beginning / different ones: n r = 512, v = 268, B = 1 and v = 320, B = 100,
// d = 2048 129 / 94 us and 162 / 143, 3072 136 / 135 and 203 / 201, 4096 175 / 174 and 256 / 248; n r = 320, v = 256, B = 64, d = 2048 99 / 78, 4096 166 / 138, 4064
// (8192 - 64 bytes) 276 / 233.  Others spread over the channels by themselves, and wrapping round only costs: v = 320, B = 40, d = 2592 224 / 241,
// 3744 0.92, B = 64, d = 3360 0.94, B = 100, d = 2240 0.93 of the speed, few more than 1.02.  Tiles of more positions, which ask for W in 64-byte halves of lines,
// gain wherever rows are of whole lines (B = 256, d = 2112 to 4096 1.04 to 1.14, B = 160 0.99 to 1.06) and lose nothing elsewhere (0.99 to 1.01).
// Rows of less than 4 KB: nothing (n r = 256, B = 1, d = 1024 39.6 us either way).
inline bool starts_differ(long long row_bytes, int positions) {
  const long long off = row_bytes % 8192;
  return row_bytes >= 4096 && (positions > 128 || row_bytes % 2048 == 0 || off <= 64 || off >= 8192 - 64);
}
// Positions per tile of the fused kernel.  A decode-sized batch is one tile (W is then read once).  Larger ones
// take 256, unless fewer are enough or the narrower tiles all run at once on the 256 CUs: a K stage of those is
// shorter, and that many CUs would stand idle.  Measured with 256 positions and with the width chosen here: FF, n = 8,
// d = 4096, B = 512 92 / 41 us, B = 4096 101 / 83 us; CP n = 4, r = 16, d = 2048, B = 250 66 / 42 us; fp32 CP n = 4, r = 8,
// d = 2048, B = 200 660 / 148 us; CP n = 16, r = 32, d = 4096, B = 100 309 / 264 us (fp32,
// d = 2048: 1249 / 678 us).
// (bf16 batches of 33 to 64 positions keep their one tile from 33 slabs on: they are bound by reading W, which two
// tiles read twice and not from its 128-byte stage-major copy - 128 slabs 107 / 114 us.)
// (Where this says 256, launches that walk their tiles choose anew among 256, 192 and 128: walk_positions, unembed.hip.)
inline int unembed_positions(int B, int n, int r, int dtype) {
  constexpr long long CUS = 256;                 // (not asked of the device: the size of a workspace follows from this, and that
                                                 // query works, and stays the same, where there is none or none is in use yet)
  const long long slabs = (long long)n * r;
  if (B <= 32) return 32;
  if (slabs * ((B + 31LL) / 32) <= CUS && (B > 64 || dtype == MTPC_F32 || slabs <= 32)) return 32;
  if (B <= 64 || slabs * ((B + 63LL) / 64) <= CUS) return 64;
  if (B <= 128 || slabs * ((B + 127LL) / 128) <= CUS) return 128;
  return 256;
}
// dst[slab][stage][row][stage_bytes] = the stage_bytes of row `row` of slab `slab` of W that K stage `stage` covers
// Stage-major copy of `slabs` matrices of v rows (row_bytes used bytes, row_stride bytes apart): per matrix
// [row_bytes / stage_bytes][v][stage_bytes].  W for the decode tiles (128-byte stages), h for the
// 256-position tiles (one matrix, 64-byte stages).
hipError_t launch_pack_rows(const void* src, void* dst, long long slabs, int v, int row_bytes, long long row_stride,
                            int stage_bytes, hipStream_t st);
constexpr int H_STAGE_BYTES = 64;
constexpr int PACK_STAGE_BYTES = 128;
hipError_t launch_univariate(const UnivariateArgs& a, int dtype, hipStream_t st);

// Flag bits of operands that are multiplied as terms.  WIDE: a row holds values too far apart for two fp16 terms.  WHOLE: a
// value is beyond SPLIT_LARGE, where sums of products of bf16 terms may overflow.  Infinite and NaN values are both.
// STOP: beside WIDE, where only launches after the one that raises it look at it.  DONE: the planes of three terms have been written
// for a forward pass; UNDONE: not all of them, since that raised WHOLE.
constexpr int SPLIT_WIDE = 1, SPLIT_WHOLE = 2, SPLIT_STOP = 4, SPLIT_DONE = 8, SPLIT_UNDONE = 16;
// Exponents of the rows of a matrix (W, h or its transpose) stored as planes of two fp16 terms of `elements` values: right behind them.  (Planes
// have room for six bytes per value in every workspace: four are those terms, six are three bf16 terms.)
inline int* plane_exps(void* planes, long long elements) { return (int*)((char*)planes + 4 * elements); }
// fp32 rows as planes of two fp16 terms (unembed.hip, k_split_rows): `slabs` matrices of v rows, each [2 d/32][v][64 bytes] or,
// with dst_rows > 0, all rows of one matrix of so many, and the exponents of all rows.  Rows from `rows1` on (one slab) are
// the `rows2` of src2 and then zeros.  cols [2][d]: incremented by the small values (SPLIT_SMALL) and the zeros of each column
hipError_t launch_split_rows(const void* src, void* dst, long long slabs, int v, int d, long long row_stride, int* exps,
                             int* flag, int guard, hipStream_t st, long long dst_rows = 0, int rows1 = 0x7fffffff,
                             const void* src2 = nullptr, int rows2 = 0, int first = 0, int skip = 0, int* cols = nullptr);
// Up to two matrices as planes of three bf16 terms (split3), the layouts as above with 3 for 2.  Forward pass (whole = 0): where *flag
// is SPLIT_WIDE alone; else (1) where it is SPLIT_WIDE, without the first done_rows rows that a forward pass has done
struct Split3Job {
  const void* src; void* dst;
  long long slabs; int v, d; long long row_stride, dst_rows;
  int rows1; const void* src2; int rows2;
  int done_rows;
};
hipError_t launch_split3(const Split3Job& j0, const Split3Job& j1, int* flag, int whole, hipStream_t st);

// ---- small kernels (circuits.hip) -----------------------------------------
// launch_call_params of more than SUMUNIT_SMALL_B positions with sum units (unembed.hip)
hipError_t launch_params_mfma(const ParamArgs& p, int dtype, hipStream_t st);

struct CircuitArgs {
  int family;           // mtpc_family
  int rows;             // B*T evidence rows
  int T;                // rows per position (logw / contextual layers are indexed by row / T)
  int n, r;
  float* e;             // [rows][n][r]: the evidence, or (table set) room for it
  const float* table;   // nullptr, or log phi [B][n][r][v], whose entries at the tokens x [rows][n] are the evidence
  const int* x;
  int v;
  const float* logw;    // [B][r] (nullptr for FF)
  const float* layers;  // normalised linear probabilities, HMM: [nb][L][j][j'], BTree: [nb][L][j][k] (transposed)
  const float* layers_nat;  // BTree with shared layers: the same in natural layout [L][k][j], or nullptr
  int L;                // number of stored layers (1 = homogeneous)
  int contextual;       // 1: layers has a leading position axis
  float* out;           // prefix ? [rows][n] : [rows]
  int prefix;
};
hipError_t launch_circuit(const CircuitArgs& a, hipStream_t st);

// latent draws of Alg. 1 (top-down over sum units)
struct LatentArgs {
  int family, B, S, n, r;
  const float* logw;    // [B][r]
  const float* layers;  // normalised linear, natural layout [nb][L][k][j]
  int L, contextual;
  uint32_t seed_lo, seed_hi, offset;
  int greedy;           // 1: every sum unit takes its largest weight
  int* zleaf;           // [B][S][n] state that indexes leaf i
  int* latents;         // [B][S][n_lat] or nullptr
  int* zero;            // launch_latents only: nzero ints it also sets to zero (the counters of the
  int nzero;            // bucketing that follows, which saves that a launch of its own), or nullptr
};
hipError_t launch_latents(const LatentArgs& a, hipStream_t st);
// batches up to this many positions compute their sum units one workgroup per position
constexpr int SUMUNIT_SMALL_B = 128;
// The same draws in the launch that computes log omega (B <= SUMUNIT_SMALL_B, families with sum
// units): writes logw [B][r] and the latents.  The normalised layers a.layers must be complete before it - or (sumunit_latents_layers)
// they come out of p.logits in the same launch, which draws from a copy in LDS and writes p.out_nat and p.out_tr; a.layers is not read then.
hipError_t launch_sumunit_latents(const ParamArgs& p, int dtype, const LatentArgs& a, hipStream_t st);
inline bool sumunit_latents_layers(int r, int nb, int L) { return nb == 1 && L > 0 && r <= 64 && (size_t)L * r * r * 4 <= 128 * 1024; }

// log marginal of the latent that indexes each leaf: logm[b][i][j]
struct LatentMarginalArgs {
  int family, B, n, r;
  const float* logw;
  const float* layers;  // natural layout
  int L, contextual;
  float* logm;          // [B][n][r]
};
hipError_t launch_latent_marginals(const LatentMarginalArgs& a, hipStream_t st);

// evidence of drafted tokens from the table the sampling pass wrote:
// e[(b*S+s)][i][j] = logphi[b][i][j][x] with x = drafts[b][s][i]
struct GatherArgs {
  int B, S, v, n, r;
  const int* x;         // [B][S][n]
  float* e;             // [B*S][n][r]
};
hipError_t launch_gather_table(const GatherArgs& a, const float* logphi, hipStream_t st);

// token draws of Alg. 1 from the table of normalised input units: token i of draft (b,s)
// comes from the row log phi[b][i][zleaf[b][s][i]][:]
struct DrawArgs {
  int B, S, v, n, r;
  const float* logphi;  // [B][n][r][v]
  const int* zleaf;     // [B][S][n] selected input unit of every token
  int* drafts;          // [B][S][n]
  uint32_t seed_lo, seed_hi, offset;
  int greedy;           // most likely token instead of a draw (smallest id on ties)
  int compact;          // logphi is [B*S*n][v]: one row of (unnormalised) logits per token
};
hipError_t launch_draw_table(const DrawArgs& a, hipStream_t st);

// logits of the selected input unit of every token: out[(b,s,i)][:] = W[i][zleaf[b][s][i]] h[b]
struct RowLogitArgs {
  const void* h;
  long long ld_h;
  const void* W;
  int B, S, d, v, n, r;
  const int* zleaf;     // [B][S][n]
  float* out;           // [B*S*n][v]
};
hipError_t launch_rows_logits(const RowLogitArgs& a, int dtype, hipStream_t st);
// The same below a CP (zleaf unused): every workgroup computes the sum units of its position and draws the draft's latent by itself;
// the latents are also left in `latents` [B][S].  Where rows_latents() says so.
struct RowLatentArgs {
  const void* Wsum;
  uint32_t seed_lo, seed_hi, offset;
  int greedy;
  int* latents;
};
hipError_t launch_rows_latents(const RowLogitArgs& a, const RowLatentArgs& la, int dtype, hipStream_t st);
// As long as every workgroup has a CU to itself (draft and verification, r = 64, v = 256, n = 8, d = 1024, bf16, 64 workgroups to a
// position: B = 4 23.8 -> 21.6 us, B = 8 26.3 -> 34.0; v = 320, n = 16, B = 1 23.8 -> 22.1, B = 2 25.4 -> 34.3), and up to 64 MB
// of Wsum out of the L2s together (r = 64, d = 4096, B = 1: bf16, 84 MB, 26.2 with and without).
inline bool rows_latents(long long drafts, int d, int v, int n, int r, int dtype) {
  const long long groups = drafts * n * ((v + 31) / 32);
  return groups <= 256 && groups * r * d * (dtype == MTPC_BF16 ? 2 : 4) <= 64ll << 20;
}

// Buckets of the (b, s, i) triples by (i, selected input unit): bucket g = i*r + z holds
// list[row_off[g] .. row_off[g+1]) = the draft rows b*S+s whose token i comes from unit z
// (in no particular order), and is covered by tiles tile_off[g] .. tile_off[g+1]-1 of
// `tile` rows each.
struct BucketArgs {
  int B, S, n, r, tile;
  const int* zleaf;     // [B][S][n]
  int* count;           // [n*r] scratch
  int cleared;          // count is already zero (launch_latents did it)
  int* slot;            // [B*S*n] scratch: rank of a triple inside its bucket
  int* row_off;         // [n*r + 1]
  int* tile_off;        // [n*r + 1]
  int* tile_bucket;     // [B*S*n / tile + n*r] bucket of every tile
  int* list;            // [B*S*n]
};
hipError_t launch_buckets(const BucketArgs& a, hipStream_t st);

// token draws through the buckets: one slab per tile, h rows gathered
struct DrawGatherArgs {
  const void* h;
  long long ld_h;
  const void* W;
  const void* Wp;       // stage-major copy of W in the 64-byte stages of these tiles, or nullptr
  int B, S, d, v, n, r;
  const int* row_off;
  const int* tile_off;
  const int* tile_bucket;
  const int* list;
  int* drafts;          // [B][S][n]
  uint32_t seed_lo, seed_hi, offset;
  int greedy;
  int tile;             // rows per tile the buckets were cut into: DRAW_GATHER_TILE or (bf16) DRAW_GATHER_TILE_WIDE
};
hipError_t launch_draw_gather(const DrawGatherArgs& a, int dtype, hipStream_t st);
constexpr int DRAW_GATHER_TILE = 128;   // rows per tile of the gathered draw kernel
// ... and of its wider bf16 tile, for buckets that would leave a nearly empty last tile of 128 rows behind
// (a tile costs nearly the same whatever it holds, so what counts is the number of rounds over the CUs)
constexpr int DRAW_GATHER_TILE_WIDE = 192;
constexpr int GATHER_STAGE_BYTES = 64;  // ... and the bytes of a row it takes per stage

// Verification step of a speculative-decoding cycle (Alg. 2, acceptance loop on)
struct VerifyArgs {
  int family, B, n, r, v, mode;
  const float* logphi;  // [B][n][r][v]
  const int* drafts;    // [B][n]
  const float* prefix;  // [B][n]
  const float* p;       // [B][n+1][v]
  const float* logw;    // [B][r] (nullptr for FF, or when the kernel computes it itself, see h)
  const void* h;        // with h set (B <= SUMUNIT_SMALL_B): log omega = log_softmax(Wsum h[b]) is computed
  long long ld_h;       // by the position's own workgroup
  const void* Wsum;
  int d, bf16;
  const float* lay_nat; // normalised linear layers [nb][L][k][j]
  const float* lay_tr;  // the same transposed [nb][L][j][k] (BTree only, not where verify_rows)
  const float* raw;     // verify_rows: nullptr, or the logits of the layers, which the kernel normalises itself (no lay_nat then)
  long long raw_layer_stride, raw_batch_stride;
  int L, contextual;
  uint32_t seed_lo, seed_hi, offset;
  int* accepted;        // [B]
  int* token;           // [B]
};
hipError_t launch_verify(const VerifyArgs& a, hipStream_t st);
// Whether the verification of a few positions keeps a position's layers in LDS (k_verify_row); L: stored layers.  LDS in floats
constexpr int VERIFY_ROW_THREADS = 1024;
inline size_t verify_row_floats(int family, int n, int r, int L, int v) {
  const bool lay = family == MTPC_HMM || family == MTPC_BTREE;
  return VERIFY_ROW_THREADS * 2 + (lay ? (size_t)L * r * (r + 1) : 0) + (size_t)n * r * (lay ? 2 : 1) + n + 2 * (size_t)r + (size_t)v;
}
inline bool verify_rows(int family, int B, int n, int r, int L, int v) {
  return B <= 256 && r <= 64 && verify_row_floats(family, n, r, L > 0 ? L : 0, v) * 4 <= 152 * 1024;
}

// ---- training step (grad.hip, backward.hip) ----------------------------------
// Recompute pass: dLT[(i*r+j)*v + a][b] = Ge[b][i][j] * (1[a == x_bi] - phi[b,i,j,a]) in the
// dtype of h; columns b in [B, ldb) are written as zero.
struct GradLogitsArgs {
  const void* h; long long ld_h; const void* W;
  int B, d, v, n, r;
  const int* targets;   // [B][n]
  const float* Ge;      // [B][n][r] gradient of the loss w.r.t. the evidence
  void* dLT;            // [n*r*v][ldb]
  long long ldb;        // >= B, a multiple of 32
};
hipError_t launch_unembed_grad(const GradLogitsArgs& a, int dtype, hipStream_t st);

// Logit gradient from stored probabilities: for m = (i*r+j)*v + a < M
//   val = Ge[b][i][j] * (1[a == x_bi] - phiT[m][b]);   rows M <= m < Mx of dLT are passed through.
// Writes dLT[m][b] (m < M, b < ldb, zero for b >= B) and dL[b][m] (b < B, m < ldM, zero for m >= Mx).
struct GradPhiArgs {
  const float* phiT; long long ld_phi;
  const int* targets; const float* Ge;
  int B, n, r, v;
  long long M, Mx, ldM, ldb;
  long long dl_end;     // dL is written for m < dl_end (a multiple of 4); columns beyond belong to others
  void* dLT; void* dL;
  // 1: both are written stage-major in 64-byte stages, as the contractions read their 320-row operands:
  // rows m < M of dLT as [ldb * esz / 64][M][64 bytes] (the sum-unit rows M..Mx-1 stay where they are, behind
  // it), dL as [ldM * esz / 64][B][64 bytes] (then dl_end = ldM: every column is written here)
  int staged;
  // 1 (fp32, staged): both as planes of two fp16 terms, stages of 32 columns per term (tile_gemm_run_split):
  // dLT [2 ldb/32][M][64 bytes], dL [2 ldM/32][B][64 bytes], scaled by rows (largest_exp of rows and top).
  // The rows of dL are those of dL[b][m] 2^Wexp[m]: they meet rows of W without their scale.  Where *flag is SPLIT_WIDE: as
  // planes of three bf16 terms, 3 for 2, without scales
  int planes;
  const void* dslT;     // the sum-unit rows M..Mx-1 of dLT, [Mx - M][ldb] in the dtype of h
  int* flag;            // planes: SPLIT_*, raised for the elements
  int* top;             // planes: scratch [ldb], cleared (k_grad_exps)
  int* rows;            // planes: scratch [M], cleared
  float* most;          // planes: scratch [B], the largest |Ge| of every position (launch_live_positions)
  const unsigned* weights;      // planes: of h's rows in the planes of h^T (launch_transpose) [ldb]
  const int* cols;      // planes: counts of the columns of [W; Wsum] (launch_split_rows)
  int* Wexp;            // planes: exponents of the rows of W and, behind them, of Wsum [Mx] (launch_transpose, along_rows)
  // 1 (staged, bf16): no dL; dLT [ldb/32][ldM][64 bytes], the sum-unit rows and zeros behind the others; and rows tail_row ..
  // ldM - 1 of [W; Wsum; 0], [ldM][d], are copied to `tail`
  int rows_only;
  const void* W;
  const void* Wsum;
  int d, tail_row;
  void* tail;
};
hipError_t launch_grad_from_phi(const GradPhiArgs& a, int dtype, hipStream_t st);
// (planes) what has to come first: which positions have a gradient; and, once h^T and [W; Wsum] are split, the scales of the rows
// of both and whether the terms do
hipError_t launch_live_positions(const GradPhiArgs& a, hipStream_t st);
hipError_t launch_grad_exps(const GradPhiArgs& a, hipStream_t st);

// An operand of a contraction given along its rows: K runs down the rows, columns lie in chunks of 32 (64 bytes).  Element
// (k, 32 c + x) is at base + c * chunk + k * row + 2 x; rows from kmain (a multiple of 32) on come from `tail` instead,
// rows and chunks the same distances apart.  term (planes of fp16 terms): how far the second term lies behind the first.
struct KRows {
  const void* base;
  const void* tail;
  unsigned chunk, row, term;
  unsigned bytes, tail_bytes;
  int kmain;
};

// C[M][N] (fp32, row stride ldc; optionally split by rows over two buffers) = A[M][K] * B[N][K]^T, both operands K-contiguous
// with row strides lda / ldb (elements); K a multiple of 32 (bf16) or 16 (fp32).
struct GemmArgs {
  const void* A; long long lda; int M;
  const void* Bm; long long ldb; int N;
  const void* Bs;       // Bm stage-major, [K * esz / 64][N][64 bytes] (read instead of Bm), or nullptr
  const void* As;       // A stage-major, [K * esz / 64][As_rows][64 bytes] with As_rows >= M (read instead of A), or nullptr
  int As_rows;
  int K;
  float* C; long long ldc;
  // output rows are dealt to up to three buffers: [0, split) -> C, [split, split + n2) -> C2,
  // [split3, M) -> C3; rows in between are computed and dropped
  int split; int n2; float* C2;
  int split3; float* C3;
  // split over K (few output tiles, long K): ksplit > 1 workgroups per tile each take kchunk
  // columns and write their partial tile to partial[ks][M][ldc]; a second kernel adds the
  // partials in a fixed order into C (single output buffer only)
  int ksplit; int kchunk; float* partial;
  int planes;           // fp32 only: As and Bs hold two fp16 terms per value, [2 K/32][rows][64 bytes]
  const int* Atop;      // ... and these the largest elements of A's rows (largest_exp), and the exponents of B's (nullptr: 0)
  const int* Be;
  const int* flag;      // planes: where SPLIT_WIDE is set they are three bf16 terms, 3 for 2 (in Bk.chunk as well), without exponents
  // operands given along their rows instead, their K rows of M and N columns: both (bf16), or the second one beside A's planes.
  // base nullptr: as above
  KRows Ak, Bk;
};
hipError_t launch_gemm_tn(const GemmArgs& a, int dtype, hipStream_t st);
// After two products of planes: where *flag is SPLIT_WIDE and SPLIT_WHOLE, forms every result that is not finite anew as an fp32
// sum of the whole values (see split3).  Single output buffer C only.
hipError_t launch_gemm_nonfinite(const GemmArgs& a, const GemmArgs& b, const int* flag, hipStream_t st);
// number of K splits that fills the 256 CUs best for an M x N output (1: none)
inline int gemm_ksplit(int M, int N, int K) {
  const long long tiles = (long long)((M + 255) / 256) * ((N + 255) / 256);
  if (tiles >= 384) return 1;
  const int cand[] = {1, 2, 3, 4, 6, 8, 12, 16};
  int best = 1;
  double best_cost = 1e30;
  for (int ks : cand) {
    if (ks > 1 && K / ks < 2048) break;
    // rounds over the CUs, each 1/ks long, plus a little for writing and adding the partials
    const double cost = (double)((tiles * ks + 255) / 256) / ks + 0.02 * ks;
    if (cost < best_cost - 1e-9) { best_cost = cost; best = ks; }
  }
  return best;
}

// dst[c][col0 + r] = src[r][c] for r < R, c < C; dst[c][col0 + r] = 0 for R <= r < Rpad.
struct TransposeArgs {
  const void* src; long long ld_src; int R, C;
  void* dst; long long ld_dst; long long col0; int Rpad;
  // 0: dst[c][col0 + r].  Else the destination is stage-major in 64-byte stages with this many rows,
  // [columns * esz / 64][stage_rows][64 bytes] (the form the contraction kernels read an operand in)
  int stage_rows;
  // 1 (fp32, stage_rows set, col0 = 0, Rpad a multiple of 32): two fp16 terms per value, [2 columns/32][stage_rows][64 bytes]
  int planes;
  int* flag;            // planes: SPLIT_*
  // planes, the transpose: src's rows whose `live` is 0 are zeros in the planes and none of the largest values of dst's
  // rows; `weights` gets the sums of their scaled magnitudes.  Both [Rpad], 0 beyond R
  const int* live; unsigned* weights;
  // planes: rows of dst get scales of their own, left behind the planes (plane_exps); src^T in fp32 goes to plain, [C][ld_plain],
  // columns up to Rpad
  void* plain; long long ld_plain;
  // no transpose, but [src; src2] (R and R2 rows of C values, dense) and zeros behind them as an operand that is read along its
  // rows (KRows): planes [2 C/32][Rpad][64 bytes] with the scales of the rows in `exps`, of which the first row0 have been
  // written (0 or R)
  int along_rows;
  const void* src2; int R2; int row0;
  int* exps;
  int* cols;            // counts of its columns (launch_split_rows)
};
hipError_t launch_transpose(const TransposeArgs& a, int dtype, hipStream_t st);

// Reverse pass through the circuit: from the evidence and the loss coefficients to
// the gradient w.r.t. the evidence, the sum-unit logits (written transposed, in the
// dtype of h, as r rows of ldb columns) and the layer logits; also the loss itself.
struct CircuitBwdArgs {
  int family, rows, n, r;
  const float* e;        // [rows][n][r]
  const float* logw;     // [rows][r] (nullptr for FF)
  const float* coef;     // [rows][n]
  const float* lay_nat;  // normalised linear layers [L][k][j] (static only)
  const float* lay_tr;   // the same transposed [L][j][k]
  int L;
  float* pi;             // scratch [rows][steps][r] (layer gradients only; steps = n-1 for the HMM)
  float* gam;            // scratch [rows][steps][r]
  float* G;              // scratch [L][r][r]
  float* Gpart;          // scratch: per block of LAYER_GRAD_ROWS rows, [steps][r][r] outer-product partials
                         // (shared layers) or [L*r*r] column sums (bias gradient of layers computed from h)
  int* clear; int nclear;       // ints set to 0 for the launches that follow (which saves a launch of its own)
  // layers of every position (computed from h): lay_nat / lay_tr hold [rows][L][r][r] and the
  // gradient w.r.t. the logits of position b goes to dlog[b*ld_dlog + (l*r + z)*r + z'] in the
  // dtype of h (dlog_cols columns, zero beyond L*r*r); dlayers then receives the column sums
  int contextual;
  void* dlog; long long ld_dlog; int dlog_cols;
  float* dlog32;         // fp32 accumulators [rows][L*r*r] (tree; a matrix shared by all steps; a caller's
                         // per-position gradient buffer), converted into dlog at the end when dlog is set
  float* ct;             // binary tree: scratch [rows][steps][r], output of every program step
  float* adj;            // binary tree: scratch [rows][n-1][r], adjoints of the node values
  float* Ge;             // [rows][n][r]
  void* dslT;            // [r][ldb] or nullptr
  long long ldb;
  int bf16;
  float* loss;           // [rows]
  float* dlayers;        // [L][r][r] gradient w.r.t. the layer logits (accumulated), or nullptr
};
hipError_t launch_circuit_bwd(const CircuitBwdArgs& a, hipStream_t st);
constexpr int LAYER_GRAD_ROWS = 256;   // rows whose contribution to a layer gradient one workgroup sums

// Raises a kernel's dynamic-LDS limit the first time the kernel is launched on a device.  This
// is the library's only process-wide state: one bit per kernel and device, set once the call
// has succeeded; threads that race here make the same idempotent call.
template <auto Kern>
inline hipError_t allow_lds(int bytes) {
  static std::atomic<unsigned long long> done{0};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const unsigned long long bit = (dev >= 0 && dev < 64) ? 1ull << dev : 0ull;
  if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
  e = hipFuncSetAttribute((const void*)Kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess) done.fetch_or(bit, std::memory_order_release);
  return e;
}

// Compute units of the current device (asked once per device).
inline hipError_t cu_count(int* n) {
  static std::atomic<int> known[64];
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const bool slot = dev >= 0 && dev < 64;
  int v = slot ? known[dev].load(std::memory_order_acquire) : 0;
  if (v == 0) {
    e = hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    if (slot) known[dev].store(v, std::memory_order_release);
  }
  *n = v;
  return hipSuccess;
}

hipError_t launch_philox_uniforms(int B, int S, int slots, uint32_t seed_lo, uint32_t seed_hi,
                                  uint32_t offset, float* out, hipStream_t st);

// ---- device helpers --------------------------------------------------------
#if defined(__HIPCC__)
// Philox4x32-10 (Salmon et al., SC'11): 10 rounds of two 32x32->64 multiplies.
__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                              uint32_t k0, uint32_t k1, uint32_t out[4]) {
  const uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u, W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
  for (int rnd = 0; rnd < 10; ++rnd) {
    if (rnd > 0) { k0 += W0; k1 += W1; }
    uint32_t hi0 = __umulhi(M0, c0), lo0 = M0 * c0;
    uint32_t hi1 = __umulhi(M1, c2), lo1 = M1 * c2;
    uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
    c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
  }
  out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// Uniform of (position b, draft s, slot t): counter (t/4, b, s, offset), word t%4,
// u = (word >> 8) * 2^-24 in [0, 1).
__device__ __forceinline__ float philox_uniform(uint32_t seed_lo, uint32_t seed_hi, uint32_t offset,
                                                uint32_t b, uint32_t s, uint32_t slot) {
  uint32_t w[4];
  philox4x32_10(slot >> 2, b, s, offset, seed_lo, seed_hi, w);
  uint32_t sel = slot & 3u;
  uint32_t word = sel == 0 ? w[0] : sel == 1 ? w[1] : sel == 2 ? w[2] : w[3];
  return (float)(word >> 8) * 5.9604644775390625e-8f;
}

// A scaled x (|x| < 2^15) as two fp16 terms of 11 significant bits, the second one the nearest of what the first leaves: their
// sum is off by at most half a unit of x's 23rd bit, or 2^-25.  An infinite or NaN x is its own first term and the second is 0:
// products of single terms may then be NaN (infinity times a second term of 0) where the product of the values is an
// infinity, so such operands are noted, and what they take part in is left to fp32 multiply-adds.
__device__ __forceinline__ void split2(float x, unsigned short (&t)[2]) {
  const _Float16 hi = (_Float16)x;
  const bool finite = (__float_as_uint(x) & 0x7f800000u) != 0x7f800000u;
  const _Float16 lo = (_Float16)(finite ? x - (float)hi : 0.f);
  t[0] = __builtin_bit_cast(unsigned short, hi);
  t[1] = __builtin_bit_cast(unsigned short, lo);
}
// x as the exact sum of three bf16 terms (8 significant bits each: 24 in all), the next one the nearest bf16 of
// what is left.  A finite x keeps finite terms (next to the largest value the nearest bf16 would be infinite:
// the one below is taken); an infinite or NaN x is its own first term, the others are 0.
// Terms below 2^-126 lose low bits, which matters to values below 2^-110 only.
// Where an operand is infinite, or so large that products overflow, the products of single terms can be infinities of
// both signs or infinity times zero: NaN where the product of the values is an infinity.  Operands beyond SPLIT_LARGE are
// therefore noted (SPLIT_WHOLE), and what they take part in is left to fp32 multiply-adds.
constexpr float SPLIT_LARGE = 0x1p60f;     // two values up to it: products below 2^120
__device__ __forceinline__ void split3(float x, unsigned short (&t)[3]) {
  auto bits = [](float y) { return (unsigned)__builtin_bit_cast(unsigned short, (__bf16)y) << 16; };
  const unsigned ux = __float_as_uint(x);
  const bool finite = (ux & 0x7f800000u) != 0x7f800000u;
  unsigned u1 = bits(x);
  if ((u1 & 0x7f800000u) == 0x7f800000u && finite) u1 = ux & 0xffff0000u;
  const float r1 = finite ? x - __uint_as_float(u1) : 0.f;
  const unsigned u2 = bits(r1);
  const float r2 = r1 - __uint_as_float(u2);
  t[0] = (unsigned short)(u1 >> 16);
  t[1] = (unsigned short)(u2 >> 16);
  t[2] = (unsigned short)(bits(r2) >> 16);
}
// Flag bits, set by one atomic where they are not set yet
__device__ __forceinline__ void raise_flag(int* flag, int bits) {
  if (bits != 0 && (__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & bits) != bits) atomicOr(flag, bits);
}
// scaled values below this (about 2^-18 of their row's largest) have fewer than 22 bits left
constexpr float SPLIT_SMALL = 0.125f;
// exponent E with x 2^-E in [2^14, 2^15), for the largest |x| of a row.  A row of zeros has one below every other: where
// exponents of rows meet in a maximum (k_grad_exps) it must not win
constexpr int SPLIT_ZERO_ROW = -100000;
__device__ __forceinline__ int split_exp(float largest) {
  return largest > 0.f ? __builtin_amdgcn_frexp_expf(largest) - 15 : SPLIT_ZERO_ROW;
}
// the same from its bits, which are an integer like any other to an atomic.  (0: as for fp32's smallest value, which is what a
// row may hold whose scaled largest is below that.)
__device__ __forceinline__ int largest_exp(int bits) { return __builtin_amdgcn_frexp_expf(__uint_as_float((unsigned)max(bits, 1))) - 15; }

__device__ __forceinline__ float neg_inf() { return -__builtin_inff(); }

// Reductions inside aligned groups of G lanes (G a power of two <= 64); every lane of the group
// gets the result.  The steps inside a row of 16 lanes are data-parallel-primitive moves on the
// operand path (swap neighbours, swap pairs, mirror 8, mirror 16: once the smaller blocks agree, a
// mirror pairs each block with the other one), only the steps across rows go through the LDS
// crossbar - a chain of circuit steps is a chain of these reductions, and a crossbar step costs
// about ten times a move.  All source lanes lie inside the group, so groups that have left do not
// matter.
template <int CTRL>
__device__ __forceinline__ int dpp_move(int x) {
  return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xF, 0xF, true);
}
template <class Op>
__device__ __forceinline__ float group_reduce(float x, int G, Op op) {
  if (G >= 2) x = op(x, __int_as_float(dpp_move<0xB1>(__float_as_int(x))));     // quad_perm [1,0,3,2]
  if (G >= 4) x = op(x, __int_as_float(dpp_move<0x4E>(__float_as_int(x))));     // quad_perm [2,3,0,1]
  if (G >= 8) x = op(x, __int_as_float(dpp_move<0x141>(__float_as_int(x))));    // row_half_mirror
  if (G >= 16) x = op(x, __int_as_float(dpp_move<0x140>(__float_as_int(x))));   // row_mirror
  if (G >= 32) x = op(x, __shfl_xor(x, 16));
  if (G >= 64) x = op(x, __shfl_xor(x, 32));
  return x;
}
__device__ __forceinline__ float group_max(float x, int G) {
  return group_reduce(x, G, [](float a, float b) { return fmaxf(a, b); });
}
__device__ __forceinline__ float group_sum(float x, int G) {
  return group_reduce(x, G, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ int group_min(int x, int G) {
  if (G >= 2) x = min(x, dpp_move<0xB1>(x));
  if (G >= 4) x = min(x, dpp_move<0x4E>(x));
  if (G >= 8) x = min(x, dpp_move<0x141>(x));
  if (G >= 16) x = min(x, dpp_move<0x140>(x));
  if (G >= 32) x = min(x, __shfl_xor(x, 16));
  if (G >= 64) x = min(x, __shfl_xor(x, 32));
  return x;
}

// ---- evaluation order of the binary tree (Eq. BTree) ---------------------------
// The order in which the tree's nodes are evaluated does not depend on the data: a
// kernel writes it once as a short program, one step per sum-layer application.
struct TreeStep {
  short m;        // inner node whose layer is applied (0: root, uses log omega instead of a layer)
  short lsrc;     // left operand: >= 0 heap index of a fully observed child, -1 path value, -2 all-ones
  short rsrc;     // right operand, same coding
  short out;      // >= 0: store as full value of node `out`; -1: becomes the path value; -2 - i: emit prefix i
};

__device__ inline int build_tree_program(TreeStep* prog, int n, int prefix) {
  int t = 0;
  for (int m = n - 2; m >= 1; --m) prog[t++] = TreeStep{(short)m, (short)(2 * m + 1), (short)(2 * m + 2), (short)m};
  if (!prefix) {
    prog[t++] = TreeStep{0, 1, 2, (short)(-2 - (n - 1))};
    return t;
  }
  for (int i = 0; i < n; ++i) {
    int idx = n - 1 + i, size = 1;
    while (idx > 0) {
      const int m = (idx - 1) >> 1;
      size <<= 1;
      const int first = (m - (n / size - 1)) * size, last = first + size - 1;
      if (m > 0 && last <= i) { idx = m; continue; }          // fully observed: stored value
      const int half = size >> 1;
      const int l_last = first + half - 1, r_first = first + half;
      const short ls = (l_last <= i) ? (short)(2 * m + 1) : (short)-1;
      const short rs = (r_first > i) ? (short)-2 : (last <= i ? (short)(2 * m + 2) : (short)-1);
      prog[t++] = TreeStep{(short)m, ls, rs, (short)(m > 0 ? -1 : -2 - i)};
      idx = m;
    }
  }
  return t;
}
#endif

inline int tree_program_steps(int n, int prefix) {
  if (!prefix) return n - 2 + 1;
  int lg = 0;
  while ((1 << lg) < n) ++lg;
  return n - 2 + n * lg;          // upper bound: at most log2(n) steps per prefix
}

}  // namespace mtpc
