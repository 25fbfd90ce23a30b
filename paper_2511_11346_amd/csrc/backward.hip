// Small kernels of the training step: layout changes between the two big
// contractions and the reverse pass through the circuit layers (Sec. 4.1 loss:
// a linear combination of prefix log-marginals, loss = sum_j g_j P_j with
// g_j = coef_{j+1} - coef_j, coef_n = 0).
#include "mtpc_internal.h"

namespace mtpc {
namespace {

__device__ __forceinline__ unsigned short to_bf16_rne(float x) {
  unsigned u = __float_as_uint(x);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (unsigned short)((u >> 16) | 0x40);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}
// a.nclear ints of a.clear to 0, by a whole grid
__device__ __forceinline__ void clear_ints(const CircuitBwdArgs& a) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < a.nclear; i += gridDim.x * blockDim.x) a.clear[i] = 0;
}
__device__ __forceinline__ float wsum(float x) { return group_sum(x, 64); }
__device__ __forceinline__ float wmax(float x) { return group_max(x, 64); }

// 64 x 64 element tiles through LDS; T is the 2- or 4-byte element type.
template <typename T>
__global__ __launch_bounds__(256) void k_transpose(const TransposeArgs a) {
  __shared__ T tile[64][64 + (sizeof(T) == 2 ? 2 : 1)];
  const int c0 = blockIdx.x * 64, r0 = blockIdx.y * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;       // 4 rows per pass
  const T* src = (const T*)a.src;
  T* dst = (T*)a.dst;
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int r = r0 + ty + 4 * k, c = c0 + tx;
    T val = 0;
    if (r < a.R && c < a.C) val = src[(long long)r * a.ld_src + c];
    tile[ty + 4 * k][tx] = val;
  }
  __syncthreads();
#pragma unroll
  for (int k0 = 0; k0 < 16; ++k0) {
    const int c = c0 + ty + 4 * k0, r = r0 + tx;
    if (c < a.C && r < a.Rpad) {
      constexpr int EPS = 64 / (int)sizeof(T);         // elements of a row per stage
      const long long k = a.col0 + r;
      if (a.stage_rows) dst[(k / EPS * a.stage_rows + c) * EPS + k % EPS] = tile[tx][ty + 4 * k0];
      else dst[(long long)c * a.ld_dst + k] = tile[tx][ty + 4 * k0];
    }
  }
}

// The same with 16-byte accesses on both sides (VE = 16 / sizeof(T) elements per thread);
// needs 16-byte aligned rows on both sides (checked by the launcher).
template <typename T>
__global__ __launch_bounds__(256) void k_transpose_vec(const TransposeArgs a) {
  constexpr int VE = 16 / sizeof(T);
  constexpr int TPR = 64 / VE;                       // threads per tile row
  struct alignas(16) Vec { T v[VE]; };
  __shared__ T tile[64][64 + VE + (sizeof(T) == 2 ? 2 : 1)];
  const int c0 = blockIdx.x * 64, r0 = blockIdx.y * 64;
  const int tx = threadIdx.x % TPR, ty = threadIdx.x / TPR;
  const T* src = (const T*)a.src;
  T* dst = (T*)a.dst;
  for (int rr = ty; rr < 64; rr += 256 / TPR) {
    const int r = r0 + rr, c = c0 + tx * VE;
    Vec x;
#pragma unroll
    for (int t = 0; t < VE; ++t) x.v[t] = 0;
    if (r < a.R) {
      if (c + VE <= a.C) x = *(const Vec*)(src + (long long)r * a.ld_src + c);
      else
        for (int t = 0; t < VE; ++t)
          if (c + t < a.C) x.v[t] = src[(long long)r * a.ld_src + c + t];
    }
#pragma unroll
    for (int t = 0; t < VE; ++t) tile[rr][tx * VE + t] = x.v[t];
  }
  __syncthreads();
  for (int cc = ty; cc < 64; cc += 256 / TPR) {
    const int c = c0 + cc, r = r0 + tx * VE;
    if (c >= a.C) continue;
    Vec x;
#pragma unroll
    for (int t = 0; t < VE; ++t) x.v[t] = tile[tx * VE + t][cc];
    constexpr int EPS = 64 / (int)sizeof(T);           // elements of a row per stage (a multiple of VE)
    const long long k = a.col0 + r;
    T* o = a.stage_rows ? dst + (k / EPS * a.stage_rows + c) * EPS + k % EPS : dst + (long long)c * a.ld_dst + k;
    if (r + VE <= a.Rpad) *(Vec*)o = x;
    else
      for (int t = 0; t < VE; ++t)
        if (r + t < a.Rpad) o[t] = x.v[t];
  }
}

// src^T in fp32 (a.plain) and, as planes of two fp16 terms with scales of its rows (split2), in a.dst.  A workgroup takes 16
// columns of src, all R rows, once: 64 bytes of each of 16 rows at a time through LDS; the largest value of a column is known
// when its last row has passed, and the columns, read back, are split.
// Rows of src whose `live` is 0 (positions without a gradient, which add nothing to any sum) are left out of the planes and
// the scales.  Raises SPLIT_WIDE for columns with more than one small value in 16 (as k_split_rows does for rows), and
// adds to a.weights the scaled magnitudes of every row of src, for check_planes.
__global__ __launch_bounds__(512) void k_transpose_split(const TransposeArgs a, int* __restrict__ exps) {
  typedef __attribute__((ext_vector_type(4))) float f32x4_t;
  typedef __attribute__((ext_vector_type(4))) int i32x4_t;
  constexpr int U = 4, RT = 128;                     // steps of RT rows in flight
  __shared__ float tile[16][RT * U + 1];
  __shared__ unsigned s_max[16];
  __shared__ int s_small[16], s_none[16];
  const int tid = threadIdx.x, lane = tid & 63, c0 = blockIdx.x * 16;
  const float* const src = (const float*)a.src;
  float* const plain = (float*)a.plain;
  if (tid < 16) { s_max[tid] = 0; s_small[tid] = 0; s_none[tid] = 0; }
  unsigned largest = 0;
  for (int r0 = 0; r0 < a.Rpad; r0 += RT * U) {
    // four threads to the 64 bytes of a row
    f32x4_t x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = r0 + RT * u + (tid >> 2);
      x[u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      if (r < a.R) x[u] = *(const f32x4_t*)(src + (long long)r * a.ld_src + c0 + 4 * (tid & 3));
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int c = 0; c < 4; ++c) tile[4 * (tid & 3) + c][RT * u + (tid >> 2)] = x[u][c];
    __syncthreads();
    // 32 threads to a column, four neighbouring rows each
    const int c = tid >> 5;
    unsigned m = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int rl = RT * u + 4 * (tid & 31), r = r0 + rl;
      if (r >= a.Rpad) continue;
      const i32x4_t live = *(const i32x4_t*)(a.live + r);
      f32x4_t y;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        y[t] = tile[c][rl + t];
        const unsigned v = __float_as_uint(y[t]) & 0x7fffffffu;
        largest = max(largest, v);
        m = max(m, v < 0x7f800000u && live[t] > 0 ? v : 0u);
      }
      *(f32x4_t*)(plain + (long long)(c0 + c) * a.ld_plain + r) = y;
    }
    if (m != 0) atomicMax(&s_max[c], m);
  }
  raise_flag(a.flag, largest >= 0x7f800000u ? SPLIT_WIDE | SPLIT_WHOLE : largest > __float_as_uint(SPLIT_LARGE) ? SPLIT_WHOLE : 0);
  __syncthreads();                                   // (and the workgroup's stores are visible to it)
  // four threads to the 64 bytes of a column's stage, 16 columns behind each other
  const int c = (tid >> 2) & 15, ch = tid & 3;
  const int E = split_exp(__uint_as_float(s_max[c]));
  if (tid < 64 && ch == 0) exps[c0 + c] = E;
  const float* const col = plain + (long long)(c0 + c) * a.ld_plain + ch * 8;
  unsigned short* const dst = (unsigned short*)a.dst + (long long)(c0 + c) * 32 + ch * 8;
  int small = 0, none = 0;                           // (small: with those that are 0)
  for (int k = tid >> 6; k < a.Rpad / 32; k += 8) {
    const f32x4_t y0 = *(const f32x4_t*)(col + k * 32), y1 = *(const f32x4_t*)(col + k * 32 + 4);
    const i32x4_t l0 = *(const i32x4_t*)(a.live + k * 32 + ch * 8), l1 = *(const i32x4_t*)(a.live + k * 32 + ch * 8 + 4);
    struct alignas(16) Oct { unsigned short v[8]; } o[2];
    unsigned w[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const float x = (t < 4 ? l0[t & 3] : l1[t & 3]) > 0 ? (t < 4 ? y0[t & 3] : y1[t & 3]) : 0.f, y = __builtin_amdgcn_ldexpf(x, -E);
      none += x == 0.f;
      small += fabsf(y) < SPLIT_SMALL;
      w[t] = (unsigned)fminf(fabsf(y), 32768.f);
      unsigned short q[2];
      split2(y, q);
      o[0].v[t] = q[0]; o[1].v[t] = q[1];
    }
#pragma unroll
    for (int p = 0; p < 2; ++p) *(Oct*)(dst + (2LL * k + p) * a.stage_rows * 32) = o[p];
    // the sum over the 16 columns, rows halved at every exchange but the last: one row to a lane (of two)
#pragma unroll
    for (int o2 = 4, n = 4; n >= 1; o2 <<= 1, n >>= 1)
#pragma unroll
      for (int t = 0; t < n; ++t) {
        const bool up = lane & o2;
        const unsigned mine = up ? w[t + n] : w[t], other = up ? w[t] : w[t + n];
        w[t] = mine + (unsigned)__shfl_xor((int)other, o2);
      }
    const unsigned sum = w[0] + (unsigned)__shfl_xor((int)w[0], 32);
    const int r = k * 32 + ch * 8 + (lane & 4) + (lane & 8) / 4 + (lane & 16) / 16;
    if (lane < 32 && sum > 0) atomicAdd(a.weights + r, sum);
  }
  atomicAdd(&s_small[c], small - none);
  atomicAdd(&s_none[c], none);
  __syncthreads();
  if (tid < 16 && s_small[tid] > (a.Rpad - s_none[tid]) / 16) raise_flag(a.flag, SPLIT_WIDE);
}

// What the counts of single rows and columns of an operand cannot say, by one workgroup of k_grad_exps (whether a position has a
// gradient is known by then, and what the others add to a.top does not change that).
// h^T has a scale per feature, so a position may be small in most of them.  The terms are off by 2^-40 of the scale in each, which
// has to be little beside that position's values alone (what an entry of dW sums is this position's alone where its
// gradients are the largest), and beside it all other positions' terms of the gradient are as far off as theirs
// make them: sqrt(B) times 2^-40 of an average position, as a random walk.  Both stay below 2^-23 where the position's
// magnitudes add up to 2^-17 of d scales (which a value has of 2^14 to 2^15 units: d / 4), and of sqrt(B) average positions.
// [W; Wsum] has a scale per row: a column may be small in most rows, which decides about that column of dh.
// The gradient has a scale per token, which is at most the largest of all positions' gradients, so a position may be small in all of them,
// and a feature that only such positions have makes a column of dW of nothing else.  Its M entries are off by 2^-42 of that largest
// one, to be compared with the position's own gradients: below 2^-20 of them where those are sqrt(M) 2^-22 of the largest.
__device__ __forceinline__ void check_planes(const GradPhiArgs& a, float (&s_sum)[4], float (&s_cnt)[4], float (&s_most)[4]) {
  const int tid = threadIdx.x;
  float sum = 0.f, cnt = 0.f, most = 0.f;
  for (int b = tid; b < a.B; b += 256)
    if (a.top[b] > 0) { sum += (float)a.weights[b]; cnt += 1.f; most = fmaxf(most, a.most[b]); }
  sum = wsum(sum); cnt = wsum(cnt); most = wmax(most);
  if ((tid & 63) == 0) { s_sum[tid >> 6] = sum; s_cnt[tid >> 6] = cnt; s_most[tid >> 6] = most; }
  __syncthreads();
  sum = s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3];
  cnt = s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3];
  most = fmaxf(fmaxf(s_most[0], s_most[1]), fmaxf(s_most[2], s_most[3]));
  const float least = fmaxf((float)a.d * 0.25f, sum / fmaxf(cnt, 1.f) * sqrtf((float)a.B) * 0x1p-17f);
  bool wide = false;
  const float faint = most * sqrtf((float)a.M) * 0x1p-22f;
  for (int b = tid; b < a.B; b += 256) wide |= a.top[b] > 0 && ((float)a.weights[b] < least || (a.most[b] > 0.f && a.most[b] < faint));
  for (int k = tid; k < a.d; k += 256) wide |= a.cols[k] > ((int)a.ldM - a.cols[a.d + k]) / 16;
  if (wide) raise_flag(a.flag, SPLIT_WIDE);
}

// The logit gradient from the stored probabilities where only dLT is wanted: no transpose, so no LDS.  A thread takes eight
// neighbouring positions of a row, 16 threads 512 bytes of probabilities, a wave four rows: 256 bytes of each of four chunks of
// dLT.  A workgroup takes 128 positions of `rows` rows, 16 at a time.  Bound by memory: 8.1 GB in 1.73 ms (4.7 TB/s) where both layouts
// take 10.7 GB and 2.30 ms (n r v = 327,680, B = 4096); with 32 positions of 16 rows to a wave - lines of probabilities 16 KB apart -
// it took 2.07 ms.
// The workgroups behind those write the rows of [W; Wsum; 0] from tail_row on, which the contraction along W's rows reads
// beside W's whole stages of 32 rows.
__global__ __launch_bounds__(256) void k_grad_rows(const GradPhiArgs a, int rows, int row_blocks) {
  typedef __attribute__((ext_vector_type(4))) float f32x4_t;
  struct alignas(16) Oct { unsigned short v[8]; };
  if ((int)blockIdx.y >= row_blocks) {
    const long long t = ((long long)(blockIdx.y - row_blocks) * gridDim.x + blockIdx.x) * 256 + threadIdx.x;
    const int per = a.d / 8;
    const long long m = a.tail_row + t / per, c = t % per * 8;
    if (m >= a.ldM) return;
    Oct o{};
    if (m < a.M) o = *(const Oct*)((const unsigned short*)a.W + m * a.d + c);
    else if (m < a.Mx) o = *(const Oct*)((const unsigned short*)a.Wsum + (m - a.M) * a.d + c);
    *(Oct*)((unsigned short*)a.tail + (m - a.tail_row) * a.d + c) = o;
    return;
  }
  const int b = blockIdx.x * 128 + (threadIdx.x & 15) * 8;
  if (b >= a.ldb) return;
  unsigned short* const out = (unsigned short*)a.dLT + (long long)(b / 32) * a.ldM * 32 + b % 32;
  int cur_slab = -1, x[8];
  float g[8];
#pragma unroll 4
  for (int k = 0; k < rows / 16; ++k) {
    const long long m = (long long)blockIdx.y * rows + k * 16 + (threadIdx.x >> 4);
    if (m >= a.ldM) return;
    Oct o{};
    if (m < a.M) {
      const f32x4_t* p = (const f32x4_t*)(a.phiT + m * a.ld_phi + b);
      const f32x4_t p0 = __builtin_nontemporal_load(p), p1 = __builtin_nontemporal_load(p + 1);
      const int slab = (int)(m / a.v), av = (int)(m - (long long)slab * a.v);
      if (slab != cur_slab) {
        cur_slab = slab;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          x[c] = -1; g[c] = 0.f;
          if (b + c < a.B) {
            x[c] = a.targets[(long long)(b + c) * a.n + slab / a.r];
            g[c] = a.Ge[(long long)(b + c) * a.n * a.r + slab];
          }
        }
      }
#pragma unroll
      for (int c = 0; c < 8; ++c)
        if (x[c] != -1) o.v[c] = to_bf16_rne(g[c] * ((av == x[c] ? 1.f : 0.f) - (c < 4 ? p0[c & 3] : p1[c & 3])));
    } else if (m < a.Mx) {
      o = *(const Oct*)((const unsigned short*)a.dslT + (m - a.M) * a.ldb + b);        // sum-unit rows, written by the reverse pass
    }
    *(Oct*)(out + m * 32) = o;
  }
}

// a.top: 1, the least, for a position that has a gradient, else 0, and the largest of its gradients (a.most).  A wave to a position.  (Before everything that reads the
// probabilities: the transpose of h asks for it, and between k_grad_exps and k_grad_from_phi, which finds what is left of the
// probabilities in the last cache, that costs the latter a third where they fit.)
__global__ __launch_bounds__(256) void k_live_positions(const GradPhiArgs a) {
  const int b = blockIdx.x * 4 + (threadIdx.x >> 6), t = threadIdx.x & 63, nr = a.n * a.r;
  if (b >= a.B) return;                              // (all 64)
  bool some = false;
  float most = 0.f;                                  // of the gradients of its evidence
  for (int i = t; i < nr; i += 64) {
    const float g = a.targets[(long long)b * a.n + i / a.r] != -1 ? fabsf(a.Ge[(long long)b * nr + i]) : 0.f;
    some |= g != 0.f;
    most = fmaxf(most, g);
  }
  for (int j = t; j < (int)(a.Mx - a.M); j += 64) some |= ((const float*)a.dslT)[j * a.ldb + b] != 0.f;
  some = __any(some);
  most = wmax(most);
  if (t == 0) { a.top[b] = some; a.most[b] = most; }
}

// What the scales of the two planes that k_grad_from_phi writes (see split2) follow from: the largest magnitude of a row of dLT over
// all positions (a.rows), and of a row of dL, whose elements carry the scales of W's rows, over all tokens (a.top), as bits.
// One more read of the probabilities.  The first workgroups take CH positions of `count` blocks of up to 64 rows of one slab: the
// gradients and targets of the slab, apart in memory, go through LDS (fetched by every wave for its rows of any slabs, this
// took 330 us for 562 MB of probabilities), and so do the maxima of the positions, which leave with one atomic of the workgroup
// each.  (A bound on a position's maximum from its gradients and the largest exponent of each slab is not enough: a row of W far
// above the others may belong to a token without probability.)  The next ones add the sum-unit rows of 16 positions each to
// a.top, and the last one looks at the other operands (check_planes).
__global__ __launch_bounds__(256, 4) void k_grad_exps(const GradPhiArgs a, int row_blocks, int count) {
  typedef __attribute__((ext_vector_type(4))) float f32x4_t;
  typedef __attribute__((ext_vector_type(4))) int i32x4_t;
  constexpr int CH = 512;
  __shared__ __align__(16) float s_g[CH];
  __shared__ __align__(16) int s_x[CH];
  __shared__ int s_top[CH];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nr = a.n * a.r;
  // what the largest magnitude of some elements, as bits (above infinity: NaN), and the largest of a position's say about them
  auto note = [&](unsigned big, int top) {
    raise_flag(a.flag, big >= 0x7f800000u || top >= 0x7f800000 ? SPLIT_WIDE | SPLIT_WHOLE : big > __float_as_uint(SPLIT_LARGE) ? SPLIT_WHOLE : 0);
  };
  const int groups = (row_blocks + count - 1) / count;
  if ((int)blockIdx.x < groups) {
    constexpr int RW = 16;                           // rows of a wave (those of the four waves alternate)
    const int parts = (a.v + 63) / 64, c0 = blockIdx.y * CH;
    unsigned largest = 0;
    int slab = -1;
#pragma unroll
    for (int q = 0; q < CH / 256; ++q) s_top[tid + q * 256] = 0;
    f32x4_t ph[RW];
    auto fetch = [&](int g, int b) {                 // rows of this wave in block g, positions b ..  (b beyond the last position: any)
      const int s = g / parts, r0 = (g - s * parts) * 64 + wave;
      const float* phi = a.phiT + (long long)s * a.v * a.ld_phi + min((long long)b + 4 * lane, a.ldb - 4);
#pragma unroll
      for (int k = 0; k < RW; ++k) ph[k] = *(const f32x4_t*)(phi + (long long)min(r0 + 4 * k, a.v - 1) * a.ld_phi);
    };
    const int end = min(row_blocks, (int)(blockIdx.x + 1) * count);
    fetch(blockIdx.x * count, c0);
#pragma unroll 1
    for (int g = blockIdx.x * count; g < end; ++g) {
      const int s = g / parts, r0 = (g - s * parts) * 64 + wave;
      unsigned big[RW];
      int we[RW];                                    // (of a row that is not there: of a row of zeros)
#pragma unroll
      for (int k = 0; k < RW; ++k) {
        big[k] = 0;
        const int row = r0 + 4 * k;
        we[k] = __builtin_amdgcn_readfirstlane(row < a.v ? a.Wexp[(long long)s * a.v + row] : SPLIT_ZERO_ROW);
      }
      if (s != slab) {
        slab = s;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < CH / 256; ++q) {
          const int i = tid + q * 256, b = c0 + i;
          const int bc = min(b, a.B - 1);
          const int x = a.targets[(long long)bc * a.n + slab / a.r];
          const float ge = a.Ge[(long long)bc * nr + slab];
          s_x[i] = x;
          s_g[i] = b < a.B && x != -1 ? ge : 0.f;
        }
        __syncthreads();
      }
#pragma unroll 1
      for (int o = 0; o < CH && c0 + o < a.B; o += 256) {
        const int i = o + 4 * lane;
        const f32x4_t ge = *(const f32x4_t*)(s_g + i);
        const i32x4_t x = *(const i32x4_t*)(s_x + i);
        float top[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < RW; ++k)
#pragma unroll
          for (int c = 0; c < 4; ++c) {              // (no gradient beyond the last position, whose probabilities may be anything)
            const float y = ge[c] != 0.f ? fabsf(ge[c] * ((r0 + 4 * k == x[c] ? 1.f : 0.f) - ph[k][c])) : 0.f;
            big[k] = max(big[k], __float_as_uint(y));
            top[c] = fmaxf(top[c], __builtin_amdgcn_ldexpf(y, we[k]));
          }
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (top[c] > 0.f) atomicMax(&s_top[i + c], (int)__float_as_uint(top[c]));
        const bool more = o + 256 < CH && c0 + o + 256 < a.B;
        fetch(more ? g : min(g + 1, end - 1), more ? c0 + o + 256 : c0);
      }
      // the largest of each row over the lanes, rows halved at every exchange: lane l ends up with row l / 4
#pragma unroll
      for (int o = 32, R = RW / 2; o >= 4; o >>= 1, R >>= 1)
#pragma unroll
        for (int k = 0; k < R; ++k) {
          const bool up = lane & o;
          const unsigned mine = up ? big[k + R] : big[k], other = up ? big[k] : big[k + R];
          big[k] = max(mine, (unsigned)__shfl_xor((int)other, o));
        }
      unsigned y = big[0];
      y = max(y, (unsigned)__shfl_xor((int)y, 1));
      y = max(y, (unsigned)__shfl_xor((int)y, 2));
      const int row = r0 + 4 * (lane >> 2);
      if ((lane & 3) == 0 && row < a.v && y > 0) atomicMax(a.rows + (long long)s * a.v + row, y);
      largest = max(largest, y);
    }
    __syncthreads();
    // (few of a position's maxima are above those of the workgroups before)
    int have[CH / 256], most = 0;
#pragma unroll
    for (int q = 0; q < CH / 256; ++q)
      have[q] = __hip_atomic_load(a.top + min(c0 + tid + q * 256, a.B - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int q = 0; q < CH / 256; ++q) {
      const int top = s_top[tid + q * 256];          // (0 beyond the last position)
      most = max(most, top);
      if (top > have[q]) atomicMax(a.top + c0 + tid + q * 256, top);
    }
    note(largest, most);
    return;
  }
  if (blockIdx.y > 0) return;
  __shared__ float s_sum[4], s_cnt[4], s_most[4];
  if (blockIdx.x == gridDim.x - 1) {
    check_planes(a, s_sum, s_cnt, s_most);
    return;
  }
  const int b = ((int)blockIdx.x - groups) * 16 + (tid >> 4), t = tid & 15;
  const int r2 = (int)(a.Mx - a.M);
  unsigned big = 0;
  int top = 0;
  if (b < a.B)
    for (int j = t; j < r2; j += 16) {
      const float y = fabsf(((const float*)a.dslT)[j * a.ldb + b]);
      big = max(big, __float_as_uint(y));
      top = max(top, (int)__float_as_uint(__builtin_amdgcn_ldexpf(y, a.Wexp[a.M + j])));
    }
#pragma unroll
  for (int o = 1; o < 16; o <<= 1) top = max(top, __shfl_xor(top, o));
  if (b < a.B && t == 0 && top > 0) atomicMax(a.top + b, top);
  note(big, top);
}

// 64 (m) x 128 (b) tiles: logit gradient from the stored probabilities, written in both
// layouts (dLT along b straight away, dL along m after a transpose through LDS).  A thread
// moves four neighbouring elements at a time (16-byte loads, 8- or 16-byte stores).
// PLANES (fp32): both layouts as planes of two fp16 terms, as tile_gemm_run_split reads them, whose rows have the scales of a.rows
// and a.top (largest_exp); or of three bf16 terms where *a.flag says so.
template <typename T, int PLANES>
__device__ __forceinline__ void grad_from_phi(const GradPhiArgs& a, const int* __restrict__ rows, const int* __restrict__ top, T (&tile)[64][128 + 4]) {
  struct alignas(4 * sizeof(T)) Quad { T v[4]; };
  // four neighbours along K, to row `row` of a staged matrix of `rows` rows; e[c]: the power of two x[c] is multiplied with
  auto put_planes = [](void* dst, long long k, long long rows, long long row, const Quad& x, const int (&e)[4]) {
    constexpr int TERMS = PLANES == 3 ? 3 : 2;
    struct alignas(8) Half { unsigned short v[4]; } o[TERMS];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      unsigned short q[TERMS];
      if constexpr (PLANES == 3) split3((float)x.v[c], q);
      else split2(__builtin_amdgcn_ldexpf((float)x.v[c], e[c]), q);
#pragma unroll
      for (int p = 0; p < TERMS; ++p) o[p].v[c] = q[p];
    }
#pragma unroll
    for (int p = 0; p < TERMS; ++p) *(Half*)((unsigned short*)dst + ((k / 32 * TERMS + p) * rows + row) * 32 + k % 32) = o[p];
  };
  const long long m0 = (long long)blockIdx.y * 64;
  const int b0 = blockIdx.x * 128;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;      // 32 column quads x 8 rows per pass
  const int b = b0 + 4 * tx;                                    // first of the thread's four positions
  T* dLT = (T*)a.dLT;
  T* dL = (T*)a.dL;
  auto conv = [](float x) -> T {
    if constexpr (sizeof(T) == 2) return to_bf16_rne(x); else return x;
  };
  const bool col_ok = b < a.ldb;                                // ldb is a multiple of 4: all four or none
  int cur_slab = -1, x[4] = {-1, -1, -1, -1};
  float g[4] = {0.f, 0.f, 0.f, 0.f};
  bool bad = false;
#pragma unroll 2
  for (int k = 0; k < 8; ++k) {
    const int ml = ty + 8 * k;
    const long long m = m0 + ml;
    Quad out;
#pragma unroll
    for (int c = 0; c < 4; ++c) out.v[c] = conv(0.f);
    if (m < a.M && col_ok) {
      const int slab = (int)(m / a.v), av = (int)(m - (long long)slab * a.v);
      if (slab != cur_slab) {                      // rows of a tile mostly share their slab
        cur_slab = slab;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          x[c] = -1; g[c] = 0.f;
          if (b + c < a.B) {
            x[c] = a.targets[(long long)(b + c) * a.n + slab / a.r];
            g[c] = a.Ge[(long long)(b + c) * a.n * a.r + slab];
          }
        }
      }
      // (the probabilities are read once, here: as a stream)
      typedef __attribute__((ext_vector_type(4))) float f32x4_t;
      const f32x4_t ph = __builtin_nontemporal_load((const f32x4_t*)(a.phiT + m * a.ld_phi + b));
      const float pv[4] = {ph[0], ph[1], ph[2], ph[3]};
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (b + c < a.B && x[c] != -1) out.v[c] = conv(g[c] * ((av == x[c] ? 1.f : 0.f) - pv[c]));
      constexpr int EPS = 64 / (int)sizeof(T);     // elements of a row per stage (b is a multiple of 4)
      if constexpr (PLANES != 0) {
        const int e = PLANES == 2 ? -largest_exp(rows[m]) : 0;
        put_planes(a.dLT, b, a.M, m, out, {e, e, e, e});
      } else if (a.staged) *(Quad*)(dLT + ((long long)(b / EPS) * a.M + m) * EPS + b % EPS) = out;
      else *(Quad*)(dLT + m * a.ldb + b) = out;
    } else if (m < a.Mx && col_ok) {
      out = *(const Quad*)((const T*)a.dslT + (m - a.M) * a.ldb + b);   // sum-unit rows, written by the reverse pass
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      tile[ml][4 * tx + c] = out.v[c];
      if constexpr (PLANES == 3) bad |= !(fabsf(out.v[c]) <= SPLIT_LARGE);
    }
  }
  if constexpr (PLANES == 3)
    if (bad) raise_flag(a.flag, SPLIT_WHOLE);
  __syncthreads();
  const int mq = threadIdx.x & 15, br = threadIdx.x >> 4;        // 16 row quads x 16 positions per pass
  int we[4] = {0, 0, 0, 0};
  if constexpr (PLANES == 2)
#pragma unroll
    for (int c = 0; c < 4; ++c) we[c] = a.Wexp[min(m0 + 4 * mq + c, a.Mx - 1)];
#pragma unroll 2
  for (int k = 0; k < 8; ++k) {
    const int bl = br + 16 * k;
    const long long m = m0 + 4 * mq;
    if (b0 + bl < a.B && m < a.dl_end) {                        // dl_end is a multiple of 4
      Quad out;
#pragma unroll
      for (int c = 0; c < 4; ++c) out.v[c] = tile[4 * mq + c][bl];
      constexpr int EPS = 64 / (int)sizeof(T);
      if constexpr (PLANES != 0) {
        const int e = PLANES == 2 ? largest_exp(top[b0 + bl]) : 0;
        put_planes(a.dL, m, a.B, b0 + bl, out, {we[0] - e, we[1] - e, we[2] - e, we[3] - e});
      } else if (a.staged) *(Quad*)(dL + ((m / EPS) * a.B + (b0 + bl)) * EPS + m % EPS) = out;
      else *(Quad*)(dL + (long long)(b0 + bl) * a.ldM + m) = out;
    }
  }
}
template <typename T, bool PLANES = false>
__global__ __launch_bounds__(256) void k_grad_from_phi(const GradPhiArgs a, const int* __restrict__ rows, const int* __restrict__ top) {
  __shared__ T tile[64][128 + 4];
  if constexpr (!PLANES) grad_from_phi<T, 0>(a, rows, top, tile);
  else if ((*a.flag & SPLIT_WIDE) == 0) grad_from_phi<T, 2>(a, rows, top, tile);
  else grad_from_phi<T, 3>(a, rows, top, tile);       // (which raises SPLIT_WHOLE only)
}

// acc_u = sum_k sh[k] * M[k*r + unit_u] for the lane's units (lane, lane + 64); M is an
// r x r matrix in global memory read along its contiguous axis, eight rows in flight.
__device__ __forceinline__ void wave_matvec(const float* __restrict__ M, const float* sh, int r, int lane,
                                            float& acc0, float& acc1) {
  const bool u1 = lane + 64 < r;
  const int c0 = min(lane, r - 1), c1 = min(lane + 64, r - 1);
  acc0 = acc1 = 0.f;
  for (int k0 = 0; k0 < r; k0 += 8) {
    float w0[8], w1[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const long long k = min(k0 + u, r - 1);
      w0[u] = M[k * r + c0];
      w1[u] = u1 ? M[k * r + c1] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (k0 + u < r) {
        const float x = sh[k0 + u];
        acc0 = fmaf(x, w0[u], acc0);
        acc1 = fmaf(x, w1[u], acc1);
      }
  }
}

// One wave per evidence row; lane l holds units l and l + 64.
__global__ __launch_bounds__(256) void k_circuit_bwd(const CircuitBwdArgs a) {
  clear_ints(a);
  __shared__ float sP[4][64];
  __shared__ float sX[4][128];
  __shared__ float sPi[4][128], sC[4][128];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long long row = (long long)blockIdx.x * 4 + wave;
  const int n = a.n, r = a.r;
  const bool u0 = lane < r, u1 = lane + 64 < r;
  auto put_dsl = [&](float v0, float v1) {          // transposed, in the dtype of h
    if (a.dslT == nullptr || row >= a.ldb) return;
    if (a.bf16) {
      unsigned short* d = (unsigned short*)a.dslT;
      if (u0) d[(long long)lane * a.ldb + row] = to_bf16_rne(v0);
      if (u1) d[(long long)(lane + 64) * a.ldb + row] = to_bf16_rne(v1);
    } else {
      float* d = (float*)a.dslT;
      if (u0) d[(long long)lane * a.ldb + row] = v0;
      if (u1) d[(long long)(lane + 64) * a.ldb + row] = v1;
    }
  };
  if (row >= a.rows) {                              // padding columns of the transposed output
    put_dsl(0.f, 0.f);
    return;
  }
  const float* e = a.e + row * n * r;
  const float* coef = a.coef + row * n;
  float* Ge = a.Ge + row * n * r;
  auto g_of = [&](int j) { return (j + 1 < n ? coef[j + 1] : 0.f) - coef[j]; };
  const float ninf = neg_inf();

  if (a.family == MTPC_FF) {
    // P_j = e_0 + .. + e_j: d loss / d e_i = sum_{j >= i} g_j = -coef_i
    float P = 0.f, loss = 0.f;
    for (int j = 0; j < n; ++j) {
      P += e[j];
      loss += g_of(j) * P;
      if (lane == 0) Ge[j] = -coef[j];
    }
    if (lane == 0) a.loss[row] = loss;
    return;
  }
  const float* lw = a.logw + row * r;
  const float w0 = u0 ? lw[lane] : ninf, w1 = u1 ? lw[lane + 64] : ninf;

  if (a.family == MTPC_CP) {
    // s_j[z] = log omega_z + sum_{i<=j} e_i[z],  P_j = LSE_z s_j,  dP_j/de_i[z] = softmax(s_j)[z] (i <= j)
    float s0 = w0, s1 = w1, loss = 0.f;
    for (int j = 0; j < n; ++j) {
      if (u0) s0 += e[j * r + lane];
      if (u1) s1 += e[j * r + lane + 64];
      const float m = wmax(fmaxf(s0, s1));
      const float P = m + __logf(wsum((u0 ? __expf(s0 - m) : 0.f) + (u1 ? __expf(s1 - m) : 0.f)));
      if (lane == 0) sP[wave][j] = P;
      loss += g_of(j) * P;
    }
    __builtin_amdgcn_wave_barrier();
    float a0 = 0.f, a1 = 0.f;                       // sum_{j >= i} g_j softmax(s_j)
    for (int j = n - 1; j >= 0; --j) {
      const float P = sP[wave][j], g = g_of(j);
      if (u0) { a0 += g * __expf(s0 - P); Ge[j * r + lane] = a0; s0 -= e[j * r + lane]; }
      if (u1) { a1 += g * __expf(s1 - P); Ge[j * r + lane + 64] = a1; s1 -= e[j * r + lane + 64]; }
    }
    // log omega = log_softmax(sum-unit logits): d/dlogit_z = G_z - omega_z sum_z' G_z'
    const float tot = wsum((u0 ? a0 : 0.f) + (u1 ? a1 : 0.f));
    put_dsl(a0 - __expf(w0) * tot, a1 - __expf(w1) * tot);
    if (lane == 0) a.loss[row] = loss;
    return;
  }

  if (a.family == MTPC_HMM) {
    // forward messages (Eq. HMM) alpha_j, kept in Ge[j] until the reverse pass replaces them
    // by their adjoints.  With pi_j = softmax(alpha_j), pred_j = pi_j T_j (predicted next
    // state) and gam_j = adj(alpha_{j+1}) / pred_j:
    //   adj(alpha_j) = g_j pi_j + pi_j * (T_j gam_j),   d loss / d log T_j[z][z'] = pi_j[z] T_j[z][z'] gam_j[z'].
    float* sh = sX[wave];
    const long long lstep = a.L > 1 ? (long long)r * r : 0;
    const long long lrow = a.contextual ? row * a.L * r * r : 0;       // this position's own layers
    const float* lay_nat = a.lay_nat + lrow;
    const float* lay_tr = a.lay_tr ? a.lay_tr + lrow : nullptr;   // shared layers only
    float al0 = w0 + (u0 ? e[lane] : 0.f), al1 = w1 + (u1 ? e[lane + 64] : 0.f);
    float loss = 0.f;
    for (int j = 0; j < n; ++j) {
      if (j > 0) {
        const float m = wmax(fmaxf(al0, al1));
        const float ms = m == ninf ? 0.f : m;
        if (u0) sh[lane] = __expf(al0 - ms);
        if (u1) sh[lane + 64] = __expf(al1 - ms);
        __builtin_amdgcn_wave_barrier();
        float s0, s1;
        wave_matvec(lay_nat + (j - 1) * lstep, sh, r, lane, s0, s1);
        __builtin_amdgcn_wave_barrier();
        al0 = u0 ? ms + __logf(s0) + e[j * r + lane] : ninf;
        al1 = u1 ? ms + __logf(s1) + e[j * r + lane + 64] : ninf;
      }
      if (u0) Ge[j * r + lane] = al0;
      if (u1) Ge[j * r + lane + 64] = al1;
      const float m = wmax(fmaxf(al0, al1));
      const float P = m + __logf(wsum((u0 ? __expf(al0 - m) : 0.f) + (u1 ? __expf(al1 - m) : 0.f)));
      if (lane == 0) sP[wave][j] = P;
      loss += g_of(j) * P;
    }
    __builtin_amdgcn_wave_barrier();
    float ad0 = 0.f, ad1 = 0.f;                     // adjoint of alpha_{j+1}
    float nx0 = 0.f, nx1 = 0.f;                     // alpha_{j+1} - e_{j+1}
    for (int j = n - 1; j >= 0; --j) {
      const float P = sP[wave][j], g = g_of(j);
      const float cur0 = u0 ? Ge[j * r + lane] : ninf, cur1 = u1 ? Ge[j * r + lane + 64] : ninf;
      const float pi0 = u0 ? __expf(cur0 - P) : 0.f, pi1 = u1 ? __expf(cur1 - P) : 0.f;
      float n0 = g * pi0, n1 = g * pi1;
      if (j < n - 1) {
        const float pr0 = __expf(nx0 - P), pr1 = __expf(nx1 - P);          // predicted next state
        const float gm0 = (u0 && pr0 > 0.f) ? ad0 / pr0 : 0.f, gm1 = (u1 && pr1 > 0.f) ? ad1 / pr1 : 0.f;
        if (u0) sh[lane] = gm0;
        if (u1) sh[lane + 64] = gm1;
        __builtin_amdgcn_wave_barrier();
        float c0, c1;
        if (!a.contextual) {
          wave_matvec(lay_tr + j * lstep, sh, r, lane, c0, c1);            // (T_j gam)[z] via T_j^T
        } else {
          // this position's own transition matrix (natural layout only): lanes run over z',
          // the loop over z; (T gam)_z is a wave reduction, and the softmax backward of
          // pi_z T[z][z'] gam_z' is pi_z T[z][z'] (gam_z' - (T gam)_z), written along z'
          if (u0) sPi[wave][lane] = pi0;
          if (u1) sPi[wave][lane + 64] = pi1;
          __builtin_amdgcn_wave_barrier();
          const float* Tj = lay_nat + j * lstep;
          // one matrix per step: written once, in the dtype of h, straight into the logit-gradient
          // block; a matrix shared by the steps (or a caller's per-position buffer): fp32 accumulation
          const long long o = row * a.ld_dlog + (long long)j * r * r;
          float* acc32 = a.dlog32 ? a.dlog32 + row * (long long)a.L * r * r + j * lstep : nullptr;
          for (int z = 0; z < r; ++z) {
            const float t0 = u0 ? Tj[z * r + lane] : 0.f, t1 = u1 ? Tj[z * r + lane + 64] : 0.f;
            const float cz = wsum(t0 * gm0 + t1 * gm1);
            const float pz = sPi[wave][z];
            if (lane == 0) sC[wave][z] = cz;
            if (u0) {
              const float val = pz * t0 * (gm0 - cz);
              if (acc32) acc32[z * r + lane] += val;
              else if (a.bf16) ((unsigned short*)a.dlog)[o + z * r + lane] = to_bf16_rne(val);
              else ((float*)a.dlog)[o + z * r + lane] = val;
            }
            if (u1) {
              const float val = pz * t1 * (gm1 - cz);
              if (acc32) acc32[z * r + lane + 64] += val;
              else if (a.bf16) ((unsigned short*)a.dlog)[o + z * r + lane + 64] = to_bf16_rne(val);
              else ((float*)a.dlog)[o + z * r + lane + 64] = val;
            }
          }
          __builtin_amdgcn_wave_barrier();
          c0 = u0 ? sC[wave][lane] : 0.f;
          c1 = u1 ? sC[wave][lane + 64] : 0.f;
        }
        __builtin_amdgcn_wave_barrier();
        n0 += pi0 * c0;
        n1 += pi1 * c1;
        if (a.pi != nullptr) {
          float* pp = a.pi + (row * (n - 1) + j) * r;
          float* gp = a.gam + (row * (n - 1) + j) * r;
          if (u0) { pp[lane] = pi0; gp[lane] = gm0; }
          if (u1) { pp[lane + 64] = pi1; gp[lane + 64] = gm1; }
        }
      }
      nx0 = u0 ? cur0 - e[j * r + lane] : ninf;
      nx1 = u1 ? cur1 - e[j * r + lane + 64] : ninf;
      ad0 = n0; ad1 = n1;
      if (u0) Ge[j * r + lane] = n0;
      if (u1) Ge[j * r + lane + 64] = n1;
    }
    if (a.dlog != nullptr && a.dlog32 == nullptr)   // padding columns of the block
      for (int c = (n - 1) * r * r + lane; c < a.dlog_cols; c += 64) {
        if (a.bf16) ((unsigned short*)a.dlog)[row * a.ld_dlog + c] = 0;
        else ((float*)a.dlog)[row * a.ld_dlog + c] = 0.f;
      }
    const float tot = wsum((u0 ? ad0 : 0.f) + (u1 ? ad1 : 0.f));
    put_dsl(ad0 - __expf(w0) * tot, ad1 - __expf(w1) * tot);
    if (lane == 0) a.loss[row] = loss;
    return;
  }
}

// Binary tree (Eq. BTree), one wave per evidence row.  The forward pass walks the
// tree program (full node values bottom-up, then the path of every prefix) and keeps
// the output of every step; the reverse pass walks it backwards.  For a step
// c[k] = log sum_j A[k][j] exp(x[j]) with x the sum of its two operands:
//   xi[j] = exp(x[j] - max x),  delta[k] = adj(c)[k] exp(max x - c[k]),
//   adj(x)[j] = xi[j] sum_k A[k][j] delta[k],   d loss / d log A[k][j] = delta[k] A[k][j] xi[j],
// and adj(x) goes to both operands (leaf: evidence gradient; stored node: its
// adjoint; path value: the adjoint consumed by the previous step of the path).
__global__ __launch_bounds__(256) void k_btree_bwd(const CircuitBwdArgs a, int nsteps_max) {
  clear_ints(a);
  extern __shared__ TreeStep bprog[];
  __shared__ float sX[4][128];
  __shared__ float sPi[4][128];
  __shared__ int s_nsteps;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long long row = (long long)blockIdx.x * 4 + wave;
  const int n = a.n, r = a.r;
  const bool u0 = lane < r, u1 = lane + 64 < r;
  if (threadIdx.x == 0) s_nsteps = build_tree_program(bprog, n, 1);
  __syncthreads();
  const int T = s_nsteps;
  auto put_dsl = [&](float v0, float v1) {
    if (a.dslT == nullptr || row >= a.ldb) return;
    if (a.bf16) {
      unsigned short* d = (unsigned short*)a.dslT;
      if (u0) d[(long long)lane * a.ldb + row] = to_bf16_rne(v0);
      if (u1) d[(long long)(lane + 64) * a.ldb + row] = to_bf16_rne(v1);
    } else {
      float* d = (float*)a.dslT;
      if (u0) d[(long long)lane * a.ldb + row] = v0;
      if (u1) d[(long long)(lane + 64) * a.ldb + row] = v1;
    }
  };
  if (row >= a.rows) {
    put_dsl(0.f, 0.f);
    return;
  }
  const float ninf = neg_inf();
  const float* e = a.e + row * n * r;
  const float* coef = a.coef + row * n;
  float* Ge = a.Ge + row * n * r;
  float* ct = a.ct + row * nsteps_max * r;           // output of every step
  float* ad = a.adj + row * (long long)(n - 1) * r;   // adjoints of the stored node values
  float* sh = sX[wave];
  const float* lw = a.logw + row * r;
  const float w0 = u0 ? lw[lane] : ninf, w1 = u1 ? lw[lane + 64] : ninf;
  const long long lstep = a.L > 1 ? (long long)r * r : 0;
  const long long lrow = a.contextual ? row * a.L * r * r : 0;        // this position's own layers
  auto g_of = [&](int j) { return (j + 1 < n ? coef[j + 1] : 0.f) - coef[j]; };
  // value of an operand for the lane's two units; path values live in ct[t-1]
  auto operand = [&](int src, int t, float& x0, float& x1) {
    if (src == -2) { x0 = u0 ? 0.f : ninf; x1 = u1 ? 0.f : ninf; return; }
    const float* p;
    if (src == -1) p = ct + (long long)(t - 1) * r;
    else if (src >= n - 1) p = e + (long long)(src - (n - 1)) * r;
    else p = ct + (long long)(n - 2 - src) * r;      // node m is the output of up-pass step n-2-m
    x0 = u0 ? p[lane] : ninf;
    x1 = u1 ? p[lane + 64] : ninf;
  };

  // ---- forward
  float loss = 0.f;
  for (int t = 0; t < T; ++t) {
    const TreeStep st = bprog[t];
    float l0, l1, r0, r1;
    operand(st.lsrc, t, l0, l1);
    operand(st.rsrc, t, r0, r1);
    float x0 = l0 + r0, x1 = l1 + r1;
    if (st.m == 0) {
      x0 += w0; x1 += w1;
      const float m = wmax(fmaxf(x0, x1));
      const float P = m + __logf(wsum((u0 ? __expf(x0 - m) : 0.f) + (u1 ? __expf(x1 - m) : 0.f)));
      loss += g_of(-2 - st.out) * P;
      if (lane == 0) ct[(long long)t * r] = P;       // the root step keeps its scalar
      continue;
    }
    const float m = wmax(fmaxf(x0, x1));
    const float ms = m == ninf ? 0.f : m;
    if (u0) sh[lane] = __expf(x0 - ms);
    if (u1) sh[lane + 64] = __expf(x1 - ms);
    __builtin_amdgcn_wave_barrier();
    float s0, s1;
    if (!a.contextual) {
      wave_matvec(a.lay_tr + (st.m - 1) * lstep, sh, r, lane, s0, s1);     // sum_j A[k][j] xi[j] via A^T
    } else {
      // this position's own layer, natural layout only: lanes run over j, one wave reduction per k
      const float* A = a.lay_nat + lrow + (st.m - 1) * lstep;
      const float xa = u0 ? sh[lane] : 0.f, xb = u1 ? sh[lane + 64] : 0.f;
      s0 = s1 = 0.f;
      for (int k = 0; k < r; ++k) {
        const float v = wsum((u0 ? A[k * r + lane] * xa : 0.f) + (u1 ? A[k * r + lane + 64] * xb : 0.f));
        if (k == lane) s0 = v;
        if (k == lane + 64) s1 = v;
      }
    }
    __builtin_amdgcn_wave_barrier();
    if (u0) ct[(long long)t * r + lane] = ms + __logf(s0);
    if (u1) ct[(long long)t * r + lane + 64] = ms + __logf(s1);
  }
  // ---- reverse
  for (int idx = lane; idx < (n - 1) * r; idx += 64) ad[idx] = 0.f;
  for (int idx = lane; idx < n * r; idx += 64) Ge[idx] = 0.f;
  __builtin_amdgcn_wave_barrier();
  float gw0 = 0.f, gw1 = 0.f;                        // gradient w.r.t. log omega
  float pv0 = 0.f, pv1 = 0.f;                        // adjoint of the path value of the step above
  auto scatter = [&](int src, float a0, float a1) {
    if (src == -2) return;
    if (src == -1) { pv0 = a0; pv1 = a1; return; }
    float* p = src >= n - 1 ? Ge + (long long)(src - (n - 1)) * r : ad + (long long)(src - 1) * r;
    if (u0) p[lane] += a0;
    if (u1) p[lane + 64] += a1;
  };
  for (int t = T - 1; t >= 0; --t) {
    const TreeStep st = bprog[t];
    float l0, l1, r0, r1;
    operand(st.lsrc, t, l0, l1);
    operand(st.rsrc, t, r0, r1);
    float x0 = l0 + r0, x1 = l1 + r1;
    float xb0, xb1;                                  // adjoint of x
    if (st.m == 0) {
      const float P = ct[(long long)t * r], g = g_of(-2 - st.out);
      xb0 = u0 ? g * __expf(x0 + w0 - P) : 0.f;
      xb1 = u1 ? g * __expf(x1 + w1 - P) : 0.f;
      gw0 += xb0; gw1 += xb1;
    } else {
      float cb0, cb1;                                // adjoint of this step's output
      if (st.out >= 0) {
        cb0 = u0 ? ad[(long long)(st.out - 1) * r + lane] : 0.f;
        cb1 = u1 ? ad[(long long)(st.out - 1) * r + lane + 64] : 0.f;
      } else {
        cb0 = pv0; cb1 = pv1;
      }
      const float m = wmax(fmaxf(x0, x1));
      const float ms = m == ninf ? 0.f : m;
      const float xi0 = u0 ? __expf(x0 - ms) : 0.f, xi1 = u1 ? __expf(x1 - ms) : 0.f;
      const float c0 = u0 ? ct[(long long)t * r + lane] : 0.f, c1 = u1 ? ct[(long long)t * r + lane + 64] : 0.f;
      const float d0 = (u0 && cb0 != 0.f) ? cb0 * __expf(ms - c0) : 0.f;
      const float d1 = (u1 && cb1 != 0.f) ? cb1 * __expf(ms - c1) : 0.f;
      if (u0) sh[lane] = d0;
      if (u1) sh[lane + 64] = d1;
      __builtin_amdgcn_wave_barrier();
      float s0, s1;
      if (!a.contextual) {
        wave_matvec(a.lay_nat + (st.m - 1) * lstep, sh, r, lane, s0, s1);   // sum_k A[k][j] delta[k]
      } else {
        // one pass over this position's layer gives both sum_k A[k][j] delta[k] and the softmax
        // backward of its logits, delta_k A[k][j] (xi_j - (A xi)_k) with (A xi)_k = exp(c_k - max x),
        // accumulated in fp32 per position (a layer is applied by several steps)
        if (u0) sPi[wave][lane] = c0 == ninf ? 0.f : __expf(c0 - ms);
        if (u1) sPi[wave][lane + 64] = c1 == ninf ? 0.f : __expf(c1 - ms);
        __builtin_amdgcn_wave_barrier();
        const float* A = a.lay_nat + lrow + (st.m - 1) * lstep;
        float* dl = a.dlog32 + row * (long long)a.L * r * r + (st.m - 1) * lstep;
        s0 = s1 = 0.f;
        for (int k = 0; k < r; ++k) {
          const float dk = sh[k], sk = sPi[wave][k];
          if (u0) {
            const float w = A[k * r + lane];
            s0 = fmaf(w, dk, s0);
            dl[k * r + lane] += dk * w * (xi0 - sk);
          }
          if (u1) {
            const float w = A[k * r + lane + 64];
            s1 = fmaf(w, dk, s1);
            dl[k * r + lane + 64] += dk * w * (xi1 - sk);
          }
        }
      }
      __builtin_amdgcn_wave_barrier();
      xb0 = xi0 * s0; xb1 = xi1 * s1;
      if (a.pi != nullptr) {
        float* pp = a.pi + (row * nsteps_max + t) * r;
        float* gp = a.gam + (row * nsteps_max + t) * r;
        if (u0) { pp[lane] = d0; gp[lane] = xi0; }
        if (u1) { pp[lane + 64] = d1; gp[lane + 64] = xi1; }
      }
    }
    __builtin_amdgcn_wave_barrier();
    scatter(st.lsrc, xb0, xb1);
    scatter(st.rsrc, xb0, xb1);
    __builtin_amdgcn_wave_barrier();
  }
  const float tot = wsum((u0 ? gw0 : 0.f) + (u1 ? gw1 : 0.f));
  put_dsl(gw0 - __expf(w0) * tot, gw1 - __expf(w1) * tot);
  if (lane == 0) a.loss[row] = loss;
}

constexpr int BTREE_BWD_LDS = 156 * 1024;
// The same for shared layers of R = 16, 32 or 64 units, 16 evidence rows per workgroup and one wave per block of
// 16 units: a layer applied to 16 rows is a matrix product, A xi on the way up and A^T delta on the way back
// (v_mfma_f32_16x16x4_f32, the operand layout of k_btree_mfma: lane (row = l mod 16, g = l div 16) holds units
// 16 b + 4 g + i).  A path of the program (one prefix) is walked back as soon as its P_j is known, so that path
// values, node values and node adjoints all stay in LDS; node values are walked back at the end.  Every wave
// forms whole vectors where a product needs them and owns the 16 units it computed everywhere else: adjoints
// and gradients are added by their owner alone, in program order.
// Bound by its chain of dependent steps (the forward kernel's 1,700 cycles each, twice), not by the products or by
// memory; a lane per unit and a wave per row took 1.02 ms for 4,096 rows at R = 64, n = 16, this takes 0.24 ms.
struct BwdOp { short t, q; };   // program step; q: its place on a path (0 first), -1 - q: walked back

template <int R>
constexpr size_t btree_bwd_lds(int n, int T) {
  int lg = 0;
  while ((1 << lg) < n) ++lg;
  const size_t slots = 2 * (size_t)(n > 2 ? n - 2 : 0) + lg + 2;
  return slots * 16 * (R + 4) * 4 + (size_t)(n + lg) * 16 * 4 + (size_t)T * sizeof(TreeStep) + 2 * (size_t)T * sizeof(BwdOp);
}

template <int R>
__global__ __launch_bounds__(4 * R) void k_btree_bwd_mfma(const CircuitBwdArgs a, int nsteps_max) {
  clear_ints(a);
  typedef __attribute__((ext_vector_type(4))) float f32x4_t;
  constexpr int NB = R / 16, RS = R + 4;
  extern __shared__ __align__(16) float wsm[];
  __shared__ int s_nops;
  const int n = a.n, n2 = max(n - 2, 0);
  int lg = 0;
  while ((1 << lg) < n) ++lg;
  const int lane = threadIdx.x & 63, rl = lane & 15, g = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int own = 16 * wv + 4 * g;                   // first of this lane's four units
  float* val = wsm;                                  // [n-2] values of nodes 1 ..
  float* adj = val + (size_t)n2 * 16 * RS;           // [n-2] their adjoints
  float* path = adj + (size_t)n2 * 16 * RS;          // [lg] values of the current path
  float* padj = path + (size_t)lg * 16 * RS;         // [2] adjoint of the path value, alternating
  float* mxs = padj + (size_t)2 * 16 * RS;           // [n-2 + lg][16] row maxima of the steps' operands
  TreeStep* prog = (TreeStep*)(mxs + (size_t)(n + lg) * 16);
  BwdOp* ops = (BwdOp*)(prog + nsteps_max);
  if (threadIdx.x == 0) {
    const int T = build_tree_program(prog, n, 1);
    int k = 0;
    for (int t = 0; t < n2; ++t) ops[k++] = BwdOp{(short)t, 0};
    for (int t = n2; t < T;) {                       // a path: up to and with its root step, then back
      int e = t;
      while (prog[e].m != 0) ++e;
      for (int s = t; s <= e; ++s) ops[k++] = BwdOp{(short)s, (short)(s - t)};
      for (int s = e - 1; s >= t; --s) ops[k++] = BwdOp{(short)s, (short)(-1 - (s - t))};
      t = e + 1;
    }
    for (int t = n2 - 1; t >= 0; --t) ops[k++] = BwdOp{(short)t, -1};
    s_nops = k;
  }
  const long long row = (long long)blockIdx.x * 16 + rl;
  const bool live = row < a.rows;
  const long long rc = live ? row : (long long)a.rows - 1;       // clamped: loads stay in bounds
  const float* e = a.e + rc * n * R + 4 * g;
  const float* coef = a.coef + rc * n;
  float* Ge = a.Ge + rc * n * R + own;
  const size_t lstep = a.L > 1 ? (size_t)R * R : 0;
  const float* lay_n = a.lay_nat + (size_t)(16 * wv + rl) * R + 4 * g;
  const float* lay_t = a.lay_tr + (size_t)(16 * wv + rl) * R + 4 * g;
  const size_t at = (size_t)rl * RS;                 // this row inside a slot
  const float ninf = neg_inf();
  const f32x4_t zero = f32x4_t{0.f, 0.f, 0.f, 0.f};
  f32x4_t lw[NB], gw[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    lw[b] = *(const f32x4_t*)(a.logw + rc * R + 16 * b + 4 * g);
    gw[b] = zero;
  }
  for (int s = 0; s < n2; ++s) *(f32x4_t*)(adj + (size_t)s * 16 * RS + at + own) = zero;
  if (live)
    for (int i = 0; i < n; ++i) *(f32x4_t*)(Ge + (size_t)i * R) = zero;
  __syncthreads();
  const int nops = __builtin_amdgcn_readfirstlane(s_nops);

  // lanes l, l ^ 16, l ^ 32, l ^ 48 share a row
  auto across = [](float x, auto f) { x = f(x, __shfl_xor(x, 16)); return f(x, __shfl_xor(x, 32)); };
  auto fadd = [](float x, float y) { return x + y; };
  auto fmx = [](float x, float y) { return fmaxf(x, y); };
  // a step of the walk, the same for every lane: in scalar registers
  struct Op { int t, q, m, lsrc, rsrc, out; };
  auto read_op = [&](int k) {
    const int w = __builtin_amdgcn_readfirstlane(*(const int*)(ops + min(k, nops - 1)));
    Op o;
    o.t = (short)(w & 0xffff); o.q = w >> 16;
    const int2 raw = *(const int2*)(prog + o.t);
    const int w0 = __builtin_amdgcn_readfirstlane(raw.x), w1 = __builtin_amdgcn_readfirstlane(raw.y);
    o.m = (short)(w0 & 0xffff); o.lsrc = w0 >> 16; o.rsrc = (short)(w1 & 0xffff); o.out = w1 >> 16;
    return o;
  };
  // where the value an operand names sits (path values: the step before on the path)
  auto slot = [&](int src, int q) { return src == -1 ? path + (size_t)(q - 1) * 16 * RS : val + (size_t)(src - 1) * 16 * RS; };
  // layer rows and leaf evidence of the next step are fetched a step ahead
  f32x4_t An[NB], nl[NB], nr[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) An[b] = nl[b] = nr[b] = zero;
  auto prefetch = [&](int k, const Op& o) {
    if (k >= nops) return;
    if (o.lsrc >= n - 1) {
#pragma unroll
      for (int b = 0; b < NB; ++b) nl[b] = *(const f32x4_t*)(e + (size_t)(o.lsrc - (n - 1)) * R + 16 * b);
    }
    if (o.rsrc >= n - 1) {
#pragma unroll
      for (int b = 0; b < NB; ++b) nr[b] = *(const f32x4_t*)(e + (size_t)(o.rsrc - (n - 1)) * R + 16 * b);
    }
    if (o.m > 0) {
      const float* A = (o.q < 0 ? lay_t : lay_n) + (size_t)(o.m - 1) * lstep;
#pragma unroll
      for (int b = 0; b < NB; ++b) An[b] = *(const f32x4_t*)(A + 16 * b);
    }
  };
  float loss = 0.f;
  Op cur = read_op(0);
  prefetch(0, cur);
  for (int k = 0; k < nops; ++k) {
    const Op st = cur;
    const bool back = st.q < 0;
    const int q = back ? -1 - st.q : st.q;
    const bool up = st.t < n2;                       // a stored node (else: on a path, or its root)
    // the operands' sum
    f32x4_t x[NB], Ac[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      f32x4_t l = zero, r = zero;
      if (st.lsrc >= n - 1) l = nl[b];
      else if (st.lsrc != -2) l = *(const f32x4_t*)(slot(st.lsrc, q) + at + 16 * b + 4 * g);
      if (st.rsrc >= n - 1) r = nr[b];
      else if (st.rsrc != -2) r = *(const f32x4_t*)(slot(st.rsrc, q) + at + 16 * b + 4 * g);
      x[b] = l + r;
      Ac[b] = An[b];
    }
    cur = read_op(k + 1);
    prefetch(k + 1, cur);
    // adds the adjoint of x (this lane's four units) to an operand
    auto scatter = [&](int src, const f32x4_t& v) {
      if (src == -2) return;
      if (src == -1) *(f32x4_t*)(padj + (size_t)((q - 1) & 1) * 16 * RS + at + own) = v;
      else if (src >= n - 1) {
        if (live) *(f32x4_t*)(Ge + (size_t)(src - (n - 1)) * R) += v;
      } else *(f32x4_t*)(adj + (size_t)(src - 1) * 16 * RS + at + own) += v;
    };
    float* mslot = mxs + (size_t)(up ? st.m - 1 : n2 + q) * 16 + rl;
    if (!back) {
      if (st.m == 0) {
#pragma unroll
        for (int b = 0; b < NB; ++b) x[b] += lw[b];
      }
      float m = ninf;
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) m = fmaxf(m, x[b][i]);
      m = across(m, fmx);
      const float ms = (m == ninf) ? 0.f : m;
      if (st.m == 0) {
        // P_j = LSE(x), adjoint of x: g_j softmax(x); the root's weights take the same
        float sum = 0.f;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int i = 0; i < 4; ++i) sum += __expf(x[b][i] - m);
        const float P = m + __logf(across(sum, fadd));
        const int j = -2 - st.out;
        const float gj = (j + 1 < n ? coef[j + 1] : 0.f) - coef[j];
        loss += gj * P;
        f32x4_t mine = zero;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          f32x4_t v;
#pragma unroll
          for (int i = 0; i < 4; ++i) v[i] = gj * __expf(x[b][i] - P);
          gw[b] += v;
          if (b == wv) mine = v;
        }
        scatter(st.lsrc, mine);
        scatter(st.rsrc, mine);
      } else {
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int i = 0; i < 4; ++i) x[b][i] = __expf(x[b][i] - ms);
        f32x4_t S = zero;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int i = 0; i < 4; ++i) S = __builtin_amdgcn_mfma_f32_16x16x4f32(Ac[b][i], x[b][i], S, 0, 0, 0);
        f32x4_t res;
#pragma unroll
        for (int i = 0; i < 4; ++i) res[i] = ms + __logf(S[i]);
        *(f32x4_t*)((up ? val + (size_t)(st.m - 1) * 16 * RS : path + (size_t)q * 16 * RS) + at + own) = res;
        if (wv == 0 && g == 0) *mslot = ms;
      }
    } else {
      // delta = adj(c) exp(max - c), whole; xi = exp(x - max), this wave's units
      const float ms = *mslot;
      const float* cs = (up ? val + (size_t)(st.m - 1) * 16 * RS : path + (size_t)q * 16 * RS) + at;
      const float* bs = (up ? adj + (size_t)(st.m - 1) * 16 * RS : padj + (size_t)(q & 1) * 16 * RS) + at;
      f32x4_t S = zero, xi = zero, dmine = zero;
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const f32x4_t c = *(const f32x4_t*)(cs + 16 * b + 4 * g), cb = *(const f32x4_t*)(bs + 16 * b + 4 * g);
        f32x4_t d;
#pragma unroll
        for (int i = 0; i < 4; ++i) d[i] = cb[i] != 0.f ? cb[i] * __expf(ms - c[i]) : 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) S = __builtin_amdgcn_mfma_f32_16x16x4f32(Ac[b][i], d[i], S, 0, 0, 0);
        if (b == wv) {
          dmine = d;
#pragma unroll
          for (int i = 0; i < 4; ++i) xi[i] = __expf(x[b][i] - ms);
        }
      }
      if (a.pi != nullptr && live) {
        *(f32x4_t*)(a.pi + (row * nsteps_max + st.t) * R + own) = dmine;
        *(f32x4_t*)(a.gam + (row * nsteps_max + st.t) * R + own) = xi;
      }
      const f32x4_t xb = xi * S;
      scatter(st.lsrc, xb);
      scatter(st.rsrc, xb);
    }
    __syncthreads();
  }
  // the sum units' logits: G_z - omega_z sum G
  float tot = 0.f;
#pragma unroll
  for (int b = 0; b < NB; ++b) tot += (gw[b][0] + gw[b][1]) + (gw[b][2] + gw[b][3]);
  tot = across(tot, fadd);
  if (a.dslT != nullptr && row < a.ldb) {
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      if (b != wv) continue;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float v = live ? gw[b][i] - __expf(lw[b][i]) * tot : 0.f;
        const long long o = (long long)(own + i) * a.ldb + row;
        if (a.bf16) ((unsigned short*)a.dslT)[o] = to_bf16_rne(v); else ((float*)a.dslT)[o] = v;
      }
    }
  }
  if (live && wv == 0 && g == 0) a.loss[row] = loss;
}

template <int R>
static hipError_t launch_btree_bwd_mfma(const CircuitBwdArgs& a, int T, hipStream_t st) {
  const size_t lds = btree_bwd_lds<R>(a.n, T);
  if (hipError_t e = allow_lds<k_btree_bwd_mfma<R>>(BTREE_BWD_LDS); e != hipSuccess) return e;
  const long long rows = a.dslT ? a.ldb : a.rows;
  hipLaunchKernelGGL(k_btree_bwd_mfma<R>, dim3((unsigned)((rows + 15) / 16)), dim3(4 * R), lds, st, a, T);
  return hipGetLastError();
}

// 16 rows of a window fit in LDS up to n = 16 (32 at R = 16).
static bool btree_bwd_mfma_takes(const CircuitBwdArgs& a, int T) {
  if (a.contextual || a.lay_tr == nullptr || a.n > 64) return false;
  const size_t lds = a.r == 64 ? btree_bwd_lds<64>(a.n, T) : a.r == 32 ? btree_bwd_lds<32>(a.n, T) : a.r == 16 ? btree_bwd_lds<16>(a.n, T) : ~(size_t)0;
  return lds <= (size_t)BTREE_BWD_LDS;
}

// part[by][j][z][z'] = sum over the rows of block by of pi[b][j][z] * gam[b][j][z'] for step j.
// Thread t owns outputs t, t + 256, ...: NO of them.  Nothing is accumulated across workgroups
// here: k_layer_reduce adds the partial tiles in a fixed order, so that the layer gradients are
// the same bits on every run.
template <int NO>
__global__ __launch_bounds__(256) void k_layer_outer(const float* pi, const float* gam, int rows, int steps,
                                                     int r, int rows_per_block, float* part) {
  __shared__ float sp[16][128], sg[16][128];
  const int j = blockIdx.x, tid = threadIdx.x;
  const long long b0 = (long long)blockIdx.y * rows_per_block;
  const long long b1 = min((long long)rows, b0 + rows_per_block);
  float acc[NO];
#pragma unroll
  for (int q = 0; q < NO; ++q) acc[q] = 0.f;
  for (long long c0 = b0; c0 < b1; c0 += 16) {
    __syncthreads();
    for (int idx = tid; idx < 16 * r; idx += 256) {
      const long long b = c0 + idx / r;
      const int z = idx % r;
      const bool ok = b < b1;
      sp[idx / r][z] = ok ? pi[(b * steps + j) * r + z] : 0.f;
      sg[idx / r][z] = ok ? gam[(b * steps + j) * r + z] : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NO; ++q) {
      const int o = tid + q * 256;
      if (o < r * r) {
        const int z = o / r, zz = o - z * r;
        float s = 0.f;
#pragma unroll
        for (int t = 0; t < 16; ++t) s = fmaf(sp[t][z], sg[t][zz], s);
        acc[q] += s;
      }
    }
  }
  float* dst = part + ((long long)blockIdx.y * steps + j) * r * r;
#pragma unroll
  for (int q = 0; q < NO; ++q) {
    const int o = tid + q * 256;
    if (o < r * r) dst[o] = acc[q];
  }
}

// G[l][o] = sum over the steps j that apply layer l (ascending), and for each over the row blocks
// (ascending), of part[by][j][o].  HMM: step j applies layer j (layer 0 when one matrix is shared).
// Tree mode (tree_n > 0): step j applies the layer of node prog[j].m (root steps: none).
__global__ __launch_bounds__(256) void k_layer_reduce(const float* part, int steps, int nby, int r, int L,
                                                      float* G, int tree_n) {
  extern __shared__ TreeStep oprog[];
  __shared__ int s_cnt;
  const int rr = r * r;
  if (tree_n > 0) {
    if (threadIdx.x == 0) s_cnt = build_tree_program(oprog, tree_n, 1);
    __syncthreads();
  }
  const int nsteps = tree_n > 0 ? s_cnt : steps;
  const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (long long)L * rr) return;
  const int l = (int)(idx / rr), o = (int)(idx - (long long)l * rr);
  float s = 0.f;
  for (int j = 0; j < nsteps; ++j) {
    int layer = tree_n > 0 ? oprog[j].m - 1 : j;
    if (layer < 0) continue;
    if (L == 1) layer = 0;
    if (layer != l) continue;
    for (int by = 0; by < nby; ++by) s += part[((long long)by * steps + j) * rr + o];
  }
  G[idx] = s;
}

// softmax backward of every layer row: dlogit[l][z][:] = T (.) (G - sum_z' T G); one wave per row
__global__ __launch_bounds__(256) void k_layer_finish(const float* G, const float* T, int nrows, int r,
                                                      float* dlayers) {
  const int lane = threadIdx.x & 63;
  const long long row = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= nrows) return;
  const bool u0 = lane < r, u1 = lane + 64 < r;
  const float t0 = u0 ? T[row * r + lane] : 0.f, t1 = u1 ? T[row * r + lane + 64] : 0.f;
  const float g0 = u0 ? G[row * r + lane] : 0.f, g1 = u1 ? G[row * r + lane + 64] : 0.f;
  const float s = wsum(t0 * g0 + t1 * g1);
  if (u0) dlayers[row * r + lane] = t0 * (g0 - s);
  if (u1) dlayers[row * r + lane + 64] = t1 * (g1 - s);
}

// part[by][c] = sum_b src[b][c] over the rows of block by (src in the dtype of h, fp32 sums);
// k_colsum_reduce adds the blocks in ascending order (no atomics: the same bits on every run)
template <typename T>
__global__ __launch_bounds__(256) void k_colsum(const T* src, long long ld, int rows, int cols, float* part) {
  __shared__ float red[4][64];
  const int c = blockIdx.x * 64 + (threadIdx.x & 63), ty = threadIdx.x >> 6;
  const int b0 = blockIdx.y * 256;
  float s = 0.f;
  if (c < cols)
    for (int b = b0 + ty; b < min(rows, b0 + 256); b += 4) {
      if constexpr (sizeof(T) == 2) s += __uint_as_float(((unsigned)src[(long long)b * ld + c]) << 16);
      else s += src[(long long)b * ld + c];
    }
  red[ty][threadIdx.x & 63] = s;
  __syncthreads();
  if (ty == 0 && c < cols)
    part[(long long)blockIdx.y * cols + c] =
        (red[0][threadIdx.x] + red[1][threadIdx.x]) + (red[2][threadIdx.x] + red[3][threadIdx.x]);
}

__global__ __launch_bounds__(256) void k_colsum_reduce(const float* part, int nby, int cols, float* out) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= cols) return;
  float s = 0.f;
  for (int by = 0; by < nby; ++by) s += part[(long long)by * cols + c];
  out[c] = s;
}

// dst[b][c] (dtype of h, row stride ld) = src[b][c] for c < cols, 0 for cols <= c < cols_pad
template <typename T>
__global__ __launch_bounds__(256) void k_convert_block(const float* src, int rows, int cols, int cols_pad, T* dst,
                                                       long long ld) {
  const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
  if (t >= (long long)rows * cols_pad) return;
  const long long b = t / cols_pad;
  const int c = (int)(t - b * cols_pad);
  const float v = c < cols ? src[b * cols + c] : 0.f;
  if constexpr (sizeof(T) == 2) dst[b * ld + c] = to_bf16_rne(v); else dst[b * ld + c] = v;
}

__global__ __launch_bounds__(256) void k_fill_zero(float* p, long long n) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0.f;
}

}  // namespace

hipError_t launch_transpose(const TransposeArgs& a, int dtype, hipStream_t st) {
  if (a.C < 1 || a.Rpad < 1) return hipSuccess;
  const dim3 grid((a.C + 63) / 64, (a.Rpad + 63) / 64);
  if (a.along_rows) {
    if (dtype != MTPC_F32 || !a.planes || a.ld_src != a.C) return hipErrorInvalidValue;
    if (a.row0 >= a.Rpad) return hipSuccess;
    const char* src = (const char*)a.src + (long long)a.row0 * a.C * 4;
    return launch_split_rows(src, (char*)a.dst + a.row0 * 64LL, 1, a.Rpad - a.row0, a.C, a.C * 4LL, a.exps + a.row0, a.flag, 1, st, a.Rpad,
                             a.R - a.row0, a.src2, a.R2, 0, 1, a.cols);
  }
  if (a.planes) {
    if (a.live == nullptr || a.weights == nullptr) return hipErrorInvalidValue;
    if (dtype != MTPC_F32 || a.stage_rows != a.C || a.C % 16 != 0 || a.col0 != 0 || a.Rpad % 32 != 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_transpose_split, dim3(a.C / 16), dim3(512), 0, st, a, plane_exps(a.dst, (long long)a.C * a.Rpad));
    return hipGetLastError();
  }
  const int esz = dtype == MTPC_BF16 ? 2 : 4, ve = 16 / esz;
  const bool vec = a.ld_src % ve == 0 && a.ld_dst % ve == 0 && a.col0 % ve == 0 &&
                   (((uintptr_t)a.src | (uintptr_t)a.dst) & 15) == 0;
  if (vec) {
    if (dtype == MTPC_BF16) hipLaunchKernelGGL(k_transpose_vec<unsigned short>, grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL(k_transpose_vec<float>, grid, dim3(256), 0, st, a);
  } else {
    if (dtype == MTPC_BF16) hipLaunchKernelGGL(k_transpose<unsigned short>, grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL(k_transpose<float>, grid, dim3(256), 0, st, a);
  }
  return hipGetLastError();
}

hipError_t launch_grad_from_phi(const GradPhiArgs& a, int dtype, hipStream_t st) {
  const dim3 grid((unsigned)((a.ldb + 127) / 128), (unsigned)((a.ldM + 63) / 64));
  if (a.rows_only) {
    if (dtype != MTPC_BF16 || !a.staged) return hipErrorInvalidValue;
    const long long cols = (a.ldb + 127) / 128;
    int rows = 256;                                  // fewer where that leaves CUs without a workgroup
    while (rows > 16 && cols * ((a.ldM + rows - 1) / rows) < 1024) rows /= 2;
    const long long row_blocks = (a.ldM + rows - 1) / rows;
    const long long tail_blocks = ((a.ldM - a.tail_row) * (a.d / 8) + 256 * cols - 1) / (256 * cols);
    hipLaunchKernelGGL(k_grad_rows, dim3((unsigned)cols, (unsigned)(row_blocks + tail_blocks)), dim3(256), 0, st, a, rows, (int)row_blocks);
  } else if (dtype == MTPC_BF16) hipLaunchKernelGGL(k_grad_from_phi<unsigned short>, grid, dim3(256), 0, st, a, nullptr, nullptr);
  else if (a.planes) {
    hipLaunchKernelGGL((k_grad_from_phi<float, true>), grid, dim3(256), 0, st, a, a.rows, a.top);
  } else hipLaunchKernelGGL(k_grad_from_phi<float>, grid, dim3(256), 0, st, a, nullptr, nullptr);
  return hipGetLastError();
}

hipError_t launch_live_positions(const GradPhiArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(k_live_positions, dim3((a.B + 3) / 4), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_grad_exps(const GradPhiArgs& a, hipStream_t st) {
  const int rb = a.n * a.r * ((a.v + 63) / 64), bb = a.Mx > a.M ? (a.B + 15) / 16 : 0, chunks = (a.B + 511) / 512;
  // four workgroups per CU; two blocks of rows each as soon as that leaves one, since a position's atomic is what they share
  const long long all = (long long)rb * chunks;
  const int count = (int)std::min((long long)rb, std::max((all + 1023) / 1024, all >= 512 ? 2LL : 1LL));
  hipLaunchKernelGGL(k_grad_exps, dim3((rb + count - 1) / count + bb + 1, chunks), dim3(256), 0, st, a, rb, count);
  return hipGetLastError();
}

hipError_t launch_circuit_bwd(const CircuitBwdArgs& a, hipStream_t st) {
  const long long rows = a.dslT ? a.ldb : a.rows;
  const int r = a.r;
  const bool tree = a.family == MTPC_BTREE;
  const int T = tree ? tree_program_steps(a.n, 1) : a.n - 1;
  const size_t prog_bytes = tree ? (size_t)T * sizeof(TreeStep) : 0;
  const bool ctx = a.contextual && a.dlog != nullptr;        // layers computed from h (R): bias gradient = column sums
  const bool layers = !a.contextual && a.dlayers != nullptr && ((a.family == MTPC_HMM && a.n > 1) || (tree && a.n > 2));
  if (a.contextual && a.dlog32 != nullptr) {       // per-position fp32 accumulators
    const long long cnt = (long long)a.rows * a.L * r * r;
    hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, st, a.dlog32, cnt);
  }
  if (tree && btree_bwd_mfma_takes(a, T)) {
    const hipError_t e = r == 64 ? launch_btree_bwd_mfma<64>(a, T, st) : r == 32 ? launch_btree_bwd_mfma<32>(a, T, st)
                                                                                 : launch_btree_bwd_mfma<16>(a, T, st);
    if (e != hipSuccess) return e;
  } else if (tree) hipLaunchKernelGGL(k_btree_bwd, dim3((unsigned)((rows + 3) / 4)), dim3(256), prog_bytes, st, a, T);
  else hipLaunchKernelGGL(k_circuit_bwd, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st, a);
  if (layers) {
    const int steps = T, rpb = LAYER_GRAD_ROWS;
    const int nby = (a.rows + rpb - 1) / rpb;
    const dim3 grid(steps, (unsigned)nby);
    const int no = (r * r + 255) / 256;
    if (no <= 1) hipLaunchKernelGGL(k_layer_outer<1>, grid, dim3(256), 0, st, a.pi, a.gam, a.rows, steps, r, rpb, a.Gpart);
    else if (no <= 4) hipLaunchKernelGGL(k_layer_outer<4>, grid, dim3(256), 0, st, a.pi, a.gam, a.rows, steps, r, rpb, a.Gpart);
    else if (no <= 16) hipLaunchKernelGGL(k_layer_outer<16>, grid, dim3(256), 0, st, a.pi, a.gam, a.rows, steps, r, rpb, a.Gpart);
    else hipLaunchKernelGGL(k_layer_outer<64>, grid, dim3(256), 0, st, a.pi, a.gam, a.rows, steps, r, rpb, a.Gpart);
    const long long cnt = (long long)a.L * r * r;
    hipLaunchKernelGGL(k_layer_reduce, dim3((unsigned)((cnt + 255) / 256)), dim3(256), prog_bytes, st, a.Gpart, steps, nby,
                       r, a.L, a.G, tree ? a.n : 0);
    const int nrows = a.L * r;
    hipLaunchKernelGGL(k_layer_finish, dim3((nrows + 3) / 4), dim3(256), 0, st, a.G, a.lay_nat, nrows, r, a.dlayers);
  }
  if (ctx && a.dlog32 != nullptr) {
    const int cols = a.L * r * r;
    const long long cnt = (long long)a.rows * a.dlog_cols;
    const dim3 g((unsigned)((cnt + 255) / 256));
    if (a.bf16) hipLaunchKernelGGL(k_convert_block<unsigned short>, g, dim3(256), 0, st, a.dlog32, a.rows, cols,
                                   a.dlog_cols, (unsigned short*)a.dlog, a.ld_dlog);
    else hipLaunchKernelGGL(k_convert_block<float>, g, dim3(256), 0, st, a.dlog32, a.rows, cols, a.dlog_cols,
                            (float*)a.dlog, a.ld_dlog);
  }
  if (ctx && a.dlayers != nullptr) {               // bias gradient = column sums of the logit gradients
    const int cols = a.L * r * r;
    const int nby = (a.rows + LAYER_GRAD_ROWS - 1) / LAYER_GRAD_ROWS;
    const dim3 grid((cols + 63) / 64, nby);
    if (a.bf16) hipLaunchKernelGGL(k_colsum<unsigned short>, grid, dim3(256), 0, st, (const unsigned short*)a.dlog,
                                   a.ld_dlog, a.rows, cols, a.Gpart);
    else hipLaunchKernelGGL(k_colsum<float>, grid, dim3(256), 0, st, (const float*)a.dlog, a.ld_dlog, a.rows, cols,
                            a.Gpart);
    hipLaunchKernelGGL(k_colsum_reduce, dim3((cols + 255) / 256), dim3(256), 0, st, a.Gpart, nby, cols, a.dlayers);
  }
  return hipGetLastError();
}

}  // namespace mtpc
