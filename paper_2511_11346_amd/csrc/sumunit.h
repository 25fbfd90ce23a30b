// Sum-unit weights of one position (Sec. 3.3: log omega = log_softmax(Wsum h)), as a piece of
// device code that the kernels needing them for a handful of positions share: the stand-alone
// kernel, the one that goes on to draw the latents, and the verification step.
#pragma once

#include "mtpc_internal.h"

namespace mtpc {

typedef __attribute__((ext_vector_type(4))) int i32x4_t;

// dot of two rows of 8-element (bf16) or 4-element (fp32) 16-byte chunks
template <bool BF16>
__device__ __forceinline__ float dot_chunk(const i32x4_t& a, const i32x4_t& b) {
  float s = 0.f;
  if constexpr (BF16) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const uint32_t ua = (uint32_t)a[t], ub = (uint32_t)b[t];
      s = fmaf(__uint_as_float(ua << 16), __uint_as_float(ub << 16), s);
      s = fmaf(__uint_as_float(ua & 0xFFFF0000u), __uint_as_float(ub & 0xFFFF0000u), s);
    }
  } else {
#pragma unroll
    for (int t = 0; t < 4; ++t) s = fmaf(__int_as_float(a[t]), __int_as_float(b[t]), s);
  }
  return s;
}

// Loads out of one row of `bytes` bytes whose address is the same in all lanes: an offset of 32 bits per lane is all that stands in
// vector registers (addresses of 64 bits for each of 24 loads in flight did not fit beside them), and what lies behind the row
// reads as zero.
struct RowLoad {
  __amdgpu_buffer_rsrc_t rsrc;
  __device__ __forceinline__ RowLoad(const char* row, int bytes) : rsrc(__builtin_amdgcn_make_buffer_rsrc((void*)row, 0, bytes, 0x00020000)) {}
  __device__ __forceinline__ i32x4_t operator()(int offset) const {
    return __builtin_bit_cast(i32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rsrc, offset, 0, 0));
  }
};

// log omega[b][:] into sc[0..r) (LDS, 128 floats) by a workgroup of NW waves: they split the r rows
// of Wsum, the position's hidden vector stays in registers (up to 8 chunks of 16 bytes per lane per
// pass: d <= 4096 bf16 / 2048 fp32 in one pass), Q rows at a time so that many loads are in flight
// (a workgroup that does nothing else takes 16 waves: one compute unit then has all of a 32 x 4096
// Wsum in flight at once instead of in two rounds).  Ends with a barrier: every thread may read sc
// afterwards.
template <bool BF16, int NW = 4>
__device__ __forceinline__ void sumunit_position(const void* h, long long ld_h, const void* Wsum, int b, int d, int r,
                                                 float* sc) {
  constexpr int ESZ = BF16 ? 2 : 4;
  constexpr int EPC = 16 / ESZ;
  constexpr int Q = NW > 8 ? 2 : 4;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const char* hb = (const char*)h + (long long)b * ld_h * ESZ;
  const int nch = d / EPC;
  for (int c0 = 0; c0 < nch; c0 += 512) {
    const int at = (c0 + lane) * 16;
    i32x4_t hv[8];
    const RowLoad hl(hb, d * ESZ);
#pragma unroll
    for (int t = 0; t < 8; ++t) hv[t] = hl(at + t * 1024);
    for (int j0 = wave * Q; j0 < r; j0 += NW * Q) {
      // all of the loads in flight together, which the barrier behind them makes the compiler keep to (it waited for one after the
      // other: the logits of one draft, k_rows_logits below a CP, 16.2 -> 8.3 us)
      i32x4_t wv[Q][8];
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const RowLoad wl((const char*)Wsum + (long long)min(j0 + q, r - 1) * d * ESZ, d * ESZ);
#pragma unroll
        for (int t = 0; t < 8; ++t) wv[q][t] = wl(at + t * 1024);
      }
      __builtin_amdgcn_sched_barrier(0);
      float acc[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        acc[q] = 0.f;
#pragma unroll
        for (int t = 0; t < 8; ++t) asm volatile("" : "+v"(hv[t]));      // (its halves taken apart anew, not kept over the rows: 64 registers)
#pragma unroll
        for (int t = 0; t < 8; ++t) acc[q] += dot_chunk<BF16>(wv[q][t], hv[t]);
      }
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const float v = group_sum(acc[q], 64);
        if (lane == 0 && j0 + q < r) { if (c0 == 0) sc[j0 + q] = v; else sc[j0 + q] += v; }
      }
    }
  }
  __syncthreads();
  if (wave == 0) {
    const float s0 = lane < r ? sc[lane] : neg_inf();
    const float s1 = lane + 64 < r ? sc[lane + 64] : neg_inf();
    const float m = group_max(fmaxf(s0, s1), 64);
    float e = 0.f;
    if (s0 > neg_inf()) e += __expf(s0 - m);
    if (s1 > neg_inf()) e += __expf(s1 - m);
    e = group_sum(e, 64);
    const float lse = m + __logf(e);
    if (lane < r) sc[lane] = s0 - lse;
    if (lane + 64 < r) sc[lane + 64] = s1 - lse;
  }
  __syncthreads();
}

// softmax over the last axis of one row (of one r x r layer) of the sum layers, by a wave: row k of layer l of position block b,
// counted through all nb * L * r of them; the natural copy [k][j], the transposed one [j][k], or both
__device__ __forceinline__ void normalise_layer_row(const float* logits, long long ls, long long bs, long long row, int L, int r,
                                                    float* out_nat, float* out_tr) {
  const int lane = threadIdx.x & 63;
  const int k = (int)(row % r);
  const int l = (int)((row / r) % L);
  const long long b = row / ((long long)r * L);
  const float* src = logits + b * bs + (long long)l * ls + (long long)k * r;
  const float x0 = lane < r ? src[lane] : neg_inf();
  const float x1 = lane + 64 < r ? src[lane + 64] : neg_inf();
  const float m = group_max(fmaxf(x0, x1), 64);
  const float ms = (m == neg_inf()) ? 0.f : m;
  const float e0 = x0 > neg_inf() ? expf(x0 - ms) : 0.f;
  const float e1 = x1 > neg_inf() ? expf(x1 - ms) : 0.f;
  const float tot = group_sum(e0 + e1, 64);
  const float inv = tot > 0.f ? 1.f / tot : 0.f;
  const long long base = (b * L + l) * (long long)r * r;
  if (out_nat) {
    if (lane < r) out_nat[base + (long long)k * r + lane] = e0 * inv;
    if (lane + 64 < r) out_nat[base + (long long)k * r + lane + 64] = e1 * inv;
  }
  if (out_tr) {
    if (lane < r) out_tr[base + (long long)lane * r + k] = e0 * inv;
    if (lane + 64 < r) out_tr[base + (long long)(lane + 64) * r + k] = e1 * inv;
  }
}

// What stands beside the sum units in the launch of a call's parameters: workgroup w of those behind theirs, NT threads each.
constexpr int PARAM_COPIES = 4, PARAM_CLEARS = 16;       // 16-byte pieces of h, and ints, of a thread
inline __host__ __device__ long long param_blocks_copy(const ParamArgs& p, int NT) {
  return p.hs == nullptr ? 0 : ((long long)p.B * (p.row_bytes / 16) + NT * PARAM_COPIES - 1) / (NT * PARAM_COPIES);
}
inline __host__ __device__ long long param_blocks_layers(const ParamArgs& p, int NT) { return ((long long)p.nb * p.L * p.r + NT / 64 - 1) / (NT / 64); }
inline long long param_blocks(const ParamArgs& p, int NT) {
  return param_blocks_copy(p, NT) + param_blocks_layers(p, NT) + (p.nclear + NT * PARAM_CLEARS - 1) / (NT * PARAM_CLEARS);
}
template <int NT>
__device__ __forceinline__ void params_beside(const ParamArgs& p, long long w) {
  const int tid = threadIdx.x;
  const long long copies = param_blocks_copy(p, NT), layers = param_blocks_layers(p, NT);
  if (w < copies) {
    // (as k_pack_rows: neighbouring threads read 64 bytes of neighbouring rows and write one run)
    const long long total = (long long)p.B * (p.row_bytes / 16);
    const long long t0 = w * (NT * PARAM_COPIES) + tid;
    const unsigned stage_chunks = (unsigned)p.B * 4;
    const long long row_stride = p.ld_h * (p.row_bytes / p.d);
    i32x4_t x[PARAM_COPIES];
#pragma unroll
    for (int c = 0; c < PARAM_COPIES; ++c) {
      const unsigned t = (unsigned)min(t0 + c * NT, total - 1);      // (of less than 4 GiB of h)
      const unsigned stage = t / stage_chunks, u = t - stage * stage_chunks;
      x[c] = *(const i32x4_t*)((const char*)p.h + (long long)(u >> 2) * row_stride + (long long)stage * 64 + (u & 3) * 16);
    }
#pragma unroll
    for (int c = 0; c < PARAM_COPIES; ++c)
      if (t0 + c * NT < total) *(i32x4_t*)((char*)p.hs + (t0 + c * NT) * 16) = x[c];
  } else if (w < copies + layers) {
    const long long row = (w - copies) * (NT / 64) + (tid >> 6);
    if (row < (long long)p.nb * p.L * p.r) normalise_layer_row(p.logits, p.layer_stride, p.batch_stride, row, p.L, p.r, p.out_nat, p.out_tr);
  } else {
    const long long t0 = (w - copies - layers) * (NT * PARAM_CLEARS) + tid;
#pragma unroll
    for (int c = 0; c < PARAM_CLEARS; ++c)
      if (t0 + c * NT < p.nclear) p.clear[t0 + c * NT] = 0;
  }
}

}  // namespace mtpc
