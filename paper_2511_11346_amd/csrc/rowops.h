// Operations on the r <= 64 units of one row (position, window), one unit to a lane, that the kernels of few rows share: reductions
// over the units and products with an r x r layer, by groups of G * P lanes of one wave.
#pragma once

#include "mtpc_internal.h"

namespace mtpc {

// G: r rounded up to a power of two, at least 8.  Lane (k, part) = (lane % G, lane / G) of a group holds unit k, every part the same;
// P parts share the terms of a product.
template <int G, int P>
struct RowOps {
  static_assert(P == 64 / G || P == 1, "a wave, or groups of G lanes");
  static constexpr int JP = G / P;                       // terms of an output that a lane sums
  // a lane's share of a layer in registers before the operand is there; 64 units: from LDS beside it
  static constexpr bool AHEAD = JP <= 16;
  struct Weights { float w[AHEAD ? JP : 1]; const float* p; };

  static __device__ __forceinline__ void both16(float x, float& p, float& q) {
    const auto t = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    p = __uint_as_float(t[0]); q = __uint_as_float(t[1]);
  }
  static __device__ __forceinline__ void both32(float x, float& p, float& q) {
    const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    p = __uint_as_float(t[0]); q = __uint_as_float(t[1]);
  }
  template <class Op>
  static __device__ __forceinline__ float over_units(float x, Op op) {
    x = op(x, __int_as_float(dpp_move<0xB1>(__float_as_int(x))));     // (as group_reduce)
    x = op(x, __int_as_float(dpp_move<0x4E>(__float_as_int(x))));
    x = op(x, __int_as_float(dpp_move<0x141>(__float_as_int(x))));
    if constexpr (G >= 16) x = op(x, __int_as_float(dpp_move<0x140>(__float_as_int(x))));
    if constexpr (G >= 32) { float p, q; both16(x, p, q); x = op(p, q); }
    if constexpr (G >= 64) { float p, q; both32(x, p, q); x = op(p, q); }
    return x;
  }
  static __device__ __forceinline__ float sum_units(float x) { return over_units(x, [](float y, float z) { return y + z; }); }
  static __device__ __forceinline__ float max_units(float x) { return over_units(x, [](float y, float z) { return fmaxf(y, z); }); }
  static __device__ __forceinline__ float sum_parts(float x) {
    if constexpr (P > 1) {
      if constexpr (G <= 8) x += __int_as_float(dpp_move<0x128>(__float_as_int(x)));    // row_ror:8
      if constexpr (G <= 16) { float p, q; both16(x, p, q); x = p + q; }
      if constexpr (G <= 32) { float p, q; both32(x, p, q); x = p + q; }
    }
    return x;
  }

  // Lane (k, part)'s weights of the outputs sum_j x_j W(j, k): element (j, k) is at Wl[j * sj + k * sk].  What multiplies no unit: any.
  static __device__ __forceinline__ Weights weights(const float* Wl, int k, int part, int r, int sj, int sk) {
    Weights o;
    o.p = Wl + min(k, r - 1) * sk;
    if constexpr (AHEAD) {
#pragma unroll
      for (int u = 0; u < JP; ++u) o.w[u] = o.p[min(part + P * u, r - 1) * sj];
    }
    return o;
  }
  // That product; x is unit k's, 0 for k >= r.  xs: G * P floats of LDS of the group's own, 16-byte aligned
  static __device__ __forceinline__ float product(float x, const Weights& w, float* xs, int k, int part, int r, int sj) {
    if (part == 0) xs[(k % P) * JP + k / P] = x;
    __builtin_amdgcn_wave_barrier();
    constexpr int C = JP < 4 ? JP : 4, U = JP < 16 ? JP : 16;          // sums side by side; terms at a time
    float acc[C];
#pragma unroll
    for (int c = 0; c < C; ++c) acc[c] = 0.f;
#pragma unroll 1
    for (int u0 = 0; u0 < JP; u0 += U) {
      float xv[U], wv[U];
#pragma unroll
      for (int u = 0; u < U; u += C) {
        if constexpr (C == 4) {
          typedef __attribute__((ext_vector_type(4))) float vec4_t;
          const vec4_t t = *(const vec4_t*)(xs + part * JP + u0 + u);
#pragma unroll
          for (int c = 0; c < 4; ++c) xv[u + c] = t[c];
        } else {
          xv[u] = xs[part * JP + u0 + u];
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) wv[u] = AHEAD ? w.w[AHEAD ? u : 0] : w.p[min(part + P * (u0 + u), r - 1) * sj];
#pragma unroll
      for (int u = 0; u < U; ++u) acc[u % C] = fmaf(xv[u], wv[u], acc[u % C]);
    }
    __builtin_amdgcn_wave_barrier();
    float y = acc[0];
    if constexpr (C == 4) y = (acc[0] + acc[1]) + (acc[2] + acc[3]);
    return sum_parts(y);
  }
};

// The HMM's forward message on linear values: x_k 2^exponent times the exponentials of what has been taken out of it before.  Its values
// sum to 2^ROW_SCALE .. 2^(ROW_SCALE + 1), and the exponentials of the evidence, relative to its largest, come times 2^ROW_EVIDENCE: no
// result overflows, and units down to 2^-126 of the largest keep their precision through a step, which is what a chain of logarithms
// whose products are formed relative to the largest unit keeps.
constexpr int ROW_SCALE = 32, ROW_EVIDENCE = 64;
// exp(d) 2^scale, d <= 0: the scale goes in before a small exponential underflows
__device__ __forceinline__ float scaled_exp(float d, int scale) {
  const bool low = d < -64.f;
  const float t = __builtin_amdgcn_ldexpf(expf(low ? 0.5f * d : d), low ? scale / 2 : scale);
  return low ? t * t : t;
}
// values c with sum s > 0 to the message's scale; 2^shift is what they were multiplied with
__device__ __forceinline__ float to_row_scale(float c, float s, int& shift) {
  shift = s > 0.f ? ROW_SCALE + 1 - __builtin_amdgcn_frexp_expf(s) : 0;
  return __builtin_amdgcn_ldexpf(c, shift);
}
// The first observation, out of logarithms: root weights and evidence may be further apart than any linear values reach, and yet
// make up for each other.  lw, e: unit k's.  Returns the scaled message, its sum before the scaling in s (whose exponent is `exponent`
// still), what it was scaled by in `shift` and the largest logarithm in `taken`.
template <class Ops>
__device__ __forceinline__ float observe_first(float lw, float e, bool live, float& s, int& exponent, int& shift, float& taken) {
  const double l = (double)lw + (double)e;                   // (one rounding, of what is left relative to the largest)
  const float most = Ops::max_units(live ? (float)l : neg_inf());
  taken = most == neg_inf() ? 0.f : most;
  const float c = live ? scaled_exp((float)(l - (double)taken), ROW_SCALE) : 0.f;
  s = Ops::sum_units(c);
  exponent = -ROW_SCALE;
  return to_row_scale(c, s, shift);
}
// One observation: y (unit k's, 0 for k >= r) times exp(evidence).  ew: exp(evidence - its maximum `taken`) 2^ROW_EVIDENCE, e: the
// evidence itself.  The rest as above.
template <class Ops>
__device__ __forceinline__ float observe(float y, float ew, float e, bool live, float& s, int& exponent, int& shift, float& taken) {
  float c = live ? y * ew : 0.f;
  s = Ops::sum_units(c);
  exponent -= ROW_EVIDENCE;
  if (s < 0x1p40f) {
    // the units that are left have next to none of the evidence (or none: nothing is left of the row): exponentials relative to
    // the largest product.  (From 2^40 on what a linear evidence of less than 2^-126 makes of a unit, 2^-93 at the most, is
    // less than 2^-126 of the largest.)
    const float l = live && y > 0.f ? logf(y) + e : neg_inf();
    const float most = Ops::max_units(l);
    if (most != neg_inf()) {
      c = scaled_exp(l - most, ROW_SCALE);
      s = Ops::sum_units(c);
      exponent += ROW_EVIDENCE - ROW_SCALE;
      taken = most;
    }
  }
  return to_row_scale(c, s, shift);
}

}  // namespace mtpc
