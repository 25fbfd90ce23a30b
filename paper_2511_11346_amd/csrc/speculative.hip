// Verification step of a speculative-decoding cycle (Alg. 2 from the acceptance
// loop on, and the greedy variant of Sec. 3.4).  One workgroup per position:
//   1. the acceptance tests, all at once (the conditional of a drafted token is a
//      difference of two prefix log-marginals), first failure = rejected position j;
//   2. the circuit's conditional q(. | x_1..x_j) over the whole vocabulary: a
//      mixture of the input units of position j whose weights lambda are the
//      circuit's message into that leaf given the accepted tokens (CP: posterior
//      of the component; HMM: one-step prediction of the forward message; binary
//      tree: product of layer-transposed messages down the path to the leaf, with
//      fully observed left siblings evaluated bottom-up and right siblings = 1);
//   3. one draw from max(0, p - q) / Z (or from p after n acceptances).
// Everything is O(n r^2 + r v) per position and latency-bound: k_verify_row fetches
// whatever a rejection may need before it knows where there is one; k_verify, where
// that does not fit, spreads a matrix-vector product over all 256 threads so that every
// layer costs one memory round trip.
#include <algorithm>
#include <climits>

#include "mtpc_internal.h"
#include "rowops.h"
#include "sumunit.h"

namespace mtpc {
namespace {

// Draft index of the verification step's random numbers: drafting calls use 0 .. S-1 with S a
// signed 32-bit count, so this counter word is never theirs and equal (seed, offset) cannot hand
// an acceptance test the uniform that drew the token it tests.
constexpr uint32_t VERIFY_DRAFT_INDEX = 0xffffffffu;

__device__ __forceinline__ float wmax(float x) { return group_max(x, 64); }
__device__ __forceinline__ float wsum(float x) { return group_sum(x, 64); }
// block-wide reductions of 256 threads; `red` holds 4 floats
__device__ __forceinline__ float block_max(float x, float* red) {
  x = wmax(x);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  return fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}
__device__ __forceinline__ float block_sum(float x, float* red) {
  x = wsum(x);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

// out[t] = log sum_k exp(c[k]) M[k*r + t] for t = threadIdx.x < r (others get -inf).
// c: r log-domain values in LDS; M: r x r linear probabilities in global memory,
// t contiguous.  The 256 threads form 256/G column groups that split the k range,
// sixteen loads in flight each.  x (128), part (256), red (4) are LDS scratch.
__device__ float matvec_log(const float* c, const float* __restrict__ M, int r, int G, float* x, float* part,
                            float* red) {
  const int tid = threadIdx.x;
  const float mx = block_max(tid < r ? c[tid] : neg_inf(), red);
  const float ms = (mx == neg_inf()) ? 0.f : mx;
  if (tid < r) x[tid] = __expf(c[tid] - ms);
  __syncthreads();
  const int parts = 256 / G, t = tid % G, pt = tid / G;
  const int per = (r + parts - 1) / parts;
  const int k0 = pt * per, k1 = min(r, k0 + per);
  const int tc = min(t, r - 1);
  float acc = 0.f;
  for (int kb = k0; kb < k1; kb += 16) {
    float w[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) w[u] = M[(long long)min(kb + u, r - 1) * r + tc];
#pragma unroll
    for (int u = 0; u < 16; ++u)
      if (kb + u < k1) acc = fmaf(x[kb + u], w[u], acc);
  }
  part[tid] = acc;
  __syncthreads();
  float s = 0.f;
  if (tid < r)
    for (int q = 0; q < parts; ++q) s += part[q * G + tid];
  return tid < r ? ms + __logf(s) : neg_inf();          // log 0 = -inf
}

// The same product in two halves, for chains of products whose layers are known in advance:
// mv_load fetches this thread's 16 weights of a layer (its column t, its part of the k range;
// needs ceil(r / (256 / G)) <= 16), mv_apply multiplies.  Loading the next layer before
// applying the current one takes the L2 round trip out of the chain.
struct MvWeights { float w[16]; };

__device__ __forceinline__ void mv_load(const float* __restrict__ M, int r, int G, MvWeights& o) {
  const int tid = threadIdx.x, parts = 256 / G, t = tid % G, pt = tid / G;
  const int per = (r + parts - 1) / parts, k0 = pt * per, tc = min(t, r - 1);
#pragma unroll
  for (int u = 0; u < 16; ++u) o.w[u] = M[(long long)min(k0 + u, r - 1) * r + tc];
}

__device__ float mv_apply(const float* c, const MvWeights& wt, int r, int G, float* x, float* part, float* red) {
  const int tid = threadIdx.x;
  const float mx = block_max(tid < r ? c[tid] : neg_inf(), red);
  const float ms = (mx == neg_inf()) ? 0.f : mx;
  if (tid < r) x[tid] = __expf(c[tid] - ms);
  __syncthreads();
  const int parts = 256 / G, pt = tid / G;
  const int per = (r + parts - 1) / parts;
  const int k0 = pt * per, k1 = min(r, k0 + per);
  float acc = 0.f;
#pragma unroll
  for (int u = 0; u < 16; ++u)
    if (k0 + u < k1) acc = fmaf(x[k0 + u], wt.w[u], acc);
  part[tid] = acc;
  __syncthreads();
  float s = 0.f;
  if (tid < r)
    for (int q = 0; q < parts; ++q) s += part[q * G + tid];
  return tid < r ? ms + __logf(s) : neg_inf();          // log 0 = -inf
}

// Greedy verification: the most likely token of every row of p (smallest id on ties), accepted up to the first one
// that differs from the draft.  One wave per row (16 waves: the last of 17 rows at n = 16 follows in a second pass), a
// row's loads in flight together: bound by those cold reads (four waves took the n + 1 rows in turn, inside k_verify:
// 10.9 -> 4.3 us at n = 16, v = 320).
__global__ __launch_bounds__(1024) void k_verify_greedy(const VerifyArgs a) {
  __shared__ int s_arg[65];
  const int b = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const int n = a.n, v = a.v;
  const int drafted = a.drafts[(long long)b * n + min(lane, n - 1)];
  for (int s = wave; s <= n; s += nw) {
    const float* row = a.p + ((long long)b * (n + 1) + s) * v;
    float x[5];                                              // v <= 320
#pragma unroll
    for (int q = 0; q < 5; ++q) x[q] = row[min(lane + 64 * q, v - 1)];
    float best = neg_inf();
    int arg = INT_MAX;
#pragma unroll
    for (int q = 0; q < 5; ++q)
      if (lane + 64 * q < v && x[q] > best) { best = x[q]; arg = lane + 64 * q; }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      const float ob = __shfl_xor(best, o);
      const int oa = __shfl_xor(arg, o);
      if (ob > best || (ob == best && oa < arg)) { best = ob; arg = oa; }
    }
    if (lane == 0) s_arg[s] = arg == INT_MAX ? 0 : arg;
  }
  __syncthreads();
  if (wave == 0) {
    const bool rej = lane < n && drafted != s_arg[min(lane, n - 1)];
    const unsigned long long m = __ballot(rej);
    const int j = m ? __ffsll((long long)m) - 1 : n;
    if (lane == 0) { a.accepted[b] = j; a.token[b] = s_arg[j]; }
  }
}

__global__ __launch_bounds__(256) void k_verify(const VerifyArgs a, int G) {
  extern __shared__ float vsm[];
  __shared__ float s_red[4], s_x[128], s_c[128], s_part[256], s_ratio[64], s_alpha[64];
  __shared__ int s_j, s_lo, s_hi;
  __shared__ float s_lw[128];
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = a.n, r = a.r, v = a.v;
  float* s_e = vsm;                                          // [n][r] evidence of the drafted tokens
  float* s_nodes = s_e + n * r;                              // [n-1][r] binary tree: node values
  float* s_m = s_nodes + (a.family == MTPC_BTREE ? (n - 1) * r : 0);   // [v] weights of the final draw
  const int* x = a.drafts + (long long)b * n;
  const float* phi = a.logphi + (long long)b * n * r * v;
  const float* pv = a.p + (long long)b * (n + 1) * v;
  // ids outside [0, v) are the caller's error; clamping keeps every access in bounds
  auto tok_at = [&](int i) { return min(max(x[i], 0), v - 1); };

  // ---- 1. acceptance tests ---------------------------------------------------
  if (tid < n) {
    const float lq = a.prefix[(long long)b * n + tid] - (tid > 0 ? a.prefix[(long long)b * n + tid - 1] : 0.f);
    s_ratio[tid] = pv[(long long)tid * v + tok_at(tid)] / __expf(lq);
    s_alpha[tid] = philox_uniform(a.seed_lo, a.seed_hi, a.offset, (uint32_t)b, VERIFY_DRAFT_INDEX, (uint32_t)tid);
  }
  __syncthreads();
  if (wave == 0) {
    const bool rej = lane < n && s_alpha[min(lane, n - 1)] > s_ratio[min(lane, n - 1)];
    const unsigned long long m = __ballot(rej);
    if (lane == 0) s_j = m ? __ffsll((long long)m) - 1 : n;
  }
  __syncthreads();
  const int j = s_j;

  // ---- 2. weights of the final draw into s_m ---------------------------------
  if (j == n) {
    for (int t = tid; t < v; t += 256) s_m[t] = pv[(long long)n * v + t];
  } else {
    // evidence of the accepted tokens: e[i][z] = log phi[i][z][x_i], i < j
    for (int i0 = tid; i0 < j * r; i0 += 4 * 256) {
      float tmp[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int idx = min(i0 + u * 256, j * r - 1);
        tmp[u] = phi[(long long)idx * v + tok_at(idx / r)];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (i0 + u * 256 < j * r) s_e[i0 + u * 256] = tmp[u];
    }
    __syncthreads();
    const float* lw = a.logw ? a.logw + (long long)b * r : nullptr;
    if (a.h != nullptr && a.family != MTPC_FF) {             // sum units of this position, computed here
      if (a.bf16) sumunit_position<true>(a.h, a.ld_h, a.Wsum, b, a.d, r, s_lw);
      else sumunit_position<false>(a.h, a.ld_h, a.Wsum, b, a.d, r, s_lw);
      lw = s_lw;
    }
    const long long lstep = a.L > 1 ? (long long)r * r : 0;
    const long long lbase = a.contextual ? (long long)b * a.L * r * r : 0;
    const bool ahead = (r + 256 / G - 1) / (256 / G) <= 16;     // a thread's share of a layer fits mv_load
    // log-domain message into leaf j -> s_c
    if (a.family == MTPC_FF) {
      if (tid < r) s_c[tid] = 0.f;
    } else if (a.family == MTPC_CP) {
      if (tid < r) {
        float acc = lw[tid];
        for (int i = 0; i < j; ++i) acc += s_e[i * r + tid];
        s_c[tid] = acc;
      }
    } else if (a.family == MTPC_HMM) {
      if (tid < r) s_c[tid] = lw[tid] + (j > 0 ? s_e[tid] : 0.f);
      __syncthreads();
      MvWeights cur, nxt;
      if (ahead && j >= 1) mv_load(a.lay_nat + lbase, r, G, cur);
      for (int i = 1; i <= j; ++i) {                         // predict state i from state i-1
        float o;
        if (ahead) {
          if (i < j) mv_load(a.lay_nat + lbase + i * lstep, r, G, nxt);
          o = mv_apply(s_c, cur, r, G, s_x, s_part, s_red);
          cur = nxt;
        } else {
          o = matvec_log(s_c, a.lay_nat + lbase + (i - 1) * lstep, r, G, s_x, s_part, s_red);
        }
        if (i < j && tid < r) o += s_e[i * r + tid];         // ... and observe token i if accepted
        if (tid < r) s_c[tid] = o;
        __syncthreads();
      }
    } else {
      // binary tree, heap order: inner nodes 0..n-2, leaf i at n-1+i
      auto value = [&](int c, int t) {                       // fully observed child c, unit t
        return c >= n - 1 ? s_e[(c - (n - 1)) * r + t] : s_nodes[c * r + t];
      };
      int lg = 0;
      while ((1 << lg) < n) ++lg;
      auto next_left = [&](int m) {                          // next inner node below m whose leaves all lie left of leaf j
        for (--m; m >= 1; --m) {
          const int lev = 31 - __clz(m + 1);
          const int span = n >> lev;
          if ((m + 1 - (1 << lev)) * span + span - 1 < j) return m;
        }
        return 0;
      };
      MvWeights cur, nxt;
      int m = next_left(n - 1);
      if (ahead && m) mv_load(a.lay_tr + lbase + (m - 1) * lstep, r, G, cur);
      while (m) {                                            // bottom-up over those subtrees
        const int mn = next_left(m);
        if (ahead && mn) mv_load(a.lay_tr + lbase + (mn - 1) * lstep, r, G, nxt);
        if (tid < r) s_c[tid] = value(2 * m + 1, tid) + value(2 * m + 2, tid);
        __syncthreads();
        const float o = ahead ? mv_apply(s_c, cur, r, G, s_x, s_part, s_red)
                              : matvec_log(s_c, a.lay_tr + lbase + (m - 1) * lstep, r, G, s_x, s_part, s_red);
        if (tid < r) s_nodes[m * r + tid] = o;
        __syncthreads();
        cur = nxt;
        m = mn;
      }
      // top-down along the path: D_child[t] = (sum_k D_node[k] A_node[k][t]) * sibling[t]
      for (int lev = 0; lev < lg; ++lev) {
        // child of the path node at this level: the node (or leaf) one level down that covers leaf j
        const int c = lev + 1 < lg ? (1 << (lev + 1)) - 1 + (j >> (lg - lev - 1)) : n - 1 + j;
        const int node = (c - 1) >> 1;
        // the node of the next level is this level's child c: its layer can be fetched now
        if (ahead && lev + 1 < lg) mv_load(a.lay_nat + lbase + (c - 1) * lstep, r, G, nxt);
        float o;
        if (node == 0) o = tid < r ? lw[tid] : neg_inf();
        else if (ahead) o = mv_apply(s_c, cur, r, G, s_x, s_part, s_red);
        else o = matvec_log(s_c, a.lay_nat + lbase + (node - 1) * lstep, r, G, s_x, s_part, s_red);
        cur = nxt;
        if ((c & 1) == 0 && tid < r) o += value(c - 1, tid);  // left sibling: leaves < j, observed
        __syncthreads();
        if (tid < r) s_c[tid] = o;                            // right sibling: nothing observed, = 1
        __syncthreads();
      }
    }
    __syncthreads();
    // lambda = softmax(s_c) (linear) -> s_x
    {
      const float cv = tid < r ? s_c[tid] : neg_inf();
      const float mx = block_max(cv, s_red);
      const float ex = tid < r ? __expf(cv - mx) : 0.f;
      const float tot = block_sum(ex, s_red);
      if (tid < r) s_x[tid] = ex / tot;
      __syncthreads();
    }
    // q(a | x_1..x_j) = sum_z lambda_z phi[j][z][a];  weights max(0, p - q)
    for (int t0 = tid; t0 < v; t0 += 256) {
      const float* col = phi + (long long)j * r * v + t0;
      const float pt = pv[(long long)j * v + t0];
      float q = 0.f;
      for (int z0 = 0; z0 < r; z0 += 32) {                   // 32 rows of the table in flight, in groups of eight: none beyond r
        float lp[32];
#pragma unroll
        for (int g = 0; g < 32; g += 8)
          if (z0 + g < r)
#pragma unroll
            for (int u = g; u < g + 8; ++u) lp[u] = col[(long long)min(z0 + u, r - 1) * v];
#pragma unroll
        for (int g = 0; g < 32; g += 8)
          if (z0 + g < r)
#pragma unroll
            for (int u = g; u < g + 8; ++u)
              if (z0 + u < r) q = fmaf(s_x[z0 + u], __expf(lp[u]), q);
      }
      s_m[t0] = fmaxf(0.f, pt - q);
    }
  }
  __syncthreads();

  // ---- 3. inverse-CDF draw from s_m / Z ---------------------------------------
  const int C = (v + 255) / 256;                             // consecutive ids per thread
  float total = 0.f, excl = 0.f;
  for (int pass = 0; pass < 2; ++pass) {
    float ls = 0.f;
    for (int q = 0; q < C; ++q) {
      const int t = tid * C + q;
      if (t < v) ls += s_m[t];
    }
    float incl = ls;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const float up = __shfl_up(incl, o);
      if (lane >= o) incl += up;
    }
    __syncthreads();
    if (lane == 63) s_red[wave] = incl;
    __syncthreads();
    float base = 0.f;
    for (int w = 0; w < wave; ++w) base += s_red[w];
    total = (s_red[0] + s_red[1]) + (s_red[2] + s_red[3]);
    excl = base + incl - ls;
    if (total > 0.f || j == n || pass == 1) break;
    // p == q at the rejected position: the adjusted distribution is undefined, draw from p
    __syncthreads();
    for (int t = tid; t < v; t += 256) s_m[t] = pv[(long long)j * v + t];
    __syncthreads();
  }
  if (tid == 0) { s_lo = INT_MAX; s_hi = -1; }
  __syncthreads();
  const float u = philox_uniform(a.seed_lo, a.seed_hi, a.offset, (uint32_t)b, VERIFY_DRAFT_INDEX, (uint32_t)n);
  const float tgt = u * total;
  {
    float run = excl;
    int first = INT_MAX, lastpos = -1;
    for (int q = 0; q < C; ++q) {
      const int t = tid * C + q;
      if (t < v) {
        const float w = s_m[t];
        run += w;
        if (first == INT_MAX && tgt < run) first = t;
        if (w > 0.f) lastpos = t;
      }
    }
    if (first != INT_MAX) atomicMin(&s_lo, first);
    if (lastpos >= 0) atomicMax(&s_hi, lastpos);
  }
  __syncthreads();
  if (tid == 0) {
    a.accepted[b] = j;
    a.token[b] = s_lo != INT_MAX ? s_lo : max(s_hi, 0);
  }
}

// The same for a few positions (verify_rows), bound by the latency of one: whatever does not depend on the rejected position is fetched
// before it is known - acceptance tests, evidence of all drafted tokens, sum units, and the logits of all layers, of which those that turn out
// to be needed are then normalised in LDS (no launch for that) -, and the message to the rejected position is formed out of LDS, by one wave (HMM: linear values, as
// in k_circuit_row) or (binary tree, observed subtrees) a wave to a node.  G as in RowOps.
// HMM n = 16, r = 32, v = 320, B = 61: 28.9 (with the launch that normalised its layers) -> 20.3 us, CP B = 1 17.5 -> 10.4.
template <int G>
__global__ __launch_bounds__(VERIFY_ROW_THREADS) void k_verify_row(const VerifyArgs a) {
  using Ops = RowOps<G, 64 / G>;
  constexpr int NT = VERIFY_ROW_THREADS, NW = NT / 64;
  extern __shared__ __align__(16) float vsm[];
  __shared__ float s_lw[128];
  __shared__ int s_j;
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, k = lane % G, part = lane / G;
  const int n = a.n, r = a.r, v = a.v, rs = r + 1;            // (rows of r + 1: either way through a layer meets all banks)
  const bool hmm = a.family == MTPC_HMM, tree = a.family == MTPC_BTREE, live = k < r;
  const int L = hmm || tree ? a.L : 0, lstep = L > 1 ? r * rs : 0;
  const float ninf = neg_inf();
  float* const xs = vsm + wave * 64;                          // [waves][64] operands of the products
  float* const s_part = vsm + NT;                             // [NT] parts of the mixture
  float* const s_lay = s_part + NT;                           // [L][r][rs]
  float* const s_e = s_lay + (size_t)L * r * rs;              // [n][r] evidence of the drafted tokens
  float* const s_w = s_e + (size_t)n * r;                     // [n][r] HMM: its exponentials; tree: node values
  float* const s_max = s_w + (hmm || tree ? (size_t)n * r : 0);     // [n]
  float* const s_lam = s_max + n;                             // [r] weights of the mixture
  float* const s_m = s_lam + 2 * r;                           // [v] weights of the final draw
  const int* x = a.drafts + (long long)b * n;
  const float* phi = a.logphi + (long long)b * n * r * v;
  const float* pv = a.p + (long long)b * (n + 1) * v;
  // ids outside [0, v) are the caller's error; clamping keeps every access in bounds
  auto tok_at = [&](int i) { return min(max(x[i], 0), v - 1); };

  // ---- 1. acceptance tests, evidence, layers, sum units
  if (wave == 0) {
    bool rej = false;
    if (lane < n) {
      const float lq = a.prefix[(long long)b * n + lane] - (lane > 0 ? a.prefix[(long long)b * n + lane - 1] : 0.f);
      const float ratio = pv[(long long)lane * v + tok_at(lane)] / __expf(lq);
      rej = philox_uniform(a.seed_lo, a.seed_hi, a.offset, (uint32_t)b, VERIFY_DRAFT_INDEX, (uint32_t)lane) > ratio;
    }
    const unsigned long long m = __ballot(rej);
    if (lane == 0) s_j = m ? __ffsll((long long)m) - 1 : n;
  }
  // a group of G lanes to a token, and to a row of a layer, sixteen rows in flight; the first tokens' evidence is looked up while the
  // rows are on their way
  const int gi = tid / G, kc = min(k, r - 1);
  constexpr int NG = NT / G, E = G / 16 > 0 ? G / 16 : 1;     // (64 tokens)
  int tok[E];
#pragma unroll
  for (int u = 0; u < E; ++u) tok[u] = tok_at(min(gi + u * NG, n - 1));
  const float* const src = a.raw != nullptr ? a.raw + (long long)b * a.raw_batch_stride : a.lay_nat + (a.contextual ? (long long)b * L * r * r : 0);
  const long long layer_stride = a.raw != nullptr ? a.raw_layer_stride : (long long)r * r;
  const int rows = L * r;
  const bool dense = L <= 1 || layer_stride == (long long)r * r;        // (rows one behind the other)
  auto load_rows = [&](int q0, float (&y)[16]) {
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int q = min(q0 + u * NG, rows - 1);
      y[u] = dense ? src[q * r + kc] : src[q / r * layer_stride + q % r * r + kc];
    }
  };
  auto put_rows = [&](int q0, const float (&y)[16]) {
#pragma unroll
    for (int u = 0; u < 16; ++u)
      if (live && q0 + u * NG < rows) s_lay[(q0 + u * NG) * rs + k] = y[u];
  };
  float y[16], ev[E];
  if (rows > 0) load_rows(gi, y);
#pragma unroll
  for (int u = 0; u < E; ++u) ev[u] = phi[(long long)(min(gi + u * NG, n - 1) * r + kc) * v + tok[u]];
  __builtin_amdgcn_sched_barrier(0);                          // (all of these in flight before the first is waited for)
  if (rows > 0) {
    put_rows(gi, y);
    for (int q0 = gi + 16 * NG; q0 < rows; q0 += 16 * NG) {
      load_rows(q0, y);
      put_rows(q0, y);
    }
  }
#pragma unroll
  for (int u = 0; u < E; ++u)
    if (live && gi + u * NG < n) s_e[(gi + u * NG) * r + k] = ev[u];
  if (a.family == MTPC_FF) {
    if (tid < r) s_lw[tid] = 0.f;
  } else if (a.h != nullptr) {
    if (a.bf16) sumunit_position<true, NW>(a.h, a.ld_h, a.Wsum, b, a.d, r, s_lw);
    else sumunit_position<false, NW>(a.h, a.ld_h, a.Wsum, b, a.d, r, s_lw);
  } else if (tid < r) {
    s_lw[tid] = a.logw[(long long)b * r + tid];
  }
  __syncthreads();
  const int j = s_j;
  int lg = 0;
  while ((1 << lg) < n) ++lg;
  if (a.raw != nullptr && j < n) {
    // the layers that the message will meet, normalised in place (as normalise_layer_row): all of them would be 8 us of it
    auto met = [&](int l) {
      if (hmm) return l < j;                                  // (one layer for all steps: l = 0)
      if (L == 1) return true;
      const int m = l + 1, lev = 31 - __clz(m + 1), span = n >> lev, at = m + 1 - (1 << lev);     // leaves at * span ..
      return at * span <= j;                                  // left of leaf j, or over it
    };
    for (int q = gi; q < rows; q += NG) {
      if (!met(q / r)) continue;
      const float z = live ? s_lay[q * rs + k] : ninf, m = Ops::max_units(z), ms = m == ninf ? 0.f : m;
      const float e = z > ninf ? expf(z - ms) : 0.f, tot = Ops::sum_units(e);
      if (live) s_lay[q * rs + k] = e * (tot > 0.f ? 1.f / tot : 0.f);
    }
    __syncthreads();
  }

  // ---- 2. weights of the final draw into s_m
  if (j == n) {
    for (int t = tid; t < v; t += NT) s_m[t] = pv[(long long)n * v + t];
  } else {
    const int vr = (v + 63) / 64 * 64, zparts = NT / vr, t = tid % vr, zp = tid / vr;
    float pt = 0.f;
    if (tid < v) pt = pv[(long long)j * v + tid];             // (v <= 320; fetched while the weights are formed)
    const float lw = live ? s_lw[k] : ninf;
    float c = lw;                                             // log-domain message into leaf j (first wave)
    bool linear = false;
    float lam = 0.f;
    if (a.family == MTPC_CP) {
      if (wave == 0 && live)
        for (int i = 0; i < j; ++i) c += s_e[i * r + k];
    } else if (hmm) {
      for (int i = tid / G; i < j; i += NT / G) {
        const float e = live ? s_e[i * r + k] : ninf;
        const float m = Ops::max_units(e), ms = m == ninf ? 0.f : m;
        if (live) s_w[i * r + k] = scaled_exp(e - ms, ROW_EVIDENCE);
      }
      __syncthreads();
      if (wave == 0 && j > 0) {
        linear = true;
        float y = 0.f;
        for (int i = 0; i < j; ++i) {                         // observe token i, predict state i + 1
          const int ic = i * r + min(k, r - 1);
          const typename Ops::Weights w = Ops::weights(s_lay + (size_t)i * lstep, k, part, r, rs, 1);
          float s, taken;
          int exponent = 0, shift;
          const float z = i == 0 ? observe_first<Ops>(lw, s_e[ic], live, s, exponent, shift, taken)
                                 : observe<Ops>(y, s_w[ic], s_e[ic], live, s, exponent, shift, taken);
          y = Ops::product(z, w, xs, k, part, r, rs);
        }
        lam = live ? y : 0.f;
      }
    } else if (tree) {
      // heap order: inner nodes 0..n-2, leaf i at n-1+i
      auto value = [&](int q) {                               // fully observed child q
        if (!live) return ninf;
        return q >= n - 1 ? s_e[(q - (n - 1)) * r + k] : s_w[q * r + k];
      };
      auto layer = [&](float y, const typename Ops::Weights& w, int sj) {
        const float mx = Ops::max_units(y);
        const float o = Ops::product(live ? __expf(y - (mx == ninf ? 0.f : mx)) : 0.f, w, xs, k, part, r, sj);
        return live ? mx + __logf(o) : ninf;                  // log 0 = -inf
      };
      for (int lev = lg - 1; lev >= 1; --lev) {               // bottom-up: the nodes whose leaves all lie left of leaf j
        const int span = n >> lev, first = (1 << lev) - 1, count = j / span;
        for (int q = wave; q < count; q += NW) {
          const int m = first + q;
          const float o = layer(value(2 * m + 1) + value(2 * m + 2), Ops::weights(s_lay + (size_t)(m - 1) * lstep, k, part, r, 1, rs), 1);
          if (part == 0 && live) s_w[m * r + k] = o;
        }
        __syncthreads();
      }
      if (wave == 0) {
        // top-down along the path: D_child[t] = (sum_k D_node[k] A_node[k][t]) * sibling[t]
        for (int lev = 0; lev < lg; ++lev) {
          // child of the path node at this level: the node (or leaf) one level down that covers leaf j
          const int q = lev + 1 < lg ? (1 << (lev + 1)) - 1 + (j >> (lg - lev - 1)) : n - 1 + j;
          const int node = (q - 1) >> 1;
          if (node > 0) c = layer(c, Ops::weights(s_lay + (size_t)(node - 1) * lstep, k, part, r, rs, 1), rs);
          if ((q & 1) == 0) c += value(q - 1);                // left sibling: leaves < j, observed; right: nothing, = 1
        }
      }
    }
    if (wave == 0) {                                          // lambda = softmax(c), or the linear values over their sum
      const float most = Ops::max_units(c);                   // (of all lanes: not behind a condition on `live`)
      if (!linear) lam = live ? __expf(c - most) : 0.f;
      const float tot = Ops::sum_units(lam);
      if (part == 0 && live) s_lam[k] = lam / tot;
    }
    __syncthreads();
    // q(a | x_1..x_j) = sum_z lambda_z phi[j][z][a];  weights max(0, p - q)
    float q = 0.f;
    if (zp < zparts && t < v) {
      const float* col = phi + (long long)j * r * v + t;
      for (int z0 = zp; z0 < r; z0 += 16 * zparts) {          // 16 rows of the table in flight: none beyond r
        float lp[16];
#pragma unroll
        for (int u = 0; u < 16; ++u)
          if (z0 + u * zparts < r) lp[u] = col[(long long)(z0 + u * zparts) * v];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 16; ++u)
          if (z0 + u * zparts < r) q = fmaf(s_lam[z0 + u * zparts], __expf(lp[u]), q);
      }
      s_part[zp * vr + t] = q;
    }
    __syncthreads();
    if (tid < v) {
      float sum = 0.f;
      for (int w = 0; w < zparts; ++w) sum += s_part[w * vr + tid];
      s_m[tid] = fmaxf(0.f, pt - sum);
    }
  }
  __syncthreads();
  if (wave != 0) return;

  // ---- 3. inverse-CDF draw from s_m / Z, consecutive ids per lane
  constexpr int VPL = 5;                                      // v <= 320
  const int C = (v + 63) / 64;
  float m[VPL], ls = 0.f, incl = 0.f, total = 0.f;
  for (int pass = 0; pass < 2; ++pass) {
    ls = 0.f;
#pragma unroll
    for (int q = 0; q < VPL; ++q) {
      const int t = lane * C + q;
      // p == q at the rejected position: the adjusted distribution is undefined, draw from p
      m[q] = q < C && t < v ? (pass == 0 ? s_m[t] : pv[(long long)j * v + t]) : 0.f;
      ls += m[q];
    }
    incl = ls;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const float up = __shfl_up(incl, o);
      if (lane >= o) incl += up;
    }
    total = __shfl(incl, 63);
    if (total > 0.f || j == n) break;
  }
  const float tgt = philox_uniform(a.seed_lo, a.seed_hi, a.offset, (uint32_t)b, VERIFY_DRAFT_INDEX, (uint32_t)n) * total;
  float run = incl - ls;
  int first = INT_MAX, last = -1;
#pragma unroll
  for (int q = 0; q < VPL; ++q) {
    run += m[q];
    if (q < C && first == INT_MAX && tgt < run) first = lane * C + q;
    if (m[q] > 0.f) last = lane * C + q;
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    first = min(first, __shfl_xor(first, o));
    last = max(last, __shfl_xor(last, o));
  }
  if (lane == 0) {
    a.accepted[b] = j;
    a.token[b] = first < v ? first : max(last, 0);
  }
}

template <int G>
hipError_t launch_verify_row(const VerifyArgs& a, hipStream_t st) {
  if (hipError_t e = allow_lds<k_verify_row<G>>(152 * 1024); e != hipSuccess) return e;
  const int L = a.family == MTPC_HMM || a.family == MTPC_BTREE ? std::max(a.L, 0) : 0;
  hipLaunchKernelGGL(k_verify_row<G>, dim3(a.B), dim3(VERIFY_ROW_THREADS), verify_row_floats(a.family, a.n, a.r, L, a.v) * 4, st, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_verify(const VerifyArgs& a, hipStream_t st) {
  if (a.mode == MTPC_VERIFY_GREEDY) {
    hipLaunchKernelGGL(k_verify_greedy, dim3(a.B), dim3(a.n < 16 ? (a.n + 1) * 64 : 1024), 0, st, a);
    return hipGetLastError();
  }
  if (verify_rows(a.family, a.B, a.n, a.r, a.L, a.v)) {
    if (a.r <= 8) return launch_verify_row<8>(a, st);
    if (a.r <= 16) return launch_verify_row<16>(a, st);
    return a.r <= 32 ? launch_verify_row<32>(a, st) : launch_verify_row<64>(a, st);
  }
  int G = 1;
  while (G < a.r) G <<= 1;                                   // r <= 128 -> at least two column groups
  const size_t smem = ((size_t)a.n * a.r + (a.family == MTPC_BTREE ? (size_t)(a.n - 1) * a.r : 0) + a.v) * 4;
  if (hipError_t e = allow_lds<k_verify>(96 * 1024); e != hipSuccess) return e;
  hipLaunchKernelGGL(k_verify, dim3(a.B), dim3(256), smem, st, a, G);
  return hipGetLastError();
}

}  // namespace mtpc
