// Router scoring (Eq. 8), wavefront-level top-N_k selection and the gate of Eq. 9, for flat layers
// and for the two-level hierarchy of Sec. 4.4.  Two scoring kernels feed the same selection code
//   router_simt_kernel  one token per workgroup, fp32 FMA dot products (fp32 layers, decode batches)
//   router_gemm_kernel  bf16 MFMA partial products over (32-token tile, K slice) workgroups, followed by
//                       route_tile_kernel, which sums the slices in order, selects, and emits each
//                       64-token tile's per-group histogram (prefill batches)
// and score_route_kernel does both for prefill batches of a flat layer.
#include <algorithm>
#include <cstdlib>
#include "../../include/cmoe.h"
#include "cmoe_internal.h"
#include "decode_device.h"
#include "device_utils.h"
#include "lds_limit.h"
#include "place_device.h"

namespace cmoe {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float floatx16_t __attribute__((ext_vector_type(16)));

struct RouteIO {
  int32_t* sel_group;     // [T][S_dyn]
  float* sel_weight;      // [T][S_dyn]
  int32_t* topk_out;      // flat: [T][N_k]; hierarchy: [T][outer_top_k][N_k]; may be null
  int32_t* outer_out;     // [T][outer_top_k] or null
  float* scores_out;      // [T][n_scored] or null
  const float* gate_u;    // [n_scored] or null
  const float* gate_b;    // [n_scored] or null
  const float* lin_off;   // [n_lin] or null
  int32_t S_dyn;
};

// ---- selection -----------------------------------------------------------------------------------------
// One wave with one token picks the best lane, its next best and so on (wave_argmax), a short chain per round whatever
// the number of candidates: whole forward at d = 4096, 32 experts, top-1 19.8 us and top-2 17.0, by rank 21.1 and 18.3.
// A workgroup with a tile of tokens selects by rank: the k-th largest of n keys is the one that exactly k - 1 keys
// beat.  Counting for every key how many beat it (a larger key, or an equal one with a lower index) takes n
// independent compares per key and no exchange between lanes, and every winner knows its place in the list at once:
// 32 tokens, 28 experts, top-4 in one workgroup 17.6 -> 12.5 us for the whole launch, the hierarchy's 4096 tokens
// 18.6 -> 10.2.
// Keys are compared as ordered integers, a total order for every bit pattern (a NaN cannot make two experts share
// a rank or leave one empty); -0 counts as +0.
__device__ __forceinline__ uint32_t rank_key(float f) { return ordered_key(f + 0.0f); }

// How many of n keys in LDS (as float bits) beat key j.  The reads of eight candidates are in flight together (one at a
// time, with a gate parameter from memory for each: 31.6 us per forward of 5 tokens, 31 experts; now 28.2).
__device__ __forceinline__ int lds_rank(const float* keys, int n, int j) {
  const uint32_t key = __float_as_uint(keys[j]);
  int rank = 0;
  for (int q0 = 0; q0 < n; q0 += 8) {
    uint32_t o[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) o[u] = __float_as_uint(keys[q0 + u < n ? q0 + u : q0]);
#pragma unroll
    for (int u = 0; u < 8; ++u) rank += (q0 + u < n && (o[u] > key || (o[u] == key && q0 + u < j))) ? 1 : 0;
  }
  return rank;
}

// Gate parameters (Eq. 9) of all scored experts in LDS: requested when a kernel starts, stored when its first loads
// are back, so that no selection waits for them.
struct GateLds { float u[MAX_SCORED], b[MAX_SCORED]; };
__device__ __forceinline__ float2 request_gate(const RouterDev& r, const RouteIO& io, int tid) {
  float2 g = make_float2(0.0f, 0.0f);
  if (r.use_gate && tid < r.n_scored) {
    if (io.gate_u) g.x = io.gate_u[tid];
    if (io.gate_b) g.y = io.gate_b[tid];
  }
  return g;
}
__device__ __forceinline__ void store_gate(GateLds& gl, float2 g, int tid) {
  if (tid < MAX_SCORED) {
    gl.u[tid] = g.x;
    gl.b[tid] = g.y;
  }
}

// Top-N_k among the routed experts held by lanes [lo, lo + n) (one lane per expert), Eq. 9:
// key = s (binary gate) or Softmax(s) + b; gate = 1 + Softmax(s) * u.  Emits N_k (group, weight)
// entries in descending key order, ties to the lowest expert id.  Executed by a full wave.
__device__ __forceinline__ void select_routed(const RouterDev& r, const RouteIO& io, float skey, int lo, int n,
                                              float scale, int group_base, int64_t t, int& n_entries,
                                              int32_t* topk_ptr, int32_t* hist) {
  const int lane = threadIdx.x & 63;
  const bool in_range = lane >= lo && lane < lo + n;
  float key = skey, sp = 0.0f, gate_u = 0.0f, gate_b = 0.0f;
  if (r.use_gate) {
    if (io.gate_u && in_range) gate_u = io.gate_u[lane];     // (needed last, requested first)
    if (io.gate_b && in_range) gate_b = io.gate_b[lane];
    const float mx = wave_max(in_range ? skey : -INFINITY);
    const float ex = in_range ? expf(skey - mx) : 0.0f;
    const float sum = wave_sum(ex);
    sp = ex / sum;
    key = sp + gate_b;
  }
  const uint32_t rkey = rank_key(key);
  bool active = in_range;
  for (int k = 0; k < r.top_k; ++k) {
    const int w = wave_argmax(rkey, active);                  // uniform
    if (lane == w) {
      float gate = 1.0f;
      if (r.use_gate && io.gate_u) gate = 1.0f + sp * gate_u;
      const int g = group_base + (lane - lo);
      io.sel_group[t * io.S_dyn + n_entries + k] = g;
      io.sel_weight[t * io.S_dyn + n_entries + k] = scale * gate;
      if (topk_ptr) topk_ptr[k] = lane - lo;
      if (hist) atomicAdd(&hist[g], 1);
      active = false;
    }
  }
  n_entries += r.top_k;
}

// Route one token from its pre-activations `pre` (LDS: n_sw_rows SwiGLU rows in blocks of IL gate /
// IL up rows, then n_lin_rows linear logits).  Executed by a full wave; all control flow is uniform.
__device__ __forceinline__ void route_token(const RouterDev& r, const RouteIO& io, const float* pre, int64_t t,
                                            int32_t* hist) {
  const int lane = threadIdx.x & 63;
  float s = 0.0f;
  if (lane < r.n_scored) {
    const int blk = lane / IL, c = lane % IL;
    const float g = pre[blk * 2 * IL + c], u = pre[blk * 2 * IL + IL + c];
    s = silu_f32(g) * u;                                                     // Eq. 8
    if (io.scores_out) io.scores_out[t * r.n_scored + lane] = s;
  }
  const float skey = r.score_abs ? fabsf(s) : s;
  int n_entries = 0;
  if (r.outer_top_k == 0) {
    select_routed(r, io, skey, 0, r.n_scored, 1.0f, r.n_always, t, n_entries,
                  io.topk_out ? io.topk_out + t * r.top_k : nullptr, hist);
    return;
  }
  // two-level: outer linear logits -> top outer_top_k -> softmax over the selected logits
  float logit = -INFINITY;
  bool active = lane < r.n_lin;
  if (active) logit = pre[r.n_sw_rows + lane] + (io.lin_off ? io.lin_off[lane] : 0.0f);
  const uint32_t okey = rank_key(logit);
  int oe[MAX_OUTER_TOPK];
  float ol[MAX_OUTER_TOPK];
  for (int i = 0; i < r.outer_top_k; ++i) {
    const int w = wave_argmax(okey, active);
    oe[i] = w;
    ol[i] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(logit), w));
    if (lane == w) active = false;
  }
  float den = 0.0f;
  for (int i = 0; i < r.outer_top_k; ++i) den += expf(ol[i] - ol[0]);
  for (int i = 0; i < r.outer_top_k; ++i) {
    const int e = oe[i];
    const float w_e = expf(ol[i] - ol[0]) / den;
    const int gbase = e * r.groups_per_outer;
    if (lane == 0 && io.outer_out) io.outer_out[t * r.outer_top_k + i] = e;
    if (r.sub_has_shared) {
      if (lane == 0) {
        io.sel_group[t * io.S_dyn + n_entries] = gbase;
        io.sel_weight[t * io.S_dyn + n_entries] = w_e;
        if (hist) atomicAdd(&hist[gbase], 1);
      }
      ++n_entries;
    }
    if (r.top_k > 0)
      select_routed(r, io, skey, e * r.n_r_sub, r.n_r_sub, w_e, gbase + r.sub_has_shared, t, n_entries,
                    io.topk_out ? io.topk_out + (t * r.outer_top_k + i) * r.top_k : nullptr, hist);
  }
}

// ---- a tile of tokens ----------------------------------------------------------------------------------
// Rounds of arg-max by a wave per token instead of ranks where top_k times this is less than n * n: a round costs the same
// whatever n is, the ranks of all candidates n * n compares.  us per forward by rank / by rounds, d = 1024, 64 tokens:
// 32 experts top-1 34.9 / 30.2, top-3 36.2 / 32.1, top-6 37.3 / 35.7; 16 experts top-1 1.03 times, top-3 0.97 times;
// 8 experts top-4 0.94 times.  Even at n * n / top_k of 128 to 170 for 40 to 2048 tokens.
constexpr int SELECT_ROUNDS_PER_N2 = 160;

// One thread per (token, candidate), all threads of the workgroup (which all must call: barriers).  `sc`: what
// score_tile left, [tok][ld_sc]; `pre`: the tile's pre-activations [tok][ld], of which the linear logits
// behind the n_sw_rows SwiGLU rows are read and the rows, no longer needed, then hold exp(s - max) [n_scored], the
// outer choice [2 n_outer] and Softmax(s) [n_scored] (n_sw_rows is at least twice n_scored, and a hierarchy has 32 linear
// rows).  Sums run in the order ((j = 0 mod 4) + (1 mod 4)) + ((2 mod 4) + (3 mod 4)).
__device__ __forceinline__ void route_select_tile(const RouterDev& r, const RouteIO& io, float* sc, int ld_sc,
                                                  float* pre, int ld, int n_tok, int64_t t0, int32_t* hist,
                                                  const GateLds& gl, int tid, int n_threads) {
  const int n_outer = r.outer_top_k > 0 ? r.outer_top_k : 1;
  // a token's outer choice: n_outer logits, then n_outer expert ids
  auto outer_of = [&](int tok) { return r.n_sw_rows > 0 ? pre + tok * ld + r.n_scored : sc + tok * ld_sc; };
  if (r.outer_top_k > 0) {
    for (int idx = tid; idx < n_tok * r.n_lin; idx += n_threads) {
      const int tok = idx / r.n_lin, e = idx - tok * r.n_lin;
      const float* lin = pre + tok * ld + r.n_sw_rows;
      const float mine = lin[e] + (io.lin_off ? io.lin_off[e] : 0.0f);
      const uint32_t key = rank_key(mine);
      int rank = 0;
      for (int i = 0; i < r.n_lin; ++i) {
        const uint32_t o = rank_key(lin[i] + (io.lin_off ? io.lin_off[i] : 0.0f));
        rank += (o > key || (o == key && i < e)) ? 1 : 0;
      }
      if (rank < n_outer) {
        float* ob = outer_of(tok);
        ob[rank] = mine;
        ob[n_outer + rank] = __int_as_float(e);
        if (io.outer_out) io.outer_out[(t0 + tok) * n_outer + rank] = e;
      }
    }
    __syncthreads();
  }
  const bool routed = r.top_k > 0;                                     // (0: the dense form of a hierarchy)
  const int n = !routed ? 1 : r.outer_top_k > 0 ? r.n_r_sub : r.n_scored;   // candidates per choice
  const int per_tok = n_outer * n;
  auto first_of = [&](int tok, int i) {                               // first candidate of the token's i-th choice
    return r.outer_top_k > 0 ? __float_as_int(outer_of(tok)[n_outer + i]) * n : 0;
  };
  const int sp0 = r.n_scored + (r.outer_top_k > 0 ? 2 * n_outer : 0);
  if (r.use_gate && routed) {
    for (int idx = tid; idx < n_tok * per_tok; idx += n_threads) {
      const int tok = idx / per_tok, c = idx - tok * per_tok, i = c / n, j = c - i * n;
      const int lo = first_of(tok, i);
      const float* s = sc + tok * ld_sc + lo;
      float mx = -INFINITY;
      for (int q0 = 0; q0 < n; q0 += 8)
#pragma unroll
        for (int u = 0; u < 8; ++u) mx = fmaxf(mx, s[q0 + u < n ? q0 + u : q0]);
      pre[tok * ld + lo + j] = expf(s[j] - mx);
    }
    __syncthreads();
    for (int idx = tid; idx < n_tok * per_tok; idx += n_threads) {
      const int tok = idx / per_tok, c = idx - tok * per_tok, i = c / n, j = c - i * n;
      const int lo = first_of(tok, i);
      const float* ex = pre + tok * ld + lo;
      float part[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      for (int q = 0; q < n; q += 4)
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (q + u < n) part[u] += ex[q + u];
      const float sp = ex[j] / ((part[0] + part[1]) + (part[2] + part[3]));
      pre[tok * ld + sp0 + lo + j] = sp;
      sc[tok * ld_sc + lo + j] = __uint_as_float(rank_key(sp + gl.b[lo + j]));      // (the scores are used up)
    }
    __syncthreads();
  }
  // choice i of token tok: its weight, first entry and first group; then candidate j, the choice's rank-th
  auto choice = [&](int tok, int i, int lo, float& w_e, int& entry, int& gbase) {
    w_e = 1.0f;
    entry = 0;
    gbase = r.n_always;
    if (r.outer_top_k > 0) {
      const float* ob = outer_of(tok);
      float den = 0.0f;
      for (int q = 0; q < n_outer; ++q) den += expf(ob[q] - ob[0]);
      w_e = expf(ob[i] - ob[0]) / den;
      gbase = (lo / n) * r.groups_per_outer + r.sub_has_shared;
      entry = i * (r.sub_has_shared + r.top_k) + r.sub_has_shared;
    }
  };
  auto emit = [&](int tok, int i, int lo, int j, int rank, float w_e, int entry, int gbase) {
    const int64_t t = t0 + tok;
    float gate = 1.0f;
    if (r.use_gate && io.gate_u) gate = 1.0f + pre[tok * ld + sp0 + lo + j] * gl.u[lo + j];
    io.sel_group[t * io.S_dyn + entry + rank] = gbase + j;
    io.sel_weight[t * io.S_dyn + entry + rank] = w_e * gate;
    if (io.topk_out) io.topk_out[(t * n_outer + i) * r.top_k + rank] = j;
    atomicAdd(&hist[gbase + j], 1);
  };
  if (r.outer_top_k == 0 && r.top_k * SELECT_ROUNDS_PER_N2 < n * n) {
    // few of many: a wave per token, best first (the ranks of all candidates cost n * n compares per token)
    const int lane = tid & 63;
    for (int tok = tid >> 6; tok < n_tok; tok += n_threads >> 6) {
      bool active = lane < n;
      const uint32_t key = active ? __float_as_uint(sc[tok * ld_sc + lane]) : 0u;
      for (int k = 0; k < r.top_k; ++k) {
        const int w = wave_argmax(key, active);
        if (lane == w) {
          emit(tok, 0, 0, lane, k, 1.0f, 0, r.n_always);
          active = false;
        }
      }
    }
    return;
  }
  for (int idx = tid; idx < n_tok * per_tok; idx += n_threads) {
    const int tok = idx / per_tok, c = idx - tok * per_tok, i = c / n, j = c - i * n;
    const int lo = first_of(tok, i);
    float w_e;
    int entry, gbase;
    choice(tok, i, lo, w_e, entry, gbase);
    if (r.sub_has_shared && r.outer_top_k > 0 && j == 0) {
      io.sel_group[(t0 + tok) * io.S_dyn + entry - 1] = gbase - 1;
      io.sel_weight[(t0 + tok) * io.S_dyn + entry - 1] = w_e;
      atomicAdd(&hist[gbase - 1], 1);
    }
    if (!routed) continue;
    const int rank = lds_rank(sc + tok * ld_sc + lo, n, j);
    if (rank < r.top_k) emit(tok, i, lo, j, rank, w_e, entry, gbase);
  }
}

// Scores of a tile of tokens, all threads of the workgroup in parallel (the exponentials are the
// expensive part of routing): Swish(gate_j) * up_j from pre[tok][...] (Eq. 8).  sc[tok][j] gets what the selection
// needs of it: the score to rank by, of which Eq. 9 takes the softmax, or without a gate its key.
__device__ __forceinline__ void score_tile(const RouterDev& r, const RouteIO& io, const float* pre, int ld_pre,
                                           float* sc, int ld_sc, int n_tok, int64_t t0, int tid, int n_threads) {
  for (int idx = tid; idx < n_tok * r.n_scored; idx += n_threads) {
    const int tok = idx / r.n_scored, j = idx - tok * r.n_scored;
    const int blk = j / IL, c = j % IL;
    const float g = pre[tok * ld_pre + blk * 2 * IL + c], u = pre[tok * ld_pre + blk * 2 * IL + IL + c];
    const float s = silu_f32(g) * u;
    const float ranked = r.score_abs ? fabsf(s) : s;
    sc[tok * ld_sc + j] = r.use_gate ? ranked : __uint_as_float(rank_key(ranked));
    if (io.scores_out) io.scores_out[(t0 + tok) * r.n_scored + j] = s;
  }
}

// ---- one token per workgroup ---------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void router_simt_kernel(RouterDev r, RouteIO io, const T* __restrict__ x,
                                                          const T* __restrict__ wr, int d) {
  extern __shared__ float smem[];
  float* xs = smem;                      // [d]
  float* pre = smem + d;                 // [n_sw_rows + n_lin_rows]
  const int64_t t = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int i = tid; i < d; i += 256) xs[i] = Elem<T>::ld(x + t * d + i);
  const int n_rows = r.n_sw_rows + r.n_lin_rows;
  for (int i = tid; i < n_rows; i += 256) pre[i] = 0.0f;
  __syncthreads();
  // The rows in use, four at a time per wave: one chain of round trips for all of them (row by row, 14 rows of d = 256, 64
  // tokens: the launch 6.6 us, now 4.3).
  const int n_used = 2 * r.n_scored + r.n_lin;
  for (int u0 = wave; u0 < n_used; u0 += 16) {
    const T* w[4];
    int row[4];
    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int u = u0 + 4 * q < n_used ? u0 + 4 * q : u0, e = u >> 1;
      row[q] = u < 2 * r.n_scored ? (e / IL) * 2 * IL + e % IL + (u & 1) * IL : r.n_sw_rows + u - 2 * r.n_scored;
      w[q] = wr + (int64_t)row[q] * d;
    }
#pragma unroll 4
    for (int i = lane; i < d; i += 64) {
      const float xv = xs[i];
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[q] = fmaf(xv, Elem<T>::ld(w[q] + i), acc[q]);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float sum = wave_sum(acc[q]);
      if (lane == 0 && u0 + 4 * q < n_used) pre[row[q]] = sum;
    }
  }
  __syncthreads();
  if (wave == 0) route_token(r, io, pre, t, nullptr);
}

// ---- prefill scoring: bf16 MFMA, split over tokens and over K ----------------------------------
// P[ks][t][row] = X[t][K slice ks] * Wr[row][K slice ks]^T for a 32-token tile.  The grid is
// (token tiles, K slices) so that even a 2048-token batch fills the chip; inside a workgroup each of
// the four waves takes every fourth 64-wide chunk of the slice and multiplies straight out of global
// memory, then the four partial sums are added in a fixed order through LDS.  NT = n_rows / 32 <= 5.
constexpr int RT_TOK = 32;

template <int NT>
__global__ __launch_bounds__(256) void router_gemm_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ wr,
                                                          int d, int64_t T, int k_slice, float* __restrict__ partial) {
  __shared__ float red[RT_TOK][NT * 32 + 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t t0 = (int64_t)blockIdx.x * RT_TOK;
  const int ks = blockIdx.y;
  const int l32 = lane & 31, lh = lane >> 5;
  floatx16_t acc[NT];
#pragma unroll
  for (int ni = 0; ni < NT; ++ni)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[ni][i] = 0.0f;
  int64_t t = t0 + l32;
  if (t >= T) t = T - 1;                                     // duplicate the last token; never stored
  const bf16_t* arow = x + t * d + lh * 8;
  const bf16_t* brow = wr + (int64_t)l32 * d + lh * 8;
  const int k_begin = ks * k_slice;
  const int k_end = (k_begin + k_slice < d) ? k_begin + k_slice : d;     // host guarantees multiples of 64
  // software pipeline over this wave's 64-wide chunks: the loads of the next chunk are issued before the MFMAs of the
  // current one.  (Because they are conditional, the compiler counts as if they had not been issued: the MFMAs of a chunk also wait
  // for the next one, and a wave makes a round trip per chunk.)
  bf16x8_t a0[4], a1[4], b0[NT][4], b1[NT][4];
  auto load_chunk = [&](int kc, bf16x8_t (&a)[4], bf16x8_t (&b)[NT][4]) {
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4) {
      a[s4] = *reinterpret_cast<const bf16x8_t*>(arow + kc + s4 * 16);
#pragma unroll
      for (int ni = 0; ni < NT; ++ni) b[ni][s4] = *reinterpret_cast<const bf16x8_t*>(brow + (int64_t)ni * 32 * d + kc + s4 * 16);
    }
  };
  auto mma_chunk = [&](bf16x8_t (&a)[4], bf16x8_t (&b)[NT][4]) {
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4)
#pragma unroll
      for (int ni = 0; ni < NT; ++ni) acc[ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[s4], b[ni][s4], acc[ni], 0, 0, 0);
  };
  int kc = k_begin + wave * 64;
  if (kc < k_end) load_chunk(kc, a0, b0);
  while (kc < k_end) {
    if (kc + 256 < k_end) load_chunk(kc + 256, a1, b1);
    mma_chunk(a0, b0);
    kc += 256;
    if (kc >= k_end) break;
    if (kc + 256 < k_end) load_chunk(kc + 256, a0, b0);
    mma_chunk(a1, b1);
    kc += 256;
  }
  for (int wsel = 0; wsel < 4; ++wsel) {
    if (wave == wsel) {
#pragma unroll
      for (int ni = 0; ni < NT; ++ni)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int row = (i / 4) * 8 + lh * 4 + (i % 4);
          const int col = ni * 32 + l32;
          if (wsel == 0) red[row][col] = acc[ni][i];
          else red[row][col] += acc[ni][i];
        }
    }
    __syncthreads();
  }
  const int n_rows = NT * 32;
  for (int i = tid; i < RT_TOK * n_rows; i += 256) {
    const int row = i / n_rows, col = i - row * n_rows;
    if (t0 + row < T) partial[((int64_t)ks * T + t0 + row) * n_rows + col] = red[row][col];
  }
}

// Row block rb holds rows in use: n_scored gate and up rows in groups of 32 + 32, then n_lin linear rows.
__device__ __forceinline__ bool row_block_used(const RouterDev& r, int rb) {
  const int lin = rb - r.n_sw_rows / 16;
  return lin >= 0 ? lin * 16 < r.n_lin : (rb / 4) * IL + (rb & 1) * 16 < r.n_scored;
}

// Adds the K-slice partials [slice][T][n_rows] of tokens t0 .. t0+rows-1 in slice order into pre[row][ld]
// (LDS; rows past T become zero, and so do row blocks that hold no router row).  n_rows is a multiple of 4: float4 loads of SL
// slices of V vectors per thread, all asked for before the sums.  Another die wrote them, and a round trip there is a tenth of a small
// batch's selection launch (16 experts, d = 4096, 4 slices of four vectors, then the other 4 / all 8 of two: 4 tokens 39.5 / 38.8 us
// per forward, 8 tokens 47.7 / 46.9; 8 experts, d = 8192, 5 tokens 74.3 / 74.7, 12 tokens 100.0 / 98.4; 8 outer experts, d = 4096, 4
// tokens 158.8 / 157.4).  As compiled a vector is two round trips: the first slice, whose conditional load has the addition to zero
// folded in, is awaited before the others are asked for, and the second vector's first slice awaits them.
template <int SL, int V>
__device__ __forceinline__ void sum_partials_of(const RouterDev& r, const float* __restrict__ partial, int n_slices, int64_t T, int64_t t0,
                                                int rows, int n_rows, float* pre, int ld, int tid, int n_threads) {
  const int vec_per_row = n_rows >> 2;
  const int n_vec = rows * vec_per_row;
  for (int i0 = tid; i0 < n_vec; i0 += V * n_threads) {
    float4 part[V][SL];
#pragma unroll
    for (int u = 0; u < V; ++u) {
      const int i = i0 + u * n_threads;
      const int row = i / vec_per_row, cv = i - row * vec_per_row;
      const bool used = i < n_vec && t0 + row < T && row_block_used(r, cv >> 2);
#pragma unroll
      for (int q = 0; q < SL; ++q) {
        part[u][q] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (used && q < n_slices) part[u][q] = *reinterpret_cast<const float4*>(partial + ((int64_t)q * T + t0 + row) * n_rows + cv * 4);
      }
    }
#pragma unroll
    for (int u = 0; u < V; ++u) {
      const int i = i0 + u * n_threads;
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int q = 0; q < SL; ++q) {
        v.x += part[u][q].x; v.y += part[u][q].y; v.z += part[u][q].z; v.w += part[u][q].w;
      }
      if (i < n_vec) {
        const int row = i / vec_per_row, cv = i - row * vec_per_row;
        float* dst = pre + row * ld + cv * 4;
        dst[0] = v.x; dst[1] = v.y; dst[2] = v.z; dst[3] = v.w;
      }
    }
  }
}
// The tile router's (at most eight slices; the front end of small batches always has eight).
__device__ __forceinline__ void sum_partials(const RouterDev& r, const float* __restrict__ partial, int n_slices, int64_t T, int64_t t0,
                                             int rows, int n_rows, float* pre, int ld, int tid, int n_threads) {
  if (n_slices <= 4) sum_partials_of<4, 4>(r, partial, n_slices, T, t0, rows, n_rows, pre, ld, tid, n_threads);
  else sum_partials_of<8, 2>(r, partial, n_slices, T, t0, rows, n_rows, pre, ld, tid, n_threads);
}

// Sum the K-slice partials in slice order, then score, select and histogram a 64-token tile.
constexpr int LD_SC = MAX_SCORED + 1;            // row stride of a tile's scores in LDS
constexpr int RT_THREADS = 1024;
__global__ __launch_bounds__(RT_THREADS) void route_tile_kernel(RouterDev r, RouteIO io, const float* __restrict__ partial,
                                                                int n_slices, int64_t T, int32_t* __restrict__ tile_counts,
                                                                int G) {
  extern __shared__ float pre[];                 // [TOK_TILE][n_rows + 1], then scores [TOK_TILE][LD_SC]
  __shared__ int32_t hist[MAX_GROUPS];
  __shared__ GateLds gl;
  const int tid = threadIdx.x;
  const int n_rows = r.n_sw_rows + r.n_lin_rows;
  const int ld = n_rows + 1;
  float* sc = pre + TOK_TILE * ld;
  const int64_t t0 = (int64_t)blockIdx.x * TOK_TILE;
  const float2 gate = request_gate(r, io, tid);
  sum_partials(r, partial, n_slices, T, t0, TOK_TILE, n_rows, pre, ld, tid, RT_THREADS);
  for (int i = tid; i < MAX_GROUPS; i += RT_THREADS) hist[i] = 0;
  store_gate(gl, gate, tid);
  __syncthreads();
  const int n_tok = (T - t0 < TOK_TILE) ? (int)(T - t0) : TOK_TILE;
  score_tile(r, io, pre, ld, sc, LD_SC, n_tok, t0, tid, RT_THREADS);
  __syncthreads();
  route_select_tile(r, io, sc, LD_SC, pre, ld, n_tok, t0, hist, gl, tid, RT_THREADS);
  __syncthreads();
  for (int g = tid; g < G; g += RT_THREADS) tile_counts[(int64_t)blockIdx.x * G + g] = hist[g];
}

// ---- scoring and selection in one launch (prefill batches of flat layers) ------------------------------------
// A workgroup of eight waves owns TB * 16 tokens and all of K: the partial sums that router_gemm_kernel leaves in memory
// for route_tile_kernel stay in its LDS.  What bounds it is the latency of the router matrix (0.5 MB at d = 4096, 64 rows) that
// every workgroup pulls through L2 in operand order (1 KB of consecutive memory per MFMA operand): as compiled a wave asks for
// the second of two chunks of K (2 x 64) when the first is there, then for the next first one, and awaits both, so that a
// workgroup takes in about 50 KB per us.  Where it pays: see score_route_units.
//
// The sums are those of the two launches, bit for bit: K falls into n_slices slices of k_slice, a slice into four
// classes of 64-wide chunks (chunk number mod 4), each of which is one chain of MFMAs; ((c0 + c1) + c2) + c3 is
// the slice, and the slices are added in order.  Wave w runs the (slice, class) units w * UPW .. + UPW - 1.
//
// NB: blocks of 16 rows that hold router rows, of the four of a group of 64 (32 gate rows, then 32 up rows).  Up to 16 scored
// experts fill two, the first gate and the first up block, and a workgroup pulls half as much.
template <int UPW, int TB, bool ONE, int NB>
__global__ __launch_bounds__(512) void score_route_kernel(RouterDev r, RouteIO io, const bf16_t* __restrict__ x,
                                                          const bf16_t* __restrict__ wrt, int d, int64_t T, int n_slices,
                                                          int k_slice, int32_t* __restrict__ counts, int G) {
  constexpr int NTOK = TB * 16, LDP = 64 + 4;
  constexpr int BSTEP = 4 / NB;                                // row block of operand b: b * BSTEP
  extern __shared__ __attribute__((aligned(16))) float sr_smem[];
  __shared__ int32_t hist[MAX_GROUPS];
  __shared__ GateLds gl;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, kq = lane >> 4;
  const int n_rows = r.n_sw_rows;
  const int ld = n_rows + 1;
  float* slice_sum = sr_smem;                                  // [n_slices][NTOK][LDP]
  float* pre = sr_smem + n_slices * NTOK * LDP;                // [NTOK][ld]
  float* sc = pre + NTOK * ld;                                 // [NTOK][LD_SC]
  const int64_t t0 = (int64_t)blockIdx.x * NTOK;
  for (int i = tid; i < MAX_GROUPS; i += 512) hist[i] = 0;
  const float2 gate = request_gate(r, io, tid);
  const bf16_t* xr[TB];
#pragma unroll
  for (int tb = 0; tb < TB; ++tb) {
    int64_t t = t0 + tb * 16 + r16;
    if (t >= T) t = T - 1;                                     // (a copy of the last token; never used)
    xr[tb] = x + t * d + kq * 8;
  }
  const int n_units = 4 * n_slices, n_i = k_slice / 256, kt = d / 32;
  const int unit0 = wave * UPW;
  struct Chunk { bf16x8_t w[2][NB], a[2][TB]; };
  Chunk c0, c1;
  for (int rg = 0; rg < n_rows / 64; ++rg) {
    auto load_chunk = [&](Chunk& c, int k, int i) {            // chunk i of this wave's k-th unit
      const int q = unit0 + k;
      if (q >= n_units) return;
      const int kc = (q >> 2) * k_slice + (q & 3) * 64 + i * 256;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
          c.w[h][b] = *reinterpret_cast<const bf16x8_t*>(wrt + (((int64_t)(rg * 4 + b * BSTEP) * kt + (kc >> 5) + h) * 64 + lane) * 8);
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) c.a[h][tb] = *reinterpret_cast<const bf16x8_t*>(xr[tb] + kc + h * 32);
      }
    };
    floatx4_t acc[UPW][NB][TB];
#pragma unroll
    for (int k = 0; k < UPW; ++k)
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int tb = 0; tb < TB; ++tb)
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[k][b][tb][i] = 0.0f;
    auto mma_chunk = [&](const Chunk& c, floatx4_t (&ac)[NB][TB]) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int tb = 0; tb < TB; ++tb) ac[b][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(c.w[h][b], c.a[h][tb], ac[b][tb], 0, 0, 0);
    };
    load_chunk(c0, 0, 0);
#pragma unroll
    for (int k = 0; k < UPW; ++k) {
      if (unit0 + k >= n_units) break;                         // (uniform)
      if constexpr (ONE) {                                     // one chunk per unit: the buffers alternate with the units
        if (k & 1) {
          if (k + 1 < UPW) load_chunk(c0, k + 1, 0);
          mma_chunk(c1, acc[k]);
        } else {
          if (k + 1 < UPW) load_chunk(c1, k + 1, 0);
          mma_chunk(c0, acc[k]);
        }
      } else {
        for (int i = 0; i < n_i; i += 2) {
          load_chunk(c1, k, i + 1);
          mma_chunk(c0, acc[k]);
          if (i + 2 < n_i) load_chunk(c0, k, i + 2);
          else if (k + 1 < UPW) load_chunk(c0, k + 1, 0);
          mma_chunk(c1, acc[k]);
        }
      }
    }
    // D layout: a lane holds router rows 16 b * BSTEP + kq * 4 .. + 3 of token tb * 16 + r16
#pragma unroll
    for (int c = 0; c < 4; ++c) {
#pragma unroll
      for (int k = 0; k < UPW; ++k) {
        const int q = unit0 + k;
        if (q >= n_units || (q & 3) != c) continue;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int tb = 0; tb < TB; ++tb) {
            floatx4_t* dst = reinterpret_cast<floatx4_t*>(slice_sum + ((q >> 2) * NTOK + tb * 16 + r16) * LDP + b * (16 * BSTEP) + kq * 4);
            *dst = c == 0 ? acc[k][b][tb] : *dst + acc[k][b][tb];
          }
      }
      __syncthreads();
    }
    for (int idx = tid; idx < NTOK * 16 * NB; idx += 512) {
      const int tok = idx / (16 * NB), c = idx % (16 * NB), row = (c & 15) + (c >> 4) * (16 * BSTEP);
      float v = 0.0f;
      for (int sl = 0; sl < n_slices; ++sl) v += slice_sum[(sl * NTOK + tok) * LDP + row];
      pre[tok * ld + rg * 64 + row] = v;
    }
    __syncthreads();
  }
  const int n_tok = (T - t0 < NTOK) ? (int)(T - t0) : NTOK;
  store_gate(gl, gate, tid);
  score_tile(r, io, pre, ld, sc, LD_SC, n_tok, t0, tid, 512);
  __syncthreads();
  route_select_tile(r, io, sc, LD_SC, pre, ld, n_tok, t0, hist, gl, tid, 512);
  __syncthreads();
  for (int g = tid; g < G; g += 512) counts[(int64_t)blockIdx.x * G + g] = hist[g];
}

// ---- decode front end ------------------------------------------------------------------------------
// For batches of at most one 64-token tile scoring is one launch and selection + permutation a second one.
// (Fusing all three behind a device-wide arrival counter was tried: on this multi-die part a device-scope
// release/acquire pair writes back and invalidates the whole L2, which costs far more than a launch.)
//
// decode_score_kernel: a workgroup per (16 router rows, eighth of K, 16 tokens), v_mfma_f32_16x16x32_bf16 with the router rows
// as the A operand.  Its four waves take a quarter of the slice each, and their sums are added in wave order through
// LDS; the eight K-slice partials of a row go to pre_g[slice][token][row] and are added in slice order by route_place_kernel.
// The router matrix comes cold from HBM, so the launch is bound by memory latency.  As compiled the form that also copies the
// tokens has all loads of a run in flight at once; in the other one the test for the last step stands between a step's products and the
// next step's loads, a round trip per K step of a wave (four at d = 4096, eight at 8192).  (With a wave per slice, 32
// loads behind one another, up to 16 tokens and router_gemm_kernel beyond / now, us per forward: d = 4096, 16 experts, one token
// 22.9 / 21.5, 4 tokens 42.5 / 39.5, 16 tokens 58.1 / 55.0, 32 tokens 69.6 / 65.5; d = 8192, 8 experts, 2 tokens 67.2 / 59.9, 5 tokens
// 79.6 / 74.3; d = 5120, 16 experts, 30 tokens 84.0 / 75.3; 8 outer experts, d = 4096, 4 tokens 161.5 / 158.8.)
// Rows that pad the groups of 32 experts or the outer logits are left out; their partials are not written, and
// the sums that are made of them are not used.
constexpr int DEC_SLICES = 8;

// CH: K steps of a wave's quarter per run.  COPY: the tokens also go to xt, [K step of 32][token][32].
template <int CH, bool COPY>
__global__ __launch_bounds__(256) void decode_score_kernel(RouterDev r, const bf16_t* __restrict__ x, const bf16_t* __restrict__ wr,
                                                           int tiled, int d, int T, int n_rows, float* __restrict__ pre_g,
                                                           bf16_t* __restrict__ xt) {
  __shared__ float red[4][16][20];                             // [wave][token][row]
  const int rb = blockIdx.x, slice = blockIdx.y, t0 = blockIdx.z * 16;
  if (!row_block_used(r, rb)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, kq = lane >> 4;
  const int steps = d / (DEC_SLICES * 32), per = (steps + 3) / 4;
  const int first = wave * per, n = steps - first < per ? steps - first : per;
  const int k0 = slice * steps + first;
  // (tiled: the copy in operand order, K step k of row block rb is the 1 KB at ((rb * d / 32 + k) * 64 + lane) * 8)
  const bf16_t* w = tiled ? wr + (((int64_t)rb * (d >> 5) + k0) * 64 + lane) * 8 : wr + (int64_t)(rb * 16 + r16) * d + k0 * 32 + kq * 8;
  const int wadv = tiled ? 512 : 32;
  const int t = t0 + r16;
  const bf16_t* xr = x + (int64_t)(t < T ? t : T - 1) * d + k0 * 32 + kq * 8;      // (past the last token: a copy, never stored)
  floatx4_t acc = {0.0f, 0.0f, 0.0f, 0.0f};
  for (int c = 0; c < n; c += CH) {
    bf16x8_t a[CH], b[CH];
#pragma unroll
    for (int s = 0; s < CH; ++s) {
      const int k = c + s < n ? c + s : n - 1;
      a[s] = *reinterpret_cast<const bf16x8_t*>(w + k * wadv);
      b[s] = *reinterpret_cast<const bf16x8_t*>(xr + k * 32);
    }
#pragma unroll
    for (int s = 0; s < CH; ++s) {
      if (c + s >= n) break;
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[s], b[s], acc, 0, 0, 0);
      // (the first row block's workgroups also leave the copy)
      if (COPY && rb == 0 && t < T) *reinterpret_cast<bf16x8_t*>(xt + ((int64_t)(k0 + c + s) * T + t) * 32 + kq * 8) = b[s];
    }
  }
  *reinterpret_cast<floatx4_t*>(&red[wave][r16][kq * 4]) = acc;      // D layout: rows kq*4 .. + 3 of column (token) r16
  __syncthreads();
  const int tok = tid >> 4, row = tid & 15;
  if (t0 + tok < T)
    pre_g[((int64_t)slice * T + t0 + tok) * n_rows + rb * 16 + row] =
        ((red[0][tok][row] + red[1][tok][row]) + red[2][tok][row]) + red[3][tok][row];
}

// The same partials computed inside a workgroup of eight waves instead of by a launch of its own: wave w takes
// K slice w of every block of 16 router rows, in decode_score_kernel's four chains (the router read from its copy in
// operand order), so the values are the same bits; they go to LDS as part[slice][token][row].  For at most 16 tokens.  The caller
// puts a barrier between this and the first read of `part`.
template <int KSTEPS>
__device__ __forceinline__ void score_slices_in_workgroup(const bf16_t* __restrict__ x, const bf16_t* __restrict__ wr,
                                                          int d, int T, int n_rows, float* part) {
  const int lane = threadIdx.x & 63, slice = threadIdx.x >> 6;
  const int r16 = lane & 15, kq = lane >> 4;
  const int kbase = slice * (KSTEPS * 32) + kq * 8;
  const bool ok = r16 < T;
  bf16x8_t b[KSTEPS];
  const bf16_t* xr = x + (int64_t)(ok ? r16 : 0) * d + kbase;
#pragma unroll
  for (int ks = 0; ks < KSTEPS; ++ks) {
    if (ok) b[ks] = *reinterpret_cast<const bf16x8_t*>(xr + ks * 32);
    else {
#pragma unroll
      for (int i = 0; i < 8; ++i) b[ks][i] = (__bf16)0.0f;
    }
  }
  for (int row0 = 0; row0 < n_rows; row0 += 16) {
    // wr is the copy in operand order: K step kk of row block rb is the 1 KB at ((rb * d/32 + kk) * 64 + lane) * 8
    const bf16_t* wop = wr + (((int64_t)(row0 >> 4) * (d >> 5) + slice * KSTEPS) * 64 + lane) * 8;
    bf16x8_t a[KSTEPS];
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) a[ks] = *reinterpret_cast<const bf16x8_t*>(wop + ks * 512);
    constexpr int PER = (KSTEPS + 3) / 4;
    floatx4_t acc[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[q][i] = 0.0f;
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) acc[ks / PER] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[ks], b[ks], acc[ks / PER], 0, 0, 0);
    if (ok) *reinterpret_cast<floatx4_t*>(part + ((int64_t)slice * T + r16) * n_rows + row0 + kq * 4) = ((acc[0] + acc[1]) + acc[2]) + acc[3];
  }
}

// route_place_kernel: a batch that fits one 64-token tile is selected and permuted by one workgroup:
// its threads add the K-slice partials of the pre-activations in slice order, score and select, then wave 0
// assigns the slots and wave 1 publishes the lists.  Histogram and routed entries are handed over in LDS (the
// workspace copies of the entries are not written: nothing after this kernel reads them).
// Every thread of the workgroup must call (barriers).
// `pre`: dynamic shared memory, [T][n_rows + 1] pre-activations, then scores [T][MAX_SCORED + 1].
// What a workgroup that runs gate/up units of routed group `group` learns from selecting the tile itself
// (route_place_body with `mine` set): the group's tokens in ascending order (its slots, by the placement rule),
// their number, and where the group's rows of H start (the exclusive prefix of count x padded width over the
// groups in id order, as place_lists computes it).
struct OwnSegment {
  int32_t tok[16];
  int32_t cnt;
  long long h_off;
};

__device__ __forceinline__ void route_place_body(const RouterDev& r, RouteIO io, const PlaceArgs& pl,
                                                 const float* __restrict__ partial, int T, float* pre,
                                                 int group = -1, OwnSegment* mine = nullptr) {
  __shared__ int32_t hist[MAX_GROUPS];
  __shared__ int32_t sel_g[TOK_TILE * MAX_DYN];
  __shared__ float sel_w[TOK_TILE * MAX_DYN];
  __shared__ GateLds gl;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n_threads = blockDim.x;
  const int n_rows = r.n_sw_rows + r.n_lin_rows;
  const int ld = n_rows + 1;
  float* sc = pre + T * ld;
  LaneWidths lw;
  if (wave <= 1) lw = load_lane_widths(pl, lane);          // needed last, requested first
  if (mine) {                                              // (nothing of the tile's routing is written by this workgroup)
    io.topk_out = nullptr;
    io.outer_out = nullptr;
    io.scores_out = nullptr;
  }
  const float2 gate = request_gate(r, io, tid);
  sum_partials_of<DEC_SLICES, 2>(r, partial, DEC_SLICES, T, 0, T, n_rows, pre, ld, tid, n_threads);
  for (int i = tid; i < MAX_GROUPS; i += n_threads) hist[i] = 0;
  store_gate(gl, gate, tid);
  __syncthreads();
  io.sel_group = sel_g;
  io.sel_weight = sel_w;
  if (T == 1) {
    // one token: wave 0 scores and selects it with one lane per expert
    if (wave == 0) route_token(r, io, pre, 0, hist);
    __syncthreads();
    if (wave == 0) place_slots(pl, 0, single_tile_counts(pl, hist, lane), sel_g, sel_w, lane);
    if (wave == 1) place_lists(pl, single_tile_counts(pl, hist, lane), lane, lw);
    return;
  }
  score_tile(r, io, pre, ld, sc, LD_SC, T, 0, tid, n_threads);
  __syncthreads();
  route_select_tile(r, io, sc, LD_SC, pre, ld, T, 0, hist, gl, tid, n_threads);
  __syncthreads();
  if (mine) {
    // T <= 16 tokens, G <= 64 groups (the caller checked): lane g holds group g's count and width, lane t token t
    if (wave == 0) {
      const int cnt = lane < pl.n_always ? T : (lane < pl.G ? hist[lane] : 0);
      const long long ah = (long long)cnt * lw.w[0];
      const long long h_incl = wave_incl_scan(ah);
      if (lane == group) {
        mine->cnt = cnt;
        mine->h_off = h_incl - ah;
      }
      bool has = false;
      if (lane < T)
        for (int i = 0; i < pl.S_dyn; ++i) has = has || sel_g[lane * pl.S_dyn + i] == group;
      const unsigned long long m = __ballot(has);
      if (has) mine->tok[__popcll(m & ((1ull << lane) - 1ull))] = lane;
    }
    __syncthreads();
    return;
  }
  if (wave == 0) place_slots(pl, 0, single_tile_counts(pl, hist, lane), sel_g, sel_w, lane);
  if (wave == 1) place_lists(pl, single_tile_counts(pl, hist, lane), lane, lw);
}

__global__ __launch_bounds__(RT_THREADS) void route_place_kernel(RouterDev r, RouteIO io, PlaceArgs pl,
                                                          const float* __restrict__ partial, int T) {
  extern __shared__ float pre[];
  route_place_body(r, io, pl, partial, T, pre);
}

// The same launch with company: workgroup 0 selects and places, the others run the gate/up units of the
// always-on (shared-expert) group, which need nothing from the router.  Selection and placement are one
// workgroup's chain of dependent steps, 8 us long at one token; the shared expert's share of the gate/up
// stream (half of the bytes at one token) is read meanwhile instead of afterwards, with no hand-off between
// workgroups and no second stream.  The gate/up work list then leaves that group out.
template <int KSTEPS, bool RUNS>
__global__ __launch_bounds__(512) void route_place_shared_kernel(RouterDev r, RouteIO io, PlaceArgs pl,
                                                                 const float* __restrict__ partial, int T,
                                                                 DecArgs da) {
  extern __shared__ float pre[];
  __shared__ DecGateUpRed<1> red;
  if (blockIdx.x == 0) {
    route_place_body(r, io, pl, partial, T, pre);
    return;
  }
  decode_gate_up<1, KSTEPS, RUNS>(da, da.groups[0].w1_row0, (int)blockIdx.x - 1, 0, T, da.groups[0].width_pad, 0, red);
}

// The same for the batches of 2 to 64 tokens that run streamed units.
template <int MAXT, int CS, int NEUR>
__global__ __launch_bounds__(512) void route_place_stream_kernel(RouterDev r, RouteIO io, PlaceArgs pl, const float* __restrict__ partial,
                                                                 int T, DecArgs da) {
  extern __shared__ float pre[];
  if (blockIdx.x == 0) {
    route_place_body(r, io, pl, partial, T, pre);
    return;
  }
  stream_gate_up<MAXT, CS, NEUR>(da, da.groups[0].w1_row0, (int)blockIdx.x - 1, 0, T, da.groups[0].width_pad, 0, pre);
}

// One token on a flat layer: the launch that selects and places also runs *every* gate/up unit, the routed
// ones included.  Workgroup 0 is route_place_kernel's body; workgroups 1 .. U_s run the shared group's units;
// workgroup 1 + U_s + k * U_r + j runs unit j of the k-th selected expert, which it finds by itself: its wave 0
// adds the K-slice partials of the router pre-activations in the same order as workgroup 0 does, scores them
// with the same arithmetic and runs the same top-N_k, so every workgroup arrives at the same experts with no
// hand-off between workgroups.  What it needs is 8 slices x the router rows (a few KB, the same few lines for
// all workgroups), not the router matrix.  The rows of H follow the placement rule: segments in ascending
// group id, so the expert's row of H starts after the shared group's and after the rows of the selected
// experts with smaller ids.  One launch and its gap less than scoring + (selection, shared units) + routed
// units; the separate gate/up launch is skipped.
template <int KSTEPS, bool RUNS>
__global__ __launch_bounds__(512) void route_place_all_kernel(RouterDev r, RouteIO io, PlaceArgs pl,
                                                              const float* __restrict__ partial,
                                                              DecArgs da, int units_shared, int units_routed,
                                                              const bf16_t* __restrict__ wr) {
  extern __shared__ float pre[];
  __shared__ DecGateUpRed<1> red;
  __shared__ int32_t my_sel_g[MAX_DYN];
  __shared__ float my_sel_w[MAX_DYN];
  const int n_rows = r.n_sw_rows + r.n_lin_rows;
  const int b = (int)blockIdx.x - 1;
  if (b >= 0 && b < units_shared) {
    decode_gate_up<1, KSTEPS, RUNS>(da, da.groups[0].w1_row0, b, 0, 1, da.groups[0].width_pad, 0, red);
    return;
  }
  if constexpr (!RUNS) {                                   // (own_scores asks for one run)
    if (wr) {
      // no scoring launch: every workgroup that needs the pre-activations computes the K-slice partials itself
      // (the router matrix is a few hundred KB that all of them find in L2 after the first) and keeps them in
      // LDS behind the selection's arrays
      float* part = pre + ((n_rows + 1 + MAX_SCORED + 1 + 3) & ~3);      // 16-byte aligned
      score_slices_in_workgroup<KSTEPS>(da.x, wr, da.d, 1, n_rows, part);
      __syncthreads();
      partial = part;
    }
  }
  if (blockIdx.x == 0) {
    route_place_body(r, io, pl, partial, 1, pre);
    return;
  }
  const int k = (b - units_shared) / units_routed, local = (b - units_shared) % units_routed;
  const int tid = threadIdx.x;
  // (where every group's rows lie, requested before the choice is known)
  int row0[MAX_GROUPS / 64];
#pragma unroll
  for (int q = 0; q < MAX_GROUPS / 64; ++q) {
    if (q > 0 && 64 * q >= da.G) break;
    row0[q] = da.groups[min((tid & 63) + 64 * q, da.G - 1)].w1_row0;
  }
  const int wp = da.groups[r.n_always].width_pad;          // (the routed groups have one width)
  if (tid < 64) {
    for (int row = tid; row < n_rows; row += 64) {
      // all slices in flight together (one after the other: 16 experts, d = 4096 21.5 us per forward, now 19.8)
      float v[DEC_SLICES], acc = 0.0f;
#pragma unroll
      for (int sl = 0; sl < DEC_SLICES; ++sl) v[sl] = partial[(int64_t)sl * n_rows + row];     // T = 1: [slice][row]
#pragma unroll
      for (int sl = 0; sl < DEC_SLICES; ++sl) acc += v[sl];
      pre[row] = acc;
    }
    wave_lds_sync();
    RouteIO mine = io;
    mine.sel_group = my_sel_g;
    mine.sel_weight = my_sel_w;
    mine.topk_out = nullptr;
    mine.outer_out = nullptr;
    mine.scores_out = nullptr;
    route_token(r, mine, pre, 0, nullptr);
  }
  __syncthreads();
  const int g = __builtin_amdgcn_readfirstlane(my_sel_g[k]);
  int rank = 0;
  for (int i = 0; i < r.top_k; ++i) rank += my_sel_g[i] < g ? 1 : 0;
  int w1_row0 = __builtin_amdgcn_readlane(row0[0], g & 63);
#pragma unroll
  for (int q = 1; q < MAX_GROUPS / 64; ++q)
    if (g >= 64 * q) w1_row0 = __builtin_amdgcn_readlane(row0[q], g & 63);
  const int64_t hoff = (r.n_always ? (int64_t)da.groups[0].width_pad : 0) + (int64_t)rank * wp;
  decode_gate_up<1, KSTEPS, RUNS>(da, w1_row0, local, 0, 1, wp, hoff, red);
}

// Two to sixteen tokens on a flat layer, the same idea: workgroup 0 selects and places the batch, the next
// workgroups run the shared group's units, and every unit of *every* routed expert has a workgroup that
// selects the whole batch by itself (route_place_kernel's selection on the scorer's partials, 16 KB that all
// workgroups share in L2), learns which tokens chose its expert and where the expert's rows of H start, and runs
// its unit on them; the workgroups of experts nobody chose leave.  The separate gate/up launch, which could not
// start before selection and placement had finished in one workgroup, is gone.  Bit-identical to the two launches
// and slower than them almost everywhere (us per forward at 2, 4, 8, 16 tokens: 16 experts of 688 35.0, 38.0, 48.8, 59.3
// against 29.6, 39.7, 43.1, 55.8; 32 of 448 40.1, 43.5, 51.2, 68.2 against 32.0, 41.7, 45.0, 61.7), so it is off unless
// the tuning switch front_tile asks for it.
template <int KSTEPS, bool RUNS>
__global__ __launch_bounds__(512) void route_place_tile_all_kernel(RouterDev r, RouteIO io, PlaceArgs pl,
                                                                   const float* __restrict__ partial, int T,
                                                                   DecArgs da, int units_shared, int units_routed) {
  extern __shared__ float pre[];
  __shared__ DecGateUpRed<1> red;
  __shared__ OwnSegment own;
  const int b = (int)blockIdx.x - 1;
  if (b >= 0 && b < units_shared) {
    decode_gate_up<1, KSTEPS, RUNS>(da, da.groups[0].w1_row0, b, 0, T, da.groups[0].width_pad, 0, red);
    return;
  }
  if (blockIdx.x == 0) {
    route_place_body(r, io, pl, partial, T, pre);
    return;
  }
  const int g = r.n_always + (b - units_shared) / units_routed, local = (b - units_shared) % units_routed;
  route_place_body(r, io, pl, partial, T, pre, g, &own);
  const int cnt = own.cnt;
  if (cnt == 0) return;
  da.slot2tok = own.tok;                          // slot j of this group = its j-th token in ascending order
  decode_gate_up<1, KSTEPS, RUNS>(da, da.groups[g].w1_row0, local, 0, cnt, da.groups[g].width_pad, own.h_off, red);
}

// Per-tile histogram of the routed entries (used when the scoring kernel did not produce one).
__global__ __launch_bounds__(64) void tile_count_kernel(const int32_t* __restrict__ sel_group, int64_t T, int S_dyn,
                                                        int G, int32_t* __restrict__ tile_counts) {
  __shared__ int32_t hist[MAX_GROUPS];
  const int lane = threadIdx.x;
  for (int i = lane; i < MAX_GROUPS; i += 64) hist[i] = 0;
  __syncthreads();
  const int64_t t = (int64_t)blockIdx.x * TOK_TILE + lane;
  if (t < T)
    for (int i = 0; i < S_dyn; ++i) atomicAdd(&hist[sel_group[t * S_dyn + i]], 1);
  __syncthreads();
  for (int g = lane; g < G; g += 64) tile_counts[(int64_t)blockIdx.x * G + g] = hist[g];
}

PlaceArgs make_place_args(const Engine& e, int64_t T, char* ws, const WsLayout& L, int32_t* counts_out);

// The MFMA scorer needs bf16 operands, K slices of 256 and whole 32-row blocks of router rows (at most five).
static bool mfma_scorer_ok(const Engine& e) {
  const int n_rows = e.r.n_sw_rows + e.r.n_lin_rows;
  return e.dtype == 1 && e.d % 256 == 0 && n_rows % 32 == 0 && n_rows / 32 <= 5;
}

// K slices of the scorer: enough workgroups to fill 256 CUs, at least 256 of K per slice, at most the partial
// buffer's 8.
static int scorer_slices(const Engine& e, int64_t T) {
  const int64_t n_tt = (T + RT_TOK - 1) / RT_TOK;
  int n = (int)std::min<int64_t>((512 + n_tt - 1) / n_tt, 8);
  while (n > 1 && (e.d % (n * 256) != 0)) --n;
  return n;
}

// Units of (slice, class) per wave of score_route_kernel, 0: this batch takes the separate scorer.  A flat layer whose
// router has a copy in operand order, whole pairs of chunks per unit (or one chunk), and either
//  - at most two slices, i.e. a batch that fills the chip with 32 tokens per workgroup (8192 tokens of the 32-expert
//    layer: 31 us against 34 + 10), or
//  - 16 tokens per workgroup, which then pulls at most 640 KB of tokens and router rows (one takes in about 50 KB per us, see the kernel).
// us per forward in two launches / in one, d = 4096, 32 experts (64 rows, 640 KB): 70 tokens 40.3 / 39.3, 2048 78.9 / 75.0,
// 3000 352.1 / 343.2, 4096 459.7 / 450.1; d = 2048, 32 experts, 4096 tokens 128.7 / 121.3.  Up to 16 experts (32 rows): d = 1024,
// 333 tokens 36.5 / 31.4 and 4096 62.4 / 55.9; d = 5120 (480 KB) 70 tokens 105.3 / 101.9, 2048 345 / 336.
// Above 640 KB it is the tokens that decide, and the line is on the safe side for many of them.  Layers of narrow experts, ratio of two
// launches to one at 65-1000 / 1300-2048 / 3000-4096 tokens (five to eight slices): 32 rows, d = 7168 (672 KB) 1.03 / 1.08 / -, 8192
// 1.01 / 1.07 / 1.12; 64 rows, d = 5120 (800 KB) 1.01 / 1.05 / 1.08, 8192 (1.3 MB) 0.93 / 1.02 / 1.09; 128 rows, d = 2560 (720 KB) 1.02 / 1.11 /
// 1.17, 3072 (864 KB) 0.99 / 1.08 / 1.25, 4096 (1.1 MB) 0.95 / 1.09 / 1.15, 8192 (2.3 MB) 0.88 / 1.02 / 1.10.
// Row blocks in use (see the kernel) of a layer of 16 experts, d = 4096, against all four: 333 tokens 109.8 -> 104.5 us per
// forward, 2048 208.0 -> 202.7 (the launch 15.8 -> 10.5 us); d = 1024, 333 tokens 36.5 -> 31.4.
static constexpr int score_route_tokens(int upw) { return upw >= 2 ? 16 : 32; }
static int score_route_blocks(const Engine& e) { return e.r.n_scored <= 16 ? 2 : 4; }
static int score_route_units(const Engine& e, int64_t T) {
  if (!mfma_scorer_ok(e) || e.wr_tiled == nullptr || e.r.outer_top_k != 0 || e.r.n_lin_rows != 0 || e.r.n_sw_rows % 64 != 0) return 0;
  const int S = scorer_slices(e, T), n_i = e.d / S / 256;
  if (n_i != 1 && n_i % 2 != 0) return 0;
  const int rows = e.r.n_sw_rows * score_route_blocks(e) / 4;
  if (S > 2 && (int64_t)(16 + rows) * e.d > (16 + 64) * 4096) return 0;
  return (4 * S + 7) / 8;
}

CountTable router_counts(const Engine& e, int64_t T, const WsLayout& L) {
  if (const int upw = score_route_units(e, T)) return {score_route_tokens(upw), L.scores};   // (no partial sums there)
  return {TOK_TILE, L.tile_counts};
}

template <int UPW, bool ONE, int NB>
static hipError_t launch_score_route(const Engine& e, const RouteIO& io, const void* x, int64_t T, int n_slices,
                                     int32_t* counts, hipStream_t s) {
  constexpr int TB = score_route_tokens(UPW) / 16, NTOK = TB * 16;
  const size_t smem = sizeof(float) * (size_t)NTOK * (n_slices * (64 + 4) + e.r.n_sw_rows + 1 + LD_SC);
  // at most 2 UPW slices and two groups of 64 rows
  constexpr size_t most = sizeof(float) * NTOK * (2 * UPW * (64 + 4) + 128 + 1 + LD_SC);
  static LdsLimit limit;
  const hipError_t err = limit.raise(reinterpret_cast<const void*>(score_route_kernel<UPW, TB, ONE, NB>), most);
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL((score_route_kernel<UPW, TB, ONE, NB>), dim3((unsigned)((T + NTOK - 1) / NTOK)), dim3(512), smem, s, e.r, io,
                     static_cast<const bf16_t*>(x), static_cast<const bf16_t*>(e.wr_tiled), e.d, T, n_slices,
                     e.d / n_slices, counts, e.G);
  return hipGetLastError();
}

// Pre-activation partials [slice][T][n_rows] of all router rows by router_gemm_kernel.
static hipError_t launch_scorer_gemm(const Engine& e, const void* x, int64_t T, float* partial, hipStream_t s, int& n_slices) {
  const int n_rows = e.r.n_sw_rows + e.r.n_lin_rows;
  const int n_tt = (int)((T + RT_TOK - 1) / RT_TOK);
  n_slices = scorer_slices(e, T);
  const int k_slice = e.d / n_slices;
  dim3 grid(n_tt, n_slices), block(256);
  const bf16_t* xx = static_cast<const bf16_t*>(x);
  const bf16_t* ww = static_cast<const bf16_t*>(e.wr);
#define CMOE_SCORER(NT) hipLaunchKernelGGL(router_gemm_kernel<NT>, grid, block, 0, s, xx, ww, e.d, T, k_slice, partial)
  switch (n_rows / 32) {
    case 1: CMOE_SCORER(1); break;
    case 2: CMOE_SCORER(2); break;
    case 3: CMOE_SCORER(3); break;
    case 4: CMOE_SCORER(4); break;
    default: CMOE_SCORER(5); break;
  }
#undef CMOE_SCORER
  return hipGetLastError();
}

// One tile of at most 64 tokens is scored in one launch and selected + placed by one workgroup in a second.  The larger
// batches need the tile's pre-activations and scores to fit the 64 KB of LDS a workgroup gets by default next to 14 KB of
// static arrays.
constexpr int FRONT_SCORE_MAX_T = 16;
bool decode_front_ok(const Engine& e, int64_t T) {
  const int n_rows = e.r.n_sw_rows + e.r.n_lin_rows;
  if (e.S_dyn <= 0 || T < 1 || T > TOK_TILE) return false;
  if (T <= FRONT_SCORE_MAX_T && decode_path_ok(e, T)) return n_rows % 16 == 0;
  return mfma_scorer_ok(e) && sizeof(float) * (size_t)T * (n_rows + 1 + MAX_SCORED + 1) <= 48 * 1024;
}

// Router scoring (one launch) and selection + permutation (one launch) of a decode batch.
hipError_t launch_decode_front(const Engine& e, const void* x, int64_t T, char* ws, const WsLayout& L,
                               int32_t* topk_out, int32_t* outer_out, float* scores_out, int32_t* counts_out,
                               hipStream_t s) {
  RouteIO io;
  io.sel_group = reinterpret_cast<int32_t*>(ws + L.sel_group);
  io.sel_weight = reinterpret_cast<float*>(ws + L.sel_weight);
  io.topk_out = topk_out;
  io.outer_out = outer_out;
  io.scores_out = scores_out;
  io.gate_u = e.gate_u;
  io.gate_b = e.gate_b;
  io.lin_off = e.lin_off;
  io.S_dyn = e.S_dyn;
  const PlaceArgs pl = make_place_args(e, T, ws, L, counts_out);
  const int n_rows = e.r.n_sw_rows + e.r.n_lin_rows;
  float* pre_g = reinterpret_cast<float*>(ws + L.scores);
  const int Ti = (int)T;
  bf16_t* xt = front_lays_tokens(e, T) ? reinterpret_cast<bf16_t*>(ws + L.y_slots) : nullptr;
  hipError_t err = hipSuccess;
  // one token, every gate/up unit in the selection launch: with front_all = 2 that launch also scores
  const bool own_scores = L.gate_up_done && tuning().front_all >= 2 && e.wr_tiled != nullptr && decode_k(e.d).nch == 1;
  if (!own_scores) {
    const dim3 grid(n_rows / 16, DEC_SLICES, (unsigned)((T + 15) / 16)), block(256);
    const bf16_t* xx = static_cast<const bf16_t*>(x);
    const int tiled = e.wr_tiled != nullptr ? 1 : 0;
    const bf16_t* ww = static_cast<const bf16_t*>(tiled ? e.wr_tiled : e.wr);
#define CMOE_SCORE(CH)                                                                                                              \
  if (xt) hipLaunchKernelGGL((decode_score_kernel<CH, true>), grid, block, 0, s, e.r, xx, ww, tiled, e.d, Ti, n_rows, pre_g, xt); \
  else hipLaunchKernelGGL((decode_score_kernel<CH, false>), grid, block, 0, s, e.r, xx, ww, tiled, e.d, Ti, n_rows, pre_g, xt)
    // (measurement aid: repeat_stage = 6 issues the scoring launch twice; it overwrites its partials)
    for (int rep = tuning().repeat_stage == 6 ? 2 : 1; rep > 0; --rep) {
      if (e.d <= 4 * 4 * DEC_SLICES * 32) { CMOE_SCORE(4); } else { CMOE_SCORE(8); }
    }
#undef CMOE_SCORE
    err = hipGetLastError();
  }
  if (err != hipSuccess) return err;
  if (tuning().skip_stage == 6) return hipSuccess;        // measurement aid: the scoring launch only
  size_t smem = sizeof(float) * (size_t)T * (n_rows + 1 + MAX_SCORED + 1);
  if (L.gate_up_done && T > 1) {
    // (the caller set this from decode_front_runs_all: 2-16 tokens, flat layer of at most 64 groups, routed
    // groups of one width, 16-neuron units)
    DecArgs da = make_dec_args(e, x, T, ws, L, nullptr);
    da.slot2tok = nullptr;                        // group 0's slots are the tokens in order
    da.work = nullptr;
    const int us = e.n_always ? e.width_pad_host[0] / 16 : 0;
    const int ur = e.width_pad_host[e.n_always] / 16;
    const dim3 grid(1 + us + (e.G - e.n_always) * ur), block(512);
    for (int rep = tuning().repeat_stage == 3 ? 2 : 1; rep > 0; --rep)       // (measurement aid, as below)
#define CMOE_LAUNCH(KS, RUNS) hipLaunchKernelGGL((route_place_tile_all_kernel<KS, RUNS>), grid, block, smem, s, e.r, io, pl, pre_g, Ti, da, us, ur)
      { CMOE_DECODE_KSTEPS(e.d, CMOE_LAUNCH) }
#undef CMOE_LAUNCH
    return hipGetLastError();
  }
  if (L.gate_up_done) {
    // (the caller set this from decode_front_runs_all: one token, flat layer, routed groups of one width)
    DecArgs da = make_dec_args(e, x, T, ws, L, nullptr);
    da.slot2tok = nullptr;                        // one token: every slot is token 0
    da.work = nullptr;
    const int us = e.n_always ? e.width_pad_host[0] / da.unit1 : 0;
    const int ur = e.width_pad_host[e.n_always] / da.unit1;
    const dim3 grid(1 + us + e.r.top_k * ur), block(512);
    const bf16_t* wr_in = own_scores ? static_cast<const bf16_t*>(e.wr_tiled) : nullptr;
    if (own_scores) smem = sizeof(float) * (size_t)(((n_rows + 1 + MAX_SCORED + 1 + 3) & ~3) + DEC_SLICES * n_rows);
    // (measurement aid: this launch is the layer's gate/up stage, so repeat_stage = 3 issues it twice; it reads
    // only the scorer's partials, the token and the weights, and every write is a plain store of a value that
    // depends on those alone, so the second launch leaves the same bits)
    for (int rep = tuning().repeat_stage == 3 ? 2 : 1; rep > 0; --rep)
#define CMOE_LAUNCH(KS, RUNS) hipLaunchKernelGGL((route_place_all_kernel<KS, RUNS>), grid, block, smem, s, e.r, io, pl, pre_g, da, us, ur, wr_in)
      { CMOE_DECODE_KSTEPS(e.d, CMOE_LAUNCH) }
#undef CMOE_LAUNCH
    return hipGetLastError();
  }
  if (L.skip_always && front_lays_tokens(e, T)) {
    // (the caller set this from decode_front_runs_shared: one always-on group, streamed gate/up units)
    DecArgs da = make_stream_args(e, x, T, ws, L);
    da.slot2tok = nullptr;                        // as below
    smem = std::max(smem, sizeof(float) * (size_t)STREAM_RED_FLOATS);
    // (units of 8 neurons while each finds a CU of its own: 17 tokens, 16 experts of 688, 63.2 -> 62.5 us per forward)
    const bool half = tuning().decode_split == 8 || (tuning().decode_split != 16 && e.width_pad_host[0] / 8 < 256);
    const dim3 grid(1 + e.width_pad_host[0] / (half ? 8 : 16)), block(512);
#define CMOE_LAUNCH_N(MAXT, CS, NEUR) hipLaunchKernelGGL((route_place_stream_kernel<MAXT, CS, NEUR>), grid, block, smem, s, e.r, io, pl, pre_g, Ti, da)
#define CMOE_LAUNCH(MAXT, CS) if (half) CMOE_LAUNCH_N(MAXT, CS, 8); else CMOE_LAUNCH_N(MAXT, CS, 16)
    CMOE_STREAM_FORM(T, e.d, CMOE_LAUNCH)
#undef CMOE_LAUNCH
#undef CMOE_LAUNCH_N
    return hipGetLastError();
  }
  if (L.skip_always) {
    // (likewise, decode units: one token whose routed units have a launch of their own, or 2 to 16 below the streamed widths)
    DecArgs da = make_dec_args(e, x, T, ws, L, nullptr);
    da.slot2tok = nullptr;                        // group 0's slots are the tokens in order; the map is not written yet
    da.work = nullptr;
    const dim3 grid(1 + e.width_pad_host[0] / da.unit1), block(512);
#define CMOE_LAUNCH(KS, RUNS) hipLaunchKernelGGL((route_place_shared_kernel<KS, RUNS>), grid, block, smem, s, e.r, io, pl, pre_g, Ti, da)
    { CMOE_DECODE_KSTEPS(e.d, CMOE_LAUNCH) }
#undef CMOE_LAUNCH
    return hipGetLastError();
  }
  hipLaunchKernelGGL(route_place_kernel, dim3(1), dim3(RT_THREADS), smem, s, e.r, io, pl, pre_g, Ti);
  return hipGetLastError();
}

bool decode_front_runs_shared(const Engine& e, int64_t T) {
  if (tuning().front_shared == 0 || e.n_always != 1 || !decode_front_ok(e, T)) return false;
  return decode_path_ok(e, T) ? T <= FRONT_SCORE_MAX_T : tiles_gate_up_streams(e, T);
}

// One token (switch front_all), or two to sixteen (switch front_tile; at most 64 groups, 16-neuron units), on a
// flat routed layer whose routed groups all have one width, at most one always-on group, the decode kernels'
// model widths (tuning switch front_shared = 0 switches this off together with the shared units in the front
// end).
bool decode_front_runs_all(const Engine& e, int64_t T) {
  if (T < 1 || T > FRONT_SCORE_MAX_T || tuning().front_shared == 0) return false;
  if (T == 1 ? tuning().front_all == 0 : (tuning().front_tile == 0 || e.G > 64 || tuning().decode_split == 8)) return false;
  if (e.r.outer_top_k != 0 || e.n_always > 1 || e.G <= e.n_always || e.S_dyn != e.r.top_k) return false;
  if (!decode_front_ok(e, T) || !decode_path_ok(e, T)) return false;
  for (int g = e.n_always; g < e.G; ++g)
    if (e.width_pad_host[g] != e.width_pad_host[e.n_always]) return false;
  return true;
}

void scorer_plan(const Engine& e, int64_t T, int32_t plan[2]) {
  const bool front = !use_simt_experts(e.dtype) && decode_front_ok(e, T), sliced = mfma_scorer_ok(e);
  plan[0] = front ? CMOE_SCORER_SMALL : score_route_units(e, T) ? CMOE_SCORER_SELECTS : sliced ? CMOE_SCORER_SPLIT : CMOE_SCORER_TOKENS;
  plan[1] = front ? DEC_SLICES : sliced ? scorer_slices(e, T) : 0;
}

// Few entries behind the scorer without a histogram: every workgroup of the placement counts them all, which a launch of
// its own takes longer for (fp32, d = 256, 64 tokens: 1.3 us and a gap for the launch, placement 5.1 us with it, 5.3 without).
bool place_counts_itself(const Engine& e, int64_t T) {
  return !mfma_scorer_ok(e) && score_route_units(e, T) == 0 && T * e.S_dyn <= 2048;
}

hipError_t launch_router(const Engine& e, const void* x, int64_t T, char* ws, const WsLayout& L,
                         int32_t* topk_out, int32_t* outer_out, float* scores_out, hipStream_t s) {
  if (e.S_dyn == 0 || T == 0) return hipSuccess;
  RouteIO io;
  io.sel_group = reinterpret_cast<int32_t*>(ws + L.sel_group);
  io.sel_weight = reinterpret_cast<float*>(ws + L.sel_weight);
  io.topk_out = topk_out;
  io.outer_out = outer_out;
  io.scores_out = scores_out;
  io.gate_u = e.gate_u;
  io.gate_b = e.gate_b;
  io.lin_off = e.lin_off;
  io.S_dyn = e.S_dyn;
  int32_t* tile_counts = reinterpret_cast<int32_t*>(ws + L.tile_counts);
  const int n_rows = e.r.n_sw_rows + e.r.n_lin_rows;
  if (const int upw = score_route_units(e, T)) {
    const int S = scorer_slices(e, T);
    const bool one = e.d / S == 256;
    tile_counts = reinterpret_cast<int32_t*>(ws + L.scores);
    const bool two = score_route_blocks(e) == 2;
#define CMOE_LAUNCH_B(UPW, ONE, NB) return launch_score_route<UPW, ONE, NB>(e, io, x, T, S, tile_counts, s)
#define CMOE_LAUNCH(UPW)                                                          \
  if (one) { if (two) CMOE_LAUNCH_B(UPW, true, 2); else CMOE_LAUNCH_B(UPW, true, 4); } \
  else { if (two) CMOE_LAUNCH_B(UPW, false, 2); else CMOE_LAUNCH_B(UPW, false, 4); }
    switch (upw) {
      case 1: CMOE_LAUNCH(1)
      case 2: CMOE_LAUNCH(2)
      case 3: CMOE_LAUNCH(3)
      default: CMOE_LAUNCH(4)
    }
#undef CMOE_LAUNCH
#undef CMOE_LAUNCH_B
  }
  if (mfma_scorer_ok(e)) {
    int n_slices = 1;
    float* partial = reinterpret_cast<float*>(ws + L.scores);
    hipError_t err = launch_scorer_gemm(e, x, T, partial, s, n_slices);
    if (err != hipSuccess) return err;
    const size_t smem = sizeof(float) * (size_t)TOK_TILE * (n_rows + 1 + MAX_SCORED + 1);
    hipLaunchKernelGGL(route_tile_kernel, dim3(L.n_tok_tiles), dim3(RT_THREADS), smem, s, e.r, io, partial, n_slices, T,
                       tile_counts, e.G);
    return hipGetLastError();
  }
  const size_t smem = sizeof(float) * (size_t)(e.d + n_rows);
  if (e.dtype == 1)
    hipLaunchKernelGGL(router_simt_kernel<bf16_t>, dim3((unsigned)T), dim3(256), smem, s, e.r, io,
                       static_cast<const bf16_t*>(x), static_cast<const bf16_t*>(e.wr), e.d);
  else
    hipLaunchKernelGGL(router_simt_kernel<float>, dim3((unsigned)T), dim3(256), smem, s, e.r, io,
                       static_cast<const float*>(x), static_cast<const float*>(e.wr), e.d);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess || place_counts_itself(e, T)) return err;
  hipLaunchKernelGGL(tile_count_kernel, dim3(L.n_tok_tiles), dim3(64), 0, s, io.sel_group, T, e.S_dyn, e.G,
                     tile_counts);
  return hipGetLastError();
}

}  // namespace cmoe
