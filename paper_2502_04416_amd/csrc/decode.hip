// Expert kernels for decode batches (T <= 16 tokens, bf16; the fused down + combine kernel up to 64):
// weight streaming bound by HBM bandwidth.
//
// Every expert group with at least one token is cut into units of 16 neurons (gate/up) or 16 output
// columns (down).  The weights of a unit are the A operand of v_mfma_f32_16x16x32_bf16 and are read
// straight from global memory exactly once, 64 contiguous bytes per row and instruction; the tokens
// of the group (at most 16, gathered through slot2tok) are the B operand and stay in registers for
// the whole unit.  The reduction dimension is split over the waves of a workgroup so that a unit
// keeps many independent loads in flight; the partial sums are added in a fixed order through LDS.
// This is the per-neuron form of the FFN, F(x) = sum_i h_i w_i (Eq. 1), evaluated only for the
// neurons of the experts some token selected (Eq. 4).
#include <algorithm>
#include <cstdlib>
#include "cmoe_internal.h"
#include "decode_device.h"
#include "device_utils.h"
#include "gemm_device.h"
#include "work_item.h"

namespace cmoe {

// The LDS operations of one wave complete in issue order: waiting for them (and keeping the compiler from
// moving LDS accesses across) is enough to order a wave's own LDS updates.
__device__ __forceinline__ void wave_lds_sync_decode() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_wave_barrier();
}

// Which unit is this workgroup?  Returns false when past the end of the list.
__device__ __forceinline__ bool find_unit(const DecArgs& p, int units_single, WorkItem& it) {
  const int u = blockIdx.x;
  if (p.single) {
    if (u >= units_single) return false;
    const GroupDev gd = p.groups[0];
    it = {0, u, 0, (int)p.T, gd.width_pad, gd.w1_row0, 0, gd.w2_off};
    return true;
  }
  const GroupLanes gl = request_groups(p.work, p.seg_off, p.groups, p.h_off, p.G);
  if (u >= p.work[p.G]) return false;
  it = find_item(gl, p.G, u);
  return true;
}

// ---- gate/up: H[slot][n] = Swish(x . wgate_n) * (x . wup_n) for 16 neurons of one group ---------------
template <int NTT, int KSTEPS, bool RUNS>
__global__ __launch_bounds__(512) void decode_gate_up_kernel(DecArgs p) {
  __shared__ DecGateUpRed<NTT> red;
  WorkItem it;
  if (!find_unit(p, p.single ? p.groups[0].width_pad / p.unit1 : 0, it)) return;
  decode_gate_up<NTT, KSTEPS, RUNS>(p, it.w1_row0, it.local, it.seg0, it.cnt, it.wp, it.hoff, red);
}

// ---- down: Y[slot][c] = sum_n H[slot][n] * Wdown[n][c] for 16 output columns of one group --------------
// 4 waves; wave w takes the 32-wide K steps w, w+4, ...
template <int NTT>
__global__ __launch_bounds__(256) void decode_down_kernel(DecArgs p) {
  __shared__ float red[4][NTT][16][17];
  WorkItem it;
  if (!find_unit(p, p.single ? p.d / 16 : 0, it)) return;
  const int seg0 = it.seg0, cnt = it.cnt, wp = it.wp;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r16 = lane & 15, kq = lane >> 4;
  const int c0 = it.local * 16;
  const bf16_t* wrow = p.w2 + it.w2_off +
                       (p.tiled ? tiled_offset(c0 + r16, kq * 8, wp / TILE_K) : (int64_t)(c0 + r16) * wp + kq * 8);
  const int kadv = p.tiled ? TILE_ELEMS : 32;                 // elements from one K step's operand to the next
  const bf16_t* hrow[NTT];
  bool hok[NTT];
#pragma unroll
  for (int tt = 0; tt < NTT; ++tt) {
    const int col = tt * 16 + r16;
    hok[tt] = col < cnt;
    hrow[tt] = p.h + it.hoff + (int64_t)(hok[tt] ? col : 0) * wp + kq * 8;
  }
  floatx4_t acc[NTT];
#pragma unroll
  for (int tt = 0; tt < NTT; ++tt)
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[tt][i] = 0.0f;
  const int n_steps = wp / 32;
  int ks = wave;
  // eight K steps of this wave at a time: their loads are independent and all in flight together
  for (; ks + 28 < n_steps; ks += 32) {
    bf16x8_t a[8], b[NTT][8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      a[u] = ld_frag(wrow + (ks + 4 * u) * kadv);
#pragma unroll
      for (int tt = 0; tt < NTT; ++tt) b[tt][u] = hok[tt] ? ld_frag(hrow[tt] + (ks + 4 * u) * 32) : zero_frag();
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int tt = 0; tt < NTT; ++tt) acc[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u], b[tt][u], acc[tt], 0, 0, 0);
  }
  for (; ks + 12 < n_steps; ks += 16) {
    bf16x8_t a[4], b[NTT][4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      a[u] = ld_frag(wrow + (ks + 4 * u) * kadv);
#pragma unroll
      for (int tt = 0; tt < NTT; ++tt) b[tt][u] = hok[tt] ? ld_frag(hrow[tt] + (ks + 4 * u) * 32) : zero_frag();
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int tt = 0; tt < NTT; ++tt) acc[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u], b[tt][u], acc[tt], 0, 0, 0);
  }
  for (; ks < n_steps; ks += 4) {
    const bf16x8_t a = ld_frag(wrow + ks * kadv);
#pragma unroll
    for (int tt = 0; tt < NTT; ++tt) {
      const bf16x8_t b = hok[tt] ? ld_frag(hrow[tt] + ks * 32) : zero_frag();
      acc[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[tt], 0, 0, 0);
    }
  }
#pragma unroll
  for (int tt = 0; tt < NTT; ++tt)
#pragma unroll
    for (int i = 0; i < 4; ++i) red[wave][tt][kq * 4 + i][r16] = acc[tt][i];
  __syncthreads();
  for (int e = tid; e < NTT * 256; e += 256) {
    const int tt = e >> 8, tok = (e >> 4) & 15, cc = e & 15;       // column fastest: contiguous stores
    const int col = tt * 16 + tok;
    if (col >= cnt) continue;
    const float s = (red[0][tt][cc][tok] + red[1][tt][cc][tok]) + (red[2][tt][cc][tok] + red[3][tt][cc][tok]);
    p.y[(int64_t)(seg0 + col) * p.d + c0 + cc] = f32_to_bf16(s);
  }
}

// ---- down + combine: y[t][c] = sum over the token's slots of weight * sum_n H[slot][n] * Wdown[n][c] ---------
// One workgroup owns 16 output columns of every token, so the weighted sum over a token's experts (Eq. 4,
// Eq. 10) needs no second pass and no per-slot outputs in memory.  Its work items are (non-empty group,
// chunk of DC_CH K steps); wave w takes items w, w + 16, ... and adds its weighted partial products into
// accumulators of its own in LDS, which are summed in wave order at the end: the result does not depend on
// timing.  All loads of an item are in flight together.
constexpr int DC_CH = 8;
constexpr int DC_WAVES = 16;
// What an item needs of its group, in LDS: every lane requests all of it for its two groups at once, one round trip where the
// offsets, then the widths, then (per item) offsets, width and places again were four.  us per forward before / now, with operands as
// buffer loads: d = 4096, 16 experts, 4 tokens 38.8 / 38.6, 24 tokens 62.3 / 61.8; 32 experts, 32 tokens 67.7 / 67.9; d = 8192, one token
// 61.7 / 61.2; d = 5120, one token 27.9 / 27.4; 8 outer experts, d = 4096, 4 tokens 157.4 / 156.1.
struct DownGroups {
  int32_t item0[MAX_GROUPS + 1];                  // prefix of work items over groups
  int32_t seg0[MAX_GROUPS], cnt[MAX_GROUPS], wp[MAX_GROUPS];
  int64_t w2_off[MAX_GROUPS], h_off[MAX_GROUPS];
};
// 16 bytes per lane from base + off (bytes; zeros where off >= size).
__device__ __forceinline__ bf16x8_t ld_frag_buffer(const bf16_t* base, uint32_t size, uint32_t off) {
#if defined(__HIP_DEVICE_COMPILE__)
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(base), 0, size, 0x00020000);
  return __builtin_bit_cast(bf16x8_t, __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, 0, 0));
#else
  return zero_frag();
#endif
}
// Called by one wave.
__device__ __forceinline__ void load_down_groups(const DecArgs& p, int G, DownGroups& dg, int lane) {
  constexpr int GPL = MAX_GROUPS / 64;
  int s0[GPL], s1[GPL];
  GroupDev gd[GPL];
  int64_t ho[GPL];
#pragma unroll
  for (int k = 0; k < GPL; ++k) {
    if (k > 0 && 64 * k >= G) break;
    const int g = min(lane + 64 * k, G - 1);
    s0[k] = p.seg_off[g];
    s1[k] = p.seg_off[g + 1];
    gd[k] = p.groups[g];
    ho[k] = p.h_off[g];
  }
  int run0 = 0;
#pragma unroll
  for (int k = 0; k < GPL; ++k) {
    if (k > 0 && 64 * k >= G) break;
    const int g = lane + 64 * k;
    const int cnt = g < G ? s1[k] - s0[k] : 0, n = cnt > 0 ? cdiv(gd[k].width_pad / 32, DC_CH) : 0;
    const int inc = wave_incl_scan(n);
    if (g < G) {
      dg.item0[g] = run0 + inc - n;
      dg.seg0[g] = s0[k];
      dg.cnt[g] = cnt;
      dg.wp[g] = gd[k].width_pad;
      dg.w2_off[g] = gd[k].w2_off;
      dg.h_off[g] = ho[k];
    }
    run0 += wave_last(inc);
  }
  if (lane == 0) dg.item0[G] = run0;
}

template <int NTT>
__global__ __launch_bounds__(DC_WAVES * 64) void decode_down_combine_kernel(DecArgs p, const float* __restrict__ w_by_slot,
                                                                            bf16_t* __restrict__ y_out) {
  __shared__ float yacc[DC_WAVES][NTT * 16][17];
  __shared__ DownGroups dg;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, kq = lane >> 4;
  const int c0 = blockIdx.x * 16;
  if (wave == 0) load_down_groups(p, p.G, dg, lane);
  float* mine = &yacc[wave][0][0];
  for (int e = lane; e < NTT * 16 * 17; e += 64) mine[e] = 0.0f;
  __syncthreads();
  const int n_items = dg.item0[p.G];
  // With two token tiles the next item's operands take the registers of this one's and are on their way while its products are
  // added.  us per forward, requested when the item begins / ahead: d = 4096, 32 experts, 32 tokens 68.2 / 67.9, 16 experts, 32 tokens
  // 65.9 / 65.5; one tile, 8 tokens, 16 experts 46.6 / 47.0, d = 8192, 5 tokens 74.5 / 74.9.
  // With four token tiles an item's rows go through the registers two tiles at a time, its weights once.
  constexpr int NP = NTT < 2 ? NTT : 2;
  constexpr bool AHEAD = NTT == 2;
  bf16x8_t a[DC_CH], b[NP][DC_CH];
  int tok[NP];
  float wt[NP];
  int seg0 = 0, cnt = 0, wp = 0, ns = 0;          // the item whose operands are requested: slots, width, K steps
  const bf16_t *wbase = nullptr, *hbase = nullptr;
  uint32_t wsize = 0, hsize = 0;
  // A load past the width returns zeros but takes its turn all the same.  With one token tile, where a wave's items are many
  // short chains (narrow experts), an item of at most four steps leaves the second half of its operands out.  us per forward, all
  // eight steps / now: d = 1024, 64 experts of 64, top-12, 16 tokens 26.9 / 23.0; 64 of 32, top-6 21.6 / 18.2; d = 512, 64 of 128,
  // top-16, 12 tokens 31.3 / 27.7; 8 outer experts of 8 of 32, 16 tokens 20.9 / 18.3; experts of 256 (eight steps) even.
  constexpr int HALF = DC_CH / 2;
  constexpr bool SHORT_ITEMS = NTT == 1;
  auto request_rows = [&](int first_tile) {
#pragma unroll
    for (int tt = 0; tt < NP; ++tt) {
      const int col = (first_tile + tt) * 16 + r16;
      if ((first_tile + tt) * 16 >= cnt) continue;      // (uniform: most items have at most 16 tokens)
      const int at = seg0 + min(col, cnt - 1);
      const uint32_t row = (uint32_t)(col * wp * 2 + kq * 16);
#pragma unroll
      for (int s = 0; s < HALF; ++s) b[tt][s] = ld_frag_buffer(hbase, hsize, row + (s < ns ? (uint32_t)(s * 64) : DMA_NONE));
      if (!SHORT_ITEMS || ns > HALF) {
#pragma unroll
        for (int s = HALF; s < DC_CH; ++s) {
          if (SHORT_ITEMS) a[s] = ld_frag_buffer(wbase, wsize, (uint32_t)(r16 * 64 + kq * 16 + s * (TILE_ELEMS * 2)));
          b[tt][s] = ld_frag_buffer(hbase, hsize, row + (s < ns ? (uint32_t)(s * 64) : DMA_NONE));
        }
      }
      tok[tt] = p.slot2tok[at];
      wt[tt] = w_by_slot[at];
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // Operands as buffer loads: rows past the group's tokens and steps past its width lie past the buffer's size and read
  // as zeros, so that nothing branches and all loads of an item leave together.  (Weights of bf16 layers are tiled.)
  auto request = [&](int u) {
    const int g = find_group(dg.item0, p.G, u);
    const int ks0 = (u - __builtin_amdgcn_readfirstlane(dg.item0[g])) * DC_CH;
    seg0 = __builtin_amdgcn_readfirstlane(dg.seg0[g]);
    cnt = __builtin_amdgcn_readfirstlane(dg.cnt[g]);
    wp = __builtin_amdgcn_readfirstlane(dg.wp[g]);
    ns = min(DC_CH, wp / 32 - ks0);
    wbase = uniform_ptr(p.w2 + dg.w2_off[g] + (int64_t)((c0 / 16) * (wp / 32) + ks0) * TILE_ELEMS);
    hbase = uniform_ptr(p.h + dg.h_off[g] + ks0 * 32);
    wsize = (uint32_t)ns * (TILE_ELEMS * 2);
    hsize = (uint32_t)(cnt * wp - ks0 * 32) * 2u;
#pragma unroll
    for (int s = 0; s < (SHORT_ITEMS ? HALF : DC_CH); ++s) a[s] = ld_frag_buffer(wbase, wsize, (uint32_t)(r16 * 64 + kq * 16 + s * (TILE_ELEMS * 2)));
    request_rows(0);
  };
  if (AHEAD && wave < n_items) request(wave);
  for (int u = wave; u < n_items; u += DC_WAVES) {
    if (!AHEAD) request(u);
    const int n = cnt;
#pragma unroll
    for (int t0 = 0; t0 < NTT; t0 += NP) {
      if (t0 * 16 >= n) break;
      if (t0 > 0) request_rows(t0);
      floatx4_t acc[NP];
      int at[NP];                                 // token of the lane's row, -1: there is none
      float by[NP];
#pragma unroll
      for (int tt = 0; tt < NP; ++tt) {
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[tt][i] = 0.0f;
        at[tt] = (t0 + tt) * 16 + r16 < n ? tok[tt] : -1;
        by[tt] = wt[tt];
        if ((t0 + tt) * 16 >= n) continue;
#pragma unroll
        for (int s = 0; s < HALF; ++s) acc[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[s], b[tt][s], acc[tt], 0, 0, 0);
        if (!SHORT_ITEMS || ns > HALF) {
#pragma unroll
          for (int s = HALF; s < DC_CH; ++s) acc[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[s], b[tt][s], acc[tt], 0, 0, 0);
        }
      }
      if (AHEAD && u + DC_WAVES < n_items) request(u + DC_WAVES);
      // accumulator element i: output column (lane/16)*4 + i, token of segment position lane%16
#pragma unroll
      for (int tt = 0; tt < NP; ++tt)
        if (at[tt] >= 0) {
#pragma unroll
          for (int i = 0; i < 4; ++i) yacc[wave][at[tt]][kq * 4 + i] += by[tt] * acc[tt][i];
        }
    }
  }
  __syncthreads();
  for (int e = tid; e < (int)p.T * 16; e += DC_WAVES * 64) {
    const int t = e >> 4, cc = e & 15;
    float s = 0.0f;
#pragma unroll
    for (int w = 0; w < DC_WAVES; ++w) s += yacc[w][t][cc];
    y_out[(int64_t)t * p.d + c0 + cc] = f32_to_bf16(s);
  }
}


// ---- neuron-level activation sparsity inside the routed experts (Sec. 5; Eq. 1 restricted to surviving neurons) ----
// A hidden activation h_n of a routed group survives iff |h_n| * scale_n >= tau, decided on the bf16 value the
// gate/up kernels stored (scale_n = 1, or the L2 norm of the neuron's row of W_down).
__device__ __forceinline__ bool neuron_survives(bf16_t v, int mode, float scale, float tau) {
  const float key = fabsf(bf16_to_f32(v)) * (mode == 2 ? scale : 1.0f);
  return key >= tau;                                          // (a NaN is dropped)
}

// Every batch but the one- and two-token ones: the dropped activations are zeroed in H after the gate/up
// contraction, so that the layer computes the same function at every batch size; one workgroup per slot row.
__global__ __launch_bounds__(256) void mask_hidden_kernel(bf16_t* __restrict__ h, const GroupDev* __restrict__ groups,
                                                          const int32_t* __restrict__ seg_off,
                                                          const int64_t* __restrict__ h_off,
                                                          const float* __restrict__ nscale, int G, int n_always, int mode,
                                                          float tau) {
  const int row = blockIdx.x;
  if (row >= seg_off[G]) return;
  const int g = find_group(seg_off, G, row);
  if (g < n_always) return;                                   // shared experts are never sparsified
  const int wp = groups[g].width_pad;
  const int64_t base = h_off[g] + (int64_t)(row - seg_off[g]) * wp;
  const int n0 = groups[g].w1_row0 / 2;
  for (int n = threadIdx.x; n < wp; n += 256)
    if (!neuron_survives(h[base + n], mode, nscale[n0 + n], tau)) h[base + n] = 0;
}

// One or two tokens: down projection + weighted sum over slots that reads only the surviving neurons' weights.
// A workgroup owns 16 output columns of both tokens.  The always-on groups go through the matrix cores as in
// decode_down_combine_kernel.  For a routed group every thread looks at one neuron: if it survives, the thread
// reads the 32 bytes of that neuron's row of the neuron-major copy of W_down that belong to the workgroup's
// columns and adds h_n * w_n (Eq. 1); the rows of dropped neurons are never touched.  The per-thread sums are
// added across the wave by exchanges in a fixed pattern, across waves in wave order: deterministic.
// Column blocks are dealt so that the four workgroups sharing a 128-byte line of a row run on one XCD.
constexpr int DS_WAVES = 16;
__global__ __launch_bounds__(DS_WAVES * 64) void decode_down_sparse_kernel(DecArgs p, const float* __restrict__ w_by_slot,
                                                                           bf16_t* __restrict__ y_out,
                                                                           const bf16_t* __restrict__ w2n,
                                                                           const float* __restrict__ nscale, int n_always,
                                                                           int mode, float tau, int cb_per_xcd) {
  __shared__ float yacc[DS_WAVES][2][16];
  __shared__ DownGroups dg;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r16 = lane & 15, kq = lane >> 4;
  const int cb = (blockIdx.x & 7) * cb_per_xcd + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= cb_per_xcd || cb >= p.d / 16) return;
  const int c0 = cb * 16;
  if (lane < 32) yacc[wave][lane >> 4][lane & 15] = 0.0f;
  if (n_always == 0 && tid == 0) dg.item0[0] = 0;
  if (wave == 0 && n_always > 0) load_down_groups(p, n_always, dg, lane);
  __syncthreads();
  // ---- always-on groups: 16 columns x 8 K steps per work item, matrix cores ----
  const int n_items = dg.item0[n_always];
  for (int u = wave; u < n_items; u += DS_WAVES) {
    const int g = find_group(dg.item0, n_always, u);
    const int ks0 = (u - dg.item0[g]) * DC_CH;
    const int seg0 = p.seg_off[g], cnt = p.seg_off[g + 1] - seg0;
    const int wp = p.groups[g].width_pad;
    const int ns = min(DC_CH, wp / 32 - ks0);
    const int kadv = p.tiled ? TILE_ELEMS : 32;
    const bf16_t* wrow = p.w2 + p.groups[g].w2_off +
                         (p.tiled ? tiled_offset(c0 + r16, ks0 * 32 + kq * 8, wp / TILE_K)
                                  : (int64_t)(c0 + r16) * wp + kq * 8 + ks0 * 32);
    const bool ok = r16 < cnt;
    const bf16_t* hrow = p.h + p.h_off[g] + kq * 8 + ks0 * 32 + (int64_t)(ok ? r16 : 0) * wp;
    bf16x8_t a[DC_CH], b[DC_CH];
#pragma unroll
    for (int s = 0; s < DC_CH; ++s) {
      a[s] = s < ns ? ld_frag(wrow + s * kadv) : zero_frag();
      b[s] = (ok && s < ns) ? ld_frag(hrow + s * 32) : zero_frag();
    }
    const int tok = ok ? p.slot2tok[seg0 + r16] : -1;
    const float wt = ok ? w_by_slot[seg0 + r16] : 0.0f;
    floatx4_t acc;
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] = 0.0f;
#pragma unroll
    for (int s = 0; s < DC_CH; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[s], b[s], acc, 0, 0, 0);
    if (tok >= 0) {
#pragma unroll
      for (int i = 0; i < 4; ++i) yacc[wave][tok][kq * 4 + i] += wt * acc[i];
    }
  }
  // ---- routed groups: one neuron per thread, surviving rows only ----
  float a0[16], a1[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) { a0[i] = 0.0f; a1[i] = 0.0f; }
  const int routed_row0 = p.groups[n_always].w1_row0 / 2;
  for (int g = n_always; g < p.G; ++g) {
    const int seg0 = p.seg_off[g], cnt = p.seg_off[g + 1] - seg0;
    if (cnt == 0) continue;
    const int wp = p.groups[g].width_pad;
    const int64_t hoff = p.h_off[g];
    const int n0 = p.groups[g].w1_row0 / 2;
    for (int col = 0; col < cnt; ++col) {
      const int tok = p.slot2tok[seg0 + col];
      const float wt = w_by_slot[seg0 + col];
      for (int n = tid; n < wp; n += DS_WAVES * 64) {
        const bf16_t hv = p.h[hoff + (int64_t)col * wp + n];
        if (!neuron_survives(hv, mode, nscale[n0 + n], tau)) continue;
        const uint4* src = reinterpret_cast<const uint4*>(w2n + (int64_t)(n0 - routed_row0 + n) * p.d + c0);
        const uint4 q0 = src[0], q1 = src[1];
        const uint32_t w[8] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w};
        const float coef = wt * bf16_to_f32(hv);
        if (tok == 0) {
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            a0[2 * i] = fmaf(coef, __uint_as_float(w[i] << 16), a0[2 * i]);
            a0[2 * i + 1] = fmaf(coef, __uint_as_float(w[i] & 0xffff0000u), a0[2 * i + 1]);
          }
        } else {
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            a1[2 * i] = fmaf(coef, __uint_as_float(w[i] << 16), a1[2 * i]);
            a1[2 * i + 1] = fmaf(coef, __uint_as_float(w[i] & 0xffff0000u), a1[2 * i + 1]);
          }
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    a0[i] = wave_sum(a0[i]);
    a1[i] = wave_sum(a1[i]);
  }
  wave_lds_sync_decode();                                   // the MFMA part's LDS updates of this wave are done
  if (lane == 0) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      yacc[wave][0][i] += a0[i];
      yacc[wave][1][i] += a1[i];
    }
  }
  __syncthreads();
  for (int e = tid; e < (int)p.T * 16; e += DS_WAVES * 64) {
    const int t = e >> 4, cc = e & 15;
    float s = 0.0f;
#pragma unroll
    for (int w = 0; w < DS_WAVES; ++w) s += yacc[w][t][cc];
    y_out[(int64_t)t * p.d + c0 + cc] = f32_to_bf16(s);
  }
}

// Up to 16 tokens (one MFMA token tile) the weight-streaming kernels are the fastest form of both
// contractions; from 17 tokens on the routed layer chooses between streamed units and tiles (streams_small_batch), and the
// dense one is 10-20 us faster on skinny tiles (measured at d = 4096).
constexpr int DECODE_MAX_T = 16;
// Above d = 4096 the batches from five tokens on choose as those from 17 on do below it: a line between what routed layers gain and
// lose by it.  us per forward with these launches up to 4 / up to 16 tokens, routed (the gate/up contraction on streamed units
// either way): d = 5120, 16 experts, top-3, 5 tokens 62.3 / 58.1, 16 tokens 79.6 / 75.5; d = 6144, 8, top-2 64.0 / 63.2 and 94.5 / 89.0;
// d = 7680, 16, top-2 70.8 / 70.6 and 90.0 / 88.7; d = 8192, 16, top-3 86.9 / 88.5 and 104.1 / 105.9; d = 10240 109.9 / 112.6 and
// 143.1 / 144.7.  The dense layer: d = 5120 79.3 / 71.4 and 80.6 / 90.8, d = 8192 119.5 / 104.0 and 120.2 / 121.9.
constexpr int DECODE_MAX_T_RUNS = 4;
bool decode_path_ok(const Engine& e, int64_t T) {
  if (e.dtype != 1 || T < 1 || T > (decode_k(e.d).nch > 1 ? DECODE_MAX_T_RUNS : DECODE_MAX_T)) return false;
  return decode_k(e.d).ksteps != 0;
}

// The fused down + combine kernel serves routed bf16 batches with more than one slot per token, whichever kernel produced the
// hidden activations (the decode_fuse tuning switch selects the separate kernels, for comparison): every one of at most 32
// tokens, and of 33 to 64 tokens those whose d / 16 workgroups are about one per CU (d = 3072 to 4096) and whose hidden activations,
// which every workgroup reads, come to at most 16 rows per row of weights and to little more than what the launches it replaces
// cost: over 3700 calls it gained 2.6 us + 1.9 us per 10000 rows of weights and lost 1.5 us (4096 / d)^2 per 100000 neurons
// of hidden activations (the fewer workgroups there are, the more CUs stand by).  us per forward, separate kernels / this one, where it is
// taken: d = 3584, 16 experts of 604, top-3, 48 tokens 55.4 / 53.6; d = 4096, 16 of 691, top-3, 33 67.2 / 65.1, 64 72.1 / 72.1; 32 with
// four shared, top-4, 33 72.7 / 66.9, 64 77.3 / 74.4; 8 with two shared, top-1, 33 89.4 / 65.3, 64 91.7 / 91.6; 8 outer experts of 8, 33
// 439 / 408, 64 438 / 417.  Where it is not: d = 3072, 16 of 2496, top-3, 64 157.8 / 175.3; d = 4096, 16 of 3328, top-4,
// 64 254.9 / 268.5; whole experts, two of eight, d = 3072, 33 378 / 387, 64 395 / 435, d = 4096, 48 485 / 500.  Other widths: d = 1024,
// 16 experts, 40 tokens 26.8 / 27.3; d = 2048, 32 experts, 33 tokens 33.1 / 31.6, 64 tokens 39.2 / 39.5, 8 outer experts, 33 tokens 67.9 /
// 70.9; d = 5120, 16 experts, 40 tokens 87.2 / 88.6; d = 8192, 8 experts, 33 tokens 120.5 / 122.5, 64 tokens 128.7 / 140.4.
constexpr int DOWN_COMBINE_ALL_T = 32, DOWN_COMBINE_MAX_T = 64;
bool decode_fuses_combine(const Engine& e, int64_t T) {
  if (tuning().decode_fuse == 0 || use_simt_experts(e.dtype) || e.dtype != 1 || T < 1 || T > DOWN_COMBINE_MAX_T || e.d % 16 != 0) return false;
  if ((e.G == 1 && e.n_always == 1) || e.S_all() <= 1) return false;
  if (T <= DOWN_COMBINE_ALL_T) return true;
  int64_t widths = 0;
  for (int g = 0; g < e.G; ++g) widths += e.width_pad_host[g];
  const int64_t hidden = T * e.h_per_token;
  return e.d >= 3072 && e.d <= 4096 && hidden <= 16 * widths && hidden * 4096 * 4096 <= (10 * widths + 200000) * e.d * e.d;
}

// 8-neuron units when they still number at most one per CU (the always-on groups count unless the routing
// front end runs them).  Measured at one token: four routed experts of 448 neurons (224 units of 8) 10.1 ->
// 8.9 us for the gate/up launch, three of 688 (258 units of 8) 12.0 -> 14.8 us; at 16 tokens 28.7 -> 32.4 us.
// CMOE_DECODE_SPLIT = 8 / 16 forces a size.
int decode_unit_neurons(const Engine& e, int64_t T) {
  const int forced = tuning().decode_split;
  if (forced == 8 || forced == 16) return forced;
  if (decode_gate_up_streams(e, T)) return stream_neurons(e, T);
  if (decode_front_runs_all(e, T)) return 16;     // (measured: 27.9 against 31.4 us and 30.4 against 31.6 us at one token)
  const int64_t dyn_groups = std::min<int64_t>(T * e.S_dyn, e.G - e.n_always);
  int64_t units8 = e.G > e.n_always ? dyn_groups * (e.width_pad_host[e.n_always] / 8) : 0;
  if (!decode_front_runs_shared(e, T))
    for (int g = 0; g < e.n_always; ++g) units8 += e.width_pad_host[g] / 8;
  return units8 <= 256 ? 8 : 16;
}

int64_t decode_unit_bound(const Engine& e, int64_t T, int which) {
  const int64_t dyn_groups = std::min<int64_t>(T * e.S_dyn, e.G - e.n_always);
  const int64_t per_group = which == 1 ? e.max_width_pad / decode_unit_neurons(e, T) : e.d / 16;
  return std::max<int64_t>((e.n_always + dyn_groups) * per_group, 1);
}

template <int NTT>
static hipError_t launch_gate_up(const DecArgs& a, int64_t n_blocks, hipStream_t s) {
  dim3 grid((unsigned)n_blocks), block(512);
#define CMOE_GATE_UP(KS, RUNS) hipLaunchKernelGGL((decode_gate_up_kernel<NTT, KS, RUNS>), grid, block, 0, s, a)
  CMOE_DECODE_KSTEPS(a.d, CMOE_GATE_UP)
#undef CMOE_GATE_UP
  return hipGetLastError();
}

DecArgs make_dec_args(const Engine& e, const void* x, int64_t T, char* ws, const WsLayout& L, void* y) {
  DecArgs a;
  a.x = static_cast<const bf16_t*>(x);
  a.w1 = static_cast<const bf16_t*>(e.w1);
  a.w2 = static_cast<const bf16_t*>(e.w2);
  a.h = reinterpret_cast<bf16_t*>(ws + L.h);
  a.y = e.direct_output() ? static_cast<bf16_t*>(y) : reinterpret_cast<bf16_t*>(ws + L.y_slots);
  a.groups = e.groups;
  a.seg_off = reinterpret_cast<const int32_t*>(ws + L.seg_off);
  a.work = nullptr;
  a.h_off = reinterpret_cast<const int64_t*>(ws + L.h_off);
  a.G = e.G;
  a.d = e.d;
  a.ldw = e.ldw1;
  a.tiled = e.w_tiled;
  a.T = T;
  a.single = (e.G == 1 && e.n_always == 1) ? 1 : 0;
  a.slot2tok = a.single ? nullptr : reinterpret_cast<const int32_t*>(ws + L.slot2tok);
  a.unit1 = decode_unit_neurons(e, T);
  a.nch = decode_k(e.d).nch;
  a.x_row = e.d;
  a.x_step = 32;
  return a;
}

// Down contraction + weighted sum over slots in one launch (callers check decode_fuses_combine first).
hipError_t launch_decode_down_combine(const Engine& e, int64_t T, char* ws, const WsLayout& L, void* y, hipStream_t s) {
  const DecArgs a = make_dec_args(e, nullptr, T, ws, L, y);
  const float* wbs = reinterpret_cast<const float*>(ws + L.w_by_slot);
  bf16_t* yo = static_cast<bf16_t*>(y);
  if (T > 32) hipLaunchKernelGGL((decode_down_combine_kernel<4>), dim3(e.d / 16), dim3(DC_WAVES * 64), 0, s, a, wbs, yo);
  else if (T > 16) hipLaunchKernelGGL((decode_down_combine_kernel<2>), dim3(e.d / 16), dim3(DC_WAVES * 64), 0, s, a, wbs, yo);
  else hipLaunchKernelGGL((decode_down_combine_kernel<1>), dim3(e.d / 16), dim3(DC_WAVES * 64), 0, s, a, wbs, yo);
  return hipGetLastError();
}

bool decode_sparse_down_ok(const Engine& e, int64_t T) {
  return e.sparse_mode != 0 && e.w2n != nullptr && T >= 1 && T <= 2 && decode_fuses_combine(e, T);
}

hipError_t launch_decode_down_sparse(const Engine& e, int64_t T, char* ws, const WsLayout& L, void* y, hipStream_t s) {
  const DecArgs a = make_dec_args(e, nullptr, T, ws, L, y);
  const float* wbs = reinterpret_cast<const float*>(ws + L.w_by_slot);
  const int per_xcd = cdiv(e.d / 16, 8);
  hipLaunchKernelGGL(decode_down_sparse_kernel, dim3(8 * per_xcd), dim3(DS_WAVES * 64), 0, s, a, wbs, static_cast<bf16_t*>(y),
                     static_cast<const bf16_t*>(e.w2n), e.nscale, e.n_always, e.sparse_mode, e.sparse_tau, per_xcd);
  return hipGetLastError();
}

hipError_t launch_mask_hidden(const Engine& e, int64_t T, char* ws, const WsLayout& L, hipStream_t s) {
  if (e.sparse_mode == 0 || e.nscale == nullptr || e.G <= e.n_always) return hipSuccess;
  hipLaunchKernelGGL(mask_hidden_kernel, dim3((unsigned)(T * e.S_all())), dim3(256), 0, s, reinterpret_cast<bf16_t*>(ws + L.h),
                     e.groups, reinterpret_cast<const int32_t*>(ws + L.seg_off), reinterpret_cast<const int64_t*>(ws + L.h_off),
                     e.nscale, e.G, e.n_always, e.sparse_mode, e.sparse_tau);
  return hipGetLastError();
}

hipError_t launch_experts_decode(const Engine& e, const void* x, int64_t T, char* ws, const WsLayout& L, void* y,
                                 hipStream_t s, int stage) {
  DecArgs a = make_dec_args(e, x, T, ws, L, y);
  if (stage != 2) {
    a.work = reinterpret_cast<const int32_t*>(ws + L.work1);
    const int64_t nb = a.single ? e.max_width_pad / a.unit1 : decode_unit_bound(e, T, 1);
    hipError_t err = decode_gate_up_streams(e, T) ? launch_stream_gate_up(e, x, T, ws, L, a.unit1, (int)nb, s) : launch_gate_up<1>(a, nb, s);
    if (err != hipSuccess || stage == 1) return err;
  }
  if (decode_fuses_combine(e, T)) return launch_decode_down_combine(e, T, ws, L, y, s);
  a.work = reinterpret_cast<const int32_t*>(ws + L.work2);
  const int64_t nb = a.single ? e.d / 16 : decode_unit_bound(e, T, 2);
  hipLaunchKernelGGL((decode_down_kernel<1>), dim3((unsigned)nb), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace cmoe
