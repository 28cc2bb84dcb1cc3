// Token -> expert permutation and the gate-weighted combine.
//
// place_kernel: from the routed (group, weight) entries of every token and the per-tile histograms,
// a wave per 64-token tile computes, with an exclusive prefix scan over groups and over preceding
// tiles, the slot of each entry.  Segments are contiguous per group and token-ascending inside a
// group, so the layout is a pure function of the routing decisions.  Tile 0 also publishes the segment
// offsets, counts, the work lists of the two grouped GEMMs and each group's offset in the ragged
// hidden-activation buffer.  Nothing is copied back to the host.
//
// combine_kernel: y[t] = sum over the token's slots of weight * Y[slot]  (Eq. 4 / Eq. 10), a gather,
// so there are no floating-point atomics and the result does not depend on scheduling.
#include "cmoe_internal.h"
#include "decode_device.h"
#include "device_utils.h"
#include "place_device.h"

namespace cmoe {

// One workgroup per tile.  The histograms of all tiles are added up by all its waves (one wave took 16 rows of the table
// per round trip: 5 us of dependent rounds at 128 tiles), then wave 0 assigns the tile's slots while, in the first
// workgroup, wave 1 publishes the lists: 9.1 -> 7.6 us at 2048 tokens, 11.9 -> 8.4 at 8192.
constexpr int PLACE_WAVES = 8;
__global__ __launch_bounds__(PLACE_WAVES * 64) void place_kernel(PlaceArgs p) {
  constexpr int GPL = MAX_GROUPS / 64;
  __shared__ int32_t part[PLACE_WAVES][2][MAX_GROUPS];
  __shared__ int32_t sel_g[TOK_TILE * MAX_DYN];
  __shared__ float sel_w[TOK_TILE * MAX_DYN];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, tile = blockIdx.x;
  const LaneWidths lw = load_lane_widths(p, lane);
  // the tile's routed entries are consecutive
  const int64_t e0 = (int64_t)tile * TOK_TILE * p.S_dyn, n_e = p.T * p.S_dyn - e0;
  for (int i = threadIdx.x; i < TOK_TILE * p.S_dyn && i < n_e; i += PLACE_WAVES * 64) {
    sel_g[i] = p.sel_group[e0 + i];
    sel_w[i] = p.sel_weight[e0 + i];
  }
  if (p.count_here) {
    int32_t(*flat)[MAX_GROUPS] = part[0];                      // tot, prev; the other waves' parts stay zero
    for (int i = threadIdx.x; i < PLACE_WAVES * 2 * MAX_GROUPS; i += PLACE_WAVES * 64) (&part[0][0][0])[i] = 0;
    __syncthreads();
    const int n = (int)(p.T * p.S_dyn);
    for (int i = threadIdx.x; i < n; i += PLACE_WAVES * 64) {
      const int g = p.sel_group[i];
      atomicAdd(&flat[0][g], 1);
      if (i < e0) atomicAdd(&flat[1][g], 1);
    }
  }
  const int per = (p.n_counts + PLACE_WAVES - 1) / PLACE_WAVES;
  const int first = wave * per, end = first + per < p.n_counts ? first + per : p.n_counts;
  const int row0 = tile * p.counts_per_tile;                   // the tile's first row of the table
#pragma unroll
  for (int k = 0; k < GPL; ++k) {
    const int g = lane + 64 * k;
    if (64 * k >= p.G || p.count_here) continue;
    int tot = 0, prev = 0;
    if (g < p.G && g >= p.n_always) {
      // independent loads, eight in flight at a time (the compiler does not batch them by itself)
      int i = first;
      for (; i + 8 <= end; i += 8) {
        int c[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) c[q] = p.tile_counts[(int64_t)(i + q) * p.G + g];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          tot += c[q];
          prev += (i + q < row0) ? c[q] : 0;
        }
      }
      for (; i < end; ++i) {
        const int c = p.tile_counts[(int64_t)i * p.G + g];
        tot += c;
        prev += (i < row0) ? c : 0;
      }
    }
    part[wave][0][g] = tot;
    part[wave][1][g] = prev;
  }
  __syncthreads();
  if (wave > 1 || (wave == 1 && tile != 0)) return;
  TileCounts tc;
#pragma unroll
  for (int k = 0; k < GPL; ++k) {
    const int g = lane + 64 * k;
    tc.tot[k] = 0;
    tc.prev[k] = 0;
    if (64 * k >= p.G) continue;
    if (g < p.n_always) tc.tot[k] = (int)p.T;
#pragma unroll
    for (int w = 0; w < PLACE_WAVES; ++w) {
      tc.tot[k] += part[w][0][g];
      tc.prev[k] += part[w][1][g];
    }
  }
  if (wave == 0) place_slots(p, tile, tc, sel_g, sel_w, lane);
  else place_lists(p, tc, lane, lw);
}

PlaceArgs make_place_args(const Engine& e, int64_t T, char* ws, const WsLayout& L, int32_t* counts_out) {
  PlaceArgs p;
  p.sel_group = reinterpret_cast<const int32_t*>(ws + L.sel_group);
  p.sel_weight = reinterpret_cast<const float*>(ws + L.sel_weight);
  p.groups = e.groups;
  p.seg_off = reinterpret_cast<int32_t*>(ws + L.seg_off);
  p.counts = reinterpret_cast<int32_t*>(ws + L.counts);
  p.work1 = reinterpret_cast<int32_t*>(ws + L.work1);
  p.work2 = reinterpret_cast<int32_t*>(ws + L.work2);
  p.h_off = reinterpret_cast<int64_t*>(ws + L.h_off);
  p.slot2tok = reinterpret_cast<int32_t*>(ws + L.slot2tok);
  p.tok2slot = reinterpret_cast<int32_t*>(ws + L.tok2slot);
  p.slot_w = reinterpret_cast<float*>(ws + L.slot_w);
  p.w_by_slot = reinterpret_cast<float*>(ws + L.w_by_slot);
  p.counts_out = counts_out;
  p.T = T;
  p.G = e.G;
  p.n_always = e.n_always;
  p.S_dyn = e.S_dyn;
  const CountTable ct = router_counts(e, T, L);
  p.tile_counts = reinterpret_cast<const int32_t*>(ws + ct.offset);
  p.n_counts = (int)((T + ct.tokens - 1) / ct.tokens);
  p.counts_per_tile = TOK_TILE / ct.tokens;
  p.d = e.d;
  p.decode = (!use_simt_experts(e.dtype) && decode_path_ok(e, T)) ? 1 : 0;
  p.skip_always = L.skip_always;
  p.dec_unit1 = p.decode ? decode_unit_neurons(e, T) : 16;
  // (a decode batch has no tiles; choosing their shapes all the same takes longer than one of its launches)
  const bool tiles = p.decode == 0;
  p.bm1 = tiles ? gemm_tile(e, T, 1) : 1;
  p.bn1 = tiles ? gemm_tile(e, T, 3) : 1;
  p.bm2 = tiles ? gemm_tile(e, T, 2) : 1;
  p.bn2 = tiles ? gemm_tile(e, T, 4) : 1;
  p.dyn1 = tiles ? gemm_tile(e, T, 5) : 0;
  p.dyn2 = tiles ? gemm_tile(e, T, 6) : 0;
  p.count_here = place_counts_itself(e, T) ? 1 : 0;
  p.stream2 = tiles ? gemm_tile(e, T, 7) : 0;
  return p;
}

hipError_t launch_permute(const Engine& e, int64_t T, char* ws, const WsLayout& L, int32_t* counts_out,
                          hipStream_t s) {
  if (T == 0) return hipSuccess;
  const PlaceArgs p = make_place_args(e, T, ws, L, counts_out);
  hipLaunchKernelGGL(place_kernel, dim3(L.n_tok_tiles), dim3(PLACE_WAVES * 64), 0, s, p);
  return hipGetLastError();
}

// ---- combine --------------------------------------------------------------------------------
// One workgroup per token; threads stride over the d columns in vectors of VEC elements.
template <typename T, int VEC>
__global__ __launch_bounds__(256) void combine_kernel(const T* __restrict__ y_slots, const int32_t* __restrict__ tok2slot,
                                                      const float* __restrict__ slot_w, T* __restrict__ y, int d,
                                                      int S_all) {
  const int64_t t = blockIdx.x;
  __shared__ int32_t slots[MAX_DYN + MAX_TOPK];
  __shared__ float wts[MAX_DYN + MAX_TOPK];
  if (threadIdx.x < S_all) {
    slots[threadIdx.x] = tok2slot[t * S_all + threadIdx.x];
    wts[threadIdx.x] = slot_w[t * S_all + threadIdx.x];
  }
  __syncthreads();
  for (int c = threadIdx.x * VEC; c < d; c += 256 * VEC) {
    float acc[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] = 0.0f;
    for (int i = 0; i < S_all; ++i) {
      const T* src = y_slots + (int64_t)slots[i] * d + c;
      const float w = wts[i];
      if (VEC == 1) {
        acc[0] = fmaf(w, Elem<T>::ld(src), acc[0]);
      } else {
        T tmp[VEC];
        // (read once, past the caches: 8192 tokens of seven slots 762 -> 737 us per forward, 500 tokens of seven at d = 2048
        // 58.5 -> 53.1, 2048 tokens of four no change)
        typedef unsigned int uintx4 __attribute__((ext_vector_type(4)));
        *reinterpret_cast<uintx4*>(tmp) = __builtin_nontemporal_load(reinterpret_cast<const uintx4*>(src));
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] = fmaf(w, Elem<T>::ld(&tmp[v]), acc[v]);
      }
    }
    if (VEC == 1) {
      Elem<T>::st(y + t * d + c, acc[0]);
    } else {
      T out[VEC];
#pragma unroll
      for (int v = 0; v < VEC; ++v) Elem<T>::st(&out[v], acc[v]);
      *reinterpret_cast<uint4*>(y + t * d + c) = *reinterpret_cast<uint4*>(out);
    }
  }
}

hipError_t launch_combine(const Engine& e, int64_t T, char* ws, const WsLayout& L, void* y, hipStream_t s) {
  if (T == 0 || e.direct_output()) return hipSuccess;   // the down contraction has written y itself
  if (decode_fuses_combine(e, T)) return hipSuccess;    // the decode down kernel has already summed the slots
  const int32_t* tok2slot = reinterpret_cast<const int32_t*>(ws + L.tok2slot);
  const float* slot_w = reinterpret_cast<const float*>(ws + L.slot_w);
  dim3 grid((unsigned)T), block(256);
  if (e.dtype == 1) {
    const bf16_t* ys = reinterpret_cast<const bf16_t*>(ws + L.y_slots);
    if (e.d % 8 == 0)
      hipLaunchKernelGGL((combine_kernel<bf16_t, 8>), grid, block, 0, s, ys, tok2slot, slot_w,
                         static_cast<bf16_t*>(y), e.d, e.S_all());
    else
      hipLaunchKernelGGL((combine_kernel<bf16_t, 1>), grid, block, 0, s, ys, tok2slot, slot_w,
                         static_cast<bf16_t*>(y), e.d, e.S_all());
  } else {
    const float* ys = reinterpret_cast<const float*>(ws + L.y_slots);
    if (e.d % 4 == 0)
      hipLaunchKernelGGL((combine_kernel<float, 4>), grid, block, 0, s, ys, tok2slot, slot_w,
                         static_cast<float*>(y), e.d, e.S_all());
    else
      hipLaunchKernelGGL((combine_kernel<float, 1>), grid, block, 0, s, ys, tok2slot, slot_w,
                         static_cast<float*>(y), e.d, e.S_all());
  }
  return hipGetLastError();
}

}  // namespace cmoe
