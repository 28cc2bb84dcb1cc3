// Slot assignment of one 64-token tile (shared by the permute kernel and the decode front end).
#pragma once
#include "cmoe_internal.h"
#include "device_utils.h"

namespace cmoe {

constexpr int N_XCD = 8;              // dies with an L2 of their own; workgroup b runs on die b % 8
constexpr int TILE_FIXED_COST = 4;    // prologue + epilogue of a tile, in units of one 64-deep K step

struct PlaceArgs {
  const int32_t* sel_group;    // [T][S_dyn]
  const float* sel_weight;     // [T][S_dyn]
  const int32_t* tile_counts;  // [n_counts][G] histograms of consecutive runs of tokens, counts_per_tile rows per tile
  const GroupDev* groups;
  int32_t* seg_off;            // [G+1]
  int32_t* counts;             // [G]
  int32_t* work1;              // [G+1] prefix of work items, then [N_XCD+1] first item of each die's share
  int32_t* work2;              // same for the down contraction; with stream2 first item per group, [G] items, [G+1] deep ones
  int64_t* h_off;              // [G+1]
  int32_t* slot2tok;           // [n_slots]
  int32_t* tok2slot;           // [T][S_all]
  float* slot_w;               // [T][S_all]
  float* w_by_slot;            // [n_slots] the same weights indexed by slot
  int32_t* counts_out;         // optional user output: counts of the routed groups [G - n_always]
  int64_t T;
  int G, n_always, S_dyn, n_counts, counts_per_tile;
  int bm1, bn1, bm2, bn2, d;   // tile sizes of the grouped GEMMs (bn1 in packed gate/up rows)
  int dyn1, dyn2;              // > 0: that contraction runs tiles of dynamic height, in steps of this many rows (a
                               // ragged last tile costs its rows)
  int stream2;                 // > 0: the down contraction is the persistent one, and groups wider than this come first in its
                               // list (see there)
  int count_here;              // 1: there is no histogram, place_kernel counts the batch's entries (few)
  int decode;                  // 1: the work lists count decode units (dec_unit1 neurons / 16 output columns per unit)
  int dec_unit1;               // neurons per gate/up unit of the decode kernels (16 or 8)
  int skip_always;             // 1: no gate/up work items for the always-on groups (another launch ran them)
};

// All 64 callers are one wave: the LDS operations of a wave are carried out in the order it issued them, so
// waiting for its outstanding ones (and keeping the compiler from moving LDS accesses across this point) is
// enough to hand data between its lanes.  Deliberately not a fence: a workgroup-scope fence also waits for
// every global store the wave has in flight, which nothing here needs.
__device__ __forceinline__ void wave_lds_sync() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_wave_barrier();
}

// Padded widths of the (at most two) groups a lane looks after in place_lists; a caller with other work to
// do first requests them early so that their latency is hidden.
struct LaneWidths { int w[MAX_GROUPS / 64]; };
__device__ __forceinline__ LaneWidths load_lane_widths(const PlaceArgs& p, int lane) {
  LaneWidths lw;
#pragma unroll
  for (int k = 0; k < MAX_GROUPS / 64; ++k) {
    const int g = lane + 64 * k;
    lw.w[k] = (g < p.G) ? p.groups[g].width_pad : 0;
  }
  return lw;
}

// Tokens of the batch in each of a lane's groups, and how many of them lie in the tiles before this one.
struct TileCounts { int tot[MAX_GROUPS / 64], prev[MAX_GROUPS / 64]; };

// A batch of one tile: the counts are its own histogram (LDS).
__device__ __forceinline__ TileCounts single_tile_counts(const PlaceArgs& p, const int32_t* hist, int lane) {
  TileCounts tc;
#pragma unroll
  for (int k = 0; k < MAX_GROUPS / 64; ++k) {
    const int g = lane + 64 * k;
    tc.tot[k] = g >= p.G ? 0 : g < p.n_always ? (int)p.T : hist[g];
    tc.prev[k] = 0;
  }
  return tc;
}

// One wave assigns the slots of one 64-token tile from its routed entries sel_g / sel_w [64][S_dyn] (LDS; those of
// tokens past T are not read).  Must be called by exactly 64 threads (lane = id).  Cost is
// O(S_dyn + G/64) per lane: the prefix over groups is a wave scan (two groups per lane), and the rank of a token
// inside its group comes from a 64-bit presence mask per group that the lanes build with LDS atomics, not from a
// pass over all groups.
__device__ __forceinline__ void place_slots(const PlaceArgs& p, int tile, const TileCounts& tc, const int32_t* sel_g,
                                            const float* sel_w, int lane) {
  constexpr int GPL = MAX_GROUPS / 64;      // groups per lane
  __shared__ int32_t base[MAX_GROUPS];      // first slot of each group for this tile
  __shared__ uint32_t present[MAX_GROUPS][2];   // which lanes (tokens of the tile) have an entry for the group
  const int S_all = p.n_always + p.S_dyn;
  const int64_t t = (int64_t)tile * TOK_TILE + lane;
  const bool valid = t < p.T;
#pragma unroll
  for (int k = 0; k < GPL; ++k) {
    present[lane + 64 * k][0] = 0u;
    present[lane + 64 * k][1] = 0u;
  }
  wave_lds_sync();                          // the cleared masks are visible to every lane
  if (valid)
    for (int i = 0; i < p.S_dyn; ++i) atomicOr(&present[sel_g[lane * p.S_dyn + i]][lane >> 5], 1u << (lane & 31));
  int run0 = 0;
#pragma unroll
  for (int k = 0; k < GPL; ++k) {
    const int g = lane + 64 * k;
    if (k > 0 && 64 * k >= p.G) continue;
    const int inc = wave_incl_scan(tc.tot[k]);
    if (g < p.G) base[g] = run0 + inc - tc.tot[k] + tc.prev[k];
    run0 += wave_last(inc);
  }
  wave_lds_sync();                          // base[] and present[] are complete
  // always-on groups: identity segments
  if (valid)
    for (int a = 0; a < p.n_always; ++a) {
      const int slot = a * (int)p.T + (int)t;
      p.slot2tok[slot] = (int)t;
      p.tok2slot[t * S_all + a] = slot;
      p.slot_w[t * S_all + a] = 1.0f;
      p.w_by_slot[slot] = 1.0f;
    }
  // routed entries: stable (token-ascending) rank inside the group = lower lanes present in its mask
  const uint32_t lt_lo = lane >= 32 ? 0xffffffffu : ((1u << lane) - 1u);
  const uint32_t lt_hi = lane > 32 ? ((1u << (lane - 32)) - 1u) : 0u;
  if (valid)
    for (int i = 0; i < p.S_dyn; ++i) {
      const int g = sel_g[lane * p.S_dyn + i];
      const float w = sel_w[lane * p.S_dyn + i];
      const int slot = base[g] + __popc(present[g][0] & lt_lo) + __popc(present[g][1] & lt_hi);
      p.slot2tok[slot] = (int)t;
      p.tok2slot[t * S_all + p.n_always + i] = slot;
      p.slot_w[t * S_all + p.n_always + i] = w;
      p.w_by_slot[slot] = w;
    }
}

// One wave publishes what depends on the batch's counts alone: segment offsets, the work lists of the two
// contractions and each group's offset in the hidden-activation buffer.  Run by another wave than the slots of
// tile 0, next to it (both in one wave made that tile the last to finish).
// DECODE: the lists count decode units (p.decode).
template <bool DECODE>
__device__ __forceinline__ void place_lists_of(const PlaceArgs& p, const TileCounts& tc, int lane, const LaneWidths& lw) {
  constexpr int GPL = MAX_GROUPS / 64;
  // exclusive prefix over groups of: slots, work items of the two contractions, hidden-buffer elements
  int run0 = 0, w1_0 = 0, w2_0 = 0, w2_deep = 0;
  long long h0 = 0;
  int n1[GPL], n2[GPL], w1x[GPL], w2x[GPL];     // work items of this lane's groups and their exclusive prefix
  int rt[2][GPL], ct[2][GPL];                   // row and column tiles of the two contractions (a division is a long chain: once)
#pragma unroll
  for (int k = 0; k < GPL; ++k) {
    const int g = lane + 64 * k;
    if (k > 0 && 64 * k >= p.G) {           // nothing to add: skip this half's four scans
      n1[k] = 0; n2[k] = 0; w1x[k] = w1_0; w2x[k] = w2_0;
      continue;
    }
    const int cnt = tc.tot[k], wp = lw.w[k];
    int a1, a2;
    if (DECODE) {
      a1 = cnt > 0 ? wp / p.dec_unit1 : 0;
      a2 = cnt > 0 ? p.d / 16 : 0;
    } else {
      rt[0][k] = cdiv(cnt, p.bm1);
      ct[0][k] = cdiv(2 * wp, p.bn1);
      rt[1][k] = cdiv(cnt, p.bm2);
      ct[1][k] = cdiv(p.d, p.bn2);
      a1 = rt[0][k] * ct[0][k];
      a2 = rt[1][k] * ct[1][k];
    }
    if (g >= p.G) { a1 = 0; a2 = 0; }
    if (p.skip_always && g < p.n_always) a1 = 0;
    const long long ah = (long long)cnt * wp;
    const bool deep = !DECODE && p.stream2 > 0 && wp > p.stream2;
    const int run_i = wave_incl_scan(cnt), w1_i = wave_incl_scan(a1), w2_i = wave_incl_scan(deep ? 0 : a2);
    const long long h_i = wave_incl_scan(ah);
    const int run = run0 + run_i - cnt, w1 = w1_0 + w1_i - a1;
    int w2 = w2_0 + w2_i - a2;
    if (!DECODE && p.stream2 > 0) {
      const int deep_i = wave_incl_scan(deep ? a2 : 0);
      if (deep) w2 = w2_deep + deep_i - a2;
      w2_deep += wave_last(deep_i);
    }
    const long long h = h0 + h_i - ah;
    n1[k] = a1; n2[k] = a2; w1x[k] = w1; w2x[k] = w2;
    if (g < p.G) {
      p.seg_off[g] = run;
      p.counts[g] = cnt;
      p.work1[g] = w1;
      p.work2[g] = w2;
      p.h_off[g] = h;
      if (p.counts_out && g >= p.n_always) p.counts_out[g - p.n_always] = cnt;
    }
    run0 += wave_last(run_i);
    w1_0 += wave_last(w1_i);
    w2_0 += wave_last(w2_i);
    h0 += wave_last(h_i);
  }
  if (lane == 0) {
    p.seg_off[p.G] = run0;
    p.work1[p.G] = w1_0;
    p.work2[p.G] = w2_0;
    p.h_off[p.G] = h0;
  }
  if (!DECODE && p.stream2 > 0) {
    // the other tiles follow the deep ones: work2[g] = first tile of group g, [G] = tiles, [G + 1] = deep ones
#pragma unroll
    for (int k = 0; k < GPL; ++k) {
      const int g = lane + 64 * k;
      if (g < p.G && lw.w[k] <= p.stream2) p.work2[g] = w2_deep + w2x[k];
    }
    if (lane == 0) {
      p.work2[p.G] = w2_deep + w2_0;
      p.work2[p.G + 1] = w2_deep;
    }
  }
  if (DECODE) return;                      // (the decode kernels take their units in list order: no shares)
  // Where each XCD's share of a work list starts (entries G+1 .. G+9 of the list): contiguous ranges of
  // equal estimated cost, so that the tiles sharing operands stay in one L2 while the eight dies finish
  // together.  A tile costs its depth (K steps of 64, plus a fixed part for prologue and epilogue: the shared
  // group's down tiles are N_s times as deep as a routed expert's) times its height in 32-row blocks; with
  // tiles of dynamic height the ragged last row tile of a group costs its own blocks (at least three: below
  // that a tile is bound by fetching its weights), otherwise as much as a full one.  Inside a group the
  // boundary falls in proportion to the cost.
  __shared__ int32_t xs[2][N_XCD + 1];
  if (lane <= N_XCD) {
    xs[0][lane] = lane == N_XCD ? w1_0 : 0;
    xs[1][lane] = lane == N_XCD ? w2_0 : 0;
  }
  wave_lds_sync();
#pragma unroll
  for (int list = 0; list < 2; ++list) {
    if (list == 1 && p.stream2 > 0) break;
    const int bm = list == 0 ? p.bm1 : p.bm2, dyn = list == 0 ? p.dyn1 : p.dyn2;
    const int blocks_full = bm / 32 > 0 ? bm / 32 : 1;
    // (Which group a boundary falls into is decided in exact integers, so that every item lands in exactly
    // one share; where inside the group, in single precision: the shares need to be about equal, not exact,
    // and this wave is on the critical path of the whole forward: 64-bit divisions here doubled the
    // kernel's duration.)
    long long gc[GPL], gx[GPL];             // cost of this lane's groups and their exclusive prefix
    long long c0 = 0;
#pragma unroll
    for (int k = 0; k < GPL; ++k) {
      gc[k] = 0;
      gx[k] = c0;
      if (k > 0 && 64 * k >= p.G) continue;
      const int n_items = list == 0 ? n1[k] : n2[k];
      const int cnt = tc.tot[k], wp = lw.w[k];
      if (n_items > 0) {
        const int row_tiles = rt[list][k], col_tiles = ct[list][k];
        const int depth = (list == 0 ? cdiv(p.d, 64) : cdiv(wp, 64)) + TILE_FIXED_COST;
        const int full = row_tiles * bm == cnt ? row_tiles : row_tiles - 1, rem = cnt - full * bm;
        int last = 0;
        if (rem > 0) {
          last = blocks_full;
          if (dyn) {
            last = cdiv(rem, dyn) * (dyn / 32);           // dyn = rows per height step
            const int floor_blocks = blocks_full < 3 ? blocks_full : 3;
            if (last < floor_blocks) last = floor_blocks;
          }
        }
        gc[k] = (long long)col_tiles * depth * (full * blocks_full + last);
      }
      const long long ci = wave_incl_scan(gc[k]);
      gx[k] = c0 + ci - gc[k];
      c0 += wave_last(ci);
    }
#pragma unroll
    for (int k = 0; k < GPL; ++k) {
      if (k > 0 && 64 * k >= p.G) continue;
      const int n_items = list == 0 ? n1[k] : n2[k];
      if (n_items <= 0) continue;
      const float per_item = (float)n_items / (float)gc[k];
      static_assert(N_XCD == 8, "the share boundaries divide by a shift");
#pragma unroll
      for (int x = 1; x < N_XCD; ++x) {
        const long long t = (x * c0) >> 3;
        if (gx[k] <= t && t < gx[k] + gc[k]) {
          int local = (int)((float)(t - gx[k]) * per_item);
          if (local > n_items - 1) local = n_items - 1;
          xs[list][x] = (list == 0 ? w1x[k] : w2x[k]) + local;
        }
      }
    }
  }
  wave_lds_sync();
  if (lane <= N_XCD) {
    p.work1[p.G + 1 + lane] = xs[0][lane];
    if (p.stream2 == 0) p.work2[p.G + 1 + lane] = xs[1][lane];
  }
}

__device__ __forceinline__ void place_lists(const PlaceArgs& p, const TileCounts& tc, int lane, const LaneWidths& lw) {
  if (p.decode) place_lists_of<true>(p, tc, lane, lw);
  else place_lists_of<false>(p, tc, lane, lw);
}

}  // namespace cmoe
