// Grouped SwiGLU expert kernels for bf16 layers (Eq. 3 restricted to an expert's neurons):
//   MODE 1  H_g = Swish(X_g Wgate_g) * (X_g Wup_g)     rows of X gathered through slot2tok, K = d
//   MODE 2  Y_g = H_g Wdown_g                          K = width_pad(g), N = d
// Both are C = A * B^T with K contiguous in A and in B, computed from LDS-staged, XOR-swizzled tiles filled by direct
// global->LDS loads, in two kernels: grouped_gemm_bf16_dma (v_mfma_f32_32x32x16_bf16, 64-bit addresses) and, for the
// largest and some small tiles, grouped_gemm_bf16_ring (v_mfma_f32_16x16x32_bf16, buffer loads).  A work item is (group,
// row tile, column tile); the list of work items is a device-side prefix array written by the permute kernel, so
// ragged, empty and skewed groups need no host round trip.  Workgroups whose index is past the list exit at once.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <type_traits>
#include "cmoe_internal.h"
#include "device_utils.h"
#include "gemm_device.h"
#include "work_item.h"
#include "lds_limit.h"

namespace cmoe {

// ---- global->LDS loads and a ring of K tiles ------------------------------------------------------
// Each global_load_lds_dwordx4 moves 64 lanes x 16 bytes into 1 KB of consecutive LDS (8 tile rows);
// which global chunk a lane fetches is free, so the XOR swizzle is applied on the global side.  No
// VGPRs are spent on staging, and STAGES-1 tiles are in flight while one is multiplied.
__device__ __attribute__((aligned(16))) uint32_t g_zero_chunk[4] = {0, 0, 0, 0};
// A row of zeros as long as any K this file meets in practice.  Tile rows past the end of a group (ragged
// expert segments fill their last row tile to 50 % on average) read it instead of a real row: the result
// rows are discarded either way, but an MFMA whose operand is all zeros draws less power than one on real
// data, and on this part the clock under MFMA load is set by power.
constexpr int ZERO_ROW_ELEMS = 32768;
__device__ __attribute__((aligned(256))) bf16_t g_zero_row[ZERO_ROW_ELEMS];


__device__ __forceinline__ void dma16(const void* gsrc, bf16_t* lds_dst) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(gsrc),
                                   (__attribute__((address_space(3))) void*)(lds_dst), 16, 0, 0);
}

// LDS tile [rows][BKT] of bf16, 16-byte chunks XOR-swizzled so that the 16 rows one quarter of a
// ds_read_b128 touches fall into 16 different 16-byte bank groups (256 bytes = all 64 banks).
template <int BKT>
__device__ __forceinline__ int lds_off_t(int row, int c) {
  if (BKT == 64) return row * 64 + ((c ^ ((row >> 1) & 7)) << 3);
  return row * 32 + ((c ^ ((row >> 2) & 3)) << 3);
}

// Waves per SIMD the register allocation has to leave room for: two when two four-wave workgroups fit a CU's
// 160 KB of LDS (the compiler otherwise spends up to 512 registers on a wave that is alone on its SIMD).
constexpr int min_waves_per_simd(int bm, int bn, int bkt, int stages, int nw) {
  return (stages >= 2 && nw == 4 && bm * bn >= 256 * 128 && stages * (bm + bn) * bkt * 2 <= 80 * 1024) ? 2 : 1;
}

// DYN: the number of 32-row blocks of the tile that hold rows of the segment is found at run time and the rest
// of the kernel runs in the instantiation for exactly that many blocks per wave (MI_ACT below; the blocks are
// dealt to the WGM wave rows in turn): blocks past the end of a ragged segment are neither fetched nor
// multiplied, so a tile costs what its rows cost, in steps of 32 * WGM rows.
// Tiles up to this size ask for all groups before they know theirs (work_item.h): their launches are a round or two long.  us per
// forward, one lookup after the other / at once: 16 experts, d = 4096, 70 tokens 75.3 / 74.6, 333 tokens 102.3 / 101.7; 32 experts, d =
// 2048, 200 tokens 42.1 / 41.2; 256x256 tiles, 16 experts, 2048 tokens 200.3 / 200.8; 192x256, 32 experts, 4096 tokens 452.3 / 454.1.
constexpr int LOW_TILE_AREA = 256 * 128;

template <int BM, int BN, int BKT, int STAGES, int WGM, int WGN, int MODE, bool DYN = false>
__global__ __launch_bounds__(WGM* WGN * 64)
__attribute__((amdgpu_waves_per_eu(min_waves_per_simd(BM, BN, BKT, STAGES, WGM* WGN)))) void grouped_gemm_bf16_dma(GemmArgs p) {
  constexpr int NW = WGM * WGN;
  constexpr int TM = BM / WGM, TN = BN / WGN, MI = TM / 32, NI = TN / 32;
  constexpr int CPR = BKT / 8;                                  // 16-byte chunks per tile row
  constexpr int RPI = 64 / CPR;                                 // tile rows one 1 KB DMA instruction fills
  constexpr int A_CH = BM / RPI / NW, B_CH = BN / RPI / NW;     // DMA instructions per wave and tile
  constexpr int LPT = A_CH + B_CH;
  constexpr int STAGE_ELEMS = (BM + BN) * BKT;
  constexpr int SWZ_SHIFT = (BKT == 64) ? 1 : 2;
  // STAGES >= 2: ring of whole K tiles (A part + B part).  STAGES == 0: ring of five half tiles in the order
  // A(0) B(0) A(1) B(1) ...: while tile kt is multiplied, B(kt+1) and A(kt+2) are fetched into the two
  // halves tile kt-1 just released, and A(kt+1) is already resident, so only half a tile has to land
  // within one K step although 2.5 tiles of LDS are in use.
  constexpr bool HR = (STAGES == 0);
  constexpr int HALF = (BM > BN ? BM : BN) * BKT;
  constexpr int RING_ELEMS = HR ? 5 * HALF : STAGES * STAGE_ELEMS;
  static_assert(BKT == 32 || BKT == 64, "K tile");
  static_assert(BM % (RPI * NW) == 0 && BN % (RPI * NW) == 0, "loader");
  static_assert(MODE != 1 || TN % 64 == 0, "gate/up pairs must stay inside a wave tile");
  static_assert(HR || (STAGES >= 2 && (STAGES - 2) * LPT < 64), "ring depth");
  constexpr bool LOW_TILE = BM * BN <= LOW_TILE_AREA;
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);     // wave-uniform: LDS destinations stay scalar
  const int wm = wave / WGN, wn = wave % WGN;
  const int l32 = lane & 31, lh = lane >> 5;

  int g = 0, cnt, seg0 = 0, wp, w1_row0 = 0;
  int64_t hoff = 0, w2_off = 0;
  int n_work;
  GroupLanes gl;
  if (LOW_TILE && !p.single) gl = request_groups(p.work, p.seg_off, p.groups, p.h_off, p.G);
  if (p.single) {
    cnt = (int)p.T;
    wp = p.groups[0].width_pad;
    if (LOW_TILE) w1_row0 = p.groups[0].w1_row0;
    if (LOW_TILE) w2_off = p.groups[0].w2_off;
    const int nc = (MODE == 1) ? 2 * wp : p.d;
    n_work = ((cnt + BM - 1) / BM) * ((nc + BN - 1) / BN);
  } else {
    n_work = p.work[p.G];
  }
  // Workgroup b runs on XCD b % 8 (own L2).  Each XCD works through a contiguous range of the list so that
  // tiles sharing an operand meet in one L2: equal parts of a single-group problem, and for work lists the
  // shares of equal estimated cost that the permutation kernel left behind the prefix array.
  int wid = blockIdx.x;
  int k_part = 0;
  if (p.k_split > 1) {
    k_part = wid % p.k_split;
    wid /= p.k_split;
  }
  if (p.xcd_remap) {
    if (p.single) {
      const int chunk = (n_work + 7) >> 3;
      if ((wid >> 3) >= chunk) return;
      wid = (wid & 7) * chunk + (wid >> 3);
    } else {
      const int first = p.work[p.G + 1 + (wid & 7)], end = p.work[p.G + 2 + (wid & 7)];
      wid = first + (wid >> 3);
      if (wid >= end) return;
    }
  }
  if (wid >= n_work) return;
  int local = wid;
  if (!p.single) {
    if (LOW_TILE) {
      const WorkItem it = find_item(gl, p.G, wid);
      local = it.local;
      seg0 = it.seg0;
      cnt = it.cnt;
      wp = it.wp;
      hoff = it.hoff;
      w1_row0 = it.w1_row0;
      w2_off = it.w2_off;
    } else {
      g = find_group(p.work, p.G, wid);
      local = wid - p.work[g];
      seg0 = p.seg_off[g];
      cnt = p.seg_off[g + 1] - seg0;
      wp = p.groups[g].width_pad;
      hoff = p.h_off[g];
    }
    if (MODE == 2 && p.ws_skip && (wp == 352 || wp == 448 || wp == 704)) return;
  }
  // this workgroup's range of K tiles (all of them without a K split); from here on K and the tile
  // index count from the start of that range and the source pointers are shifted accordingly
  const int K_full = (MODE == 1) ? p.d : wp;
  int K = K_full, k_first = 0;
  if (p.k_split > 1) {
    const int kt_all = (K_full + BKT - 1) / BKT;
    const int per = (kt_all + p.k_split - 1) / p.k_split;
    k_first = (k_part * per < kt_all ? k_part * per : kt_all) * BKT;
    const int k_end = ((k_part + 1) * per < kt_all) ? (k_part + 1) * per * BKT : K_full;
    K = k_end > k_first ? k_end - k_first : 0;
  }
  const int n_cols = (MODE == 1) ? 2 * wp : p.d;
  const int n_nt = (n_cols + BN - 1) / BN;
  const int n_mt = (cnt + BM - 1) / BM;
  constexpr int GM = 8;
  const int sr = local / (GM * n_nt);
  const int rem = local - sr * (GM * n_nt);
  const int rows_in_sr = (n_mt - sr * GM) < GM ? (n_mt - sr * GM) : GM;
  const int mt = sr * GM + rem % rows_in_sr;
  const int nt = rem / rows_in_sr;

  using std::integral_constant;
  using std::false_type;
  using std::true_type;
  auto body = [&](auto act_tag) {
  constexpr int MI_ACT = decltype(act_tag)::value;              // 32-row blocks per wave that are computed
  // tile rows that are fetched: with a dynamic height the 32-row blocks of the tile are dealt to the WGM wave
  // rows in turn (wave row wm owns blocks wm, wm + WGM, ...), so MI_ACT blocks per wave cover the first
  // MI_ACT * WGM blocks of the tile; DMA instructions per wave that cover them:
  constexpr int A_ACT = DYN ? (MI_ACT * WGM * 32 + RPI * NW - 1) / (RPI * NW) : A_CH;
  auto row_block = [&](int mi) { return DYN ? mi * WGM + wm : wm * MI + mi; };
  constexpr int LPT_ACT = A_ACT + B_CH;
  // every offset a row source is read at stays below K_full rounded up to a whole K tile
  const bool use_zero_row = p.zero_pad && K_full + BKT <= ZERO_ROW_ELEMS;
  // per-lane sources: transfer i of this wave covers tile rows rg*8 .. rg*8+7, rg = wave + i*NW; the lane
  // writes physical chunk lane%8 of row rg*8 + lane/8 and therefore fetches logical chunk (lane%8) ^ swz(row)
  const bf16_t* a_src[A_ACT];
  const bf16_t* b_src[B_CH];
  int a_coff[A_ACT], b_coff[B_CH];                      // element offset of the lane's chunk inside a 64-wide K tile
#pragma unroll
  for (int i = 0; i < A_ACT; ++i) {
    const int row = (wave + i * NW) * RPI + lane / CPR;
    a_coff[i] = (((lane % CPR) ^ ((row >> SWZ_SHIFT) & (CPR - 1))) << 3);
    int r = mt * BM + row;
    const bool past = r >= cnt;
    if (past) r = cnt - 1;
    if (MODE == 1) {
      const int64_t tok = p.slot2tok ? p.slot2tok[seg0 + r] : (seg0 + r);
      a_src[i] = p.A + tok * p.d + a_coff[i] + k_first;
    } else {
      a_src[i] = p.A + hoff + (int64_t)r * wp + a_coff[i] + k_first;
    }
    if (past && use_zero_row) a_src[i] = g_zero_row + a_coff[i] + k_first;
  }
#pragma unroll
  for (int i = 0; i < B_CH; ++i) {
    const int row = (wave + i * NW) * RPI + lane / CPR;
    b_coff[i] = (((lane % CPR) ^ ((row >> SWZ_SHIFT) & (CPR - 1))) << 3);
    int n = nt * BN + row;
    const bool past = n >= n_cols;
    if (past) n = n_cols - 1;
    if (p.b_tiled) {
      // the lane's chunk of K tile kt lies 64 / 32 = 2 tiles (BKT / TILE_K) further for every kt
      const int64_t rowg = (MODE == 1) ? (int64_t)(LOW_TILE ? w1_row0 : p.groups[g].w1_row0) + n : n;
      const int64_t base = (MODE == 1) ? 0 : (LOW_TILE ? w2_off : p.groups[g].w2_off);
      const int kt32 = (MODE == 1) ? p.ldb / TILE_K : wp / TILE_K;
      b_src[i] = p.B + base + tiled_offset(rowg, k_first + b_coff[i], kt32);
    } else {
      if (MODE == 1) b_src[i] = p.B + ((int64_t)(LOW_TILE ? w1_row0 : p.groups[g].w1_row0) + n) * p.ldb + b_coff[i] + k_first;
      else b_src[i] = p.B + (LOW_TILE ? w2_off : p.groups[g].w2_off) + (int64_t)n * wp + b_coff[i] + k_first;
      if (past && use_zero_row) b_src[i] = g_zero_row + b_coff[i] + k_first;
    }
  }
  const int b_adv = p.b_tiled ? (BKT / TILE_K) * TILE_ELEMS : BKT;     // elements between a lane's chunks of two K tiles
  const int KT = (K + BKT - 1) / BKT;
  const bool k_ragged = (K % BKT) != 0;
  auto a_slot = [&](int kt) -> bf16_t* { return HR ? smem + ((2 * kt) % 5) * HALF : smem + (kt % (HR ? 1 : STAGES)) * STAGE_ELEMS; };
  auto b_slot = [&](int kt) -> bf16_t* {
    return HR ? smem + ((2 * kt + 1) % 5) * HALF : smem + (kt % (HR ? 1 : STAGES)) * STAGE_ELEMS + BM * BKT;
  };
  // one DMA instruction (index i of this wave's share) of the A or B part of tile kt
  // `maybe_last`: the tile may be the last one of a K that is not a multiple of the tile depth; its chunks
  // past K come from a block of zeros instead.  Steady-state steps never fetch the last tile and skip the test.
  auto issue_a = [&](int kt, int i, bool maybe_last) {
    const void* src = a_src[i] + kt * BKT;
    if (maybe_last && k_ragged && kt == KT - 1 && kt * BKT + a_coff[i] >= K) src = g_zero_chunk;
    dma16(src, a_slot(kt) + (wave + i * NW) * RPI * BKT);
  };
  auto issue_b = [&](int kt, int i, bool maybe_last) {
    const void* src = b_src[i] + kt * b_adv;
    if (maybe_last && k_ragged && kt == KT - 1 && kt * BKT + b_coff[i] >= K) src = g_zero_chunk;
    dma16(src, b_slot(kt) + (wave + i * NW) * RPI * BKT);
  };
  auto issue_tile_a = [&](int kt) {
#pragma unroll
    for (int i = 0; i < A_ACT; ++i) issue_a(kt, i, true);
  };
  auto issue_tile_b = [&](int kt) {
#pragma unroll
    for (int i = 0; i < B_CH; ++i) issue_b(kt, i, true);
  };

  floatx16_t acc[MI_ACT][NI];
#pragma unroll
  for (int mi = 0; mi < MI_ACT; ++mi)
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[mi][ni][i] = 0.0f;

  // prologue (a K part can be empty when the split does not divide the K tiles)
  if (HR) {
    if (KT > 0) {
      issue_tile_a(0);
      issue_tile_b(0);
    }
    if (KT > 1) issue_tile_a(1);
  } else {
#pragma unroll
    for (int st = 0; st < STAGES - 1; ++st)
      if (st < KT) { issue_tile_a(st); issue_tile_b(st); }
  }

  // One K tile: wait for it and multiply it while the loads that run ahead are issued.  AHEAD is a
  // compile-time count of what is still to be fetched, so the whole step is straight-line code:
  //   whole-tile ring: 1 = fetch tile kt+STAGES-1, 0 = nothing left
  //   half-tile ring : 2 = fetch B(kt+1) and A(kt+2), 1 = fetch B(kt+1) only, 0 = last tile
  // Instruction order inside the step is fixed by hand: memory instructions never follow one another.
  // After each MFMA comes at most one LDS fragment read of the next sub-step and at most one DMA
  // instruction, the DMA instructions spread evenly over all MFMAs of the step.  A wave that issues memory
  // instructions back to back waits for the queue to take them and cannot issue its MFMAs meanwhile
  // (measured on a skeleton of this loop: 3030 cycles per step with clustered reads, 2620 interleaved).
  auto k_tile = [&](int kt, auto ahead_tag, auto last_tag) {
    constexpr int AHEAD = decltype(ahead_tag)::value;
    constexpr bool MAYBE_LAST = decltype(last_tag)::value;   // a tile fetched in this step may be tile KT-1
    if (HR) {
      if (AHEAD >= 1) wait_vmcnt<A_ACT>();           // A(kt+1) may still be in flight; A(kt), B(kt) are older
      else wait_vmcnt<0>();
    } else {
      if (AHEAD >= 1) wait_vmcnt<HR ? 0 : (STAGES - 2) * LPT_ACT>();
      else wait_vmcnt<0>();
    }
    // Bare barrier: __syncthreads() would add a fence that drains every outstanding load (vmcnt(0)) and with
    // it the loads running ahead.  What the barrier has to order is covered by hand: this wave's parts of
    // tile kt have landed (vmcnt above), and its LDS reads of tile kt-1 were consumed by MFMAs already.
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");                   // all lanes' parts landed; the slots of tile kt-1 are free
    const bf16_t* as = a_slot(kt);
    const bf16_t* bs = b_slot(kt);
    constexpr int NKS = BKT / 16;                    // sub-steps (one MFMA depth each)
    constexpr int NMS = MI_ACT * NI;                 // MFMAs per sub-step
    constexpr int NM = NKS * NMS;                    // MFMAs per step
    // DMA instructions of this step, in issue order: half ring B(kt+1) then A(kt+2); whole ring A then B
    constexpr int N_FIRST = HR ? B_CH : A_ACT;
    constexpr int L = A_ACT + B_CH;
    auto issue_nth = [&](int i) {
      if (HR) {
        if (i < N_FIRST) issue_b(kt + 1, i, MAYBE_LAST);
        else if (AHEAD >= 2) issue_a(kt + 2, i - N_FIRST, MAYBE_LAST);
      } else {
        if (i < N_FIRST) issue_a(kt + STAGES - 1, i, MAYBE_LAST);
        else issue_b(kt + STAGES - 1, i - N_FIRST, MAYBE_LAST);
      }
    };
    // Fragments of a sub-step in the order of their first use by its MFMAs (row block mi is first needed by
    // MFMA mi * NI, column block ni by MFMA ni): A0, B0 .. B(NI-1), A1, A2, ...  LDS reads complete in issue
    // order, so the wait in front of an MFMA covers exactly the reads issued up to its own operands; with the
    // B fragments last, the first MFMA of every sub-step waited for all of them.
    bf16x8_t af[2][MI_ACT], bfr[2][NI];
    auto load_frag = [&](int ks, int k, int set) {
      const int mi = k == 0 ? 0 : k - NI;               // valid when k == 0 or k > NI
      if (k == 0 || k > NI) af[set][mi] = *reinterpret_cast<const bf16x8_t*>(as + lds_off_t<BKT>(row_block(mi) * 32 + l32, ks * 2 + lh));
      else bfr[set][k - 1] = *reinterpret_cast<const bf16x8_t*>(bs + lds_off_t<BKT>(wn * TN + (k - 1) * 32 + l32, ks * 2 + lh));
    };
#pragma unroll
    for (int f = 0; f < MI_ACT + NI; ++f) load_frag(0, f, 0);
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      const int cur = ks & 1;
#pragma unroll
      for (int j = 0; j < NMS; ++j) {
        const int mi = j / NI, ni = j % NI;
        __builtin_amdgcn_sched_barrier(0);
        // (down contraction: operands swapped, so that the accumulator block is the transpose: a lane then holds
        // four consecutive output columns of one row instead of one column of sixteen rows, and the epilogue
        // stages 8-byte pieces instead of single elements; same products, same order of accumulation)
        if constexpr (MODE == 2) acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[cur][ni], af[cur][mi], acc[mi][ni], 0, 0, 0);
        else acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[cur][mi], bfr[cur][ni], acc[mi][ni], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        // fragments of the next sub-step, spread over this sub-step's MFMAs (several per MFMA only when
        // a sub-step has fewer MFMAs than fragments)
#pragma unroll
        for (int f = 0; f < MI_ACT + NI; ++f)
          if (ks + 1 < NKS && f * NMS / (MI_ACT + NI) == j) load_frag(ks + 1, f, cur ^ 1);
        if (AHEAD >= 1) {
          const int m = ks * NMS + j;
          // (a skinny tile has more DMA instructions than MFMAs: then several follow one MFMA)
#pragma unroll
          for (int i = 0; i < L; ++i)
            if (L > NM ? (i * NM / L == m) : ((i + 1) * NM / L - 1 == m)) issue_nth(i);
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  int kt = 0;
  if (HR) {
    for (; kt + 3 < KT; ++kt) k_tile(kt, integral_constant<int, 2>{}, false_type{});   // fetches B(kt+1), A(kt+2)
    for (; kt + 2 < KT; ++kt) k_tile(kt, integral_constant<int, 2>{}, true_type{});    // A(KT-1)
    for (; kt + 1 < KT; ++kt) k_tile(kt, integral_constant<int, 1>{}, true_type{});    // B(KT-1)
    for (; kt < KT; ++kt) k_tile(kt, integral_constant<int, 0>{}, false_type{});
  } else {
    constexpr int S1 = (HR ? 2 : STAGES) - 1;             // a step fetches tile kt+S1
    for (; kt + S1 + 1 < KT; ++kt) k_tile(kt, integral_constant<int, 1>{}, false_type{});
    for (; kt + S1 < KT; ++kt) k_tile(kt, integral_constant<int, 1>{}, true_type{});
    for (; kt < KT; ++kt) k_tile(kt, integral_constant<int, 0>{}, false_type{});
  }

  // ---- K split: the raw fp32 partial sums go to this part's slab; 32 consecutive lanes hold 32
  // consecutive columns of a row, so the stores are 128-byte segments ----
  if (p.k_split > 1) {
    float* slab = p.P + (int64_t)k_part * p.p_rows * p.ldp;
    if constexpr (MODE == 2) {
      // transposed accumulator blocks: element i of block (mi, ni) = row l32 of the row block, column
      // (i / 4) * 8 + lh * 4 + i % 4 of the column block; four consecutive columns per 16-byte store
      // (the slab's row stride is d, a multiple of 8)
#pragma unroll
      for (int mi = 0; mi < MI_ACT; ++mi) {
        const int r = mt * BM + row_block(mi) * 32 + l32;
        if (r >= cnt) continue;
        float* prow = slab + (int64_t)(seg0 + r) * p.ldp;
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int col = nt * BN + wn * TN + ni * 32 + q * 8 + lh * 4;
            if (col < n_cols)
              *reinterpret_cast<float4*>(prow + col) =
                  make_float4(acc[mi][ni][4 * q], acc[mi][ni][4 * q + 1], acc[mi][ni][4 * q + 2], acc[mi][ni][4 * q + 3]);
          }
      }
      return;
    }
#pragma unroll
    for (int mi = 0; mi < MI_ACT; ++mi)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int r = mt * BM + row_block(mi) * 32 + (i / 4) * 8 + lh * 4 + (i % 4);
        if (r >= cnt) continue;
        float* prow = slab + (int64_t)(seg0 + r) * p.ldp;
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
          const int col = nt * BN + wn * TN + ni * 32 + l32;
          if (col < n_cols) prow[col] = acc[mi][ni][i];
        }
      }
    return;
  }
  // ---- epilogue: through LDS, so that global stores are 16-byte vectors along the rows ----
  // Each wave stages 32 rows of its tile at a time in a private LDS strip (row stride padded by 16 bytes
  // against bank conflicts), then every lane copies 16-byte pieces of rows out to global memory.
  constexpr int TNO = (MODE == 1) ? TN / 2 : TN;          // output columns of a wave tile
  constexpr int LDO = TNO + 8;                            // strip row stride in elements
  constexpr int CPRO = TNO / 8;                           // 16-byte pieces per strip row
  static_assert(NW * 32 * LDO <= RING_ELEMS, "epilogue strip must fit in the tile ring");
  __syncthreads();                                        // every wave is done reading the last tile
  bf16_t* strip = smem + wave * 32 * LDO;
  const int out_col0 = (MODE == 1) ? (nt * BN + wn * TN) / 2 : nt * BN + wn * TN;
  const int out_cols = (MODE == 1) ? wp : p.d;
  bf16_t* out_base = (MODE == 1) ? p.C + hoff : p.C + (int64_t)seg0 * p.d;
  const int64_t out_ld = (MODE == 1) ? wp : p.d;
#pragma unroll
  for (int mi = 0; mi < MI_ACT; ++mi) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int rr = (i / 4) * 8 + lh * 4 + (i % 4);
      if constexpr (MODE == 1) {
#pragma unroll
        for (int pi = 0; pi < NI / 2; ++pi) {
          const float gt = acc[mi][2 * pi][i], up = acc[mi][2 * pi + 1][i];
          // Swish(g) * u with the hardware exponential: the result is rounded to bf16 right after
          const float sg = gt * __frcp_rn(1.0f + __expf(-gt));
          strip[rr * LDO + pi * 32 + l32] = f32_to_bf16(sg * up);
        }
      }
    }
    if constexpr (MODE == 2) {
      // transposed blocks (see the MFMA above): this lane's row of the strip is l32, and every group of four
      // accumulator elements is four consecutive columns: one 8-byte LDS write each
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          ushort4 v;
          v.x = f32_to_bf16(acc[mi][ni][4 * q]);
          v.y = f32_to_bf16(acc[mi][ni][4 * q + 1]);
          v.z = f32_to_bf16(acc[mi][ni][4 * q + 2]);
          v.w = f32_to_bf16(acc[mi][ni][4 * q + 3]);
          *reinterpret_cast<ushort4*>(strip + l32 * LDO + ni * 32 + q * 8 + lh * 4) = v;
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");    // the strip is private to this wave: no barrier
#pragma unroll
    for (int q = lane; q < 32 * CPRO; q += 64) {
      const int rr = q / CPRO, cc = q % CPRO;
      const int r = mt * BM + row_block(mi) * 32 + rr;
      const int col = out_col0 + cc * 8;
      const uint4 v = *reinterpret_cast<const uint4*>(strip + rr * LDO + cc * 8);
      if (r < cnt && col < out_cols) *reinterpret_cast<uint4*>(out_base + (int64_t)r * out_ld + col) = v;
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");    // reads done before the strip is overwritten
  }
};   // body
  if constexpr (DYN) {
    const int rows_here = cnt - mt * BM;
    const int nb = rows_here >= BM ? MI : ((rows_here + 31) / 32 + WGM - 1) / WGM;      // blocks per wave row
    switch (nb) {
      case 1: body(integral_constant<int, 1>{}); break;
      case 2: if constexpr (MI >= 2) body(integral_constant<int, 2>{}); break;
      case 3: if constexpr (MI >= 3) body(integral_constant<int, 3>{}); break;
      case 4: if constexpr (MI >= 4) body(integral_constant<int, 4>{}); break;
      case 5: if constexpr (MI >= 5) body(integral_constant<int, 5>{}); break;
      case 6: if constexpr (MI >= 6) body(integral_constant<int, 6>{}); break;
      case 7: if constexpr (MI >= 7) body(integral_constant<int, 7>{}); break;
      default: body(integral_constant<int, MI>{}); break;
    }
  } else {
    body(integral_constant<int, MI>{});
  }
}

// ---- deep ring: the kernel of the large tiles ------------------------------------------------------------
// What bounds it: the matrix cores under the power limit at large batches (a loop of nothing but MFMAs on random
// operands holds 2.06 PFLOP/s at 2.04 GHz with the 16x16x32 instruction and 1.77 PFLOP/s at 1.76 GHz with
// 32x32x16: half the accumulator traffic per flop), bytes in flight from HBM at small ones.
//
// A 16x16x32 MFMA gives the bits of the two 32x32x16 ones of the kernel above, so the shapes stay interchangeable.
//
// Layout.  K runs in steps of 32, the depth of one MFMA.  A stage of the LDS ring is the A part and the B part
// of one step in blocks of 16 rows x 32 K (1 KB): one block is one 1 KB buffer load of a wave and one
// operand of the MFMA, and a weight block is 1 KB of consecutive memory (the tiled weight layout).  The 16-byte
// chunks of a row are XOR-swizzled with (row >> 2) & 3, on the global side, so that the 16 rows a quarter of a
// ds_read_b128 touches fall into 16 different 16-byte bank groups.
//
// Schedule.  While step kt is multiplied out of registers, the fragments of step kt + 1 are read from LDS into the
// other register set and step kt + STAGES is fetched into the slot that step kt left: a step has STAGES - 1 steps
// of time to arrive (128 KB in flight per CU for the 256 x 256 tile), its LDS reads have a quarter of a step
// to return, and nothing is waited for between the barrier and the first MFMA.  (A step of 64 whose first
// fragments were read behind its barrier, with one and a half steps in flight, took 2700-3000 cycles for 2048
// cycles of MFMA issue.)  Memory instructions never follow one another: after an MFMA comes at most one LDS
// read and one DMA instruction.
//
// Transfers are buffer loads: the lane's offset stays in one register for the whole K loop, the step's is a scalar, and
// lanes without a source (rows past a segment's end, K past its end) carry an offset past the buffer's
// size, for which the hardware delivers zeros.  A wave issues in order, so a transfer stalls its MFMAs until the
// address unit has taken it: measured 65 cycles each with 64-bit global addresses, 22-27 with buffer offsets
// (1650 against 1290 cycles per step of 1024 cycles of MFMA issue; 8192 x 22016 x 4096: 1203 -> 1364 TFLOP/s; the step
// of 64 with global addresses that this replaces: 1174).  Giving the four waves different issue slots made it
// slower in every form tried.

constexpr int ring_stage_elems(int bm, int bn, int nw) {
  return ((bm / 16 + nw - 1) / nw + (bn / 16 + nw - 1) / nw) * nw * BLK;
}
// The epilogue's strips take the ring's place: each wave stages its whole tile in rows padded by 16 bytes.
constexpr int ring_strip_elems(int bm, int bn, int wgn, int mode) { return bm * wgn * ((mode == 1 ? bn / wgn / 2 : bn / wgn) + 8); }
constexpr size_t ring_smem_bytes(int bm, int bn, int stages, int nw, int wgn, int mode) {
  const int ring = stages * ring_stage_elems(bm, bn, nw), strips = ring_strip_elems(bm, bn, wgn, mode);
  return (size_t)(ring > strips ? ring : strips) * sizeof(bf16_t);
}
// Workgroups a CU's 160 KB of LDS holds, hence waves per SIMD the register allocation has to leave room for.
constexpr int ring_groups_per_cu(int bm, int bn, int stages, int nw) {
  return (stages * ring_stage_elems(bm, bn, nw) * 2 <= 80 * 1024) ? 2 : 1;
}

// WIDE: the rows of a tile may lie 2 GB or more apart (a gather from a batch of that size): 64-bit addresses per lane.
template <int BM, int BN, int STAGES, int KU, int WGM, int WGN, int MODE, bool WIDE = false>
__global__ __launch_bounds__(WGM* WGN * 64)
__attribute__((amdgpu_waves_per_eu(ring_groups_per_cu(BM, BN, STAGES * KU, WGM* WGN) * (WGM * WGN / 4)))) void grouped_gemm_bf16_ring(GemmArgs p) {
  constexpr int NW = WGM * WGN;
  constexpr int TM = BM / WGM, TN = BN / WGN, MB = TM / 16, NB = TN / 16;
  constexpr int A_CH = (BM / 16 + NW - 1) / NW, B_CH = (BN / 16 + NW - 1) / NW;   // DMA instructions per wave and step
  constexpr int LPT = A_CH + B_CH;
  constexpr int A_ELEMS = A_CH * NW * BLK;                     // (a part that NW does not divide has spare blocks)
  constexpr int STAGE_ELEMS = ring_stage_elems(BM, BN, NW);
  static_assert(BM % (16 * WGM) == 0 && BN % (16 * WGN) == 0, "whole blocks per wave");
  static_assert(MODE != 1 || TN % 64 == 0, "gate/up pairs must stay inside a wave tile");
  static_assert(STAGES >= 3 && (STAGES - 1) * KU * LPT < 64, "ring depth");
  constexpr bool LOW_TILE = BM * BN <= LOW_TILE_AREA;
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);     // wave-uniform: LDS destinations stay scalar
  const int wm = wave / WGN, wn = wave % WGN;
  const int r16 = lane & 15, kq = lane >> 4;

  int g = 0, cnt, seg0 = 0, wp, w1_row0 = 0;
  int64_t hoff = 0, w2_off = 0;
  int n_work;
  GroupLanes gl;
  if (LOW_TILE && !p.single) gl = request_groups(p.work, p.seg_off, p.groups, p.h_off, p.G);
  if (p.single) {
    cnt = (int)p.T;
    wp = p.groups[0].width_pad;
    if (LOW_TILE) w1_row0 = p.groups[0].w1_row0;
    if (LOW_TILE) w2_off = p.groups[0].w2_off;
    const int nc = (MODE == 1) ? 2 * wp : p.d;
    n_work = ((cnt + BM - 1) / BM) * ((nc + BN - 1) / BN);
  } else {
    n_work = p.work[p.G];
  }
  // Workgroup b runs on XCD b % 8 (own L2).  Each XCD works through a contiguous range of the list so that
  // tiles sharing an operand meet in one L2: equal parts of a single-group problem, and for work lists the
  // shares of equal estimated cost that the permutation kernel left behind the prefix array.
  int wid = blockIdx.x;
  int k_part = 0;
  if (p.k_split > 1) {
    k_part = wid % p.k_split;
    wid /= p.k_split;
  }
  if (p.xcd_remap) {
    if (p.single) {
      const int chunk = (n_work + 7) >> 3;
      if ((wid >> 3) >= chunk) return;
      wid = (wid & 7) * chunk + (wid >> 3);
    } else {
      const int first = p.work[p.G + 1 + (wid & 7)], end = p.work[p.G + 2 + (wid & 7)];
      wid = first + (wid >> 3);
      if (wid >= end) return;
    }
  }
  if (wid >= n_work) return;
  int local = wid;
  if (!p.single) {
    if (LOW_TILE) {
      const WorkItem it = find_item(gl, p.G, wid);
      local = it.local;
      seg0 = it.seg0;
      cnt = it.cnt;
      wp = it.wp;
      hoff = it.hoff;
      w1_row0 = it.w1_row0;
      w2_off = it.w2_off;
    } else {
      g = find_group(p.work, p.G, wid);
      local = wid - p.work[g];
      seg0 = p.seg_off[g];
      cnt = p.seg_off[g + 1] - seg0;
      wp = p.groups[g].width_pad;
      hoff = p.h_off[g];
    }
    if (MODE == 2 && p.ws_skip && (wp == 352 || wp == 448 || wp == 704)) return;
  }
  // this workgroup's range of K steps (all of them without a K split); K counts from the start of the range
  const int K_full = (MODE == 1) ? p.d : wp;
  int K = K_full, k_first = 0;
  if (p.k_split > 1) {
    const int kt_all = (K_full + BK - 1) / BK;
    const int per = (kt_all + p.k_split - 1) / p.k_split;
    k_first = (k_part * per < kt_all ? k_part * per : kt_all) * BK;
    const int k_end = ((k_part + 1) * per < kt_all) ? (k_part + 1) * per * BK : K_full;
    K = k_end > k_first ? k_end - k_first : 0;
  }
  const int KT = (K + BK - 1) / BK;
  const int n_cols = (MODE == 1) ? 2 * wp : p.d;
  const int n_nt = (n_cols + BN - 1) / BN;
  const int n_mt = (cnt + BM - 1) / BM;
  constexpr int GM = 8;
  const int sr = local / (GM * n_nt);
  const int rem = local - sr * (GM * n_nt);
  const int rows_in_sr = (n_mt - sr * GM) < GM ? (n_mt - sr * GM) : GM;
  const int mt = sr * GM + rem % rows_in_sr;
  const int nt = rem / rows_in_sr;

  // Sources: transfer i of this wave fills block wave + i * NW; the lane writes physical chunk lane % 4 of row lane / 4
  // and therefore fetches logical chunk (lane % 4) ^ (row >> 2) & 3.  Offsets count from the tile's first row
  // (for a gather: the row of its first token; a segment's tokens ascend) and first column block.  Everything
  // past the end of the segment, of the group's columns or of K (the loop fetches STAGES steps ahead to its end)
  // is delivered as zeros.  (A product with zeros also draws less power than one with a repeated row, and the
  // clock under MFMA load is set by power.)
  const int coff = ((lane & 3) ^ ((lane >> 4) & 3)) << 3;
  const int row_first = mt * BM;                               // of the segment
  int64_t tok_first = 0;
  const bf16_t* a_base;
  int64_t a_bytes;                                             // from a_base to the end of the operand
  if (MODE == 1) {
    tok_first = __builtin_amdgcn_readfirstlane(p.slot2tok ? p.slot2tok[seg0 + row_first] : (seg0 + row_first));
    a_base = p.A + tok_first * p.d + k_first;
    a_bytes = ((p.T - tok_first) * p.d - k_first) * 2;
  } else {
    a_base = p.A + hoff + (int64_t)row_first * wp + k_first;
    a_bytes = ((int64_t)(cnt - row_first) * wp - k_first) * 2;
  }
  a_base = uniform_ptr(a_base);
  const uint32_t a_size = __builtin_amdgcn_readfirstlane((uint32_t)(a_bytes < (int64_t)DMA_NONE ? a_bytes : (int64_t)DMA_NONE));
  uint32_t a_off[A_CH];
  const bf16_t* a_src[WIDE ? A_CH : 1];
#pragma unroll
  for (int i = 0; i < A_CH; ++i) {
    const int row = (wave + i * NW) * 16 + (lane >> 2);
    const int r = row_first + row;
    const bool ok = row < BM && r < cnt;
    int64_t rel = row;                                         // row of A, relative to the first one
    if (MODE == 1 && p.slot2tok) rel = ok ? p.slot2tok[seg0 + r] - tok_first : 0;
    const int64_t off = rel * (MODE == 1 ? p.d : wp) + coff;
    a_off[i] = ok ? (uint32_t)(off * 2) : DMA_NONE;
    if constexpr (WIDE) a_src[i] = ok ? a_base + off : nullptr;
  }
  // K need not be a multiple of 32 (the weights are zero-padded, x is not): chunks of the last step past its end
  const bool k_past = (KT - 1) * BK + coff >= K;
  const int kt32 = (MODE == 1) ? p.ldb / TILE_K : wp / TILE_K;
  const int col_blk0 = nt * (BN / 16);
  const bf16_t* b_base = (MODE == 1) ? p.B + (int64_t)(LOW_TILE ? w1_row0 : p.groups[g].w1_row0) * p.ldb : p.B + (LOW_TILE ? w2_off : p.groups[g].w2_off);
  b_base = uniform_ptr(b_base + ((int64_t)col_blk0 * kt32 + k_first / TILE_K) * TILE_ELEMS);
  // column blocks the tile has: the rest of the buffer's size would be the next tile's
  const int col_blks = min(BN / 16, (n_cols + 15) / 16 - col_blk0);
  const uint32_t b_size = __builtin_amdgcn_readfirstlane((uint32_t)((col_blks * kt32 - k_first / TILE_K) * TILE_ELEMS * 2));
  uint32_t b_off[B_CH];
#pragma unroll
  for (int i = 0; i < B_CH; ++i) {
    const int blk = wave + i * NW;
    b_off[i] = blk < col_blks ? (uint32_t)((blk * kt32 * TILE_ELEMS + (lane >> 2) * TILE_K + coff) * 2) : DMA_NONE;
  }
  auto issue_a = [&](int kt, int slot, int i) {
    bf16_t* dst = smem + slot * STAGE_ELEMS + (wave + i * NW) * BLK;
    if constexpr (WIDE) {
      const bool none = a_src[i] == nullptr || kt >= KT || (kt == KT - 1 && k_past);
      dma16(none ? (const void*)g_zero_chunk : (const void*)(a_src[i] + kt * BK), dst);
    } else {
      dma16_buffer(a_base, kt < KT ? a_size : 0u, (kt == KT - 1 && k_past) ? DMA_NONE : a_off[i], (uint32_t)kt * (BK * 2), dst);
    }
  };
  auto issue_b = [&](int kt, int slot, int i) {
    dma16_buffer(b_base, kt < KT ? b_size : 0u, b_off[i], (uint32_t)kt * (TILE_ELEMS * 2), smem + slot * STAGE_ELEMS + A_ELEMS + (wave + i * NW) * BLK);
  };

  // accumulator blocks of 16 x 16 (transposed, see mfma_acc): a lane holds columns kq * 4 .. + 3 of row r16
  floatx4_t acc[MB][NB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[mb][nb][i] = 0.0f;

  // a lane's fragment of a block: row r16, logical chunk kq
  const int frag = r16 * BK + ((kq ^ (r16 >> 2)) << 3);
  constexpr int NM = MB * NB * KU, NF = (MB + NB) * KU, ND = LPT * KU;   // MFMAs, LDS reads and transfers per step
  static_assert(ND <= NM, "at most one DMA instruction after an MFMA");
  bf16x8_t af[2][KU][MB], wf[2][KU][NB];
  auto load_frag = [&](int slot, int f, int set) {            // per K32: B fragments first, then A
    const int u = f / (MB + NB), q = f % (MB + NB);
    const bf16_t* st = smem + (slot * KU + u) * STAGE_ELEMS + frag;
    if (q < NB) wf[set][u][q] = *reinterpret_cast<const bf16x8_t*>(st + A_ELEMS + (wn * NB + q) * BLK);
    else af[set][u][q - NB] = *reinterpret_cast<const bf16x8_t*>(st + (wm * MB + q - NB) * BLK);
  };
  auto issue = [&](int step, int slot, int i) {               // transfer i of a step
    const int u = i / LPT, q = i % LPT;
    if (q < A_CH) issue_a(step * KU + u, slot * KU + u, q);
    else issue_b(step * KU + u, slot * KU + u, q - A_CH);
  };

#pragma unroll
  for (int st = 0; st < STAGES; ++st)
#pragma unroll
    for (int i = 0; i < ND; ++i) issue(st, st, i);
  wait_vmcnt<(STAGES - 1) * ND>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#pragma unroll
  for (int f = 0; f < NF; ++f) load_frag(0, f, 0);

  const int n_steps = (KT + KU - 1) / KU;
  int slot = 0;                                               // of the current step
  auto step = [&](int ks, auto set_tag, auto wait_tag) {
    constexpr int SET = decltype(set_tag)::value;
    constexpr bool WAIT = decltype(wait_tag)::value;
    // Bare barrier: __syncthreads() would add a fence that drains every outstanding load.  What the barrier has to
    // order is covered by hand: this wave's parts of step ks + 1 have landed (vmcnt), and its LDS reads of step
    // ks have returned (lgkmcnt), so behind it step ks + 1 can be read and the slot of step ks refilled.
    wait_vmcnt<(STAGES - 2) * ND>();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    const int next = slot + 1 == STAGES ? 0 : slot + 1;
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      const int u = m / (MB * NB), mb = (m / NB) % MB, nb = m % NB;
      __builtin_amdgcn_sched_barrier(0);
      if (WAIT && m == NM - 1) mfma_acc<true>(acc[mb][nb], wf[SET][u][nb], af[SET][u][mb]);
      else mfma_acc<false>(acc[mb][nb], wf[SET][u][nb], af[SET][u][mb]);
      __builtin_amdgcn_sched_barrier(0);
      // fragment f of the next step follows MFMA f * (3/4 NM) / NF: the last ones have a quarter of a step to return
      const int f = (m * NF * 4 + NM * 3 - 1) / (NM * 3);
      if (f < NF && f * NM * 3 / (NF * 4) == m) load_frag(next, f, SET ^ 1);
      // (a small tile has more of them than MFMAs in three quarters of a step: then two follow one MFMA)
      if (f + 1 < NF && (f + 1) * NM * 3 / (NF * 4) == m) load_frag(next, f + 1, SET ^ 1);
      // DMA instruction i follows MFMA (i + 1) * NM / ND - 1
      const int i = ((m + 1) * ND + NM - 1) / NM - 1;
      if (i < ND && (i + 1) * NM / ND - 1 == m) issue(ks + STAGES, slot, i);
    }
    __builtin_amdgcn_sched_barrier(0);
    slot = next;
  };
  int ks = 0;
  for (; ks + 1 < n_steps; ks += 2) {
    step(ks, std::integral_constant<int, 0>{}, std::false_type{});
    step(ks + 1, std::integral_constant<int, 1>{}, std::true_type{});      // (the loop may end here)
  }
  if (ks < n_steps) step(ks, std::integral_constant<int, 0>{}, std::true_type{});
  __builtin_amdgcn_sched_barrier(0);

  // ---- K split: the raw fp32 partial sums go to this part's slab, four consecutive columns per 16-byte store
  // (the slab's row stride is d or 2 * max_width_pad, a multiple of 8) ----
  if (p.k_split > 1) {
    wait_vmcnt<0>();                                          // (no transfer into LDS may outlive the workgroup)
    float* slab = p.P + (int64_t)k_part * p.p_rows * p.ldp;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int r = mt * BM + (wm * MB + mb) * 16 + r16;
      if (r >= cnt) continue;
      float* prow = slab + (int64_t)(seg0 + r) * p.ldp;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const int col = nt * BN + wn * TN + nb * 16 + kq * 4;
        if (col < n_cols) *reinterpret_cast<floatx4_t*>(prow + col) = acc[mb][nb];
      }
    }
    return;
  }
  // ---- epilogue: through LDS, so that global stores are 16-byte vectors along the rows ----
  // Each wave stages its tile in a private LDS strip (row stride padded by 16 bytes against bank conflicts), then
  // every lane copies 16-byte pieces of rows out to global memory.
  constexpr int TNO = (MODE == 1) ? TN / 2 : TN;          // output columns of a wave tile
  constexpr int LDO = TNO + 8;                            // strip row stride in elements
  constexpr int CPRO = TNO / 8;                           // 16-byte pieces per strip row
  static_assert(NW * TM * LDO == ring_strip_elems(BM, BN, WGN, MODE), "strips");
  wait_vmcnt<0>();
  __syncthreads();                                        // every wave's reads of the ring and transfers into it are done
  bf16_t* strip = smem + wave * TM * LDO;
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    bf16_t* srow = strip + (mb * 16 + r16) * LDO + kq * 4;
    if constexpr (MODE == 1) {
      // column blocks of a gate/up pair: two of 16 gate columns, then the two of the matching up columns
#pragma unroll
      for (int pb = 0; pb < NB / 2; ++pb) {
        const floatx4_t gt = acc[mb][(pb / 2) * 4 + pb % 2], up = acc[mb][(pb / 2) * 4 + 2 + pb % 2];
        // Swish(g) * u with the hardware exponential: the result is rounded to bf16 right after
        ushort4 v;
        v.x = f32_to_bf16(gt[0] * __frcp_rn(1.0f + __expf(-gt[0])) * up[0]);
        v.y = f32_to_bf16(gt[1] * __frcp_rn(1.0f + __expf(-gt[1])) * up[1]);
        v.z = f32_to_bf16(gt[2] * __frcp_rn(1.0f + __expf(-gt[2])) * up[2]);
        v.w = f32_to_bf16(gt[3] * __frcp_rn(1.0f + __expf(-gt[3])) * up[3]);
        *reinterpret_cast<ushort4*>(srow + pb * 16) = v;
      }
    } else {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        ushort4 v;
        v.x = f32_to_bf16(acc[mb][nb][0]);
        v.y = f32_to_bf16(acc[mb][nb][1]);
        v.z = f32_to_bf16(acc[mb][nb][2]);
        v.w = f32_to_bf16(acc[mb][nb][3]);
        *reinterpret_cast<ushort4*>(srow + nb * 16) = v;
      }
    }
  }
  const int out_col0 = (MODE == 1) ? (nt * BN + wn * TN) / 2 : nt * BN + wn * TN;
  const int out_cols = (MODE == 1) ? wp : p.d;
  bf16_t* out_base = (MODE == 1) ? p.C + hoff : p.C + (int64_t)seg0 * p.d;
  const int64_t out_ld = (MODE == 1) ? wp : p.d;
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // the strip is private to this wave: no barrier
  const int row0 = mt * BM + wm * TM;
#pragma unroll 4
  for (int q = lane; q < TM * CPRO; q += 64) {
    const int rr = q / CPRO, cc = q % CPRO;
    const int r = row0 + rr;
    const int col = out_col0 + cc * 8;
    const uint4 v = *reinterpret_cast<const uint4*>(strip + rr * LDO + cc * 8);
    if (r < cnt && col < out_cols) *reinterpret_cast<uint4*>(out_base + (int64_t)r * out_ld + col) = v;
  }
}

// ---- tile configurations ---------------------------------------------------------------------
// Tile shapes (the tuning switches gemm1_cfg / gemm2_cfg select one by index).
// stages >= 2: ring of whole K tiles; stages == 0: ring of five half tiles.
struct TileCfg { int bm, bn, wgm, wgn, stages, bk; };
static const TileCfg kCfgs[] = {
    {256, 256, 2, 4, 5, 32},   // 0: deep ring (see grouped_gemm_bf16_ring), eight waves of 128x64
    {128, 128, 2, 2, 2, 64},   // 1: two stages, two workgroups per CU
    {256, 256, 2, 4, 2, 64},   // 2
    {128, 128, 2, 2, 0, 64},   // 3
    {256, 128, 4, 2, 3, 64},   // 4
    {256, 256, 2, 4, 4, 32},   // 5
    {256, 256, 2, 2, 5, 32},   // 6: deep ring, four waves of 128x128
    {64, 128, 2, 2, 4, 64},    // 7: skinny tile for batches of tens of tokens per group, four whole K tiles deep: a
                               //    CU keeps 72 KB of loads in flight, two thirds of them weights (such a launch
                               //    is bound by HBM latency x bytes in flight, not by MFMA work).  Measured against
                               //    32x128 (2 waves; 3 and 7 stages), 32x256 and 64x128 with 3 and 6 stages.
    {128, 256, 2, 2, 3, 32},   // 8: four waves of 64x128, three K tiles of 32: 72 KB of LDS and at most 256 registers,
                               //    so two workgroups share a CU and one's epilogue overlaps the other's K loop
                               //    (the short-K down contraction; 256x128 in the same arrangement was slower)
    {224, 256, 2, 2, 5, 32},   // 9: deep ring, four waves of 112x128
    {192, 256, 1, 4, 0, 64},   // 10: four waves of 192x64
    {256, 256, 1, 4, 0, 64},   // 11: four waves of 256x64 with a dynamic tile height (DYN): a ragged segment's last tile
                               //     costs its rows in steps of 32, so the tallest tile wastes the least
    {128, 256, 1, 4, 3, 32},   // 12: the arrangement of 8 (two workgroups per CU, three K tiles of 32) with four waves
                               //     of 128x64 and a dynamic tile height
    {256, 256, 2, 2, 0, 64},   // 13: shape 6 (four waves of 128x128) with a dynamic tile height in steps of 64 rows: a
                               //     wave reads each A fragment for 128 columns, which the LDS keeps up with; four
                               //     waves of 256x64 (11) read a quarter more and are bound by it
    {128, 256, 2, 2, 3, 32},   // 14: shape 8 with a dynamic tile height in steps of 64 rows
    // 15-18: the weight-stationary down contraction (ws_down.hip): work items of 128 / 256 / 512 / 1024 rows x 256 columns,
    // cost in steps of 64 rows; groups it has no instantiation for run shape 8 (128 rows) or 6 (256 rows) over
    // the same list
    {128, 256, 2, 2, 3, 32},
    {256, 256, 2, 2, 0, 32},
    {512, 256, 2, 2, 0, 32},
    {1024, 256, 2, 2, 0, 32},  // 18: the same with 1024 rows per item
    {160, 256, 2, 2, 5, 32},   // 19: deep ring, four waves of 80x128
    {128, 128, 2, 2, 5, 32},   // 20: deep ring, four waves of 64x64
    {64, 128, 2, 2, 6, 32},    // 21: deep ring in steps of 64, four waves of 32x64, two workgroups per CU
    {128, 256, 2, 2, 3, 32},   // 22: the persistent down contraction (gemm_stream.hip)
    {STREAM_ROWS, 32, 1, 8, 2, 32},   // 23: streamed gate/up units of 16 neurons (gate_up_stream.hip)
    {STREAM_ROWS, 16, 1, 8, 2, 32},   // 24: ... of 8
};
static bool cfg_is_ws(int ci) { return ci >= 15 && ci <= 18; }
static bool cfg_is_stream(int ci) { return ci == 22; }
static bool cfg_is_ring(int ci) { return kCfgs[ci].stages >= 5 && !cfg_is_stream(ci); }
static bool cfg_is_units(int ci) { return ci == 23 || ci == 24; }
bool gate_up_streams_forced() { return cfg_is_units(tuning().gemm1_cfg); }
static bool cfg_is_dyn(int ci) { return ci >= 11 && ci <= 18; }
bool ws_down_handles(int width_pad);
hipError_t launch_down_stream(const Engine& e, const GemmArgs& a, hipStream_t s);
hipError_t launch_ws_down(const Engine& e, char* ws, const WsLayout& L, const void* y_slots, int rc, int n_blocks,
                          int xcd_remap, hipStream_t s);
constexpr int kNumCfgs = sizeof(kCfgs) / sizeof(kCfgs[0]);

// Rows of x that one tile gathers can be 2 GB or more apart.
static bool wide_gather(int d, int64_t T) { return T * d * 2 >= (int64_t)DMA_NONE; }

// Routed groups of one width and load: the experts of a flat layer; the outer experts' shared groups and the
// sub-experts of a hierarchy.
struct LoadClass { int64_t groups, entries; int width_pad; };
static int load_classes(const Engine& e, int64_t T, LoadClass (&c)[2]) {
  const int routed = e.G - e.n_always;
  if (routed <= 0 || e.S_dyn <= 0) return 0;
  if (e.r.outer_top_k > 0 && e.r.sub_has_shared && e.r.top_k > 0) {
    const int64_t outer = routed / e.r.groups_per_outer, entries = T * e.r.outer_top_k;
    c[0] = {outer, entries, e.width_pad_host[e.n_always]};
    c[1] = {routed - outer, entries * e.r.top_k, e.width_pad_host[e.n_always + 1]};
    return 2;
  }
  c[0] = {routed, T * e.S_dyn, e.width_pad_host[e.n_always]};
  return 1;
}

// Which tile shape for contraction `which` (1: gate/up, 2: down) of a batch of T tokens: the tuning switches
// gemm1_cfg / gemm2_cfg when set, else the models below.
// Tile shape of the gate/up contraction: the one with the lowest estimated time = rounds x time per round,
// rounds = ceil(tiles / workgroup slots on the chip).  Relative times per round measured on the
// LLaMA-shaped layers (K = d for every shape, so the ratios carry over): 256x256 0.95 (one workgroup per CU),
// 224x256 0.875, 192x256 0.81, 160x256 0.75, 256x128 0.62, 128x128 0.66 with two per CU and, on the deep ring, 0.51
// with one (333 tokens of the 16-expert layer: 112 -> 105 us; two of the ring's per CU are slower than two of
// the other kernel's), 64x128 0.30 (one per CU; it only wins while the launch is one or two rounds, i.e. up to
// 128 tokens for the dense FFN and about 200 for the 16-expert layer).  When ragged segments fill 256-row tiles
// poorly, a lower tile with the same number of rounds does less padded work (16 experts at 4096 tokens: 820
// rows are four tiles either way, 387 -> 367 us per forward).
// Up to a model width of 2048 the 64x128 tile runs on the deep ring, two per CU: a K loop of 16 to 32 steps of 64 is
// mostly prologue, which two workgroups share (d = 1024: 32.0 -> 31.2 us per forward at 20 tokens, d = 2048, 777
// tokens: 64.4 -> 61.4; d = 4096 the other way round, 59.6 against 62.4 at 20 tokens).
// The number of row tiles of the routed groups is an estimate, the full ones plus half a tile per touched group; a
// group's last tile is filled uniformly between nothing and everything, so the sum strays by sqrt(groups / 12)
// row tiles: the rounds are averaged over the estimate and two such deviations more (none where every touched group
// has but one row tile).  (A flat margin of 8 % counted a further round where there was none: 32 experts, 2048
// tokens: 294 -> 270 us.)  A hierarchy's shared groups and its sub-experts differ in load and in width and are estimated
// apart, with 2.5 deviations for its outer choice (8 outer experts, top-2 of 6 sub-experts, d = 512, 1998 tokens: 81 -> 70
// us, before the ring 76; d = 1024, 1496 tokens: 92 -> 82; 4 outer experts, d = 2048, 753 tokens: 96 -> 86).
// 256x128 and the ring's 128x128 are taken for single rounds that nearly fill the chip, and there the groups that hold
// more than the average decide: routed loads spread about like an exponential (the library's partitions on clustered
// tokens), a group of mean load m needs a further row tile with probability exp(-bm / m), and the margin is 1.5
// deviations of that.  12 experts, top-1, 1000 tokens: 183 -> 141 us per forward; 32 experts, d = 8192, 298 tokens: 274 -> 209;
// the other way 16 experts, 158 tokens: 110 -> 121.  The other shapes' figures above hold with the plain estimate (with
// this one for all of them 46 of 368 layers and batches changed shape, 26 of them for the worse).
static int gate_up_cfg(const Engine& e, int64_t T) {
  struct Cand { int cfg, bm, bn, slots; double t; };
  const bool single = e.G == 1 && e.n_always == 1;
  const bool narrow = e.d <= 2048;
  const Cand cands[] = {{3, 128, 128, 512, 0.66}, {4, 256, 128, 256, 0.62}, {6, 256, 256, 256, 0.95},
                        {narrow ? 21 : 7, 64, 128, narrow ? 512 : 256, narrow ? 0.45 : 0.30},
                        {9, 224, 256, 256, 0.875}, {10, 192, 256, 256, 0.81}, {19, 160, 256, 256, 0.75}, {20, 128, 128, 256, 0.51}};
  LoadClass classes[2];
  const int n_classes = load_classes(e, T, classes);
  int best = 0;
  double best_t = 1e30;
  for (const Cand& c : cands) {
    // a tile of 160 rows or more for groups that average less than a quarter of it streams its weights at the
    // pace of a full tile (measured with 256 rows at 224-256 tokens on 16 experts: 61 us against 52 us with
    // 128x128)
    if (!single && c.bm >= 160 && T * e.S_dyn * 4 < (int64_t)std::min<int64_t>(e.G - e.n_always, T * e.S_dyn) * c.bm) continue;
    int64_t tiles = 0;
    double var = 0.0;
    for (int g = 0; g < e.n_always; ++g) tiles += ((T + c.bm - 1) / c.bm) * cdiv(2 * e.width_pad_host[g], c.bn);
    for (int i = 0; i < n_classes; ++i) {
      const int64_t entries = classes[i].entries;
      const int64_t touched = std::min<int64_t>(classes[i].groups, entries);
      const int64_t full = (entries + c.bm - 1) / c.bm + touched / 2, rows = std::max<int64_t>(full, touched);
      const double cols = cdiv(2 * classes[i].width_pad, c.bn);
      double dev = 0.0;                                        // tiles
      if (c.cfg == 4 || c.cfg == 20) {
        const double more = std::exp(-(double)c.bm * (double)touched / (double)entries);
        tiles += (int64_t)((double)touched / (1.0 - more) * cols + 0.5);
        dev = 1.5 * std::sqrt((double)touched * std::min(more, 1.0 / 12.0)) * cols;
      } else {
        tiles += (int64_t)((double)rows * cols);
        if (full > touched) dev = (e.r.outer_top_k > 0 ? 2.5 : 2.0) * std::sqrt((double)touched / 12.0) * cols;
      }
      var += dev * dev;
    }
    const int64_t hi = tiles + (int64_t)(std::sqrt(var) + 0.5);
    double t = 0.5 * c.t * (double)((tiles + c.slots - 1) / c.slots + (hi + c.slots - 1) / c.slots);
    // (a short K loop shows more of a tall tile's prologue and epilogue: 8 outer experts, d = 512, 2052 tokens 89 -> 78 us)
    if (narrow && c.bm >= 160 && c.bn == 256) t *= 1.1;
    if (c.cfg == 21 && hi <= 256) t = 0.30;                    // one workgroup on a CU
    // the skinny tile runs one workgroup per CU and its rounds are long: when the estimate is close to
    // spilling into a second, nearly empty round, count that round in full
    if (c.cfg == 7 && !single && tiles <= c.slots && hi > c.slots) t = 2.3 * c.t;      // (above one round of 128x128)
    if (t < best_t) {
      best_t = t;
      best = c.cfg;
    }
  }
  return best;
}

static int64_t est_tiles(const Engine& e, int64_t T, int which, int bm, int bn);

// The persistent down contraction: a work list, and at least as many K steps in every group as its ring is deep.
static bool stream_ok(const Engine& e) {
  if ((e.G == 1 && e.n_always == 1) || !e.w_tiled) return false;
  for (int g = 0; g < e.G; ++g)
    if (e.width_pad_host[g] < 3 * TILE_K) return false;
  return true;
}

// Streamed units instead of a tile: few rows per expert, counted as routed entries per expert times d (q below).  Units of 8
// neurons read the tokens twice as often for the weights they hide them behind, so their line lies lower.  us per forward on
// tiles / streamed, units of 16: d = 2048, 12 experts, top-2, 64 tokens (q 23831) 47.2 / 42.7; d = 2560, 16 experts, top-3, 48
// (24576) 57.7 / 52.6; d = 3072, 16 experts, top-3, 40 (26331) 61.2 / 56.5; d = 4096, 8 experts, top-2, 20 (23405) 72.0 / 70.1;
// 16, top-3, 32 (26214) 70.1 / 69.9, 40 (32768) 76.0 / 77.1; 32 with four shared, top-4, 40 (23405) 83.0 / 82.2, 56 (32768) 89.9 /
// 90.3; d = 5120, 16, top-2, 32 (21845) 91.4 / 88.1; 32, top-5, 24 (20480) 90.0 / 86.8, 32 (27306) 95.9 / 94.7.  Units of 8: d =
// 5632, 16 experts, top-2, 24 tokens (18022) 99.0 / 97.9, 32 (24029) 106.4 / 108.4; d = 6144, 16, top-3, 17 (20889) 87.0 / 80.0, 32
// (39321) 101.9 / 105.0; d = 8192, 8, top-2, 8 (18724) 110.8 / 105.2, 17 (39789) 125.5 / 127.2; 16, top-3, 12 (19660) 104.4 / 101.0,
// 17 (27852) 108.9 / 110.5; 32, top-5, 17 (23210) 105.7 / 102.7, 24 (32768) 112.8 / 113.9.
// Without an always-on group nothing streams beside the selection, and from d = 3584 to 5120 tiles win earlier (at 6144 and 8192
// they do not: q 23040 88.3 / 86.0, 25600 100.7 / 96.1): d = 4096, 8
// experts, top-2, 17 tokens (17408) 67.3 / 70.2; 16, top-4, 17 (17408) 65.3 / 67.1; 32, top-5, 24 (15360) 63.2 / 61.6; d = 3584, 8, top-2,
// 17 (15232) 58.5 / 56.1; d = 5120, 16, top-3, 12 (11520) 77.7 / 73.5, 24 (23040) 85.4 / 85.6; at d = 3072 48 (27648) 59.7 / 57.7.
// A hierarchy's outer experts meet more rows than its groups do on average: 17 tokens 65.3 / 66.1, 64 90 / 97.
static bool streams_small_batch(const Engine& e, int64_t T) {
  if (!stream_gate_up_ok(e, T) || e.r.outer_top_k != 0) return false;
  const int64_t limit = e.n_always == 0 && e.d > 3072 && e.d <= 5120 ? 15500 : stream_neurons(e, T) == 8 ? 23500 : 26500;
  return T * e.S_dyn * e.d <= limit * (int64_t)(e.G - e.n_always);
}

static int choose_cfg(int which, const Engine& e, int64_t T) {
  int dflt = 0;
  if (which == 1) dflt = streams_small_batch(e, T) ? (stream_neurons(e, T) == 8 ? 24 : 23) : gate_up_cfg(e, T);
  if (which == 2) {
    const bool single = e.G == 1 && e.n_always == 1;
    int k_min = 1 << 30;
    for (int g = 0; g < e.G; ++g) k_min = std::min(k_min, e.width_pad_host[g]);
    if (!single && k_min < 2048) {
      // Short K (an expert's width, up to a few tens of K steps per tile; a wider merged shared group next to
      // such experts does not change the picture): rounds x time per round, rounds = ceil(tiles /
      // workgroup slots on the chip).  Measured on 8 to 64 experts of 352 to 1792 neurons, 128 to 8192 tokens:
      // a round of 256 tiles of 256x256 (eight waves, one workgroup per CU) and a round of 512 tiles of 128x256
      // (two per CU) take the same time, a round of 512 tiles of 128x128 two thirds of it.  The 128-row tiles
      // waste less of a ragged segment, and two workgroups on a CU overlap one's epilogue with the other's
      // K loop; a single round of the two-per-CU shape costs 1.4 (both workgroups of a CU start together), a round
      // of 512 tiles of 64x128 on the deep ring 0.42 up to two of them, 0.5 beyond: the shape of batches of tens to a few hundred tokens, where
      // an expert has fewer rows than a taller tile (8 experts of 704 at d = 2048, 512 tokens: 56 -> 48 us per
      // forward; 28 of 448 at d = 4096, 64 tokens: 98.6 -> 93.5).
      const int64_t n0 = est_tiles(e, T, 2, 256, 256), n9 = est_tiles(e, T, 2, 128, 256), n3 = est_tiles(e, T, 2, 128, 128),
                    n21 = est_tiles(e, T, 2, 64, 128);
      const int64_t r0 = (n0 + 255) / 256, r9 = (n9 + 511) / 512, r3 = (n3 + 511) / 512, r21 = (n21 + 511) / 512;
      const double t0 = (double)r0, t9 = (double)r9 + (r9 == 1 ? 0.4 : 0.0), t3 = 0.66 * (double)r3, t21 = (r21 <= 2 ? 0.42 : 0.5) * (double)r21;
      dflt = (t3 < t9 && t3 < t0) ? 3 : (t9 <= t0 ? 8 : 0);
      if (k_min <= 1024 && t21 < std::min(t3, std::min(t9, t0))) dflt = 21;      // (K = 1408: 134 -> 138 us at 64 tokens)
      // The persistent kernel (128x256, two per CU) from 0.8 of a round of tiles on, for narrow experts from 0.44, where the
      // average touched group half fills a row tile.  Below, its lookup of all tiles in advance costs more than it saves
      // (8 experts of 692, d = 2048, 441 tokens, 0.17 rounds: 54 against 65 us; 27 groups of 17 rows: 76 against 89).  From there
      // on, against the shape the models above take: 12 experts of 439, d = 2048, 2295 tokens 94 -> 84 us per forward, 32 of 324 at
      // 603 tokens 119 -> 111, 16 of 300, d = 1536, 3254 tokens 80 -> 75.
      // With a K loop of more than 32 steps of 32 it takes the place of shape 8 only (8 experts of 1357, 5544 tokens: shape 0
      // 415, this one 426, shape 8 430).
      const int64_t entries = T * e.S_dyn, touched = std::min<int64_t>(e.G - e.n_always, entries);
      // In the place of shape 0, a single round of tall tiles, only where K is too short for those or an always-on group at least twice
      // as deep makes their round as long as its own tiles (shape 0 / this one: d = 2048, 8 experts of 692, one of them
      // shared, 2048 tokens 96.8 / 100.9, none, 3000 tokens 104.3 / 109.4, two, 2048 tokens 120.0 / 114.1; 12 of 439, 1400 tokens, one
      // shared 75.3 / 77.9, three 94.7 / 89.7; of 320, one, 70.7 / 71.8; 16 of 256, 1400 tokens 74.9 / 73.0; d = 1024, 16 of 176,
      // 2048 tokens 54.4 / 52.0), and never of shape 21 (d = 2048, 32 experts of 192, 400 tokens 59.9 / 62.4; d = 3072, 12 of
      // 512, 678 tokens 87.5 / 89.0).  What is left of losses against the shape it replaces are single batches between others that
      // gain (d = 8192, 16 of 704, two shared: 678 tokens 242.0 / 236.1, 800 tokens 242.9 / 248.6, 1000 tokens 291.6 / 283.2).
      const int k_max = *std::max_element(e.width_pad_host, e.width_pad_host + e.G);
      const bool in_place = dflt == 3 || dflt == 8 || (dflt == 0 && (k_min <= 256 || k_max >= 2 * k_min));
      if (stream_ok(e) && in_place && entries >= 64 * touched && n9 >= (k_min <= 640 ? 225 : 400) && (k_min <= 1024 || dflt == 8)) dflt = 22;
    } else {
      // Deep K (dense FFN, un-restructured experts): 256x256 tiles with four waves when every CU gets one;
      // below that 256x128, whose round takes 0.56 of the time, unless it would need a second round; 128x128
      // (two workgroups per CU) for batches of a few hundred tokens.
      const int64_t tiles_256 = ((T * e.S_all() + 255) / 256) * ((e.d + 255) / 256), tiles_4 = 2 * tiles_256;
      const int big = e.max_width_pad >= 2048 ? 6 : 0;
      const double t_big = (double)((tiles_256 + 255) / 256), t_4 = 0.56 * (double)((tiles_4 + 255) / 256);
      dflt = (2 * tiles_256 < 256) ? 3 : (t_big <= t_4 ? big : 4);
      if (dflt == 3 && est_tiles(e, T, 2, 128, 128) > 512 && tiles_256 <= 256) dflt = 0;
      // Batches of hundreds of tokens split K (see bf16_splitk); there 128x256 tiles with two workgroups per
      // CU stream the weights faster than 128x128 ones over part of the range (measured: dense FFN at 512 to
      // 1024 tokens 69-114 us against 83-142 us; eight experts of 14336 neurons up to 256 tokens 145-166 us
      // against 195-202 us; slower outside these ranges).
      if (dflt == 3) {
        const int64_t n8 = est_tiles(e, T, 2, 128, 256);
        if (single ? (n8 > 48 && n8 <= 160) : n8 <= 128) dflt = 8;
      }
    }
  }
  const int forced = which == 1 ? tuning().gemm1_cfg : tuning().gemm2_cfg;
  if (which == 1 && e.S_dyn > 0 && wide_gather(e.d, T)) {
    // (of the ring shapes only 6 is built with 64-bit row addresses; the others have them)
    return forced >= 0 && forced < kNumCfgs && !cfg_is_ws(forced) && !cfg_is_ring(forced) && !cfg_is_units(forced) ? forced : 6;
  }
  if (forced >= 0 && forced < kNumCfgs && !(which == 1 && (cfg_is_ws(forced) || cfg_is_stream(forced))) &&
      (!cfg_is_stream(forced) || stream_ok(e)) && (!cfg_is_units(forced) || (which == 1 && stream_gate_up_ok(e, T)))) return forced;
  if (which == 2 && tuning().ws_down != 0 && !(e.G == 1 && e.n_always == 1) && e.w_tiled && e.d % 256 == 0) {
    // The weight-stationary kernel for the groups it handles, when the batch gives it enough work items to
    // fill the chip several times over: the largest row chunk that still leaves four rounds of items (a chunk
    // pays once for loading its strip of weights into registers).  Groups of other widths keep a 128- or
    // 256-row tile of the general kernel over the same list.
    bool any = false, all = true;
    for (int g = 0; g < e.G; ++g) {
      if (ws_down_handles(e.width_pad_host[g])) any = true;
      else all = false;
    }
    if (any) {
      if (all && est_tiles(e, T, 2, 1024, 256) >= 1024) return 18;
      if (all && est_tiles(e, T, 2, 512, 256) >= 1024) return 17;
      if (est_tiles(e, T, 2, 256, 256) >= 1024) return 16;
      if (est_tiles(e, T, 2, 128, 256) >= 768 || tuning().ws_down == 2) return 15;
    }
  }
  return dflt;
}

static int cfg_index(int which, const Engine& e, int64_t T) {
  if (e.plan_T == T) return which == 1 ? e.plan1 : e.plan2;
  return choose_cfg(which, e, T);
}

int bf16_shape(int which, const Engine& e, int64_t T) { return cfg_index(which, e, T); }

void bf16_plan_tiles(Engine& e, int64_t T) {
  e.plan_T = -1;
  if (decode_path_ok(e, T)) return;
  e.plan1 = choose_cfg(1, e, T);
  e.plan2 = choose_cfg(2, e, T);
  e.plan_T = T;
}

bool tiles_gate_up_streams(const Engine& e, int64_t T) {
  return stream_gate_up_ok(e, T) && !decode_path_ok(e, T) && cfg_is_units(cfg_index(1, e, T));
}

// which = 1: BM of gate/up, 2: BM of down, 3: BN of gate/up (packed rows), 4: BN of down,
// 5 / 6: rows per height step when the gate/up / down contraction runs tiles of dynamic height, else 0,
// 7: width of the narrowest group when the down contraction is the persistent one, else 0
int bf16_gemm_tile(int which, const Engine& e, int64_t T) {
  switch (which) {
    case 1: return kCfgs[cfg_index(1, e, T)].bm;
    case 2: return kCfgs[cfg_index(2, e, T)].bm;
    case 3: return kCfgs[cfg_index(1, e, T)].bn;
    case 4: return kCfgs[cfg_index(2, e, T)].bn;
    case 5: return cfg_is_dyn(cfg_index(1, e, T)) ? 32 * kCfgs[cfg_index(1, e, T)].wgm : 0;
    case 7: return cfg_is_stream(cfg_index(2, e, T)) ? *std::min_element(e.width_pad_host, e.width_pad_host + e.G) : 0;
    default: return cfg_is_dyn(cfg_index(2, e, T)) ? 32 * kCfgs[cfg_index(2, e, T)].wgm : 0;
  }
}

// Estimated number of tiles of contraction `which` (1 gate/up, 2 down) with bm x bn tiles: exact for the
// always-on groups, and for the routed groups the full row tiles plus half a tile per touched group.
static int64_t est_tiles(const Engine& e, int64_t T, int which, int bm, int bn) {
  auto cols = [&](int g) { return which == 1 ? cdiv(2 * e.width_pad_host[g], bn) : cdiv(e.d, bn); };
  int64_t tiles = 0;
  for (int g = 0; g < e.n_always; ++g) tiles += ((T + bm - 1) / bm) * cols(g);
  if (e.G > e.n_always && e.S_dyn > 0) {
    const int64_t entries = T * e.S_dyn;
    const int64_t touched = std::min<int64_t>(e.G - e.n_always, entries);
    const int64_t rows = std::max<int64_t>((entries + bm - 1) / bm + touched / 2, touched);
    tiles += rows * cols(e.n_always);
  }
  return tiles;
}

// K split of contraction `which`: with too few tiles to give every CU one (batches of a few hundred
// tokens) several workgroups share a tile.  Powers of two up to 8, at least four K tiles per part, at
// most 64 MB of partial sums.
constexpr size_t SPLITK_MAX_BYTES = 64u << 20;
static int64_t splitk_rows(const Engine& e, int64_t T) { return T * e.S_all(); }
static int splitk_ldp(const Engine& e, int which) { return which == 1 ? 2 * e.max_width_pad : e.d; }

int bf16_splitk(const Engine& e, int64_t T, int which) {
  if (T < 1 || T > 1024 || tuning().splitk == 0) return 1;
  const int ci = cfg_index(which, e, T);
  if (cfg_is_ws(ci) || cfg_is_stream(ci) || cfg_is_units(ci)) return 1;
  const TileCfg& c = kCfgs[ci];
  const int64_t tiles = est_tiles(e, T, which, c.bm, c.bn);
  int k_min = e.d;
  if (which == 2) {
    k_min = 1 << 30;
    for (int g = 0; g < e.G; ++g) k_min = std::min(k_min, e.width_pad_host[g]);
  }
  // (On the deep ring a K tile counts 64 like the other shapes': counted in its steps of 32, parts of 128 were allowed, too
  // short to be worth their partial sums: dense FFN, d = 512, 50 tokens 24.2 -> 21.2 us, 8 experts, d = 1536, 64 tokens
  // 37.5 -> 34.3.)
  const int kt = cdiv(k_min, cfg_is_ring(ci) ? 64 : c.bk);
  const size_t per_part = (size_t)splitk_rows(e, T) * splitk_ldp(e, which) * sizeof(float);
  int ks = 1;
  // Split only while the launch stays well inside one round of workgroups (two tiles of 128 rows fit a CU, one of
  // the larger shapes): measured at 64..512 tokens, splitting a launch that already has a tile for most
  // CUs costs more (partial sums, a second launch) than the shorter K loop saves.
  const int64_t slots = (c.bm == 128 && !cfg_is_ring(ci)) ? 2 : 1;      // (the deep ring's 128x128 counts as one per CU)
  while (ks < 8 && tiles * ks * 2 <= 192 * slots && kt / (ks * 2) >= 4 && per_part * ks * 2 <= SPLITK_MAX_BYTES) ks *= 2;
  return ks;
}

// Bytes to reserve for the partial sums in a workspace for up to T tokens: the cap, because a smaller
// batch may split further than the largest one does.
size_t bf16_splitk_bytes(const Engine& e, int64_t T) {
  (void)e;
  (void)T;
  return SPLITK_MAX_BYTES;
}

// The split a launch may use: the chosen one, unless the slabs would not fit what the workspace reserved.
static int splitk_that_fits(const Engine& e, int64_t T, int which, const WsLayout& L) {
  const int ks = bf16_splitk(e, T, which);
  const size_t per_part = (size_t)splitk_rows(e, T) * splitk_ldp(e, which) * sizeof(float);
  return (ks > 1 && per_part * ks <= L.splitk_bytes) ? ks : 1;
}

// Finish of a K-split gate/up contraction: one workgroup per slot row adds the parts in order and applies
// Swish(g) * u (Eq. 3, first line) with the same arithmetic as the fused epilogue.
__global__ __launch_bounds__(256) void splitk_finish_gate_up(const float* __restrict__ P, int k_split, int64_t p_rows,
                                                             int ldp, const GroupDev* __restrict__ groups,
                                                             const int32_t* __restrict__ seg_off,
                                                             const int64_t* __restrict__ h_off, int G, int single,
                                                             bf16_t* __restrict__ H) {
  const int64_t row = blockIdx.x;
  int g = 0, seg0 = 0;
  int64_t hoff = 0;
  if (!single) {
    g = find_group(seg_off, G, (int)row);       // the group whose slot segment holds this row
    seg0 = seg_off[g];
    hoff = h_off[g];
  }
  const int wp = groups[g].width_pad;
  for (int n = threadIdx.x; n < wp; n += 256) {
    const int gc = (n / IL) * 2 * IL + (n % IL);
    float gt = 0.0f, up = 0.0f;
    for (int k = 0; k < k_split; ++k) {
      const float* prow = P + ((int64_t)k * p_rows + row) * ldp;
      gt += prow[gc];
      up += prow[gc + IL];
    }
    const float sg = gt * __frcp_rn(1.0f + __expf(-gt));
    H[hoff + (row - seg0) * wp + n] = f32_to_bf16(sg * up);
  }
}

// Finish of a K-split down contraction: C[row][c] = sum of the parts, four columns per thread.
__global__ __launch_bounds__(256) void splitk_finish_down(const float* __restrict__ P, int k_split, int64_t p_rows,
                                                          int d, bf16_t* __restrict__ C) {
  const int64_t row = blockIdx.x;
  for (int c = threadIdx.x * 4; c < d; c += 1024) {
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int k = 0; k < k_split; ++k) {
      const float4 v = *reinterpret_cast<const float4*>(P + ((int64_t)k * p_rows + row) * d + c);
      acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
    }
    bf16_t out[4] = {f32_to_bf16(acc.x), f32_to_bf16(acc.y), f32_to_bf16(acc.z), f32_to_bf16(acc.w)};
    *reinterpret_cast<uint2*>(C + row * d + c) = *reinterpret_cast<const uint2*>(out);
  }
}

template <typename K>
static hipError_t launch_kernel(K kern, size_t smem, int threads, LdsLimit& limit, const GemmArgs& a, hipStream_t s) {
  const hipError_t err = limit.raise(reinterpret_cast<const void*>(kern), smem);
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL(kern, dim3((unsigned)a.n_blocks * (unsigned)(a.k_split > 1 ? a.k_split : 1)), dim3(threads), smem, s, a);
  return hipGetLastError();
}

template <int BM, int BN, int BKT, int STAGES, int WGM, int WGN, int MODE, bool DYN = false>
static hipError_t launch_dma(const GemmArgs& a, hipStream_t s) {
  static LdsLimit limit;
  constexpr size_t smem = (STAGES == 0 ? 5 * (size_t)(BM > BN ? BM : BN) : STAGES * (size_t)(BM + BN)) * BKT * sizeof(bf16_t);
  return launch_kernel(grouped_gemm_bf16_dma<BM, BN, BKT, STAGES, WGM, WGN, MODE, DYN>, smem, WGM * WGN * 64, limit, a, s);
}

template <int BM, int BN, int STAGES, int KU, int WGM, int WGN, int MODE, bool WIDE = false>
static hipError_t launch_ring(const GemmArgs& a, hipStream_t s) {
  static LdsLimit limit;
  constexpr size_t smem = ring_smem_bytes(BM, BN, STAGES * KU, WGM * WGN, WGN, MODE);
  static_assert(smem <= 160 * 1024, "LDS of a CU");
  return launch_kernel(grouped_gemm_bf16_ring<BM, BN, STAGES, KU, WGM, WGN, MODE, WIDE>, smem, WGM * WGN * 64, limit, a, s);
}

template <int MODE>
static hipError_t launch_cfg(int ci, const GemmArgs& a, hipStream_t s) {
  switch (ci) {
    case 0: return launch_ring<256, 256, 5, 1, 2, 4, MODE>(a, s);
    case 1: return launch_dma<128, 128, 64, 2, 2, 2, MODE>(a, s);
    case 2: return launch_dma<256, 256, 64, 2, 2, 4, MODE>(a, s);
    case 3: return launch_dma<128, 128, 64, 0, 2, 2, MODE>(a, s);
    case 4: return launch_dma<256, 128, 64, 3, 4, 2, MODE>(a, s);
    case 6:
      if constexpr (MODE == 1)
        if (a.slot2tok && wide_gather(a.d, a.T)) return launch_ring<256, 256, 5, 1, 2, 2, MODE, true>(a, s);
      return launch_ring<256, 256, 5, 1, 2, 2, MODE>(a, s);
    case 7: return launch_dma<64, 128, 64, 4, 2, 2, MODE>(a, s);
    case 8: return launch_dma<128, 256, 32, 3, 2, 2, MODE>(a, s);
    case 9: return launch_ring<224, 256, 5, 1, 2, 2, MODE>(a, s);
    case 10: return launch_dma<192, 256, 64, 0, 1, 4, MODE>(a, s);
    case 11: return launch_dma<256, 256, 64, 0, 1, 4, MODE, true>(a, s);
    case 12: return launch_dma<128, 256, 32, 3, 1, 4, MODE, true>(a, s);
    case 13: return launch_dma<256, 256, 64, 0, 2, 2, MODE, true>(a, s);
    case 14: return launch_dma<128, 256, 32, 3, 2, 2, MODE, true>(a, s);
    case 19: return launch_ring<160, 256, 5, 1, 2, 2, MODE>(a, s);
    case 20: return launch_ring<128, 128, 5, 1, 2, 2, MODE>(a, s);
    case 21: return launch_ring<64, 128, 3, 2, 2, 2, MODE>(a, s);
    default: return launch_dma<256, 256, 32, 4, 2, 4, MODE>(a, s);
  }
}

hipError_t launch_experts_bf16(const Engine& e, const void* x, int64_t T, char* ws, const WsLayout& L, void* y,
                               hipStream_t s, int stage) {
  const int remap = tuning().xcd_remap;
  GemmArgs a;
  a.groups = e.groups;
  a.seg_off = reinterpret_cast<const int32_t*>(ws + L.seg_off);
  a.h_off = reinterpret_cast<const int64_t*>(ws + L.h_off);
  a.G = e.G;
  a.d = e.d;
  a.ldb = e.ldw1;
  a.b_tiled = e.w_tiled;
  a.T = T;
  a.single = (e.G == 1 && e.n_always == 1) ? 1 : 0;
  a.xcd_remap = remap;
  a.zero_pad = tuning().zero_pad;
  a.ws_skip = 0;
  // gate/up
  a.A = static_cast<const bf16_t*>(x);
  a.B = static_cast<const bf16_t*>(e.w1);
  a.C = reinterpret_cast<bf16_t*>(ws + L.h);
  a.work = reinterpret_cast<const int32_t*>(ws + L.work1);
  a.slot2tok = a.single ? nullptr : reinterpret_cast<const int32_t*>(ws + L.slot2tok);
  {
    // An XCD's share of a work list has equal estimated cost, not equal length (see place_lists): with tiles of
    // dynamic height the cheapest tile counts 3 blocks of 32 rows and a full one bm / 32, so the longest share
    // can hold that many times an eighth of the list.
    const int ci = cfg_index(1, e, T);
    const int64_t bound = gemm_work_bound(e, T, 1);
    int64_t share = (bound + 7) / 8;
    if (remap && !a.single) share = std::min<int64_t>(bound, share + 1);   // (a boundary inside a group is rounded)
    if (cfg_is_dyn(ci) && remap && !a.single) {
      const int full = kCfgs[ci].bm / 32, low = std::min(full, 3);
      share = std::min<int64_t>(bound, (bound * full + 8 * low - 1) / (8 * low) + 2);
    }
    a.n_blocks = (int)(8 * share);
  }
  a.P = reinterpret_cast<float*>(ws + L.splitk);
  a.p_rows = splitk_rows(e, T);
  a.k_split = splitk_that_fits(e, T, 1, L);
  a.ldp = splitk_ldp(e, 1);
  if (stage != 2) {
    const int ci = cfg_index(1, e, T);
    hipError_t err = cfg_is_units(ci) ? launch_stream_gate_up(e, x, T, ws, L, ci == 24 ? 8 : 16, a.n_blocks, s) : launch_cfg<1>(ci, a, s);
    if (err == hipSuccess && a.k_split > 1) {
      hipLaunchKernelGGL(splitk_finish_gate_up, dim3((unsigned)a.p_rows), dim3(256), 0, s, a.P, a.k_split, a.p_rows, a.ldp,
                         a.groups, a.seg_off, a.h_off, a.G, a.single, a.C);
      err = hipGetLastError();
    }
    if (err != hipSuccess || stage == 1) return err;
  }
  // down
  a.A = reinterpret_cast<const bf16_t*>(ws + L.h);
  a.B = static_cast<const bf16_t*>(e.w2);
  a.C = e.direct_output() ? static_cast<bf16_t*>(y) : reinterpret_cast<bf16_t*>(ws + L.y_slots);
  a.work = reinterpret_cast<const int32_t*>(ws + L.work2);
  a.slot2tok = nullptr;
  {
    // An XCD's share of the down list has equal cost, not equal length: with groups of unequal width the
    // share made of the cheapest tiles is longer than an eighth of the list.
    const int64_t bound = gemm_work_bound(e, T, 2);
    int c_min = 1 << 30, c_max = 1;
    const int ci2 = cfg_index(2, e, T);
    const int full2 = kCfgs[ci2].bm / 32, low2 = cfg_is_dyn(ci2) ? std::min(full2, 3) : full2;
    for (int g = 0; g < e.G; ++g) {
      const int c = cdiv(e.width_pad_host[g], 64) + 4;
      c_min = std::min(c_min, c * low2);
      c_max = std::max(c_max, c * full2);
    }
    const int64_t share = std::min<int64_t>(bound, (bound * c_max + 8 * c_min - 1) / (8 * c_min) + 2);
    a.n_blocks = (int)(remap && !a.single ? 8 * share : round_up64(bound, 8));
  }
  a.k_split = splitk_that_fits(e, T, 2, L);
  a.ldp = splitk_ldp(e, 2);
  {
    const int ci2 = cfg_index(2, e, T);
    if (cfg_is_stream(ci2)) return launch_down_stream(e, a, s);
    if (cfg_is_ws(ci2)) {
      bool wide = false;
      for (int g = 0; g < e.G; ++g) wide = wide || !ws_down_handles(e.width_pad_host[g]);
      hipError_t err = hipSuccess;
      if (wide) {
        a.ws_skip = 1;
        a.k_split = 1;
        err = launch_cfg<2>(kCfgs[ci2].bm == 128 ? 8 : 6, a, s);
      }
      if (err == hipSuccess) err = launch_ws_down(e, ws, L, a.C, kCfgs[ci2].bm, a.n_blocks, a.xcd_remap, s);
      return err;
    }
  }
  hipError_t err = launch_cfg<2>(cfg_index(2, e, T), a, s);
  if (err == hipSuccess && a.k_split > 1) {
    hipLaunchKernelGGL(splitk_finish_down, dim3((unsigned)a.p_rows), dim3(256), 0, s, a.P, a.k_split, a.p_rows, e.d, a.C);
    err = hipGetLastError();
  }
  return err;
}

}  // namespace cmoe
