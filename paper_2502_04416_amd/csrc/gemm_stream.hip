// Persistent down contraction of the routed layers: Y_g = H_g Wdown_g on the tiles of all groups, K = width_pad(g).
//
// What bounds it.  An expert's width is 11 to 56 K steps of 32, so a workgroup per tile spends most of its life outside
// the K loop (finding its tile, three dependent round trips; waiting for its first operands; staging the result through
// LDS), and the result it writes is as large as the operands it reads: 470 MB at 8192 tokens of seven slots, d = 4096.
//   * Two workgroups stay on every CU and walk strided parts of the work list; the K steps of a workgroup's tiles
//     form one sequence, the transfers run STAGES steps ahead of the multiplication across tile boundaries, and between two
//     tiles a workgroup does nothing but convert and store, while the CU's other one multiplies.
//   * Results go from the registers to memory: the weight rows are dealt to the MFMA's columns such that a lane holds
//     eight consecutive output columns and a store covers 256 bytes of each of four rows.  (16 rows of 64 bytes per store
//     are written at 34 GB/s per CU, 4 rows of 256 at 90.)
//   * The stores go through the caches, where the combine kernel finds what the last level could hold, unless all results
//     together are about as small as the L2s or larger than the last level can use (SLOTS_NT_BYTES, SLOTS_NT_FROM): then they are
//     non-temporal.
// Launches, 128x256 tiles of the other kernel (two per CU, a workgroup per tile) -> this one: 2048 tokens of the 16-expert
// layer 73.8 -> 71.1 us, 4096 of the 32-expert layer with four shared 152 -> 144, 8192 of the 32-expert layer 276 -> 265, 4096
// of the hierarchy 530 -> 523 (its K loops are long, and its time is theirs).
#include <algorithm>
#include <type_traits>
#include "cmoe_internal.h"
#include "device_utils.h"
#include "gemm_device.h"
#include "lds_limit.h"

namespace cmoe {

typedef unsigned int uintx4_t __attribute__((ext_vector_type(4)));

// acc = a * w: the first step of a tile.
__device__ __forceinline__ void mfma_first(floatx4_t& acc, const bf16x8_t& a, const bf16x8_t& w) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(acc) : "v"(a), "v"(w));
}

// Slot outputs up to the first size are stored past the caches: plain stores leave them dirty in the L2s, to be written back between
// this launch and the combine kernel.  us per forward, plain / non-temporal: d = 1024, 25 MB 59.0 / 58.0; d = 2048, 18 MB 81.0 /
// 80.3, 29 MB 75.5 / 74.6, 43 MB 85.0 / 82.9, 59 MB 95.0 / 95.1, 117 MB 163.5 / 166.6; d = 4096, 33 MB 149.7 / 149.5, 49 MB 194.5 /
// 195.9, 67 MB 231 / 233, 117 MB 223.2 / 228.2, 168 MB 457 / 460, 234 MB 398.2 / 403.0.  In between the last-level cache holds enough of
// them to pay the combine launch back what non-temporal stores give this one (67 MB 71.2 + 15.8 for 71.1 + 13.8); beyond the second
// size it does not: 352 MB 555.7 / 558.2 and (d = 2048) 405.4 / 411.4, 402 MB 931.4 / 934.8 and (d = 8192) 679.2 / 678.1 and 997.2 / 990.7,
// 469 MB 735.5 / 734.1 (on another box 760.8 / 749.7), 503 MB 1148.5 / 1145.9, 587 MB 888.7 / 879.4.
constexpr int64_t SLOTS_NT_BYTES = (int64_t)45 << 20, SLOTS_NT_FROM = (int64_t)380 << 20;

// 16 bytes to base + lane_off (bytes; dropped where lane_off >= size).  Lanes without a target still issue the store, so
// that the number of memory instructions of a wave is the same for every tile (see wait counts below).
template <bool NT>
__device__ __forceinline__ void store16_buffer(const bf16_t* base, uint32_t size, uint32_t lane_off, uintx4_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(base), 0, size, 0x00020000);
  __builtin_amdgcn_raw_buffer_store_b128(v, rsrc, lane_off, 0, NT ? 2 : 0);   // 2: non-temporal
#endif
}

// An accumulator from the AGPRs.  (Left to itself the register allocator fetches all of a tile's at once, and spills.)
__device__ __forceinline__ float read_acc(float acc) {
  float f;
  asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(f) : "a"(acc));
  return f;
}

__device__ __forceinline__ uintx4_t pack8(const floatx4_t& lo, const floatx4_t& hi) {
  typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
  struct { bf16x4_t l, h; } v = {__builtin_convertvector(lo, bf16x4_t), __builtin_convertvector(hi, bf16x4_t)};
  return __builtin_bit_cast(uintx4_t, v);
}

// A value the compiler cannot carry over from an earlier use: what is computed from it is computed again.
template <typename T>
__device__ __forceinline__ T opaque(T v) {
  asm volatile("" : "+v"(v));
  return v;
}

__device__ __forceinline__ uint32_t lds_addr(const bf16_t* ptr) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) bf16_t*)ptr;
}
__device__ __forceinline__ bf16x8_t lds_read16(uint32_t addr) {
  return *(const __attribute__((address_space(3))) bf16x8_t*)(uintptr_t)addr;
}

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

constexpr int BM = 128, BN = 256, STAGES = 3;

// A tile of the work list, looked up ahead of its time by one lane for 64 tiles of its workgroup.
struct TileLane {
  int wp, rows, nt, pad;                                       // K, rows of the tile that exist, column tile
  int64_t a, b, c;                                             // element offsets of its operands and its result
};

__device__ __forceinline__ TileLane decode_tile(const GemmArgs& p, int item) {
  const int lane = threadIdx.x & 63, n_nt = (p.d + BN - 1) / BN;
  // Two groups per lane: their first tile and how many they have (the list is not in the order of the groups).
  int from[2], n[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int g = lane + 64 * k;
    from[k] = g < p.G ? p.work[g] : 0;
    n[k] = g < p.G ? (p.seg_off[g + 1] - p.seg_off[g] + BM - 1) / BM * n_nt : 0;
  }
  int g = 0, local = 0;
  auto look = [&](int i, int from_k, int n_k) {
    const int at = item - __builtin_amdgcn_readlane(from_k, i & 63);
    const bool in = (unsigned)at < (unsigned)__builtin_amdgcn_readlane(n_k, i & 63);
    g = in ? i : g;
    local = in ? at : local;
  };
  for (int i = 0; i < p.G && i < 64; ++i) look(i, from[0], n[0]);
  for (int i = 64; i < p.G; ++i) look(i, from[1], n[1]);
  const int seg0 = p.seg_off[g], cnt = p.seg_off[g + 1] - seg0;
  const GroupDev gd = p.groups[g];
  const int64_t hoff = p.h_off[g];
  const int n_mt = (cnt + BM - 1) / BM;
  constexpr int GM = 8;                                        // row tiles fastest, in super-rows of 8
  const int sr = local / (GM * n_nt), rem = local - sr * (GM * n_nt);
  const int rows_in_sr = (n_mt - sr * GM) < GM ? (n_mt - sr * GM) : GM;
  const int mt = sr * GM + rem % rows_in_sr, nt = rem / rows_in_sr;
  TileLane t;
  t.wp = gd.width_pad;
  t.rows = cnt - mt * BM < BM ? cnt - mt * BM : BM;
  t.nt = nt;
  t.pad = 0;
  t.a = hoff + (int64_t)mt * BM * gd.width_pad;
  t.b = gd.w2_off + (int64_t)nt * (BN / 16) * (gd.width_pad / TILE_K) * TILE_ELEMS;
  t.c = (int64_t)(seg0 + mt * BM) * p.d + nt * BN;
  return t;
}

// Every group's K must hold at least STAGES steps (then the transfers are never more than one tile ahead of the
// multiplication).
template <bool NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void down_stream_kernel(GemmArgs p) {
  constexpr int NW = 4, WGN = 2;
  constexpr int TM = BM / 2, TN = BN / 2, MB = TM / 16, NB = TN / 16;
  constexpr int A_CH = BM / 16 / NW, B_CH = BN / 16 / NW, ND = A_CH + B_CH;   // transfers per wave and step
  constexpr int A_ELEMS = BM * BK, STAGE_ELEMS = (BM + BN) * BK;
  constexpr int NST = MB * 4;                                 // stores per wave and tile
  static_assert(BM % (16 * NW) == 0 && BN % (16 * NW) == 0 && NB == 8 && STAGES >= 3, "tile");
  static_assert((STAGES - 2) * ND + NST < 64 && (STAGES - 1) * ND < 64, "wait counts");
  extern __shared__ __attribute__((aligned(1024))) bf16_t smem[];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  const int r16 = lane & 15, kq = lane >> 4;

  // Which tiles.  The list holds the deep tiles (an always-on group's K is several experts wide), then the others.
  // Workgroup b runs on XCD b % 8 (own L2); each die gets a contiguous eighth of either part, so that the tiles in work
  // at one time are neighbours that share operands.  Inside a die the tiles are dealt in turn, deep ones first; where they
  // do not divide evenly, the workgroups without a last deep tile take deep_rounds others before the dealing goes on
  // with all.  (Contiguous shares of equal estimated cost left three dies with nothing but deep tiles, two or
  // three to a workgroup.)
  const int n_dies = p.xcd_remap ? 8 : 1, die = blockIdx.x % n_dies, me = blockIdx.x / n_dies, team = gridDim.x / n_dies;
  const int n_deep = p.work[p.G + 1], n_rest = p.work[p.G] - n_deep;
  const int deep0 = n_deep * die / n_dies, deep_n = n_deep * (die + 1) / n_dies - deep0;
  const int rest0 = (int)((int64_t)n_rest * die / n_dies), rest_n = (int)((int64_t)n_rest * (die + 1) / n_dies) - rest0;
  const int deep_more = deep_n % team;                         // workgroups with one deep tile more than the others
  const int my_deep = deep_n / team + (me < deep_more ? 1 : 0);
  const int waiting = deep_more > 0 ? team - deep_more : 0, lead = deep_more > 0 && me >= deep_more ? p.deep_rounds : 0;
  auto tile_at = [&](int j) {                                  // this workgroup's j-th tile, -1 past its last
    if (j < my_deep) return deep0 + me + j * team;
    j -= my_deep;
    const int i = j < lead ? j * waiting + me - deep_more : p.deep_rounds * waiting + (j - lead) * team + me;
    return i < rest_n ? rest0 + n_deep + i : -1;
  };

  // Sources: a transfer fills a block of 16 rows x 32 K (1 KB), lane l the 16-byte chunk at 16 l.  The activation blocks
  // are those of the deep ring (gemm_bf16.hip): chunk l % 4 of row l / 4 holds chunk (l % 4) ^ (row >> 2) & 3 of the row.
  // Weights: the MFMA's column r of block nb is to be column 8 r + nb of the wave's 128, so a read of block nb touches rows
  // nb and 8 + nb of all eight 16-row blocks beta.  Row 8 h + e of block beta therefore lies in row 8 h + (e ^ beta), which
  // makes the 64 chunks of a read cover a whole 1 KB of banks, as they do for the activations.
  TileLane* table = reinterpret_cast<TileLane*>(smem + STAGES * STAGE_ELEMS);
  const bf16_t *a_base = nullptr, *b_base = nullptr, *c_next = nullptr;
  uint32_t a_size = 0, b_size = 0;
  uint32_t a_off[A_CH], b_off[B_CH];
  int n_items = 0, fetch_item = 0, fetch_k = 0, fetch_kt = 0;               // the transfers' place in the sequence
  int kt_next = 0, rows_next = 0, nt_next = 0;                 // the tile behind the one being multiplied
  auto fetch_tile = [&]() __attribute__((always_inline)) {                                    // the transfers go on to tile fetch_item
    fetch_k = 0;
    if (fetch_item >= n_items) {                               // nothing left: zeros into slots that nobody reads
      a_size = b_size = 0;
      fetch_kt = 0x7fffffff;
      return;
    }
    const TileLane t = table[fetch_item];
    const int wp = uniform(t.wp), kt = wp / BK;
    rows_next = uniform(t.rows);
    nt_next = uniform(t.nt);
    a_base = uniform_ptr(p.A + t.a);
    b_base = uniform_ptr(p.B + t.b);
    c_next = uniform_ptr(p.C + t.c);
    kt_next = fetch_kt = kt;
    // rows past the end of the segment and column blocks past the end of the matrix lie past these sizes
    a_size = (uint32_t)(rows_next * wp * 2);
    const int blks = (p.d + 15) / 16 - nt_next * (BN / 16);
    b_size = (uint32_t)((blks < BN / 16 ? blks : BN / 16) * kt * TILE_ELEMS * 2);
    const int l = opaque(lane), row = l >> 2, chunk = ((l & 3) ^ ((l >> 4) & 3)) * 16;
#pragma unroll
    for (int i = 0; i < A_CH; ++i) {
      const int blk = wave + i * NW;
      a_off[i] = (uint32_t)((blk * 16 + row) * wp * 2 + chunk);
    }
#pragma unroll
    for (int i = 0; i < B_CH; ++i) {
      const int blk = wave + i * NW;
      b_off[i] = (uint32_t)(blk * kt * TILE_ELEMS * 2 + (row ^ (blk & 7)) * (TILE_K * 2) + chunk);
    }
  };
  auto issue = [&](int slot, int i) __attribute__((always_inline)) {                          // transfer i of step fetch_k
    bf16_t* st = smem + slot * STAGE_ELEMS;
    if (i < A_CH) dma16_buffer(a_base, a_size, a_off[i], (uint32_t)fetch_k * (BK * 2), st + (wave + i * NW) * BLK);
    else dma16_buffer(b_base, b_size, b_off[i - A_CH], (uint32_t)fetch_k * (TILE_ELEMS * 2), st + A_ELEMS + (wave + (i - A_CH) * NW) * BLK);
  };

  floatx4_t acc[MB][NB];
  bf16x8_t af[2][MB], wf[2][NB];
  const uint32_t a_frag = lds_addr(smem) + (wm * MB * BLK + r16 * BK + ((kq ^ (r16 >> 2)) << 3)) * 2;
  // block 0's row 8 (r16 & 1) of block beta = r16 / 2; the other blocks differ in bits (see the sources)
  const uint32_t w_frag = lds_addr(smem) + (A_ELEMS + wn * NB * BLK + (r16 >> 1) * BLK + ((8 * (r16 & 1)) ^ (r16 >> 1)) * BK +
                                            ((kq ^ (2 * (r16 & 1)) ^ (r16 >> 3)) << 3)) * 2;
  constexpr int NM = MB * NB, NF = MB + NB;                    // MFMAs and LDS reads per step
  uint32_t a_at, w_at;                                         // a lane's place in the slot that is read
  auto read_slot = [&](int slot) __attribute__((always_inline)) {
    // (opaque: the eight addresses a step derives from it would be kept in registers otherwise)
    a_at = opaque(a_frag + (uint32_t)slot * (STAGE_ELEMS * 2));
    w_at = opaque(w_frag + (uint32_t)slot * (STAGE_ELEMS * 2));
  };
  auto load_frag = [&](int f, int set) __attribute__((always_inline)) {      // weights first
    if (f < NB) wf[set][f] = lds_read16(w_at ^ (uint32_t)(f * BK * 2 + ((f >> 2) << 4)));
    else af[set][f - NB] = lds_read16(a_at + (uint32_t)((f - NB) * BLK * 2));
  };

  using std::integral_constant;
  using std::false_type;
  using std::true_type;
  // (a list that gives a workgroup more than 64 tiles is walked in runs of 64)
  for (int run = 0;; run += 64) {
  const int mine = tile_at(run + lane);
  n_items = __popcll(__ballot(mine >= 0));
  if (n_items == 0) break;
  if (wave == 0) table[lane] = decode_tile(p, mine >= 0 ? mine : 0);
  __syncthreads();
  fetch_item = 0;
  fetch_tile();
#pragma unroll
  for (int st = 0; st < STAGES; ++st) {
#pragma unroll
    for (int i = 0; i < ND; ++i) issue(st, i);
    ++fetch_k;
  }
  wait_vmcnt<(STAGES - 1) * ND>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  read_slot(0);
#pragma unroll
  for (int f = 0; f < NF; ++f) load_frag(f, 0);

  int slot = 0;                                                // of the current step
  // One K step.  SET: fragment registers it reads.  FIRST: of its tile.  after_stores: one of the STAGES - 1 first steps
  // behind an epilogue, whose stores are younger than the transfers waited for.
  auto step = [&](auto set_tag, auto first_tag, bool after_stores) __attribute__((always_inline)) {
    constexpr int SET = decltype(set_tag)::value;
    constexpr bool FIRST = decltype(first_tag)::value;
    if (fetch_k == fetch_kt) {
      ++fetch_item;
      fetch_tile();
    }
    // Bare barrier, as in the deep ring: this wave's parts of the next step have landed (vmcnt) and its LDS reads of
    // this step have returned, so behind it the next step can be read and this step's slot refilled.
    if (after_stores) wait_vmcnt<(STAGES - 2) * ND + NST>();
    else wait_vmcnt<(STAGES - 2) * ND>();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    const int next = slot + 1 == STAGES ? 0 : slot + 1;
    read_slot(next);
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      const int mb = m / NB, nb = m % NB;
      __builtin_amdgcn_sched_barrier(0);
      if (FIRST) mfma_first(acc[mb][nb], af[SET][mb], wf[SET][nb]);
      else if (m == NM - 1) mfma_acc<true>(acc[mb][nb], af[SET][mb], wf[SET][nb]);   // (a tile may end here)
      else mfma_acc<false>(acc[mb][nb], af[SET][mb], wf[SET][nb]);
      __builtin_amdgcn_sched_barrier(0);
      // memory instructions spread over the MFMAs: fragment f of the next step follows MFMA f * (3/4 NM) / NF, transfer i
      // MFMA (i + 1) * NM / ND - 1
      const int f = (m * NF * 4 + NM * 3 - 1) / (NM * 3);
      if (f < NF && f * NM * 3 / (NF * 4) == m) load_frag(f, SET ^ 1);
      const int i = ((m + 1) * ND + NM - 1) / NM - 1;
      if (i < ND && (i + 1) * NM / ND - 1 == m) issue(slot, i);
    }
    __builtin_amdgcn_sched_barrier(0);
    ++fetch_k;
    slot = next;
  };
  // One flat sequence of steps over the tiles of the run, in pairs (the two sets of fragment registers); a tile ends where it ends.
  int k = 0, kt = kt_next, rows = rows_next, nt = nt_next, done = 0;
  const bf16_t* c_base = c_next;
  // The tile's rows from the registers: a lane holds columns 8 r16 .. + 7 of rows 4 kq .. + 3 of every 16-row block, so a
  // store covers 256 consecutive bytes of four rows.
  auto epilogue = [&]() __attribute__((always_inline)) {
    const uint32_t c_size = (uint32_t)(rows * p.d) * 2u;
    const int l = opaque(lane), row_bytes = p.d * 2, col = wn * TN + (l & 15) * 8;
    uint32_t off = nt * BN + col < p.d ? (uint32_t)((wm * TM + (l >> 4) * 4) * row_bytes + col * 2) : DMA_NONE;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const floatx4_t lo = {read_acc(acc[mb][0][i]), read_acc(acc[mb][1][i]), read_acc(acc[mb][2][i]), read_acc(acc[mb][3][i])};
        const floatx4_t hi = {read_acc(acc[mb][4][i]), read_acc(acc[mb][5][i]), read_acc(acc[mb][6][i]), read_acc(acc[mb][7][i])};
        store16_buffer<NT>(c_base, c_size, off + (uint32_t)(i * row_bytes), pack8(lo, hi));
        __builtin_amdgcn_sched_barrier(0);
      }
      off += (uint32_t)(16 * row_bytes);
    }
  };
  auto pass = [&](auto set_tag) __attribute__((always_inline)) {
    const bool after_stores = done > 0 && k < STAGES - 1;
    if (k == 0) step(set_tag, true_type{}, after_stores);
    else step(set_tag, false_type{}, after_stores);
    if (++k < kt) return true;
    epilogue();
    if (++done == n_items) return false;
    k = 0;
    kt = kt_next;
    rows = rows_next;
    nt = nt_next;
    c_base = c_next;
    return true;
  };
  while (pass(integral_constant<int, 0>{}) && pass(integral_constant<int, 1>{})) {}
  wait_vmcnt<0>();                                             // (no transfer into LDS may outlive the run)
  __syncthreads();
  }
}

template <bool NT>
static hipError_t launch_form(const GemmArgs& a, hipStream_t s) {
  static LdsLimit limit;
  constexpr size_t smem = (size_t)STAGES * (BM + BN) * BK * sizeof(bf16_t) + 64 * sizeof(TileLane);
  static_assert(2 * smem <= 160 * 1024, "two workgroups on a CU");
  const hipError_t err = limit.raise(reinterpret_cast<const void*>(down_stream_kernel<NT>), smem);
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL(down_stream_kernel<NT>, dim3((unsigned)std::min(a.n_blocks, 512)), dim3(256), smem, s, a);
  return hipGetLastError();
}

bool down_stream_past_caches(const Engine& e, int64_t T) {
  const int64_t bytes = T * e.S_all() * e.d * (int64_t)sizeof(bf16_t);
  return bytes <= SLOTS_NT_BYTES || bytes > SLOTS_NT_FROM;
}

hipError_t launch_down_stream(const Engine& e, const GemmArgs& args, hipStream_t s) {
  GemmArgs a = args;
  // a tile costs its K steps and about six more
  const auto width = std::minmax_element(e.width_pad_host, e.width_pad_host + e.G);
  const int deep = *width.second / BK + 6, rest = *width.first / BK + 6;
  a.deep_rounds = (deep + rest / 2) / rest;
  return down_stream_past_caches(e, a.T) ? launch_form<true>(a, s) : launch_form<false>(a, s);
}

}  // namespace cmoe
