// Pieces of the decode kernels that more than one translation unit launches: the argument block and the
// gate/up contraction of one 16-neuron unit (the routing front end runs the shared expert's units in the
// launch that selects and places the tokens).
#pragma once
#include <type_traits>
#include "cmoe_internal.h"
#include "device_utils.h"

namespace cmoe {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float floatx4_t __attribute__((ext_vector_type(4)));

struct DecArgs {
  const bf16_t* x;          // [T][d]
  const bf16_t* w1;
  const bf16_t* w2;
  bf16_t* h;                // ragged hidden activations
  bf16_t* y;                // per-slot outputs [n_slots][d] (or y itself when every token has one slot)
  const GroupDev* groups;
  const int32_t* seg_off;
  const int32_t* work;      // [G+1] prefix of units
  const int64_t* h_off;
  const int32_t* slot2tok;
  int G, d;
  int ldw;                  // elements per row of w1
  int tiled;                // 1: w1 and w2 are tiled 16 x 32: the weights of one operand are 1 KB of consecutive memory
  int64_t T;
  int single;
  int unit1;                // neurons per gate/up unit: 16 or 8
  int x_row, x_step;        // stream_gate_up_unit: elements from one token to the next and from one K step of 32 to the next
  int nch;                  // a wave's K slice in runs of KSTEPS steps of 32: d = 8 * KSTEPS * 32 * nch (1 but for the _runs forms)
};

__device__ __forceinline__ bf16x8_t ld_frag(const bf16_t* p) { return *reinterpret_cast<const bf16x8_t*>(p); }
__device__ __forceinline__ bf16x8_t zero_frag() {
  bf16x8_t z;
#pragma unroll
  for (int i = 0; i < 8; ++i) z[i] = (__bf16)0.0f;
  return z;
}

// Shared memory a workgroup needs for decode_gate_up_unit.
template <int NTT>
struct DecGateUpRed { float v[8][2][NTT][16][17]; };

// H[slot][n] = Swish(x . wgate_n) * (x . wup_n) for the 16 neurons [local*16, local*16+16) of the group at packed row w1_row0, whose
// cnt <= 16*NTT tokens are the slots seg0 .. seg0+cnt-1 and whose rows of H start at element hoff.
// Called by all 512 threads of a workgroup: 8 waves, wave w multiplies the K slice [w*d/8, (w+1)*d/8).
// NTT = token tiles of 16.  KSTEPS = d/8/32.  The _runs forms below take a wave's slice in p.nch runs of KSTEPS steps
// (d above 4096: the operands of the whole slice would leave room for one workgroup per CU); as one loop for both
// cases the code of the single run came out 5-8 % slower (62 -> 67 us at 16 tokens, d = 4096).
template <int NTT, int KSTEPS>
__device__ __forceinline__ void decode_gate_up_unit(const DecArgs& p, int w1_row0, int local, int seg0, int cnt, int wp,
                                                    int64_t hoff, DecGateUpRed<NTT>& redbuf) {
  float (*red)[2][NTT][16][17] = redbuf.v;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r16 = lane & 15, kq = lane >> 4;
  const int neuron0 = local * 16;
  const int kbase = wave * (KSTEPS * 32) + kq * 8;
  // weight rows of this lane: packed row = (n / IL) * 2 * IL + n % IL (+ IL for the up row)
  const int n = neuron0 + r16;
  const int64_t grow = (int64_t)w1_row0 + (n / IL) * 2 * IL + (n % IL);
  // (grow is a multiple of 16 plus lane%16, kbase a multiple of 32 plus (lane/16)*8: one tile per K step)
  const bf16_t* wg = p.w1 + (p.tiled ? tiled_offset(grow, kbase, p.ldw / TILE_K) : grow * p.ldw + kbase);
  const bf16_t* wu = wg + (p.tiled ? (int64_t)(IL / TILE_ROWS) * (p.ldw / TILE_K) * TILE_ELEMS : (int64_t)IL * p.ldw);
  const int kadv = p.tiled ? TILE_ELEMS : 32;                 // elements from one K step's operand to the next
  // The gate rows of the unit are requested before anything else (the stream from HBM is what the kernel
  // waits for; left to itself the compiler keeps half a dozen weight loads in flight per wave), the up rows
  // as the loop goes.  Requesting those up front as well costs a third workgroup per CU and gains nothing.
  // (Loads return in order: the wait for the token index below is one for the gate rows, and the up rows follow the tokens.)
  bf16x8_t ag[KSTEPS];
#pragma unroll
  for (int ks = 0; ks < KSTEPS; ++ks) ag[ks] = ld_frag(wg + ks * kadv);
  __builtin_amdgcn_sched_barrier(0);
  // tokens (B operand), kept for the whole unit
  bf16x8_t bx[NTT][KSTEPS];
#pragma unroll
  for (int tt = 0; tt < NTT; ++tt) {
    const int col = tt * 16 + r16;
    const bool ok = col < cnt;
    int64_t tok = 0;
    if (ok) tok = p.slot2tok ? p.slot2tok[seg0 + col] : (seg0 + col);
    const bf16_t* xr = p.x + tok * p.d + kbase;
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) bx[tt][ks] = ok ? ld_frag(xr + ks * 32) : zero_frag();
  }
  floatx4_t accg[NTT], accu[NTT];
#pragma unroll
  for (int tt = 0; tt < NTT; ++tt)
#pragma unroll
    for (int i = 0; i < 4; ++i) { accg[tt][i] = 0.0f; accu[tt][i] = 0.0f; }
#pragma unroll
  for (int ks = 0; ks < KSTEPS; ++ks) {
    const bf16x8_t au = ld_frag(wu + ks * kadv);
#pragma unroll
    for (int tt = 0; tt < NTT; ++tt) {
      accg[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ag[ks], bx[tt][ks], accg[tt], 0, 0, 0);
      accu[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(au, bx[tt][ks], accu[tt], 0, 0, 0);
    }
  }
  // accumulator element i: neuron row (lane/16)*4 + i, token column lane%16
#pragma unroll
  for (int tt = 0; tt < NTT; ++tt)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      red[wave][0][tt][kq * 4 + i][r16] = accg[tt][i];
      red[wave][1][tt][kq * 4 + i][r16] = accu[tt][i];
    }
  __syncthreads();
  for (int e = tid; e < NTT * 256; e += 512) {
    const int tt = e >> 8, tok = (e >> 4) & 15, nn = e & 15;     // neuron fastest: contiguous stores
    const int col = tt * 16 + tok;
    if (col >= cnt) continue;
    float sg = 0.0f, su = 0.0f;
#pragma unroll
    for (int w = 0; w < 8; ++w) { sg += red[w][0][tt][nn][tok]; su += red[w][1][tt][nn][tok]; }
    p.h[hoff + (int64_t)col * wp + neuron0 + nn] = f32_to_bf16(silu_f32(sg) * su);
  }
}

template <int NTT, int KSTEPS>
__device__ __forceinline__ void decode_gate_up_unit_runs(const DecArgs& p, int w1_row0, int local, int seg0, int cnt, int wp,
                                                    int64_t hoff, DecGateUpRed<NTT>& redbuf) {
  float (*red)[2][NTT][16][17] = redbuf.v;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r16 = lane & 15, kq = lane >> 4;
  const int neuron0 = local * 16;
  const int kbase = wave * (KSTEPS * 32 * p.nch) + kq * 8;
  // weight rows of this lane: packed row = (n / IL) * 2 * IL + n % IL (+ IL for the up row)
  const int n = neuron0 + r16;
  const int64_t grow = (int64_t)w1_row0 + (n / IL) * 2 * IL + (n % IL);
  // (grow is a multiple of 16 plus lane%16, kbase a multiple of 32 plus (lane/16)*8: one tile per K step)
  const bf16_t* wg = p.w1 + (p.tiled ? tiled_offset(grow, kbase, p.ldw / TILE_K) : grow * p.ldw + kbase);
  const bf16_t* wu = wg + (p.tiled ? (int64_t)(IL / TILE_ROWS) * (p.ldw / TILE_K) * TILE_ELEMS : (int64_t)IL * p.ldw);
  const int kadv = p.tiled ? TILE_ELEMS : 32;                 // elements from one K step's operand to the next
  int64_t xoff[NTT];                                          // tokens (B operand), gathered
  bool ok[NTT];
  floatx4_t accg[NTT], accu[NTT];
#pragma unroll
  for (int tt = 0; tt < NTT; ++tt) {
    const int col = tt * 16 + r16;
    ok[tt] = col < cnt;
    xoff[tt] = -1;                                            // (looked up behind the first weight loads)
#pragma unroll
    for (int i = 0; i < 4; ++i) { accg[tt][i] = 0.0f; accu[tt][i] = 0.0f; }
  }
  int ch = 0;
  do {
    // The gate rows of the unit are requested before anything else (the stream from HBM is what the kernel
    // waits for; left to itself the compiler keeps half a dozen weight loads in flight per wave), the up rows
    // as the loop goes.  Requesting those up front as well costs a third workgroup per CU and gains nothing.
    bf16x8_t ag[KSTEPS];
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) ag[ks] = ld_frag(wg + ks * kadv);
    __builtin_amdgcn_sched_barrier(0);
    bf16x8_t bx[NTT][KSTEPS];
#pragma unroll
    for (int tt = 0; tt < NTT; ++tt) {
      if (ch == 0) {
        int64_t tok = 0;
        if (ok[tt]) tok = p.slot2tok ? p.slot2tok[seg0 + tt * 16 + r16] : (seg0 + tt * 16 + r16);
        xoff[tt] = tok * p.d + kbase;
      }
      const bf16_t* xr = p.x + xoff[tt] + ch * (KSTEPS * 32);
#pragma unroll
      for (int ks = 0; ks < KSTEPS; ++ks) bx[tt][ks] = ok[tt] ? ld_frag(xr + ks * 32) : zero_frag();
    }
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) {
      const bf16x8_t au = ld_frag(wu + ks * kadv);
#pragma unroll
      for (int tt = 0; tt < NTT; ++tt) {
        accg[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ag[ks], bx[tt][ks], accg[tt], 0, 0, 0);
        accu[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(au, bx[tt][ks], accu[tt], 0, 0, 0);
      }
    }
    wg += KSTEPS * kadv;
    wu += KSTEPS * kadv;
  } while (++ch < p.nch);
  // accumulator element i: neuron row (lane/16)*4 + i, token column lane%16
#pragma unroll
  for (int tt = 0; tt < NTT; ++tt)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      red[wave][0][tt][kq * 4 + i][r16] = accg[tt][i];
      red[wave][1][tt][kq * 4 + i][r16] = accu[tt][i];
    }
  __syncthreads();
  for (int e = tid; e < NTT * 256; e += 512) {
    const int tt = e >> 8, tok = (e >> 4) & 15, nn = e & 15;     // neuron fastest: contiguous stores
    const int col = tt * 16 + tok;
    if (col >= cnt) continue;
    float sg = 0.0f, su = 0.0f;
#pragma unroll
    for (int w = 0; w < 8; ++w) { sg += red[w][0][tt][nn][tok]; su += red[w][1][tt][nn][tok]; }
    p.h[hoff + (int64_t)col * wp + neuron0 + nn] = f32_to_bf16(silu_f32(sg) * su);
  }
}

// The same for 8 neurons: one MFMA operand holds the 8 gate rows (operand rows 0-7) and the 8 up rows (8-15) of
// the unit, so a unit is half as long and a launch has twice as many; taken when 16-neuron units would leave
// CUs without a workgroup (one token on a layer of few selected experts).  A load instruction covers two
// 512-byte pieces instead of 1 KB.  K slices, their order and the order of the final sum are those of the
// 16-neuron unit: H comes out bit for bit the same.
template <int NTT, int KSTEPS>
__device__ __forceinline__ void decode_gate_up_unit8(const DecArgs& p, int w1_row0, int local, int seg0, int cnt, int wp,
                                                     int64_t hoff, DecGateUpRed<NTT>& redbuf) {
  float (*red)[2][NTT][16][17] = redbuf.v;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r16 = lane & 15, kq = lane >> 4;
  const int neuron0 = local * 8;
  const int kbase = wave * (KSTEPS * 32) + kq * 8;
  const int n = neuron0 + (r16 & 7);
  const int64_t grow = (int64_t)w1_row0 + (n / IL) * 2 * IL + (n % IL) + (r16 >= 8 ? IL : 0);
  const bf16_t* wrow = p.w1 + (p.tiled ? tiled_offset(grow, kbase, p.ldw / TILE_K) : grow * p.ldw + kbase);
  const int kadv = p.tiled ? TILE_ELEMS : 32;
  bf16x8_t a[KSTEPS];
#pragma unroll
  for (int ks = 0; ks < KSTEPS; ++ks) a[ks] = ld_frag(wrow + ks * kadv);
  __builtin_amdgcn_sched_barrier(0);
  floatx4_t acc[NTT];
#pragma unroll
  for (int tt = 0; tt < NTT; ++tt) {
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[tt][i] = 0.0f;
    const int col = tt * 16 + r16;
    const bool ok = col < cnt;
    int64_t tok = 0;
    if (ok) tok = p.slot2tok ? p.slot2tok[seg0 + col] : (seg0 + col);
    const bf16_t* xr = p.x + tok * p.d + kbase;
    bf16x8_t bx[KSTEPS];
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) bx[ks] = ok ? ld_frag(xr + ks * 32) : zero_frag();
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) acc[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[ks], bx[ks], acc[tt], 0, 0, 0);
  }
  // accumulator element i: operand row (lane/16)*4 + i (0-7 gate, 8-15 up of neuron row % 8), token column lane%16
#pragma unroll
  for (int tt = 0; tt < NTT; ++tt)
#pragma unroll
    for (int i = 0; i < 4; ++i) red[wave][0][tt][kq * 4 + i][r16] = acc[tt][i];
  __syncthreads();
  for (int e = tid; e < NTT * 128; e += 512) {
    const int tt = e >> 7, tok = (e >> 3) & 15, nn = e & 7;
    const int col = tt * 16 + tok;
    if (col >= cnt) continue;
    float sg = 0.0f, su = 0.0f;
#pragma unroll
    for (int w = 0; w < 8; ++w) { sg += red[w][0][tt][nn][tok]; su += red[w][0][tt][8 + nn][tok]; }
    p.h[hoff + (int64_t)col * wp + neuron0 + nn] = f32_to_bf16(silu_f32(sg) * su);
  }
}

template <int NTT, int KSTEPS>
__device__ __forceinline__ void decode_gate_up_unit8_runs(const DecArgs& p, int w1_row0, int local, int seg0, int cnt, int wp,
                                                     int64_t hoff, DecGateUpRed<NTT>& redbuf) {
  float (*red)[2][NTT][16][17] = redbuf.v;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r16 = lane & 15, kq = lane >> 4;
  const int neuron0 = local * 8;
  const int kbase = wave * (KSTEPS * 32 * p.nch) + kq * 8;
  const int n = neuron0 + (r16 & 7);
  const int64_t grow = (int64_t)w1_row0 + (n / IL) * 2 * IL + (n % IL) + (r16 >= 8 ? IL : 0);
  const bf16_t* wrow = p.w1 + (p.tiled ? tiled_offset(grow, kbase, p.ldw / TILE_K) : grow * p.ldw + kbase);
  const int kadv = p.tiled ? TILE_ELEMS : 32;
  floatx4_t acc[NTT];
#pragma unroll
  for (int tt = 0; tt < NTT; ++tt)
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[tt][i] = 0.0f;
  int ch = 0;
  do {
    bf16x8_t a[KSTEPS];
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) a[ks] = ld_frag(wrow + ks * kadv);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int tt = 0; tt < NTT; ++tt) {
      const int col = tt * 16 + r16;
      const bool ok = col < cnt;
      int64_t tok = 0;
      if (ok) tok = p.slot2tok ? p.slot2tok[seg0 + col] : (seg0 + col);
      const bf16_t* xr = p.x + tok * p.d + kbase + ch * (KSTEPS * 32);
      bf16x8_t bx[KSTEPS];
#pragma unroll
      for (int ks = 0; ks < KSTEPS; ++ks) bx[ks] = ok ? ld_frag(xr + ks * 32) : zero_frag();
#pragma unroll
      for (int ks = 0; ks < KSTEPS; ++ks) acc[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[ks], bx[ks], acc[tt], 0, 0, 0);
    }
    wrow += KSTEPS * kadv;
  } while (++ch < p.nch);
  // accumulator element i: operand row (lane/16)*4 + i (0-7 gate, 8-15 up of neuron row % 8), token column lane%16
#pragma unroll
  for (int tt = 0; tt < NTT; ++tt)
#pragma unroll
    for (int i = 0; i < 4; ++i) red[wave][0][tt][kq * 4 + i][r16] = acc[tt][i];
  __syncthreads();
  for (int e = tid; e < NTT * 128; e += 512) {
    const int tt = e >> 7, tok = (e >> 3) & 15, nn = e & 7;
    const int col = tt * 16 + tok;
    if (col >= cnt) continue;
    float sg = 0.0f, su = 0.0f;
#pragma unroll
    for (int w = 0; w < 8; ++w) { sg += red[w][0][tt][nn][tok]; su += red[w][0][tt][8 + nn][tok]; }
    p.h[hoff + (int64_t)col * wp + neuron0 + nn] = f32_to_bf16(silu_f32(sg) * su);
  }
}

// A unit of unit1 neurons, in whichever form.  RUNS: the slice of a wave is more than one run of KSTEPS steps.
template <int NTT, int KSTEPS, bool RUNS>
__device__ __forceinline__ void decode_gate_up(const DecArgs& p, int w1_row0, int local, int seg0, int cnt, int wp, int64_t hoff,
                                               DecGateUpRed<NTT>& redbuf) {
  if constexpr (RUNS) {
    if (p.unit1 == 8) decode_gate_up_unit8_runs<NTT, KSTEPS>(p, w1_row0, local, seg0, cnt, wp, hoff, redbuf);
    else decode_gate_up_unit_runs<NTT, KSTEPS>(p, w1_row0, local, seg0, cnt, wp, hoff, redbuf);
  } else {
    if (p.unit1 == 8) decode_gate_up_unit8<NTT, KSTEPS>(p, w1_row0, local, seg0, cnt, wp, hoff, redbuf);
    else decode_gate_up_unit<NTT, KSTEPS>(p, w1_row0, local, seg0, cnt, wp, hoff, redbuf);
  }
}

// The same contraction for up to 16 * NTT rows of a group whose tokens do not stay in registers: K is walked in chunks of
// CS steps, the operands of the next chunk requested before the current one is multiplied, so that from the second chunk on
// between one and two of them are always on their way.  (The first chunk is alone: loads return in order, so waiting for the token
// index behind it is waiting for all of it.)  What bounds a unit is the stream of its weights from HBM; its tokens, NTT KB
// for every KB of gate and every KB of up rows, come from L2.  NEUR = 16, or 8 as in decode_gate_up_unit8 (gate and up rows in
// one operand).  w1_row0: the group's first packed row; row0, cnt: the unit's first slot and how many there are; columns past them repeat the first row and are not
// stored.  d must be a multiple of 256 * CS, the weights tiled.
constexpr int STREAM_RED_FLOATS = 8 * 2 * 16 * 17;
template <int NTT, int CS, int NEUR>
__device__ __forceinline__ void stream_gate_up_unit(const DecArgs& p, int w1_row0, int local, int row0, int cnt, int wp, int64_t hoff,
                                                    float* redbuf) {
  constexpr int OPS = NEUR / 8;                               // operands per K step: gate and up, or both in one
  float (*red)[OPS][16][17] = reinterpret_cast<float (*)[OPS][16][17]>(redbuf);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, kq = lane >> 4;
  const int neuron0 = local * NEUR;
  const int steps = p.d / 256, kbase = wave * steps * 32 + kq * 8, chunks = steps / CS;
  const int n = neuron0 + (r16 & (NEUR - 1));
  const int64_t grow = (int64_t)w1_row0 + (n / IL) * 2 * IL + (n % IL) + (r16 >= NEUR ? IL : 0);
  const bf16_t* w[OPS];
  w[0] = p.w1 + tiled_offset(grow, kbase, p.ldw / TILE_K);
  if (OPS == 2) w[OPS - 1] = w[0] + (int64_t)(IL / TILE_ROWS) * (p.ldw / TILE_K) * TILE_ELEMS;
  bf16x8_t a[2][OPS][CS], bx[2][NTT][CS];
  auto load_w = [&](auto buf, int c) {
    constexpr int B = decltype(buf)::value;
#pragma unroll
    for (int s = 0; s < CS; ++s)
#pragma unroll
      for (int o = 0; o < OPS; ++o) a[B][o][s] = ld_frag(w[o] + (int64_t)(c * CS + s) * TILE_ELEMS);
  };
  using B0 = std::integral_constant<int, 0>;
  using B1 = std::integral_constant<int, 1>;
  load_w(B0{}, 0);                                            // before anything else: HBM is what the unit waits for
  __builtin_amdgcn_sched_barrier(0);
  uint32_t xo[NTT];
#pragma unroll
  for (int tt = 0; tt < NTT; ++tt) {
    const int row = row0 + (tt * 16 + r16 < cnt ? tt * 16 + r16 : 0);
    xo[tt] = (uint32_t)((p.slot2tok ? p.slot2tok[row] : row) * p.x_row + kq * 8);
  }
  auto load_x = [&](auto buf, int c) {
    constexpr int B = decltype(buf)::value;
#pragma unroll
    for (int s = 0; s < CS; ++s) {
      const bf16_t* xs = p.x + (int64_t)(wave * steps + c * CS + s) * p.x_step;
#pragma unroll
      for (int tt = 0; tt < NTT; ++tt) bx[B][tt][s] = ld_frag(xs + xo[tt]);
    }
  };
  floatx4_t acc[OPS][NTT];
#pragma unroll
  for (int o = 0; o < OPS; ++o)
#pragma unroll
    for (int tt = 0; tt < NTT; ++tt)
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[o][tt][i] = 0.0f;
  auto multiply = [&](auto buf) {
    constexpr int B = decltype(buf)::value;
#pragma unroll
    for (int s = 0; s < CS; ++s)
#pragma unroll
      for (int tt = 0; tt < NTT; ++tt)
#pragma unroll
        for (int o = 0; o < OPS; ++o) acc[o][tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[B][o][s], bx[B][tt][s], acc[o][tt], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto load = [&](auto buf, int c) {
    load_w(buf, c);
    load_x(buf, c);
    __builtin_amdgcn_sched_barrier(0);                        // (requested here, not where the compiler finds a use)
  };
  load_x(B0{}, 0);
  int c = 0;
  for (; c + 2 < chunks; c += 2) {
    load(B1{}, c + 1);
    multiply(B0{});
    load(B0{}, c + 2);
    multiply(B1{});
  }
  if (c + 1 < chunks) {
    load(B1{}, c + 1);
    multiply(B0{});
    multiply(B1{});
  } else {
    multiply(B0{});
  }
  // one token tile at a time: accumulator element i is operand row (lane/16)*4 + i, token column lane%16
#pragma unroll
  for (int tt = 0; tt < NTT; ++tt) {
    if (tt > 0) __syncthreads();
#pragma unroll
    for (int o = 0; o < OPS; ++o)
#pragma unroll
      for (int i = 0; i < 4; ++i) red[wave][o][kq * 4 + i][r16] = acc[o][tt][i];
    __syncthreads();
    const int tok = tid / NEUR, nn = tid % NEUR, col = tt * 16 + tok;       // neuron fastest: contiguous stores
    if (tok < 16 && col < cnt) {
      float sg = 0.0f, su = 0.0f;
#pragma unroll
      for (int k = 0; k < 8; ++k) { sg += red[k][0][nn][tok]; su += red[k][OPS - 1][NEUR == 8 ? 8 + nn : nn][tok]; }
      p.h[hoff + (int64_t)col * wp + neuron0 + nn] = f32_to_bf16(silu_f32(sg) * su);
    }
  }
}

// A unit in the instantiation for its rows; MAXT: token tiles of the fullest unit the caller can have.
template <int MAXT, int CS, int NEUR>
__device__ __forceinline__ void stream_gate_up(const DecArgs& p, int w1_row0, int local, int row0, int cnt, int wp, int64_t hoff, float* redbuf) {
  if (MAXT == 1 || cnt <= 16) stream_gate_up_unit<1, CS, NEUR>(p, w1_row0, local, row0, cnt, wp, hoff, redbuf);
  else if (MAXT == 2 || cnt <= 32) stream_gate_up_unit<MAXT < 2 ? MAXT : 2, CS, NEUR>(p, w1_row0, local, row0, cnt, wp, hoff, redbuf);
  else stream_gate_up_unit<MAXT, NEUR == 8 ? CS : 2, NEUR>(p, w1_row0, local, row0, cnt, wp, hoff, redbuf);    // (16 neurons, four steps: spills)
}

// CALL(MAXT, CS) with the template arguments for a batch of T <= 64 tokens at model width d (a multiple of 512).
#define CMOE_STREAM_FORM(T, d, CALL)                                                            \
  if ((T) <= 16) { if ((d) % 1024 == 0) { CALL(1, 4); } else { CALL(1, 2); } }                  \
  else if ((T) <= 32) { CALL(2, 2); }                                                           \
  else { if ((d) % 1024 == 0) { CALL(4, 4); } else { CALL(4, 2); } }

// Model widths of the decode kernels: d = 8 waves x nch runs x ksteps steps of 32.  One run of an even number of
// steps up to d = 4096, above that runs of 8 or 10; zero steps for a width they do not serve.
struct DecodeK { int ksteps, nch; };
static constexpr DecodeK decode_k(int d) {
  if (d % 512 != 0) return {0, 0};
  const int ks = d / 256;
  if (ks <= 16) return {ks, 1};
  if (ks > 40) return {0, 0};
  return ks % 8 == 0 ? DecodeK{8, ks / 8} : ks % 10 == 0 ? DecodeK{10, ks / 10} : DecodeK{0, 0};
}
// Every width served is covered to its end, in runs that the dispatches below have.
static constexpr bool decode_widths_covered() {
  for (int d = 256; d <= 65536; d += 256) {
    const DecodeK k = decode_k(d);
    if (k.ksteps == 0) continue;
    if (k.ksteps * k.nch * 256 != d) return false;
    if (k.nch > 1 ? k.ksteps != 8 && k.ksteps != 10 : k.ksteps % 2 != 0 || k.ksteps > 16) return false;
  }
  return true;
}
static_assert(decode_widths_covered(), "a model width without its step count");
// CALL(KSTEPS, RUNS) with the template arguments for model width d; returns an error from the enclosing function where there
// are none.
#define CMOE_DECODE_KSTEPS(d, CALL)                \
  switch (decode_k(d).nch > 1 ? -decode_k(d).ksteps : decode_k(d).ksteps) { \
    case -8: CALL(8, true); break;                 \
    case -10: CALL(10, true); break;               \
    case 16: CALL(16, false); break;               \
    case 14: CALL(14, false); break;               \
    case 12: CALL(12, false); break;               \
    case 10: CALL(10, false); break;               \
    case 8: CALL(8, false); break;                 \
    case 6: CALL(6, false); break;                 \
    case 4: CALL(4, false); break;                 \
    case 2: CALL(2, false); break;                 \
    default: return hipErrorInvalidValue;          \
  }

// Host side (decode.hip): the argument block of a forward.
DecArgs make_dec_args(const Engine& e, const void* x, int64_t T, char* ws, const WsLayout& L, void* y);
// The same for the streamed units (gate_up_stream.hip): tokens as the scorer of the front end laid them out, if it did.
DecArgs make_stream_args(const Engine& e, const void* x, int64_t T, char* ws, const WsLayout& L);

}  // namespace cmoe
