// Small device helpers: bf16 conversion, wave reductions, the wave-level top-k.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cmoe {

typedef uint16_t bf16_t;   // storage type of a bf16 element (bit pattern)

__device__ __forceinline__ float bf16_to_f32(bf16_t v) { return __uint_as_float(((uint32_t)v) << 16); }

// round-to-nearest-even; NaN stays NaN.  The cast compiles to the hardware conversion of gfx950
// (v_cvt_pk_bf16_f32): no integer rounding sequence and no branch for the NaN case.
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
  const __bf16 h = static_cast<__bf16>(f);
  return __builtin_bit_cast(bf16_t, h);
}

// Work lists: work[0..G] is a non-decreasing prefix array (work[0] = 0, G <= 128 groups) and item u belongs
// to the last group g with work[g] <= u (empty groups are skipped).  Every lane looks at two entries and
// a ballot counts the entries that do not exceed u: one round of loads instead of the seven dependent
// ones of a binary search, which matters because every workgroup starts with this lookup.  Requires
// u < work[G]; all lanes of the wave must call it.
__device__ __forceinline__ int find_group(const int32_t* __restrict__ work, int G, int u) {
  const int lane = threadIdx.x & 63;
  const int i0 = 1 + lane, i1 = 65 + lane;
  const bool b0 = i0 <= G && work[i0] <= u;
  const bool b1 = i1 <= G && work[i1] <= u;
  return __popcll(__ballot(b0)) + __popcll(__ballot(b1));
}

// Inclusive prefix sums over the 64 lanes of a wave, all of which must call.  The partial sums move up the wave in DPP
// operands, within rows of 16 lanes, then from row to row: a scan is a chain of vector instructions, where exchanges through
// the LDS crossbar are a chain of six round trips, and selection and placement are mostly such chains.  us per forward with
// exchanges / now: d = 4096, 16 experts, one token 23.2 / 22.9, 4 tokens 43.3 / 42.4, 32 experts, 32 tokens 73.2 / 71.9, 2048 tokens
// 203.1 / 202.3; fp32, d = 256, 512 tokens 26.2 / 25.4.
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_from(int v) {               // 0 for lanes without a source
  return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, false);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ long long dpp_from(long long v) {
  const uint32_t lo = (uint32_t)dpp_from<CTRL, ROWS>((int)(uint32_t)v);
  const uint32_t hi = (uint32_t)dpp_from<CTRL, ROWS>((int)(v >> 32));
  return (long long)(((unsigned long long)hi << 32) | lo);
}
template <typename I>
__device__ __forceinline__ I wave_incl_scan(I v) {
  v += dpp_from<0x111, 0xf>(v);      // row_shr 1, 2, 4, 8
  v += dpp_from<0x112, 0xf>(v);
  v += dpp_from<0x114, 0xf>(v);
  v += dpp_from<0x118, 0xf>(v);
  v += dpp_from<0x142, 0xa>(v);      // row_bcast 15 into rows 1 and 3
  v += dpp_from<0x143, 0xc>(v);      // row_bcast 31 into rows 2 and 3
  return v;
}
// The last lane's value, e.g. a scan's total.
__device__ __forceinline__ int wave_last(int v) { return __builtin_amdgcn_readlane(v, 63); }
__device__ __forceinline__ long long wave_last(long long v) {
  return ((long long)wave_last((int)(v >> 32)) << 32) | (uint32_t)wave_last((int)(uint32_t)v);
}

template <typename T> struct Elem;
template <> struct Elem<float> {
  static __device__ __forceinline__ float ld(const float* p) { return *p; }
  static __device__ __forceinline__ void st(float* p, float v) { *p = v; }
};
template <> struct Elem<bf16_t> {
  static __device__ __forceinline__ float ld(const bf16_t* p) { return bf16_to_f32(*p); }
  static __device__ __forceinline__ void st(bf16_t* p, float v) { *p = f32_to_bf16(v); }
};

// SiLU / Swish with beta = 1 (Eq. 3): z * sigmoid(z), evaluated in fp32.
__device__ __forceinline__ float silu_f32(float z) { return z / (1.0f + expf(-z)); }

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ int wave_sum_i(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Monotone map float -> uint32 (larger float <=> larger integer; -0 < +0).
__device__ __forceinline__ uint32_t ordered_key(float f) {
  uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Wave arg-max: every lane passes (key, active), at least one lane active; returns the lane that holds the largest key
// among the active ones, ties to the lowest lane.  All 64 lanes must call.  The maximum moves up the wave in DPP operands
// (within rows of 16 lanes, then from row to row) and ends in lane 63; exchanges through the LDS crossbar are a
// longer chain (one token, d = 4096, whole forward: 32 experts, top-5 22.5 -> 21.6 us; 8 experts, top-5 45.6 -> 42.3).
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_max(uint32_t m) {
  const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, CTRL, 0xf, 0xf, true);
  return o > m ? o : m;
}
__device__ __forceinline__ int wave_argmax(uint32_t key, bool active) {
  uint32_t m = active ? key : 0u;
  m = dpp_max<0x111>(m);      // row_shr 1, 2, 4, 8
  m = dpp_max<0x112>(m);
  m = dpp_max<0x114>(m);
  m = dpp_max<0x118>(m);
  m = dpp_max<0x142>(m);      // row_bcast 15, 31
  m = dpp_max<0x143>(m);
  const uint32_t top = (uint32_t)__builtin_amdgcn_readlane((int)m, 63);
  return __ffsll((unsigned long long)__ballot(active && key == top)) - 1;
}

}  // namespace cmoe
