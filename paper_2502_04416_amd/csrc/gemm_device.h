// Arguments and device helpers shared by the grouped contraction kernels (gemm_bf16.hip, gemm_stream.hip).
#pragma once
#include "cmoe_internal.h"
#include "device_utils.h"

namespace cmoe {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float floatx16_t __attribute__((ext_vector_type(16)));
typedef float floatx4_t __attribute__((ext_vector_type(4)));

struct GemmArgs {
  const bf16_t* A;
  const bf16_t* B;
  bf16_t* C;
  const GroupDev* groups;
  const int32_t* seg_off;    // [G+1]
  const int32_t* work;       // [G+1+9], see WsLayout::work1, work2
  const int64_t* h_off;      // [G+1]
  const int32_t* slot2tok;   // MODE 1 gather; null = identity
  int G;
  int d;
  int ldb;                   // elements per row of B in MODE 1 (packed gate/up rows)
  int b_tiled;               // 1: the weight matrices are tiled 16 x 32 (see cmoe_internal.h)
  int64_t T;
  int single;                // 1: one always-on group holding all T tokens; no device schedule is read
  int n_blocks;              // grid size (multiple of 8) before the K split
  int xcd_remap;             // 1: consecutive work items run on the same XCD
  int zero_pad;              // 1: tile rows past the end of a group read zeros instead of repeating its last row
  int deep_rounds;           // persistent down contraction: tiles of the narrowest groups that take as long as one of the widest
  int ws_skip;               // 1 (down contraction): groups the weight-stationary kernel handles are left to it
  // K split: k_split > 1 workgroups share one tile, each multiplies a contiguous range of K tiles and
  // stores its fp32 partial sums to P [k_split][p_rows][ldp] (row = slot, column = column of the tile
  // grid); a finishing kernel adds the parts in order and applies the epilogue.  Used when a launch has
  // too few tiles to fill the chip (batches of a few hundred tokens).
  int k_split;
  float* P;
  int64_t p_rows;
  int ldp;
};

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

constexpr uint32_t DMA_NONE = 0x80000000u;                    // an offset past the end of every buffer used here

// A uniform pointer, in scalar registers.
__device__ __forceinline__ const bf16_t* uniform_ptr(const bf16_t* ptr) {
  const uint64_t v = reinterpret_cast<uint64_t>(ptr);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<const bf16_t*>(((uint64_t)hi << 32) | lo);
}

// 64 lanes x 16 bytes from base + lane_off + step_off (bytes; zeros where lane_off >= size) to 1 KB of LDS.
__device__ __forceinline__ void dma16_buffer(const bf16_t* base, uint32_t size, uint32_t lane_off, uint32_t step_off, bf16_t* lds_dst) {
#if defined(__HIP_DEVICE_COMPILE__)
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(base), 0, size, 0x00020000);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)(lds_dst), 16, lane_off, step_off, 0, 0);
#endif
}

// acc += w * a (w: 16 weight rows x 32 K, a: 16 activation rows x 32 K).  Written as assembly to pin the
// accumulators to the AGPRs: with the builtin the register allocator shuffles them between the two halves of the
// register file inside the K loop (96 to 470 moves per step, and spills for the 256 x 256 tile of four waves).
// The compiler does not see an MFMA here, so it puts no wait states in front of another use of the result (8 on this
// part) and may place such a use anywhere behind the block, a spill or a copy of an accumulator among them.  WAIT, set for the
// last MFMA of the last K step, therefore waits inside the block: whatever follows it finds every accumulator
// complete.  (A wait in a statement of its own came too late: the allocator had spilled an accumulator in front of it.)
// Sources come from LDS reads only (waited for by the compiler as for any use), and the accumulator is overwritten by
// nothing else inside the loop.  tests/test_kernel_code_cpu.py checks these distances in the machine code.
template <bool WAIT>
__device__ __forceinline__ void mfma_acc(floatx4_t& acc, const bf16x8_t& w, const bf16x8_t& a) {
  if constexpr (WAIT) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0\n\ts_nop 7" : "+a"(acc) : "v"(w), "v"(a) : "memory");
  else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(w), "v"(a));
}

constexpr int BK = 32;                                        // K step
constexpr int BLK = 16 * BK;                                  // elements of a 16-row block

}  // namespace cmoe
