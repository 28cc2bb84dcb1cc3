// Which group a workgroup's work item belongs to, and what it needs of that group.
#pragma once
#include "cmoe_internal.h"
#include "device_utils.h"

namespace cmoe {

// Every workgroup of a grouped launch starts with this lookup, and nothing else can be asked for before it is done.  Each lane
// requests everything about its (at most two) groups at once, before the work item is even known, so that the lookup is
// one round trip to memory (in the streamed gate/up units two: they first ask whether there is an item at all); the prefix array, then
// the group's offsets and places, then its matrix one after the other were three.
// us per forward: d = 4096, 16 experts, 4 tokens 37.3 -> 37.1, 32 tokens 64.7 -> 63.9; d = 8192, 5 tokens 93.5 -> 92.6; d = 2048, 32 experts,
// 16 tokens 23.7 -> 23.2; fp32, d = 256, 512 tokens 25.6 -> 24.6.
struct GroupLanes {
  int first[MAX_GROUPS / 64], end[MAX_GROUPS / 64];            // work items
  int slot[MAX_GROUPS / 64], slot_end[MAX_GROUPS / 64];
  GroupDev gd[MAX_GROUPS / 64];
  int64_t h[MAX_GROUPS / 64];
};
// All lanes of a wave must call both.
__device__ __forceinline__ GroupLanes request_groups(const int32_t* __restrict__ work, const int32_t* __restrict__ seg_off,
                                                     const GroupDev* __restrict__ groups, const int64_t* __restrict__ h_off, int G) {
  const int lane = threadIdx.x & 63;
  GroupLanes gl;
#pragma unroll
  for (int k = 0; k < MAX_GROUPS / 64; ++k) {
    if (k > 0 && 64 * k >= G) break;
    const int g = lane + 64 * k < G ? lane + 64 * k : G - 1;
    gl.first[k] = work[g];
    gl.end[k] = work[g + 1];
    gl.slot[k] = seg_off[g];
    gl.slot_end[k] = seg_off[g + 1];
    gl.gd[k] = groups[g];
    gl.h[k] = h_off[g];
  }
  return gl;
}

struct WorkItem {
  int g, local;                                                // group, item's number inside the group
  int seg0, cnt, wp, w1_row0;
  int64_t hoff, w2_off;
};
// Item u of the list, which is a non-decreasing prefix array: u belongs to the last group that begins at or before it (empty
// groups are skipped).  Requires u < work[G].
__device__ __forceinline__ WorkItem find_item(const GroupLanes& gl, int G, int u) {
  const int lane = threadIdx.x & 63;
  int g = __popcll(__ballot(lane < G && gl.end[0] <= u));
  GroupDev gd = gl.gd[0];
  int first = gl.first[0], slot = gl.slot[0], slot_end = gl.slot_end[0];
  int64_t h = gl.h[0];
#pragma unroll
  for (int k = 1; k < MAX_GROUPS / 64; ++k) {
    if (g < 64 * k) break;
    g += __popcll(__ballot(lane + 64 * k < G && gl.end[k] <= u));
    gd = gl.gd[k];
    first = gl.first[k];
    slot = gl.slot[k];
    slot_end = gl.slot_end[k];
    h = gl.h[k];
  }
  auto of = [&](int v) { return __builtin_amdgcn_readlane(v, g & 63); };
  auto of64 = [&](int64_t v) { return ((int64_t)of((int)(v >> 32)) << 32) | (uint32_t)of((int)(uint32_t)v); };
  WorkItem it;
  it.g = g;
  it.local = u - of(first);
  it.seg0 = of(slot);
  it.cnt = of(slot_end) - it.seg0;
  it.wp = of(gd.width_pad);
  it.w1_row0 = of(gd.w1_row0);
  it.w2_off = of64(gd.w2_off);
  it.hoff = of64(h);
  return it;
}
}  // namespace cmoe
