// Gate/up contraction of batches of 2 to 64 tokens, a few rows to a group.  The launch is bound by the stream of the touched
// experts' weights from HBM; a workgroup takes 16 or 8 neurons over all of K (stream_gate_up_unit).  Against keeping a unit's
// tokens in registers (decode_gate_up_unit): two to three workgroups fit a CU instead of one or two, weight loads never pause
// for a new run of tokens, and the tokens come from a copy laid out [K step][token][32] by the scorer, where the 16 rows of an
// operand are neighbours; in the caller's matrix they are a power of two apart at d = 4096 and 8192 and meet in one L2 channel.
// Gate/up + selection launches, d = 8192, 8 experts, 5 tokens: 63.6 -> 56.2 us.
#include "cmoe_internal.h"
#include "decode_device.h"
#include "device_utils.h"
#include "work_item.h"

namespace cmoe {

// (units of 8 neurons: at most 80 registers, three workgroups on a CU)
template <int MAXT, int CS, int NEUR>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(MAXT > 2 ? 2 : MAXT == 1 && NEUR == 8 ? 6 : 4))) void stream_gate_up_kernel(DecArgs p) {
  __shared__ float red[STREAM_RED_FLOATS];
  const int u = blockIdx.x;
  if (u >= p.work[p.G]) return;                               // (first: the grid is a bound, and if those past the list's end asked too, 8 tokens
                                                              // on 32 experts, d = 4096, took 48.0 us per forward for 46.3)
  const GroupLanes gl = request_groups(p.work, p.seg_off, p.groups, p.h_off, p.G);
  const WorkItem it = find_item(gl, p.G, u);
  stream_gate_up<MAXT, CS, NEUR>(p, it.w1_row0, it.local, it.seg0, it.cnt, it.wp, it.hoff, red);
}

bool stream_gate_up_ok(const Engine& e, int64_t T) {
  return e.dtype == 1 && !use_simt_experts(e.dtype) && e.w_tiled && e.d % 512 == 0 && T >= 2 && T <= STREAM_ROWS && e.S_dyn > 0;
}

// Units of 8 are shorter, and a last round of workgroups that does not fill the chip costs less; units of 16 read the tokens half
// as often.  us per forward with 16 / 8 neurons, d = 4096, 16 experts, top-3: 4 tokens 45.5 / 41.8, 16 tokens 59.5 / 55.4, 24 tokens
// 67.0 / 68.3; d = 5120, 16 experts, top-2: 17 tokens 75.6 / 77.7; d = 8192, 32 experts, top-5: 8 tokens 86.9 / 81.7, 24 tokens 122.9 / 120.5.
int stream_neurons(const Engine& e, int64_t T) { return T <= 16 || e.d > 5120 ? 8 : 16; }

// From d = 3072 on: below, a unit's tokens fit its registers in a few loads and a launch is too short for a stream.  us per forward
// on decode_gate_up_kernel / streamed: d = 1536, 8 experts, top-2: 2 tokens 18.7 / 19.1, 16 tokens 23.8 / 24.6; d = 2048, 32 experts,
// top-4: 2 tokens 19.2 / 19.9, 12 tokens 26.4 / 27.3; d = 2560, 32 experts, top-4: 4 tokens 25.3 / 26.3, 16 tokens 34.0 / 33.5 (8, top-2:
// 37.4 / 37.1); d = 3072, 16 experts, top-3: 4 tokens 34.0 / 33.2, 16 tokens 44.8 / 41.7; d = 3584, 8 experts, top-2: 47.0 / 41.5 and
// 53.5 / 49.4; d = 4096, 16 experts, top-3: 2 tokens 33.8 / 33.4, 16 tokens 61.9 / 55.5.  Without an always-on group next to the
// selection, two tokens are the other way round (d = 4096, 16 experts 29.5 / 30.3, 32 28.5 / 29.8), three even.  Hierarchies: d = 1024, 8
// outer experts, 16 tokens 27.1 / 27.8; d = 2048 2 to 16 tokens 27.0 / 26.5 to 45.0 / 44.8; d = 3072, 4 outer, 4 tokens 52.7 / 51.8, 16
// tokens 68.1 / 68.4.  A forced shape of streamed units counts at every width.
bool decode_gate_up_streams(const Engine& e, int64_t T) {
  if (!decode_path_ok(e, T) || !stream_gate_up_ok(e, T) || decode_front_runs_all(e, T)) return false;
  if (gate_up_streams_forced()) return true;
  return e.d >= 3072 && (T > 3 || e.n_always == 1 || e.r.outer_top_k != 0 || decode_k(e.d).nch > 1);
}

bool front_lays_tokens(const Engine& e, int64_t T) {
  return decode_front_ok(e, T) && (decode_path_ok(e, T) ? decode_gate_up_streams(e, T) : tiles_gate_up_streams(e, T));
}

DecArgs make_stream_args(const Engine& e, const void* x, int64_t T, char* ws, const WsLayout& L) {
  DecArgs a = make_dec_args(e, x, T, ws, L, nullptr);
  if (front_lays_tokens(e, T)) {
    a.x = reinterpret_cast<const bf16_t*>(ws + L.y_slots);
    a.x_row = 32;
    a.x_step = 32 * (int)T;
  }
  return a;
}

hipError_t launch_stream_gate_up(const Engine& e, const void* x, int64_t T, char* ws, const WsLayout& L, int neurons, int n_blocks, hipStream_t s) {
  DecArgs a = make_stream_args(e, x, T, ws, L);
  a.work = reinterpret_cast<const int32_t*>(ws + L.work1);
#define CMOE_LAUNCH_N(MAXT, CS, NEUR) hipLaunchKernelGGL((stream_gate_up_kernel<MAXT, CS, NEUR>), dim3((unsigned)n_blocks), dim3(512), 0, s, a)
#define CMOE_LAUNCH(MAXT, CS) if (neurons == 8) CMOE_LAUNCH_N(MAXT, CS, 8); else CMOE_LAUNCH_N(MAXT, CS, 16)
  CMOE_STREAM_FORM(T, e.d, CMOE_LAUNCH)
#undef CMOE_LAUNCH
#undef CMOE_LAUNCH_N
  return hipGetLastError();
}

}  // namespace cmoe
