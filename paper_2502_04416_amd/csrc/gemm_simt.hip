// Grouped SwiGLU expert kernels with fp32 arithmetic.  They serve the
// fp32 layers (tolerance 1e-5, where bf16 MFMA inputs would be too coarse) and follow the same work
// list, gather and ragged layouts as the bf16 MFMA kernels:
//   MODE 1  H_g = Swish(X_g Wgate_g) * (X_g Wup_g)   (Eq. 3, first line, on the group's neurons)
//   MODE 2  Y_g = H_g Wdown_g                        (Eq. 3, second line)
#include <algorithm>
#include "cmoe_internal.h"
#include "device_utils.h"
#include "work_item.h"

namespace cmoe {

template <typename T>
struct SimtArgs {
  const T* A;
  const T* B;
  T* C;
  const GroupDev* groups;
  const int32_t* seg_off;
  const int32_t* work;
  const int64_t* h_off;
  const int32_t* slot2tok;
  int G;
  int d;
  int ldb;
  int b_tiled;               // 1: B is tiled 16 x 32 (bf16 layers run here only when forced to)
  int64_t T_tokens;
  int single;
  int vec;                   // 1: rows of A and of B are 16-byte aligned and K a multiple of 4 (fp32 layers): float4 loads
};

constexpr int SB = 64;     // tile rows and tile columns
// K step.  These layers are small and a workgroup's time is the chain of its K steps, a round trip to memory each: a
// step of 64 in float4 loads, the next one's in flight while a step is multiplied, instead of 16 in scalar
// loads (d = 256, 64 tokens: 64.4 -> 56.8 us per forward).  The sums run over ascending k either way.
constexpr int SK = 64;

template <typename T, int MODE>
__global__ __launch_bounds__(256) void grouped_gemm_simt(SimtArgs<T> p) {
  __shared__ __attribute__((aligned(16))) float As[SK][SB + 4];
  __shared__ __attribute__((aligned(16))) float Bs[SK][SB + 4];
  const int tid = threadIdx.x;
  const int ty = tid >> 4, tx = tid & 15;
  int wid = blockIdx.x;
  int g = 0, local = wid, cnt, seg0 = 0, wp;
  int64_t hoff = 0;
  if (p.single) {
    cnt = (int)p.T_tokens;
    wp = p.groups[0].width_pad;
  } else {
    const GroupLanes gl = request_groups(p.work, p.seg_off, p.groups, p.h_off, p.G);
    if (wid >= p.work[p.G]) return;
    const WorkItem it = find_item(gl, p.G, wid);
    g = it.g;
    local = it.local;
    seg0 = it.seg0;
    cnt = it.cnt;
    wp = it.wp;
    hoff = it.hoff;
  }
  const int K = (MODE == 1) ? p.d : wp;
  const int n_cols = (MODE == 1) ? 2 * wp : p.d;
  const int n_nt = (n_cols + SB - 1) / SB;
  const int n_mt = (cnt + SB - 1) / SB;
  if (p.single && local >= n_mt * n_nt) return;
  const int mt = local / n_nt, nt = local % n_nt;

  // loader: thread loads k = lk .. lk + 3, and the same 16, 32 and 48 further, of one row of A and of B
  const int lrow = tid >> 2, lk = (tid & 3) * 4;
  int ar = mt * SB + lrow;
  if (ar >= cnt) ar = cnt - 1;
  const T* a_src;
  if (MODE == 1) {
    const int64_t tok = p.slot2tok ? p.slot2tok[seg0 + ar] : (seg0 + ar);
    a_src = p.A + tok * p.d;
  } else {
    a_src = p.A + hoff + (int64_t)ar * wp;
  }
  int bn = nt * SB + lrow;
  if (bn >= n_cols) bn = n_cols - 1;
  const T* b_src = (MODE == 1) ? p.B + ((int64_t)p.groups[g].w1_row0 + bn) * p.ldb
                               : p.B + p.groups[g].w2_off + (int64_t)bn * wp;
  // tiled weights: element (row, k) through the layout function instead of b_src + k
  const int64_t b_rowg = (MODE == 1) ? (int64_t)p.groups[g].w1_row0 + bn : bn;
  const T* b_base = (MODE == 1) ? p.B : p.B + p.groups[g].w2_off;
  const int b_kt32 = (MODE == 1) ? p.ldb / TILE_K : wp / TILE_K;
  // columns owned by this thread inside the 64-wide tile
  int cols[4];
  if (MODE == 1) { cols[0] = 2 * tx; cols[1] = 2 * tx + 1; cols[2] = IL + 2 * tx; cols[3] = IL + 2 * tx + 1; }
  else { cols[0] = 4 * tx; cols[1] = 4 * tx + 1; cols[2] = 4 * tx + 2; cols[3] = 4 * tx + 3; }

  float acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.0f;

  float ra[SK / 4], rb[SK / 4];
  auto load_step = [&](int k0) {
#pragma unroll
    for (int v = 0; v < SK / 16; ++v) {
      const int k = k0 + v * 16 + lk;
      if constexpr (sizeof(T) == 4) {
        if (p.vec) {
          float4 fa = make_float4(0.f, 0.f, 0.f, 0.f), fb = fa;
          if (k < K) {
            fa = *reinterpret_cast<const float4*>(a_src + k);
            fb = *reinterpret_cast<const float4*>(b_src + k);
          }
          ra[4 * v] = fa.x; ra[4 * v + 1] = fa.y; ra[4 * v + 2] = fa.z; ra[4 * v + 3] = fa.w;
          rb[4 * v] = fb.x; rb[4 * v + 1] = fb.y; rb[4 * v + 2] = fb.z; rb[4 * v + 3] = fb.w;
          continue;
        }
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        ra[4 * v + j] = (k + j < K) ? Elem<T>::ld(a_src + k + j) : 0.0f;
        rb[4 * v + j] = (k + j < K) ? Elem<T>::ld(p.b_tiled ? b_base + tiled_offset(b_rowg, k + j, b_kt32) : b_src + k + j) : 0.0f;
      }
    }
  };
  load_step(0);
  for (int k0 = 0; k0 < K; k0 += SK) {
#pragma unroll
    for (int v = 0; v < SK / 16; ++v)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        As[v * 16 + lk + j][lrow] = ra[4 * v + j];
        Bs[v * 16 + lk + j][lrow] = rb[4 * v + j];
      }
    __syncthreads();
    if (k0 + SK < K) load_step(k0 + SK);
    // 16 of K at a time, and no further than K goes: with all 64 multiplied whatever is left, experts of up to 32 neurons
    // and widths like 328 spent up to half of it on zeros (d = 328, 4 experts of 24, one token: 55.1 -> 48.8 us per forward)
    for (int kb = 0; kb < SK && k0 + kb < K; kb += 16) {
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        // (rows of 68 floats: 16-byte aligned pieces, one or two LDS reads per operand)
        float a[4], b[4];
        *reinterpret_cast<float4*>(a) = *reinterpret_cast<const float4*>(&As[kb + k][ty * 4]);
        if (MODE == 1) {
          *reinterpret_cast<float2*>(b) = *reinterpret_cast<const float2*>(&Bs[kb + k][2 * tx]);
          *reinterpret_cast<float2*>(b + 2) = *reinterpret_cast<const float2*>(&Bs[kb + k][IL + 2 * tx]);
        } else {
          *reinterpret_cast<float4*>(b) = *reinterpret_cast<const float4*>(&Bs[kb + k][4 * tx]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
      }
    }
    __syncthreads();
  }

#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = mt * SB + ty * 4 + i;
    if (r >= cnt) continue;
    if (MODE == 1) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int neuron = nt * (SB / 2) + 2 * tx + j;
        if (neuron < wp) Elem<T>::st(p.C + hoff + (int64_t)r * wp + neuron, silu_f32(acc[i][j]) * acc[i][j + 2]);
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int col = nt * SB + cols[j];
        if (col < p.d) Elem<T>::st(p.C + (int64_t)(seg0 + r) * p.d + col, acc[i][j]);
      }
    }
  }
}

// ---- small fp32 problems, on the fp32 matrix instruction -----------------------------------------------------
// What bounds it: the numerics layers are small (tens to hundreds of tokens, experts of tens of neurons), so a launch is a
// chain of memory round trips, and tiles of 64 x 64 left most of the chip idle and multiplied groups of nine rows as 64.
// Here a workgroup takes 16 rows x 32 columns (MODE 1: the gate and the up row of 16 neurons); its four waves take every
// fourth chunk of 16 of K, all of a wave's operand loads (up to 128 of K) in flight at once, straight from memory in operand
// order, and the four partial sums are added in wave order.  v_mfma_f32_16x16x4_f32 multiplies and adds in fp32 like the
// FMAs of the kernel above; a lane's float4 holds k = 4 (lane / 16) .. + 3 of a chunk, and MFMA j takes element j of
// both operands, so a chunk is summed in the order 0, 4, 8, 12, 1, 5, ...
// d = 256, 8 experts of 128, 64 tokens: gate/up 25.2 and down 14.4 us before, 5.9 and 4.4 now.
constexpr int FM = 16, FN = 32;       // rows and columns of a tile
constexpr int FC = 8;                 // chunks of a wave in flight

typedef float f32x4_t __attribute__((ext_vector_type(4)));

template <int MODE, bool VEC>
__global__ __launch_bounds__(256) void grouped_gemm_f32(SimtArgs<float> p) {
  __shared__ float red[4][FM][FN + 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r16 = lane & 15, kq = lane >> 4;
  int local = blockIdx.x, cnt, seg0 = 0, wp, w1_row0;
  int64_t hoff = 0, w2_off;
  if (p.single) {
    cnt = (int)p.T_tokens;
    wp = p.groups[0].width_pad;
    w1_row0 = p.groups[0].w1_row0;
    w2_off = p.groups[0].w2_off;
  } else {
    const GroupLanes gl = request_groups(p.work, p.seg_off, p.groups, p.h_off, p.G);
    if (local >= p.work[p.G]) return;
    const WorkItem it = find_item(gl, p.G, local);
    local = it.local;
    seg0 = it.seg0;
    cnt = it.cnt;
    wp = it.wp;
    hoff = it.hoff;
    w1_row0 = it.w1_row0;
    w2_off = it.w2_off;
  }
  const int K = (MODE == 1) ? p.d : wp;
  const int n_nt = (MODE == 1) ? wp / 16 : (p.d + FN - 1) / FN;
  const int n_mt = (cnt + FM - 1) / FM;
  if (p.single && local >= n_mt * n_nt) return;
  const int mt = local % n_mt, nt = local / n_mt;              // neighbours share the weights
  // this lane's row of A and rows of the two 16-row blocks of B (past the end: a row that exists, never stored)
  const int ar = min(mt * FM + r16, cnt - 1);
  const float *b0, *b1;
  if (MODE == 1) {
    b0 = p.B + ((int64_t)w1_row0 + (nt >> 1) * 2 * IL + (nt & 1) * 16 + r16) * p.ldb;
    b1 = b0 + (int64_t)IL * p.ldb;
  } else {
    b0 = p.B + w2_off + (int64_t)min(nt * FN + r16, p.d - 1) * wp;
    b1 = p.B + w2_off + (int64_t)min(nt * FN + 16 + r16, p.d - 1) * wp;
  }
  auto fetch = [&](const float* row, int k) {
    f32x4_t v = {0.0f, 0.0f, 0.0f, 0.0f};
    if constexpr (VEC) {
      if (k < K) v = *reinterpret_cast<const f32x4_t*>(row + k);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (k + j < K) v[j] = row[k + j];
    }
    return v;
  };
  f32x4_t acc0 = {0.0f, 0.0f, 0.0f, 0.0f}, acc1 = acc0;
  const float* a = nullptr;
  for (int k0 = wave * 16; k0 < K; k0 += FC * 64) {
    f32x4_t av[FC], b0v[FC], b1v[FC];
#pragma unroll
    for (int c = 0; c < FC; ++c)
      if (k0 + c * 64 < K) {
        b0v[c] = fetch(b0, k0 + c * 64 + kq * 4);
        b1v[c] = fetch(b1, k0 + c * 64 + kq * 4);
      }
    if (!a) {                                                  // (behind the first weights: the map is one more round trip)
      if (MODE == 1) a = p.A + (int64_t)(p.slot2tok ? p.slot2tok[seg0 + ar] : seg0 + ar) * p.d;
      else a = p.A + hoff + (int64_t)ar * wp;
    }
#pragma unroll
    for (int c = 0; c < FC; ++c)
      if (k0 + c * 64 < K) av[c] = fetch(a, k0 + c * 64 + kq * 4);
#pragma unroll
    for (int c = 0; c < FC; ++c)
      if (k0 + c * 64 < K) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(av[c][j], b0v[c][j], acc0, 0, 0, 0);
          acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(av[c][j], b1v[c][j], acc1, 0, 0, 0);
        }
      }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {                                // a lane holds rows 4 kq .. + 3 of column r16
    red[wave][kq * 4 + i][r16] = acc0[i];
    red[wave][kq * 4 + i][16 + r16] = acc1[i];
  }
  __syncthreads();
  const int row = tid >> 4, col = tid & 15, r = mt * FM + row;
  if (r >= cnt) return;
  float s0 = 0.0f, s1 = 0.0f;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    s0 += red[w][row][col];
    s1 += red[w][row][16 + col];
  }
  if (MODE == 1) {
    p.C[hoff + (int64_t)r * wp + nt * 16 + col] = silu_f32(s0) * s1;
  } else {
    float* out = p.C + (int64_t)(seg0 + r) * p.d + nt * FN + col;
    if (nt * FN + col < p.d) out[0] = s0;
    if (nt * FN + 16 + col < p.d) out[16] = s1;
  }
}

// Which kernel contraction `which` of an fp32 batch runs.  While the large tiles leave the chip idle, their launch is as long as one
// tile's chain of K steps of 64, 5.2 us each; that is what some 3500 of the small tiles take per step (a rate of 0.7 of the large
// ones' on a full chip).  The small tiles' launch costs about 1.6 us more to start, which counts where K is short.  The two
// contractions differ in tiles, so each decides for itself.  us per forward, gate/up + down in tiles of 64 + 64 rows / 64 + 16 / 16
// + 16: dense, d = 256, d_ff = 1024 at 512 tokens (gate/up 2048 small tiles, down 256) 113 / 34.1 / 26.9, 1024 tokens 113 / 40.6 /
// 44.2, 4096 tokens 157 / 124 / 157; d = d_ff = 256, 8192 tokens 63.9 / 66.1 / 80.9; d = 1024, d_ff = 4096, 128 tokens 432 / 115 /
// 91, 2048 tokens 812 / 897 / 1145; 12 experts of 128, d = 512, 1024 tokens 90.7 / 89.0 / 78.5, 4096 tokens 193 / 215 / 230.
static bool choose_f32_small(const Engine& e, int64_t T, int which) {
  if (e.dtype == 1) return false;
  const int forced = which == 1 ? tuning().f32_rows1 : tuning().f32_rows2;
  if (forced == FM || forced == SB) return forced == FM;
  // K steps of a row of small tiles of group g, and of one tile
  auto row_steps = [&](int g) { return which == 1 ? (int64_t)(e.width_pad_host[g] / 16) * cdiv(e.d, SK) : (int64_t)cdiv(e.d, FN) * cdiv(e.width_pad_host[g], SK); };
  int64_t chain = cdiv(e.d, SK), always = 0, routed = 0;
  if (which == 2) chain = cdiv(*std::max_element(e.width_pad_host, e.width_pad_host + e.G), SK);
  for (int g = 0; g < e.G; ++g) (g < e.n_always ? always : routed) += row_steps(g);
  const int64_t groups = e.G - e.n_always, entries = T * e.S_dyn, touched = std::min<int64_t>(groups, entries);
  int64_t steps = always * ((T + FM - 1) / FM);
  if (groups > 0) steps += (entries / FM + touched / 2) * routed / groups;
  return steps <= 3500 * chain - 1100;
}

static bool f32_small(const Engine& e, int64_t T, int which) {
  if (e.plan_T == T) return (which == 1 ? e.plan1 : e.plan2) != 0;
  return choose_f32_small(e, T, which);
}

void simt_plan_tiles(Engine& e, int64_t T) {
  e.plan1 = choose_f32_small(e, T, 1) ? 1 : 0;
  e.plan2 = choose_f32_small(e, T, 2) ? 1 : 0;
  e.plan_T = T;
}

template <int MODE>
static hipError_t launch_simt(const Engine& e, int64_t T, const SimtArgs<float>& a, int64_t n, hipStream_t s) {
  const dim3 grid((unsigned)n), block(256);
  if (!f32_small(e, T, MODE)) hipLaunchKernelGGL((grouped_gemm_simt<float, MODE>), grid, block, 0, s, a);
  else if (a.vec) hipLaunchKernelGGL((grouped_gemm_f32<MODE, true>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((grouped_gemm_f32<MODE, false>), grid, block, 0, s, a);
  return hipGetLastError();
}
template <int MODE>
static hipError_t launch_simt(const Engine&, int64_t, const SimtArgs<bf16_t>& a, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL((grouped_gemm_simt<bf16_t, MODE>), dim3((unsigned)n), dim3(256), 0, s, a);
  return hipGetLastError();
}

template <typename T>
static hipError_t run_simt(const Engine& e, const void* x, int64_t Tn, char* ws, const WsLayout& L, void* y,
                           hipStream_t s, int stage) {
  SimtArgs<T> a;
  a.groups = e.groups;
  a.seg_off = reinterpret_cast<const int32_t*>(ws + L.seg_off);
  a.h_off = reinterpret_cast<const int64_t*>(ws + L.h_off);
  a.G = e.G;
  a.d = e.d;
  a.ldb = e.ldw1;
  a.b_tiled = e.w_tiled;
  a.T_tokens = Tn;
  a.single = (e.G == 1 && e.n_always == 1) ? 1 : 0;
  a.A = static_cast<const T*>(x);
  a.B = static_cast<const T*>(e.w1);
  a.C = reinterpret_cast<T*>(ws + L.h);
  a.work = reinterpret_cast<const int32_t*>(ws + L.work1);
  a.slot2tok = a.single ? nullptr : reinterpret_cast<const int32_t*>(ws + L.slot2tok);
  // (the workspace and the weights are 256-byte aligned and H's rows a multiple of 32 wide; x is the caller's)
  a.vec = (sizeof(T) == 4 && !e.w_tiled && e.d % 4 == 0 && e.ldw1 % 4 == 0 && reinterpret_cast<uintptr_t>(x) % 16 == 0) ? 1 : 0;
  if (stage != 2) {
    const hipError_t err = launch_simt<1>(e, Tn, a, gemm_work_bound(e, Tn, 1), s);
    if (err != hipSuccess || stage == 1) return err;
  }
  a.vec = (sizeof(T) == 4 && !e.w_tiled) ? 1 : 0;
  a.A = reinterpret_cast<const T*>(ws + L.h);
  a.B = static_cast<const T*>(e.w2);
  a.C = e.direct_output() ? static_cast<T*>(y) : reinterpret_cast<T*>(ws + L.y_slots);
  a.work = reinterpret_cast<const int32_t*>(ws + L.work2);
  a.slot2tok = nullptr;
  return launch_simt<2>(e, Tn, a, gemm_work_bound(e, Tn, 2), s);
}

hipError_t launch_experts_simt(const Engine& e, const void* x, int64_t T, char* ws, const WsLayout& L, void* y,
                               hipStream_t s, int stage) {
  if (e.dtype == 1) return run_simt<bf16_t>(e, x, T, ws, L, y, s, stage);
  return run_simt<float>(e, x, T, ws, L, y, s, stage);
}

// which as in bf16_gemm_tile (no tiles of dynamic height and no persistent kernel here)
int simt_gemm_tile(int which, const Engine& e, int64_t T) {
  if (which >= 5) return 0;
  return !f32_small(e, T, which == 1 || which == 3 ? 1 : 2) ? SB : which <= 2 ? FM : FN;
}

}  // namespace cmoe
