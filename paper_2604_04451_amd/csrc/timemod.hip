// Timestep injection (Sec. 2.1, Fig. 2): the projected timestep embedding of one denoising step.
//   f = [cos(t w_i), sin(t w_i)], w_i = 10000^(-i / half)          sinusoidal features, freq_dim = 2 half
//   e = W2 silu(W1 f + b1) + b2                                     [D]
//   t_mod  = reshape(Wp silu(e) + bp, [6, D])                       modulation rows of every block
//   t_head = [e, e]                                                 the head adds e to both rows of its table
// Three matrix-vector products with bf16 weights and fp32 activations: HBM-bound on the weights
// (2 (D F + D D + 6 D D) bytes), one wave per output row, 16-byte weight loads.
#include "chorus_ops.h"
#include "common.h"

namespace chorus {
namespace {

// Feature i of [cos(t w), sin(t w)]
__device__ __forceinline__ float sinusoid(float t, int i, int half) {
  const int j = i < half ? i : i - half;
  const float a = t * exp2f(-(float)j / (float)half * 13.287712379549449f);  // w = 10000^(-j/half)
  float sn, cs;
  sincosf(a, &sn, &cs);
  return i < half ? cs : sn;
}

// More features than this are made in a launch of their own, once and not by every workgroup. D = 1536, with the launch /
// without: 2048 features 20.2 / 19.9 us, 4096 21.6 / 21.9, 8192 24.2 / 27.2.
constexpr int kFeatureLds = 2048;
constexpr int kSiluLdsFrom = 2560, kSiluLds = 8192;  // values of a vector in LDS, up to 32 KB
constexpr int kGemvBlocks = 1024;  // four workgroups on every compute unit

__global__ __launch_bounds__(256) void sinusoid_kernel(float t, int half, float* __restrict__ f) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < 2 * half) f[i] = sinusoid(t, i, half);
}

// out[n] = sum_k W[n][k] act(x[k]) + b[n]; act: silu (SILU_IN) or nothing. One wave per row n at a time; K % 8 == 0.
// The waves of a compute unit keep enough loads in flight between them: with four of a lane's own the call was slower (D =
// 3072 43.2 us, 40.4 with one; 1536 17.0 / 16.9). out2 (optional) receives the same values (the two head rows). FEATURES: x
// is the sinusoidal features of t (K of them), made by every workgroup for itself: one sine per thread instead of a
// launch in front of this one (4.8 us). IN_LDS: a workgroup puts act(x) into LDS once for all its rows; made again for every
// row the exponentials take longer than the weights.
template <bool SILU_IN, bool FEATURES, bool IN_LDS>
__global__ __launch_bounds__(256) void gemv_bf16w_kernel(const uint16_t* __restrict__ W, const float* __restrict__ x_in,
                                                         const float* __restrict__ b, float* __restrict__ out,
                                                         float* __restrict__ out2, int N, int K, float t) {
  extern __shared__ __attribute__((aligned(16))) float s_f[];  // [K] (IN_LDS)
  static_assert(IN_LDS || !FEATURES, "features are made in LDS");
  auto act = [](float v) { return SILU_IN ? v / (1.0f + __expf(-v)) : v; };
  if constexpr (IN_LDS) {
    for (int i = threadIdx.x; i < K; i += 256) s_f[i] = FEATURES ? sinusoid(t, i, K / 2) : act(x_in[i]);
    __syncthreads();
  }
  const float* x = IN_LDS ? s_f : x_in;
  const int lane = threadIdx.x & 63;
  for (int n = blockIdx.x * 4 + (threadIdx.x >> 6); n < N; n += gridDim.x * 4) {
    const uint16_t* w = W + (long)n * K;
    float acc = 0.f;
    for (int k = lane * 8; k < K; k += 64 * 8) {
      const u32x4 u = *reinterpret_cast<const u32x4*>(w + k);
      const f32x4 x0 = *reinterpret_cast<const f32x4*>(x + k);
      const f32x4 x1 = *reinterpret_cast<const f32x4*>(x + k + 4);
      const float xv[8] = {x0[0], x0[1], x0[2], x0[3], x1[0], x1[1], x1[2], x1[3]};
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float v = IN_LDS ? xv[j] : act(xv[j]);
        const float wv = __uint_as_float((j & 1) ? (u[j >> 1] & 0xffff0000u) : (u[j >> 1] << 16));
        acc = __builtin_fmaf(wv, v, acc);
      }
    }
    acc = wave_sum(acc);
    if (lane == 0) {
      const float r = acc + (b ? b[n] : 0.f);
      out[n] = r;
      if (out2) out2[n] = r;
    }
  }
}

// W silu(x) + b. Long vectors by way of LDS; short ones are passed on to the rows directly, whose loads then wait for nothing
// (the call from HBM, directly / through LDS: D = 1024 12.6 / 14.8 us, 1536 19.2 / 20.3, 2048 24.7 / 25.7, 3072 43.3 / 41.5, 5120
// 103.7 / 90.1, 8192 240 / 195).
void launch_gemv_silu(const uint16_t* W, const float* x, const float* b, float* out, float* out2, int N, int K, hipStream_t s) {
  const int rows = (N + 3) / 4, most = kGemvBlocks;
  if (K >= kSiluLdsFrom && K <= kSiluLds)
    hipLaunchKernelGGL((gemv_bf16w_kernel<true, false, true>), dim3((unsigned)(rows < most ? rows : most)), dim3(256), (size_t)K * 4, s, W,
                       x, b, out, out2, N, K, 0.f);
  else
    hipLaunchKernelGGL((gemv_bf16w_kernel<true, false, false>), dim3((unsigned)rows), dim3(256), 0, s, W, x, b, out, out2, N, K, 0.f);
}

}  // namespace
}  // namespace chorus

using namespace chorus;

extern "C" {

size_t chorus_time_mod_workspace_bytes(int32_t D, int32_t freq_dim) {
  if (D <= 0 || freq_dim <= 0) return 0;
  return align_up((size_t)freq_dim * 4, 256) + align_up((size_t)D * 4, 256);
}

int32_t chorus_time_mod(float t, int32_t freq_dim, int32_t D, const chorus_time_weights* w, float* t_mod, float* t_head,
                        void* ws, size_t ws_bytes, void* stream) {
  if (!w || !t_mod || !t_head || D <= 0 || freq_dim <= 0) return CHORUS_E_ARG;
  if (!w->w_t1 || !w->w_t2 || !w->w_tp) return CHORUS_E_ARG;
  if ((freq_dim & 7) != 0 || (D & 7) != 0) return CHORUS_E_SHAPE;
  if (!aligned16(w->w_t1) || !aligned16(w->w_t2) || !aligned16(w->w_tp) || !aligned16(t_mod) || !aligned16(t_head))
    return CHORUS_E_ARG;
  if (!ws || !aligned16(ws) || ws_bytes < chorus_time_mod_workspace_bytes(D, freq_dim)) return CHORUS_E_WORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  float* f = (float*)ws;
  float* h = (float*)((uint8_t*)ws + align_up((size_t)freq_dim * 4, 256));
  // h = W1 f + b1;  e = W2 silu(h) + b2 -> both head rows;  t_mod = Wp silu(e) + bp
  if (freq_dim <= kFeatureLds) {
    hipLaunchKernelGGL((gemv_bf16w_kernel<false, true, true>), dim3((unsigned)((D + 3) / 4)), dim3(256), (size_t)freq_dim * 4, s, w->w_t1,
                       (const float*)nullptr, w->b_t1, h, (float*)nullptr, D, freq_dim, t);
  } else {
    hipLaunchKernelGGL(sinusoid_kernel, dim3((unsigned)((freq_dim + 255) / 256)), dim3(256), 0, s, t, freq_dim / 2, f);
    CHORUS_LAUNCH_CHECK();
    hipLaunchKernelGGL((gemv_bf16w_kernel<false, false, false>), dim3((unsigned)((D + 3) / 4)), dim3(256), 0, s, w->w_t1, f, w->b_t1, h,
                       (float*)nullptr, D, freq_dim, 0.f);
  }
  CHORUS_LAUNCH_CHECK();
  launch_gemv_silu(w->w_t2, h, w->b_t2, t_head, t_head + D, D, D, s);
  CHORUS_LAUNCH_CHECK();
  launch_gemv_silu(w->w_tp, t_head, w->b_tp, t_mod, nullptr, 6 * D, D, s);
  CHORUS_LAUNCH_CHECK();
  return CHORUS_OK;
}

}  // extern "C"
