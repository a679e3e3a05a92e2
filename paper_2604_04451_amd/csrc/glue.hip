// Step glue around the block stack: patch embedding of the selected tokens, the
// output head fused with the sampler update on the selected tokens, and the text
// projection. The sampler (Sec. 4.1: DPM++, default settings) is DPM-Solver++ in
// data-prediction form on the rectified-flow path: chorus_head_update is its first-order
// step written as the Euler update, chorus_head_update_solver the multistep form with
// classifier-free guidance and the latent fusion of Eq. 6 folded into the same pass.
#include <cmath>
#include <type_traits>

#include "chorus_ops.h"
#include "common.h"

namespace chorus {
namespace {

// Patches of other than 64 values: one thread per (selected token, channel): the ph x pw cell of that channel, split
// into a bf16 head and a bf16 remainder so the K = C*ph*pw GEMM keeps fp32-level accuracy
__global__ __launch_bounds__(256) void patch_gather_kernel(const float* __restrict__ latent,
                                                           const int* __restrict__ token_idx, long Ls, int C, int T,
                                                           int Hl, int Wl, int ph, int pw, uint16_t* __restrict__ hi,
                                                           uint16_t* __restrict__ lo) {
  long g = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= Ls * C) return;
  long i = g / C;
  int ch = (int)(g - i * C);
  const int Wg = Wl / pw, Hg = Hl / ph;
  long n = token_idx ? (long)token_idx[i] : i;
  int wg = (int)(n % Wg), hg = (int)((n / Wg) % Hg), t = (int)(n / ((long)Wg * Hg));
  const int cell = ph * pw;
  const float* src = latent + (((long)ch * T + t) * Hl + (long)hg * ph) * Wl + (long)wg * pw;
  uint16_t* oh = hi + i * (long)(C * cell) + ch * cell;
  uint16_t* ol = lo + i * (long)(C * cell) + ch * cell;
  for (int dy = 0; dy < ph; ++dy)
    for (int dx = 0; dx < pw; ++dx) {
      float v = src[(long)dy * Wl + dx];
      uint16_t h = f32_to_bf16(v);
      oh[dy * pw + dx] = h;
      ol[dy * pw + dx] = f32_to_bf16(v - bf16_to_f32(h));
    }
}

// Where a token's cell of one channel lies: the token's original id gives its place on the grid.
struct LatentGrid {
  int C, T, Hl, Wl, ph, pw;
  __device__ __forceinline__ long cell(long token, int ch) const {
    const int Wg = Wl / pw, Hg = Hl / ph;
    const int wg = (int)(token % Wg), hg = (int)((token / Wg) % Hg), t = (int)(token / ((long)Wg * Hg));
    return (((long)ch * T + t) * Hl + (long)hg * ph) * Wl + (long)wg * pw;
  }
};

// What a step does to PW consecutive elements (from offset o, of token n) of the latent of a selected token: load()
// requests what it needs, store() finishes once the head's output for them is known. All loads stand before the first
// store, which may alias them for all the compiler knows.
struct EulerUpdate {
  static constexpr int kPasses = 1;
  float* latent;
  const float* SL;
  const uint8_t* mask_edit;
  float dsigma;
  template <int PW>
  struct Cell {
    float x[PW];
    bool keep;
  };
  // Eq. 6 on the selected tokens when a mask is given: one outside M_edit receives the source latent instead
  template <int PW>
  __device__ __forceinline__ void load(Cell<PW>& c, long n, long o) const {
    c.keep = mask_edit == nullptr || mask_edit[n] != 0;
#pragma unroll
    for (int e = 0; e < PW; ++e) c.x[e] = c.keep ? latent[o + e] : SL[o + e];
  }
  template <int PW>
  __device__ __forceinline__ void store(const Cell<PW>& c, long o, const float (&v)[PW], const float (&)[PW]) const {
#pragma unroll
    for (int e = 0; e < PW; ++e) latent[o + e] = c.keep ? c.x[e] + dsigma * v[e] : c.x[e];
  }
};

//   v = CFG ? vu + g (vc - vu) : vc;  x0 = x - sigma_s v;  D = c0 x0 + c1 x0_prev (tokens with history) or x0
//   x0_prev <- x0;  latent <- M_edit ? rho x + A D : SL
template <bool CFG>
struct SolverUpdate {
  static constexpr int kPasses = CFG ? 2 : 1;
  float* latent;
  float* x0_prev;
  const uint8_t* hist;
  const float* SL;
  const uint8_t* mask_edit;
  chorus_sampler_coef cf;
  float guidance;
  template <int PW>
  struct Cell {
    float x[PW], prev[PW], src[PW];
    bool second, keep;
  };
  template <int PW>
  __device__ __forceinline__ void load(Cell<PW>& c, long n, long o) const {
    c.second = cf.c1 != 0.f && (hist == nullptr || hist[n] != 0);
    c.keep = mask_edit == nullptr || mask_edit[n] != 0;
#pragma unroll
    for (int e = 0; e < PW; ++e) {
      c.x[e] = latent[o + e];
      c.prev[e] = c.second ? x0_prev[o + e] : 0.f;
      c.src[e] = c.keep ? 0.f : SL[o + e];
    }
  }
  template <int PW>
  __device__ __forceinline__ void store(const Cell<PW>& c, long o, const float (&vc)[PW], const float (&vu)[PW]) const {
    float x0[PW], r[PW];
#pragma unroll
    for (int e = 0; e < PW; ++e) {
      const float v = CFG ? vu[e] + guidance * (vc[e] - vu[e]) : vc[e];
      x0[e] = c.x[e] - cf.sigma_s * v;
      const float d = c.second ? cf.c0 * x0[e] + cf.c1 * c.prev[e] : x0[e];
      r[e] = c.keep ? cf.rho * c.x[e] + cf.A * d : c.src[e];
    }
#pragma unroll
    for (int e = 0; e < PW; ++e) {
      if (x0_prev) x0_prev[o + e] = x0[e];
      latent[o + e] = r[e];
    }
  }
};

// One row of a token's cell (pw elements) of one channel; vc(e) and vu(e) give the head's output at element e of it.
template <typename U, typename V, typename V2>
__device__ __forceinline__ void update_row(const U& upd, long n, long o, int pw, V vc, V2 vu) {
  if (pw == 2) {
    typename U::template Cell<2> c;
    upd.load(c, n, o);
    const float a[2] = {vc(0), vc(1)}, b[2] = {vu(0), vu(1)};
    upd.store(c, o, a, b);
  } else {
    for (int e = 0; e < pw; ++e) {
      typename U::template Cell<1> c;
      upd.load(c, n, o + e);
      const float a[1] = {vc(e)}, b[1] = {vu(e)};
      upd.store(c, o + e, a, b);
    }
  }
}

// The update alone, from v in memory: one (selected token, channel) cell per thread.
template <typename U>
__global__ __launch_bounds__(256) void unpatch_update_kernel(const float* __restrict__ vc, const float* __restrict__ vu,
                                                             const int* __restrict__ token_idx, long Ls, LatentGrid g, U upd) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= Ls * g.C) return;
  const long tok = i / g.C;
  const int ch = (int)(i - tok * g.C), cell = g.ph * g.pw;
  const long n = token_idx ? (long)token_idx[tok] : tok;
  const long row = tok * (long)(g.C * cell) + ch * cell, base = g.cell(n, ch);
  struct Mem {
    const float* p;
    __device__ __forceinline__ float operator()(int e) const { return p[e]; }
  };
  for (int dy = 0; dy < g.ph; ++dy)
    update_row(upd, n, base + (long)dy * g.Wl, g.pw, Mem{vc + row + dy * g.pw}, Mem{vu + row + dy * g.pw});
}

// ---------------------------------------------------------------------------
// Patch embedding in one pass: x[token][n] = sum_k W[n][k] patch[token][k] + b[n], the fp32 patch split into a bf16
// value and a bf16 remainder whose products share one fp32 accumulator. What it cannot do without is writing x once
// (201 MB at 32760 x 1536); as a gather and two GEMMs it wrote x, read it and wrote it again: 153 us there, now 47 (streaming stores: 70).
//
// A workgroup takes 64 tokens and a range of columns. Its four waves gather the patches (lanes along tokens, so that a
// wave reads 512 contiguous bytes per latent row) into LDS as [64][hi 64 | lo 64] bf16; each wave then holds all of it
// as MFMA fragments in registers (64 of them) and walks its own 16-column blocks: two 16-byte loads per lane of W (cached,
// 128 bytes per output column), 16 MFMAs, four stores of 16 bytes per lane. The columns are split over workgroups where
// the tokens alone do not give the chip two workgroups per compute unit.
// ---------------------------------------------------------------------------
constexpr int kEmbedTok = 64, kEmbedP = 64;
constexpr int kEmbedStride = 2 * kEmbedP + 16;  // elements per LDS row: 32 bytes of padding keep the fragment reads apart

__global__ __launch_bounds__(256) void patch_embed_kernel(const float* __restrict__ latent, const int* __restrict__ token_idx,
                                                          long Ls, LatentGrid g, const uint16_t* __restrict__ W,
                                                          const float* __restrict__ bias, int D, int cols,
                                                          float* __restrict__ x) {
  __shared__ __attribute__((aligned(16))) uint16_t sp[kEmbedTok * kEmbedStride];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const long tok0 = (long)blockIdx.x * kEmbedTok;
  const int lj = lane & 15, lg = lane >> 4;
  const int n_begin = blockIdx.y * cols, n_end = n_begin + cols < D ? n_begin + cols : D;
  {
    const long tok = tok0 + lane < Ls ? tok0 + lane : Ls - 1;  // rows past the end are gathered again and not stored
    const long base = g.cell(token_idx ? (long)token_idx[tok] : tok, 0);
    const long plane = (long)g.T * g.Hl * g.Wl;
    const int cell = g.ph * g.pw;
    float v[kEmbedP / 4];
#pragma unroll
    for (int j = 0; j < kEmbedP / 4; ++j) {
      const int p = wave * (kEmbedP / 4) + j, e = p % cell;
      v[j] = latent[base + (p / cell) * plane + (long)(e / g.pw) * g.Wl + e % g.pw];
    }
#pragma unroll
    for (int j = 0; j < kEmbedP / 4; j += 8) {
      u32x4 hi, lo;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float a = v[j + 2 * k], b = v[j + 2 * k + 1];
        hi[k] = pack_bf16x2(a, b);
        lo[k] = pack_bf16x2(a - __uint_as_float(hi[k] << 16), b - __uint_as_float(hi[k] & 0xffff0000u));
      }
      uint16_t* row = sp + lane * kEmbedStride + wave * (kEmbedP / 4) + j;
      *reinterpret_cast<u32x4*>(row) = hi;
      *reinterpret_cast<u32x4*>(row + kEmbedP) = lo;
    }
  }
  __syncthreads();
  bf16x8 a[4][4];  // [16-token block][k steps of 32: hi 0, hi 1, lo 0, lo 1]
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) a[m][ks] = *reinterpret_cast<const bf16x8*>(sp + (16 * m + lj) * kEmbedStride + 32 * ks + 8 * lg);
  constexpr int NB = 2;  // 16-column blocks at a time
  // The weights of the next blocks are requested ahead of this block's stores: memory operations complete in order, so
  // weights requested behind stores arrive when those have drained.
  bf16x8 w[2][NB][2];
  f32x4 bv[2][NB];
  auto fetch = [&](int set, int n0) {
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int n = n0 + 16 * b + lj < D ? n0 + 16 * b + lj : D - 1;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) w[set][b][ks] = *reinterpret_cast<const bf16x8*>(W + (long)n * kEmbedP + 32 * ks + 8 * lg);
      const int nc = n0 + 16 * b + 4 * lg;  // the lane's four output columns: D % 8 == 0, in or out together
      bv[set][b] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (bias && nc < D) bv[set][b] = *reinterpret_cast<const f32x4*>(bias + nc);
    }
  };
  auto block = [&](int set, int n0) {
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      f32x4 r[NB];
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[set][b][ks & 1], a[m][ks], acc, 0, 0, 0);
        r[b] = acc + bv[set][b];
      }
      const long tok = tok0 + 16 * m + lj;
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const int nc = n0 + 16 * b + 4 * lg;
        if (tok < Ls && nc < n_end) *reinterpret_cast<f32x4*>(x + tok * (long)D + nc) = r[b];
      }
    }
  };
  int n0 = n_begin + 16 * NB * wave;
  if (n0 < n_end) fetch(0, n0);
  for (; n0 < n_end; n0 += 2 * 64 * NB) {  // two turns: the sets are named, not indexed
    const int n1 = n0 + 64 * NB;
    if (n1 < n_end) fetch(1, n1);
    block(0, n0);
    if (n1 >= n_end) break;
    if (n1 + 64 * NB < n_end) fetch(0, n1 + 64 * NB);
    block(1, n1);
  }
}

// ---------------------------------------------------------------------------
// Output head and sampler update in one pass over x: LayerNorm + modulation in fp32, one rounding to bf16, the product
// with the head's weights, and the update of the tokens' latents, with the guided pass over x_uncond in the same
// workgroup. What it cannot do without is reading x (and x_uncond) once (HBM-bound: 90 us for 402 MB at 32760 x 1536 with
// guidance). Apart, the bf16 rows went to memory and back and v as well: 191 us; now 100.
//
// One workgroup of eight waves per compute unit walks over groups of 16 tokens with the head's weights in registers: a
// wave holds all 64 columns over its eighth of D (96 registers at D = 1536). Read again for every 16 tokens they were
// 805 MB through the L1s, 80 us more than the stream itself. Per group a wave normalises two rows (in registers, requested
// one group ahead) into LDS ([16][D] bf16), multiplies its eighth, and leaves a partial v; the eight partials are added in
// ascending order by the threads that update the latents, whose values were requested before the product. The barriers
// order the LDS only, so all of those requests stay in flight across them. D = 256 KS, P <= 64.
// ---------------------------------------------------------------------------
constexpr int kHeadTok = 16, kHeadThreads = 512, kHeadP = 64;
constexpr int kHeadVStride = kHeadTok + 1;
constexpr int kHeadPart = kHeadP * kHeadVStride;  // floats of one partial v
inline size_t head_lds_bytes(int D) { return (size_t)kHeadTok * (D + 16) * 2 + (size_t)2 * D * 4 + (size_t)9 * kHeadPart * 4; }

template <int KS, typename U>
__global__ __launch_bounds__(kHeadThreads, 2) void head_update_kernel(const float* __restrict__ x, const float* __restrict__ xu,
                                                                      const float* __restrict__ table,
                                                                      const float* __restrict__ t_head,
                                                                      const uint16_t* __restrict__ W,
                                                                      const float* __restrict__ bias,
                                                                      const int* __restrict__ token_idx, long Ls, int P,
                                                                      LatentGrid g, U upd) {
  constexpr int D = 256 * KS, HS = D + 16, PASSES = U::kPasses;
  extern __shared__ __attribute__((aligned(16))) uint8_t smem_raw[];
  float* s_mul = reinterpret_cast<float*>(smem_raw);  // 1 + scale
  float* s_add = s_mul + D;                           // shift
  float* s_red = s_add + D;                           // [8][kHeadP][kHeadVStride]: the waves' partial v
  float* s_vc = s_red + 8 * kHeadPart;                // [kHeadP][kHeadVStride]: v of the guided pass's first half
  uint16_t* s_h = reinterpret_cast<uint16_t*>(s_vc + kHeadPart);  // [kHeadTok][HS]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lj = lane & 15, lg = lane >> 4;
  const long ngroups = (Ls + kHeadTok - 1) / kHeadTok;
  f32x4 v[2][KS];
  auto fetch = [&](const float* src, long group, int r) {
    const long tok = group * kHeadTok + 2 * wave + r < Ls ? group * kHeadTok + 2 * wave + r : Ls - 1;
    const f32x4* row = reinterpret_cast<const f32x4*>(src + tok * (long)D);
#pragma unroll
    for (int i = 0; i < KS; ++i) v[r][i] = row[lane + 64 * i];
  };
  fetch(x, blockIdx.x, 0);
  fetch(x, blockIdx.x, 1);
  bf16x8 w[4][KS];
#pragma unroll
  for (int nb = 0; nb < 4; ++nb) {
    const int n = 16 * nb + lj < P ? 16 * nb + lj : P - 1;  // columns past P are computed again and not used
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      w[nb][ks] = *reinterpret_cast<const bf16x8*>(W + (long)n * D + wave * (D / 8) + 32 * ks + 8 * lg);
  }
  for (int i = tid; i < D; i += kHeadThreads) {
    s_mul[i] = 1.0f + table[D + i] + t_head[D + i];
    s_add[i] = table[i] + t_head[i];
  }
  lds_barrier();
  // one row of a cell per thread, where that is all there is to do: its values are requested ahead
  const bool one_each = g.pw == 2 && kHeadTok * g.C * g.ph == kHeadThreads && (long)g.C * g.T * g.Hl * g.Wl <= 0x7fffffffL;
  const int cell = g.ph * g.pw, my_t = tid % kHeadTok, my_row = tid / kHeadTok, my_ch = my_row / g.ph, my_dy = my_row - my_ch * g.ph;

  for (long group = blockIdx.x; group < ngroups; group += gridDim.x) {
    const long tok0 = group * kHeadTok;
#pragma unroll
    for (int pass = 0; pass < PASSES; ++pass) {
      const bool last = pass + 1 == PASSES;
      // requests, in the order in which they are needed: the latents of this group, then each of the next rows as soon as this
      // one's registers are free (with both rows requested behind the second one nothing was in flight while they were normalised)
      typename U::template Cell<2> mine;
      int mine_o = 0;  // 32 bits: the widest variant is at the register limit
      if (last && one_each) {
        const long tok = tok0 + my_t < Ls ? tok0 + my_t : Ls - 1;
        const long n = token_idx ? (long)token_idx[tok] : tok;
        mine_o = (int)(g.cell(n, my_ch) + (long)my_dy * g.Wl);
        upd.load(mine, n, mine_o);
      }
      auto normalise = [&](auto first, auto end) {
        float s[2], q[2];
#pragma unroll
        for (int r = first; r < end; ++r) {
          s[r] = 0.f;
#pragma unroll
          for (int i = 0; i < KS; ++i) s[r] += (v[r][i][0] + v[r][i][1]) + (v[r][i][2] + v[r][i][3]);
        }
#pragma unroll
        for (int r = first; r < end; ++r) s[r] = wave_sum(s[r]) * (1.0f / (float)D);  // the mean
#pragma unroll
        for (int r = first; r < end; ++r) {
          q[r] = 0.f;
#pragma unroll
          for (int i = 0; i < KS; ++i) {
            const float a = v[r][i][0] - s[r], b = v[r][i][1] - s[r], c = v[r][i][2] - s[r], d = v[r][i][3] - s[r];
            q[r] += (a * a + b * b) + (c * c + d * d);
          }
        }
#pragma unroll
        for (int r = first; r < end; ++r) q[r] = rsqrtf(wave_sum(q[r]) * (1.0f / (float)D) + 1e-6f);
#pragma unroll
        for (int i = 0; i < KS; ++i) {
          const f32x4 mu = reinterpret_cast<const f32x4*>(s_mul)[lane + 64 * i];
          const f32x4 ad = reinterpret_cast<const f32x4*>(s_add)[lane + 64 * i];
#pragma unroll
          for (int r = first; r < end; ++r) {
            float y[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) y[e] = (v[r][i][e] - s[r]) * q[r] * mu[e] + ad[e];
            *reinterpret_cast<uint2*>(s_h + (2 * wave + r) * HS + 4 * (lane + 64 * i)) =
                make_uint2(pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3]));
          }
        }
      };
      using R0 = std::integral_constant<int, 0>;
      using R1 = std::integral_constant<int, 1>;
      using R2 = std::integral_constant<int, 2>;
      const float* next = !last ? xu : group + gridDim.x < ngroups ? x : nullptr;
      if (next) {
        const long next_group = last ? group + gridDim.x : group;
        normalise(R0{}, R1{});
        fetch(next, next_group, 0);
        __builtin_amdgcn_sched_barrier(0);
        normalise(R1{}, R2{});
        fetch(next, next_group, 1);
      } else {
        // nothing to request: both rows' chains together (embedding and head: 98 tokens 19.3 -> 18.8 us, 32760 without
        // guidance 105.6 -> 102.4, with guidance 151.0 -> 153.0)
        normalise(R0{}, R2{});
      }
      lds_barrier();  // the 16 rows are in LDS, and the previous partial v have been read
      f32x4 acc[4];
#pragma unroll
      for (int nb = 0; nb < 4; ++nb) acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const bf16x8 h = *reinterpret_cast<const bf16x8*>(s_h + lj * HS + wave * (D / 8) + 32 * ks + 8 * lg);
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[nb][ks], h, acc[nb], 0, 0, 0);
      }
#pragma unroll
      for (int nb = 0; nb < 4; ++nb)
#pragma unroll
        for (int e = 0; e < 4; ++e) s_red[wave * kHeadPart + (16 * nb + 4 * lg + e) * kHeadVStride + lj] = acc[nb][e];
      lds_barrier();  // the partial v are complete, and no wave reads the rows any more
      struct Sum {
        const float* p;
        const float* bias;
        __device__ __forceinline__ float operator()(int e) const {
          float r = bias ? bias[e] : 0.f;
#pragma unroll
          for (int k = 0; k < 8; ++k) r += p[k * kHeadPart + e * kHeadVStride];
          return r;
        }
      };
      struct One {
        const float* p;
        __device__ __forceinline__ float operator()(int e) const { return p[e * kHeadVStride]; }
      };
      if (!last) {
        for (int i = tid; i < kHeadTok * P; i += kHeadThreads) {
          const int n = i / kHeadTok, t = i % kHeadTok;
          s_vc[n * kHeadVStride + t] = Sum{s_red + n * kHeadVStride + t, bias ? bias + n : nullptr}(0);
        }
      } else if (one_each) {
        const int n0 = my_ch * cell + my_dy * 2;
        const Sum sum{s_red + n0 * kHeadVStride + my_t, bias ? bias + n0 : nullptr};
        const One one{s_vc + n0 * kHeadVStride + my_t};
        const float vl[2] = {sum(0), sum(1)};  // of the last pass
        const float vc[2] = {PASSES == 2 ? one(0) : vl[0], PASSES == 2 ? one(1) : vl[1]};
        if (tok0 + my_t < Ls) upd.store(mine, mine_o, vc, vl);
      } else {
        int first = tid;
        asm volatile("" : "+v"(first));  // made here: the loop's addresses are not kept in registers across the groups
        for (int i = first; i < kHeadTok * g.C * g.ph; i += kHeadThreads) {
          const int t = i % kHeadTok, row = i / kHeadTok, ch = row / g.ph, dy = row - ch * g.ph;
          if (tok0 + t >= Ls) continue;
          const long n = token_idx ? (long)token_idx[tok0 + t] : tok0 + t;
          const int n0 = ch * cell + dy * g.pw;
          const Sum sum{s_red + n0 * kHeadVStride + t, bias ? bias + n0 : nullptr};
          const One one{s_vc + n0 * kHeadVStride + t};
          const long o = g.cell(n, ch) + (long)dy * g.Wl;
          if constexpr (PASSES == 2)
            update_row(upd, n, o, g.pw, one, sum);
          else
            update_row(upd, n, o, g.pw, sum, sum);
        }
      }
    }
  }
}

#define CHK(call)                       \
  do {                                  \
    int32_t st__ = (call);              \
    if (st__ != CHORUS_OK) return st__; \
  } while (0)

// The one-pass head takes widths whose weights fit the registers of eight waves and heads of up to 64 columns; the
// others (D = 5120 among them: 655 KB of weights) run LayerNorm, GEMM and update apart. So does anything misaligned, for
// those calls to refuse.
inline bool head_in_one_pass(const float* x, const float* xu, const chorus_glue_weights* gw, const float* t_head, const void* ws,
                             int D, int P) {
  return (D == 256 || D == 512 || D == 768 || D == 1024 || D == 1280 || D == 1536) && P <= kHeadP && aligned16(x) && aligned16(xu) &&
         aligned16(gw->w_head) && aligned16(gw->b_head) && aligned16(gw->head_table) && aligned16(t_head) && aligned16(ws);
}

template <typename U>
int32_t launch_head(const float* x, const float* xu, const chorus_glue_weights* gw, const float* t_head,
                    const int32_t* token_idx, int64_t Ls, int D, int P, const LatentGrid& g, const U& upd, hipStream_t s) {
  int dev = 0, cus = 0;
  CHORUS_HIP(hipGetDevice(&dev));
  CHORUS_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  const long groups = (Ls + kHeadTok - 1) / kHeadTok;
  const dim3 grid((unsigned)(groups < cus ? groups : cus));
  switch (D / 256) {
#define HEAD_CASE(KS)                                                                                                       \
  case KS: {                                                                                                                \
    auto kern = head_update_kernel<KS, U>;                                                                                  \
    static DynLdsOnce once;                                                                                                 \
    CHK(once.ensure(reinterpret_cast<const void*>(kern), (int)head_lds_bytes(256 * KS)));                                   \
    hipLaunchKernelGGL(kern, grid, dim3(kHeadThreads), head_lds_bytes(256 * KS), s, x, xu, gw->head_table, t_head,          \
                       gw->w_head, gw->b_head, token_idx, (long)Ls, P, g, upd);                                             \
    break;                                                                                                                  \
  }
    HEAD_CASE(1)
    HEAD_CASE(2)
    HEAD_CASE(3)
    HEAD_CASE(4)
    HEAD_CASE(5)
    HEAD_CASE(6)
#undef HEAD_CASE
    default: return CHORUS_E_SHAPE;
  }
  CHORUS_LAUNCH_CHECK();
  return CHORUS_OK;
}

template <typename U>
int32_t launch_unpatch(const float* vc, const float* vu, const int32_t* token_idx, int64_t Ls, const LatentGrid& g,
                       const U& upd, hipStream_t s) {
  const long n = Ls * g.C;
  hipLaunchKernelGGL(unpatch_update_kernel<U>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, vc, vu, token_idx, (long)Ls,
                     g, upd);
  CHORUS_LAUNCH_CHECK();
  return CHORUS_OK;
}

}  // namespace
}  // namespace chorus

using namespace chorus;

extern "C" {

size_t chorus_glue_workspace_bytes(int32_t D, int32_t P, int64_t Ls) {
  if (Ls < 1) Ls = 1;
  size_t embed = 2 * align_up((size_t)Ls * P * 2, 256);
  size_t head = align_up((size_t)Ls * D * 2, 256) + align_up((size_t)Ls * P * 4, 256);
  return embed > head ? embed : head;
}

int32_t chorus_patch_embed(const float* latent, int32_t C, int32_t T, int32_t Hl, int32_t Wl, int32_t ph, int32_t pw,
                           const int32_t* token_idx, int64_t Ls, const chorus_glue_weights* gw, int32_t D, float* x,
                           void* ws, size_t ws_bytes, void* stream) {
  if (Ls < 0 || C <= 0 || T <= 0 || Hl <= 0 || Wl <= 0 || ph <= 0 || pw <= 0 || D <= 0) return CHORUS_E_ARG;
  if (Ls == 0) return CHORUS_OK;
  if (!latent || !gw || !x || !gw->w_patch) return CHORUS_E_ARG;
  const int P = C * ph * pw;
  if (Hl % ph || Wl % pw || P % 64 || D % 8) return CHORUS_E_SHAPE;
  if (!token_idx && Ls > (int64_t)T * (Hl / ph) * (Wl / pw)) return CHORUS_E_SHAPE;
  if (!ws || ws_bytes < chorus_glue_workspace_bytes(D, P, Ls)) return CHORUS_E_WORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  if (P == kEmbedP && aligned16(gw->w_patch) && aligned16(gw->b_patch) && aligned16(x) && aligned16(ws)) {
    const LatentGrid g{C, T, Hl, Wl, ph, pw};
    const long tiles = (Ls + kEmbedTok - 1) / kEmbedTok;
    // columns per workgroup, a multiple of the 128 that four waves take at a time: all of them from 512 token tiles on
    const long want = (512 + tiles - 1) / tiles, most = (D + 127) / 128;
    const int cols = (int)((most + (want < most ? want : most) - 1) / (want < most ? want : most)) * 128;
    if (tiles > 0x7fffffffL) return CHORUS_E_SHAPE;
    hipLaunchKernelGGL(patch_embed_kernel, dim3((unsigned)tiles, (unsigned)((D + cols - 1) / cols)), dim3(256), 0, s, latent,
                       token_idx, (long)Ls, g, gw->w_patch, gw->b_patch, D, cols, x);
    CHORUS_LAUNCH_CHECK();
    return CHORUS_OK;
  }
  uint16_t* hi = (uint16_t*)ws;
  uint16_t* lo = (uint16_t*)((uint8_t*)ws + align_up((size_t)Ls * P * 2, 256));
  long n = Ls * C;
  hipLaunchKernelGGL(patch_gather_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, latent, token_idx, (long)Ls,
                     C, T, Hl, Wl, ph, pw, hi, lo);
  CHORUS_LAUNCH_CHECK();
  CHK(chorus_gemm_bf16(hi, gw->w_patch, Ls, D, P, CHORUS_EPI_F32, x, gw->b_patch, nullptr, nullptr, 1.f, stream));
  CHK(chorus_gemm_bf16(lo, gw->w_patch, Ls, D, P, CHORUS_EPI_RESID, x, nullptr, nullptr, nullptr, 1.f, stream));
  return CHORUS_OK;
}

int32_t chorus_head_update_region(float* latent, const float* x, int64_t Ls, const int32_t* token_idx,
                                  const chorus_glue_weights* gw, const float* t_head, float dsigma, const float* SL,
                                  const uint8_t* mask_edit, int32_t D, int32_t C, int32_t T, int32_t Hl, int32_t Wl,
                                  int32_t ph, int32_t pw, void* ws, size_t ws_bytes, void* stream) {
  if (Ls < 0 || C <= 0 || T <= 0 || Hl <= 0 || Wl <= 0 || ph <= 0 || pw <= 0 || D <= 0) return CHORUS_E_ARG;
  if ((SL != nullptr) != (mask_edit != nullptr)) return CHORUS_E_ARG;
  if (Ls == 0) return CHORUS_OK;
  if (!latent || !x || !gw || !t_head || !gw->w_head || !gw->head_table) return CHORUS_E_ARG;
  const int P = C * ph * pw;
  if (Hl % ph || Wl % pw || P % 8 || D % 64) return CHORUS_E_SHAPE;
  if (!token_idx && Ls > (int64_t)T * (Hl / ph) * (Wl / pw)) return CHORUS_E_SHAPE;
  if (!ws || ws_bytes < chorus_glue_workspace_bytes(D, P, Ls)) return CHORUS_E_WORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  const LatentGrid g{C, T, Hl, Wl, ph, pw};
  const EulerUpdate upd{latent, SL, mask_edit, dsigma};
  if (head_in_one_pass(x, nullptr, gw, t_head, ws, D, P))
    return launch_head(x, x, gw, t_head, token_idx, Ls, D, P, g, upd, s);
  uint16_t* h = (uint16_t*)ws;
  float* v = (float*)((uint8_t*)ws + align_up((size_t)Ls * D * 2, 256));
  CHK(chorus_ln_modulate(x, h, Ls, D, gw->head_table + D, t_head + D, gw->head_table, t_head, 1, stream));
  CHK(chorus_gemm_bf16(h, gw->w_head, Ls, P, D, CHORUS_EPI_F32, v, gw->b_head, nullptr, nullptr, 1.f, stream));
  return launch_unpatch(v, v, token_idx, Ls, g, upd, s);
}

int32_t chorus_head_update(float* latent, const float* x, int64_t Ls, const int32_t* token_idx,
                           const chorus_glue_weights* gw, const float* t_head, float dsigma, int32_t D, int32_t C,
                           int32_t T, int32_t Hl, int32_t Wl, int32_t ph, int32_t pw, void* ws, size_t ws_bytes,
                           void* stream) {
  return chorus_head_update_region(latent, x, Ls, token_idx, gw, t_head, dsigma, nullptr, nullptr, D, C, T, Hl, Wl, ph, pw,
                                   ws, ws_bytes, stream);
}

int32_t chorus_sampler_coefficients(const float* sigmas, int32_t n_steps, int32_t i, int32_t order,
                                    chorus_sampler_coef* out) {
  if (!sigmas || !out || n_steps < 1 || i < 0 || i >= n_steps || order < 1 || order > 2) return CHORUS_E_ARG;
  const double s = sigmas[i], t = sigmas[i + 1];
  if (!(s > 0.0 && s <= 1.0 && t >= 0.0 && t < s)) return CHORUS_E_ARG;
  const double a_s = 1.0 - s, a_t = 1.0 - t;
  double c0 = 1.0, c1 = 0.0;
  if (order == 2 && i > 0 && t > 0.0) {
    const double p = sigmas[i - 1];
    if (!(p > s && p <= 1.0)) return CHORUS_E_ARG;
    const double a_p = 1.0 - p;
    if (a_p > 0.0) {  // a history taken at sigma = 1 lies infinitely far back in lambda and has no weight
      const double lam_p = log(a_p / p), lam_s = log(a_s / s), lam_t = log(a_t / t);
      const double inv2r = (lam_t - lam_s) / (2.0 * (lam_s - lam_p));
      c0 = 1.0 + inv2r;
      c1 = -inv2r;
    }
  }
  out->sigma_s = (float)s;
  out->rho = (float)(t / s);
  out->A = (float)(a_t - t * a_s / s);
  out->c0 = (float)c0;
  out->c1 = (float)c1;
  return CHORUS_OK;
}

size_t chorus_head_solver_workspace_bytes(int32_t D, int32_t P, int64_t Ls, int32_t cfg) {
  if (Ls < 1) Ls = 1;
  return align_up((size_t)Ls * D * 2, 256) + (cfg ? 2 : 1) * align_up((size_t)Ls * P * 4, 256);
}

int32_t chorus_head_update_solver(float* latent, const float* x, const float* x_uncond, float guidance, int64_t Ls,
                                  const int32_t* token_idx, const chorus_glue_weights* gw, const float* t_head,
                                  const chorus_sampler_coef* coef, float* x0_prev, const uint8_t* hist, const float* SL,
                                  const uint8_t* mask_edit, int32_t D, int32_t C, int32_t T, int32_t Hl, int32_t Wl,
                                  int32_t ph, int32_t pw, void* ws, size_t ws_bytes, void* stream) {
  if (Ls < 0 || C <= 0 || T <= 0 || Hl <= 0 || Wl <= 0 || ph <= 0 || pw <= 0 || D <= 0) return CHORUS_E_ARG;
  if (!coef || (coef->c1 != 0.f && !x0_prev) || ((mask_edit != nullptr) != (SL != nullptr))) return CHORUS_E_ARG;
  if (Ls == 0) return CHORUS_OK;
  if (!latent || !x || !gw || !t_head || !gw->w_head || !gw->head_table) return CHORUS_E_ARG;
  if (x0_prev == latent || (SL && (SL == latent || SL == x0_prev))) return CHORUS_E_ARG;
  const int P = C * ph * pw;
  if (Hl % ph || Wl % pw || P % 8 || D % 64) return CHORUS_E_SHAPE;
  if (!token_idx && Ls > (int64_t)T * (Hl / ph) * (Wl / pw)) return CHORUS_E_SHAPE;
  const int cfg = x_uncond != nullptr;
  if (!ws || ws_bytes < chorus_head_solver_workspace_bytes(D, P, Ls, cfg)) return CHORUS_E_WORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  const LatentGrid g{C, T, Hl, Wl, ph, pw};
  const SolverUpdate<false> upd{latent, x0_prev, hist, SL, mask_edit, *coef, 1.f};
  const SolverUpdate<true> upd_cfg{latent, x0_prev, hist, SL, mask_edit, *coef, guidance};
  if (head_in_one_pass(x, x_uncond, gw, t_head, ws, D, P))
    return cfg ? launch_head(x, x_uncond, gw, t_head, token_idx, Ls, D, P, g, upd_cfg, s)
               : launch_head(x, x, gw, t_head, token_idx, Ls, D, P, g, upd, s);
  uint16_t* h = (uint16_t*)ws;
  float* v = (float*)((uint8_t*)ws + align_up((size_t)Ls * D * 2, 256));
  float* vu = (float*)((uint8_t*)v + align_up((size_t)Ls * P * 4, 256));
  CHK(chorus_ln_modulate(x, h, Ls, D, gw->head_table + D, t_head + D, gw->head_table, t_head, 1, stream));
  CHK(chorus_gemm_bf16(h, gw->w_head, Ls, P, D, CHORUS_EPI_F32, v, gw->b_head, nullptr, nullptr, 1.f, stream));
  if (!cfg) return launch_unpatch(v, v, token_idx, Ls, g, upd, s);
  CHK(chorus_ln_modulate(x_uncond, h, Ls, D, gw->head_table + D, t_head + D, gw->head_table, t_head, 1, stream));
  CHK(chorus_gemm_bf16(h, gw->w_head, Ls, P, D, CHORUS_EPI_F32, vu, gw->b_head, nullptr, nullptr, 1.f, stream));
  return launch_unpatch(v, vu, token_idx, Ls, g, upd_cfg, s);
}

size_t chorus_text_project_workspace_bytes(int32_t Lt, int32_t D) {
  return align_up((size_t)(Lt > 0 ? Lt : 1) * (size_t)(D > 0 ? D : 1) * 2, 256);
}

int32_t chorus_text_project(const uint16_t* text, int32_t Lt, int32_t text_dim, int32_t D, const uint16_t* w1,
                            const float* b1, const uint16_t* w2, const float* b2, uint16_t* ctx, void* ws,
                            size_t ws_bytes, void* stream) {
  if (Lt < 0 || text_dim <= 0 || D <= 0) return CHORUS_E_ARG;
  if (Lt == 0) return CHORUS_OK;
  if (!text || !w1 || !w2 || !ctx) return CHORUS_E_ARG;
  if (text_dim % 64 || D % 64) return CHORUS_E_SHAPE;
  if (!ws || ws_bytes < chorus_text_project_workspace_bytes(Lt, D)) return CHORUS_E_WORKSPACE;
  uint16_t* hid = (uint16_t*)ws;
  CHK(chorus_gemm_bf16(text, w1, Lt, D, text_dim, CHORUS_EPI_GELU_BF16, hid, b1, nullptr, nullptr, 1.f, stream));
  CHK(chorus_gemm_bf16(hid, w2, Lt, D, D, CHORUS_EPI_BF16, ctx, b2, nullptr, nullptr, 1.f, stream));
  return CHORUS_OK;
}

}  // extern "C"
