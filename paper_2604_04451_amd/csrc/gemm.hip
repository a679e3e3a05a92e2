// bf16 MFMA GEMM with fused epilogues: C = epi(A W^T + bias), A [M,K], W [N,K], both K-contiguous, fp32 accumulation.
//
// One kernel, `gemm_w16_kernel`, that copies its tiles straight from global memory to LDS, in five tile shapes; which shape a
// product is run on, and whether K is cut into slices, is decided by `plan_gemm` at the end of the file.
#include <cmath>

#include "chorus_ops.h"
#include "common.h"
#include "gemm.h"

namespace chorus {
namespace {

// s_waitcnt operand that waits for at most n vector memory operations in flight and for nothing else
constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0F70; }

constexpr int BK = 64;

__device__ __forceinline__ float gelu_tanh_fast(float x) {
  // 0.5 x (1 + tanh(u)) = x / (1 + exp(-2u)),  u = sqrt(2/pi) (x + 0.044715 x^3); the exponent is taken in base 2:
  // -2u log2(e) = -x (2.3022082 + 0.10294324 x^2)
  const float t = x * x;
  const float p = __builtin_fmaf(t, -0.10294324f, -2.3022082f);
  const float e = __builtin_amdgcn_exp2f(p * x);
  return x * __builtin_amdgcn_rcpf(1.0f + e);
}

struct EpiArgs {
  void* out;
  const float* bias;
  const float* gate0;
  const float* gate1;
  float scale;
};

// where the slices of K but the last leave their [M, N] results
struct PartPtrs {
  float* first;
  float* rest;
  __device__ __forceinline__ float* of(int slice, long M, int N) const {
    return slice == 0 ? first : rest + (size_t)(slice - 1) * M * N;
  }
};

// ---------------------------------------------------------------------------
// Large-problem kernel: 256 x 256 x 64 tiles, four waves (one per SIMD), each wave a 128 x 128 quadrant as 8 x 8
// accumulators of v_mfma_f32_16x16x32_bf16 (256 accumulator registers). Per unit of work a 16x16x32 MFMA reads and
// writes half the accumulator registers of a 32x32x16 one (k = 32 per instruction instead of 16), which is what the
// power-managed part rewards; a 16-byte LDS fragment (16 rows x 8 k per quarter wave) feeds eight MFMAs.
//
// Both operands stream global -> LDS directly (buffer_load_dwordx4 ... lds: no register staging, no LDS store
// instructions, one lane offset per load for all steps) into a ring of five half steps of 32 KB, the whole 160 KB: rows 0-127
// of A and of W are one half of a k-step, rows 128-255 the other. A direct load writes the 64 lanes' 16-byte pieces to
// consecutive LDS addresses, i.e. 8 unpadded rows of 128 bytes. Bank conflicts are avoided by an XOR swizzle instead of padding: the
// 16-byte chunk c of row r lives at chunk position c ^ ((r >> 1) & 7); the loading lane for position p of row r
// fetches global chunk p ^ ((r >> 1) & 7). (A 16-byte-per-lane LDS read is served 16 lanes a cycle: the four-lane
// groups of one half wave whose group index has the same bit parity, groups 0, 3, 5, 6 together and 1, 2, 4, 7. With
// lane = 16 * chunk + row those are rows 0-3 and 12-15 of one chunk with rows 4-11 of its neighbour, which this
// swizzle spreads over all 64 banks: measured, no conflict cycles.)
//
// Operand layout of v_mfma_f32_16x16x32_bf16: lane l supplies row (or column) l % 16 and the 8 k-values
// 8 (l / 16) .. + 8; it receives column l % 16 and rows 4 (l / 16) .. + 4 of the 16 x 16 result. The weight fragment is
// the row operand and the activation fragment the column operand, so a lane holds one output row m and four
// consecutive output columns n.
//
// One loop iteration per k-step, hand-laid for a single wave per SIMD (nothing else hides a gap between two MFMAs):
// half-step 0 (64 MFMAs) with the LDS reads of half-step 1's fragments; wait + barrier; half-step 1 (64 MFMAs) with the LDS
// reads of the next step's first fragments. Either half issues the 8 loads of a half step, one every eight MFMAs: those of
// half-step 0 land 1 to 1.5 steps later, those of half-step 1 half a step to a step. Every read and load stands alone
// between two MFMAs. What bounds the loop is the delivery of the operands: with all 16 loads of a step in its second half and
// two whole stages in LDS it ran at 1310 TFLOP/s (8192 x 8192 x 8192), so at 1510; with the loads aimed at two steps
// that stay in the L2 at 1530, without any loads at 1780. Measured and not taken: 16 loads in the first half of half-step
// 1 (1.04 of the time), one load per wave and step that fetches lines into the L2 four steps ahead (1.04), workgroups that
// stay and take the next tile's first steps behind the last ones of this tile's (0.99 to 1.02), later starts for some of the XCDs
// so that not all epilogues write at once (they cost what they save).
// The MFMAs are volatile assembly, in place on their accumulators: left to the register allocator every result gets
// a new home, at the price of several hundred accumulator moves per k-step.
// ---------------------------------------------------------------------------

// WBM, WBN = 16 x 16 blocks along the rows (M) and columns (N) of a wave's quadrant: 8, 8 (256 x 256 tiles), 4, 4 (128 x
// 128), 2, 2 (64 x 64) or 4, 8 (128 x 256).
// C = half steps in LDS: the loads of a half step are issued C - 4 to C - 2 half-steps before the barrier that they must have
// landed at. Five leave room for two 128 x 128 workgroups on a compute unit, which then hide each other's waits; a launch with
// fewer tiles than units has no second workgroup there, and seven (112 KB) take its place: 1200 x 1536 x 8960 100 -> 67 us. More
// measured the same: from there on the unit's L1, not the distance, sets the rate.
//
// bf16 (optionally GELU) epilogue of the 16x16 layout: 32 output rows at a time go through a private LDS region as
// [32][16 WBN] bf16 (row stride 16 WBN + 8), then leave as full row segments of the quadrant (256, 128 or 64 bytes).
template <int WBN> constexpr int e16_bf_stride() { return 16 * WBN + 8; }
template <int WBN> constexpr int e16_bf_wave() { return 32 * e16_bf_stride<WBN>(); }  // elements per wave
template <int EPI, int WBM, int WBN>
__device__ __forceinline__ void gemm16_epilogue_bf16(const f32x4 (&acc)[8][8], const EpiArgs& ep, uint16_t* cw, long m_wave0,
                                                     int n_wave0, long M, int N, int lane) {
  constexpr int E16_BF_STRIDE = e16_bf_stride<WBN>();
  constexpr int LPR = 2 * WBN, RPI = 64 / LPR;  // read-back: LPR lanes x 16 bytes per row, RPI rows per instruction
  const int lj = lane & 15, lg = lane >> 4;
  const int rrow = lane / LPR, rcol = (lane % LPR) * 8;
  float4 bias[WBN];
#pragma unroll
  for (int nb = 0; nb < WBN; ++nb) {
    const int n = n_wave0 + 16 * nb + 4 * lg;
    bias[nb] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (ep.bias && n < N) bias[nb] = *reinterpret_cast<const float4*>(ep.bias + n);
  }
#pragma unroll
  for (int mp = 0; mp < WBM / 2; ++mp) {  // pairs of 16-row blocks
#pragma unroll
    for (int mh = 0; mh < 2; ++mh)
#pragma unroll
      for (int nb = 0; nb < WBN; ++nb) {
        f32x4 a = acc[nb][2 * mp + mh];
        // one block at a time out of the accumulators: of the large tile's, fetched together, 8 to 12 bytes a lane spilled
        if (WBM == 8 && mh) asm volatile("" : "+v"(a));
        float v0 = a[0] + bias[nb].x, v1 = a[1] + bias[nb].y, v2 = a[2] + bias[nb].z, v3 = a[3] + bias[nb].w;
        if (EPI == CHORUS_EPI_GELU_BF16) {
          v0 = gelu_tanh_fast(v0); v1 = gelu_tanh_fast(v1); v2 = gelu_tanh_fast(v2); v3 = gelu_tanh_fast(v3);
        }
        uint2 w;
        w.x = pack_bf16x2(v0, v1);
        w.y = pack_bf16x2(v2, v3);
        *reinterpret_cast<uint2*>(cw + (16 * mh + lj) * E16_BF_STRIDE + 16 * nb + 4 * lg) = w;
      }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
#pragma unroll
    for (int it = 0; it < 32 / RPI; ++it) {
      const int row = RPI * it + rrow;
      const long m = m_wave0 + 32 * mp + row;
      const int n = n_wave0 + rcol;
      const u32x4 v = *reinterpret_cast<const u32x4*>(cw + row * E16_BF_STRIDE + rcol);
      // streaming store: an output tile is not read again by this kernel, and left to the default policy the written
      // lines push the operand panels that the next tiles share out of the L2 (measured: 14-19 % on the widest output)
      if (m < M && n < N) __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(ep.out) + m * N + n));
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_sched_barrier(0);
  }
}

// The same address in scalar registers: the compiler does not see that a value worked out from the workgroup's id by a
// division is one for the whole wave, and would walk over the lanes with every descriptor made from it.
__device__ __forceinline__ void* uniform_address(const uint16_t* p) {
  const uint64_t u = reinterpret_cast<uint64_t>(p);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(u >> 32)), lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)u);
  return reinterpret_cast<void*>(((uint64_t)hi << 32) | lo);
}

// fp32 gated-residual epilogue of the 16x16 layout: 16 output rows at a time through a private LDS region as
// [16][16 WBN] fp32 (row stride 16 WBN + 4), read back with 4 WBN lanes per row; the residual rows are requested before the
// LDS round trip. out[m][n] += gate[n] * scale * (acc + bias[n]).
template <int WBN> constexpr int e16_f32_stride() { return 16 * WBN + 4; }
template <int WBN> constexpr int e16_f32_wave() { return 16 * e16_f32_stride<WBN>(); }  // floats per wave
// CHAIN: what another workgroup of the tile wrote is read and what the next one reads is written past the L2s (agent scope).
template <int WBM, int WBN, bool CHAIN = false>
__device__ __forceinline__ void gemm16_epilogue_resid(const f32x4 (&acc)[8][8], const EpiArgs& ep, float* cw, long m_wave0,
                                                      int n_wave0, long M, int N, int lane) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int E16_F32_STRIDE = e16_f32_stride<WBN>();
  constexpr int LPR = 4 * WBN, RPI = 64 / LPR;  // read-back: LPR lanes x 16 bytes per row, RPI rows per instruction
  const int lj = lane & 15, lg = lane >> 4;
  const int rrow = lane / LPR, rcol = (lane % LPR) * 4;
  const int n = n_wave0 + rcol;
  const bool n_ok = n < N;
  f32x4 bias = {0.f, 0.f, 0.f, 0.f}, gate = {1.f, 1.f, 1.f, 1.f};
  if (n_ok) {
    if (ep.bias) bias = *reinterpret_cast<const f32x4*>(ep.bias + n);
    if (ep.gate0 || ep.gate1) {
      gate = f32x4{0.f, 0.f, 0.f, 0.f};
      if (ep.gate0) gate += *reinterpret_cast<const f32x4*>(ep.gate0 + n);
      if (ep.gate1) gate += *reinterpret_cast<const f32x4*>(ep.gate1 + n);
    }
    gate *= ep.scale;
  }
  float* out = reinterpret_cast<float*>(ep.out);
  constexpr int kAgent = 16;  // cache policy bit sc1
  const long m_base = m_wave0 < M ? m_wave0 : M - 1;  // never in front of the descriptor's first row
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(uniform_address(reinterpret_cast<const uint16_t*>(out + m_base * N)), 0, -1, 0x00027000);
  auto offset = [&](long m) { return ((int)(m - m_base) * N + n) * 4; };
  // The residual rows of block mb + 1 are requested before the results of block mb are stored: memory operations
  // retire in order, so a load issued behind a block's stores could only be consumed once those stores had drained.
  f32x4 cur[2][WBN];
  auto fetch = [&](int mb, f32x4 (&dst)[WBN]) {
#pragma unroll
    for (int it = 0; it < WBN; ++it) {
      long m = m_wave0 + 16 * mb + RPI * it + rrow;
      if (m > M - 1) m = M - 1;  // rows past the end read the last row (never stored)
      if constexpr (CHAIN)
        dst[it] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, offset(m) - (n_ok ? 0 : 4 * n), 0, kAgent));
      else
        dst[it] = *reinterpret_cast<const f32x4*>(out + m * N + (n_ok ? n : 0));
    }
  };
  fetch(0, cur[0]);
#pragma unroll
  for (int mb = 0; mb < WBM; ++mb) {
#pragma unroll
    for (int nb = 0; nb < WBN; ++nb) *reinterpret_cast<f32x4*>(cw + lj * E16_F32_STRIDE + 16 * nb + 4 * lg) = acc[nb][mb];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    if (mb + 1 < WBM) fetch(mb + 1, cur[(mb + 1) & 1]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int it = 0; it < WBN; ++it) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(cw + (RPI * it + rrow) * E16_F32_STRIDE + rcol);
      const long m = m_wave0 + 16 * mb + RPI * it + rrow;
      const f32x4 r = cur[mb & 1][it] + gate * (v + bias);
      if constexpr (CHAIN) {
        if (n_ok && m < M) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, r), rsrc, offset(m), 0, kAgent);
      } else {
        if (n_ok && m < M) *reinterpret_cast<f32x4*>(out + m * N + n) = r;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_sched_barrier(0);
  }
#endif
}

// Epilogue of the 4-wave 16x16 kernels: wave (wm, wn) holds rows m0 + 16 WBM wm .. + 16 WBM, columns
// n0 + 16 WBN wn .. + 16 WBN.
template <int EPI, int WBM, int WBN>
__device__ __forceinline__ void gemm16_finish(f32x4 (&acc)[8][8], const EpiArgs& ep, uint8_t* smem_raw, int wave, int wm, int wn,
                                              long m0, int n0, long M, int N, int lane) {
  constexpr int WTM = 16 * WBM, WTN = 16 * WBN;  // rows and columns of a wave's quadrant
  uint16_t* smem = reinterpret_cast<uint16_t*>(smem_raw);
  const int lj = lane & 15, lg = lane >> 4;
  if constexpr (EPI == CHORUS_EPI_BF16 || EPI == CHORUS_EPI_GELU_BF16) {
    gemm16_epilogue_bf16<EPI, WBM, WBN>(acc, ep, smem + wave * e16_bf_wave<WBN>(), m0 + wm * WTM, n0 + wn * WTN, M, N, lane);
  } else if constexpr (EPI == CHORUS_EPI_RESID) {
    gemm16_epilogue_resid<WBM, WBN>(acc, ep, reinterpret_cast<float*>(smem_raw) + wave * e16_f32_wave<WBN>(), m0 + wm * WTM,
                                    n0 + wn * WTN, M, N, lane);
  } else {
    // plain fp32: a lane stores its four consecutive columns of every block
#pragma unroll
    for (int nb = 0; nb < WBN; ++nb) {
      const int n = n0 + wn * WTN + 16 * nb + 4 * lg;
      if (n >= N) continue;
      f32x4 bias = {0.f, 0.f, 0.f, 0.f};
      if (ep.bias) bias = *reinterpret_cast<const f32x4*>(ep.bias + n);
#pragma unroll
      for (int mb = 0; mb < WBM; ++mb) {
        const long m = m0 + wm * WTM + 16 * mb + lj;
        if (m < M) *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(ep.out) + m * N + n) = acc[nb][mb] + bias;
      }
    }
  }
}

// A second product of a launch with bf16 outputs, with the same K: its tiles follow the first one's `first` tiles.
struct Twin {
  const uint16_t* A;
  const uint16_t* W;
  uint16_t* out;
  const float* bias;
  long M;
  int N, tiles_m, tiles_n, first;
  static constexpr bool kTwo = true, kChain = false;
};
struct Alone {  // no second product
  static constexpr bool kTwo = false, kChain = false;
};
// The gated residual in slices of K without scratch: every slice adds its part to the residual itself, in the order of the slices. A
// slice waits until its tile's count has reached its number. Workgroups are dealt out by each XCD for itself, so that a workgroup's
// number says nothing of what has started elsewhere; what a workgroup does is given out by ticket instead. The workgroups
// whose number leaves the same rest by `groups` (8: they share an XCD and its L2) take tickets of one counter for a range of tiles of their
// own, all of its tiles of the first slice first. So a slice only ever waits for a lower ticket of its group, whose workgroup
// has taken it and is running; that one waits for a still lower ticket or for nothing: every wait ends, whatever else runs on the GPU.
// The ticket is a round trip to memory ahead of the first load, about 1 us (by workgroup number / by ticket, us: 3271 x 1536 x 8960 84.4 /
// 86.8, 2000 59.1 / 59.5, 1100 39.3 / 40.7, 300 21.5 / 22.6, 960 x 5120 x 5120 60.3 / 61.2, 200 x 2048 x 4096 13.8 / 15.2, operands warm).
// A word a tile, zero at the start: the slices that have been added in its low four bits and, in the word of a group's first
// tile, the tickets taken in the others.
// Slices of equal length would all end together and then wait for each other's updates: each is a few steps longer than the one in
// front of it instead (3271 x 1536 x 8960, three slices of 256 x 256 tiles: 100 us with equal ones, 87 with five steps more each).
struct Chain {
  uint32_t* count;  // [tiles]
  int stagger;      // steps that a slice is longer than the one in front of it
  int tiles, groups;
  static constexpr bool kTwo = false, kChain = true;
  static constexpr uint32_t kTicket = 16, kAdded = 15;  // one ticket; the bits of the slices that have been added
};

// The 128 x 256 shape takes three quarters of the operand bytes per product of 128 x 128 tiles: for products of about 400 to
// 512 such tiles with a long K, which run two to a unit, half as many wide ones finish earlier (N = 1536, K = 8960: 5000 rows
// 132 -> 117 us; N = 5120, K = 13824, 1200 rows: 202 -> 172; with 312 tiles, 3271 rows of the former, 109 and 112).
// FAR: rows so long that a tile's last byte is out of reach of the 32-bit offsets; loads by 64-bit addresses.
template <int EPI, int WBM, int WBN, int C, bool FAR, class SECOND>
__global__ __launch_bounds__(256, 1) void gemm_w16_kernel(const uint16_t* __restrict__ A, const uint16_t* __restrict__ W,
                                                          long M, int N, int K, EpiArgs ep, PartPtrs parts, int tiles_m,
                                                          int tiles_n, SECOND twin) {
#if defined(__HIP_DEVICE_COMPILE__)  // the buffer descriptors below are types of the device compiler's alone
  static_assert((WBM == 8 || WBM == 4 || WBM == 2) && (WBN == WBM || (WBM == 4 && WBN == 8)), "quadrants of 8 x 8, 4 x 4, 2 x 2 or 4 x 8 blocks");
  static_assert(C >= 5 && (WBM + WBN) / 2 * (C - 1) < 64, "two steps and a half in LDS at least, and the loads in flight must fit the wait counter");
  constexpr int BM = 32 * WBM, BN = 32 * WBN;
  constexpr int WTM = 16 * WBM, WTN = 16 * WBN;  // rows and columns of a wave's quadrant
  constexpr int GM = 8;
  constexpr int HA = WTM * BK, HB = WTN * BK;  // elements of half a step's rows of A and of W
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem_raw[];
  uint16_t* smem = reinterpret_cast<uint16_t*>(smem_raw);  // [C][HA], [C][HB]

  // The grid's rows are the slices of K, their steps shared out as evenly as can be (never none: the host asks for no more
  // slices than steps). The last slice runs the epilogue, the others leave their plain fp32 result in `parts`. Without a
  // split there is one, and the divisions, a tenth of a microsecond of a product of one to four steps, are left out.
  int block = blockIdx.x, ntiles = gridDim.x;
  if constexpr (SECOND::kTwo) {
    ntiles = twin.first;
    if (block >= twin.first) {
      block -= twin.first;
      ntiles = gridDim.x - twin.first;
      A = twin.A;
      W = twin.W;
      M = twin.M;
      N = twin.N;
      ep.out = twin.out;
      ep.bias = twin.bias;
      tiles_m = twin.tiles_m;
      tiles_n = twin.tiles_n;
    }
  }
  const int nslices = gridDim.y;
  int slice = blockIdx.y, tile;
  if constexpr (SECOND::kChain) {
    const int g = block % twin.groups, q = twin.tiles / twin.groups, r = twin.tiles % twin.groups;
    const int of_group = q + (g < r), first_tile = g * q + (g < r ? g : r);
    if ((slice * (int)gridDim.x + block) / twin.groups >= of_group * nslices) return;  // the grid's x is a multiple of the groups
    // one of the ring's places that nothing is requested into before every wave has read it
    uint32_t* const mine = reinterpret_cast<uint32_t*>(smem + (C - 1) * HA);
    if (threadIdx.x == 0)
      mine[0] = __hip_atomic_fetch_add(twin.count + first_tile, Chain::kTicket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) / Chain::kTicket;
    __syncthreads();
    const int ticket = __builtin_amdgcn_readfirstlane((int)mine[0]);
    slice = ticket / of_group;
    tile = ticket - slice * of_group;
    tile += first_tile;
  } else {
    tile = xcd_remap(block, ntiles);
  }
  int KTN = K / BK, k_first = 0;
  if (nslices > 1) {
    auto start = [&](int i) {
      if constexpr (SECOND::kChain)
        return i * KTN / nslices - twin.stagger * i * (nslices - i) / 2;
      else
        return i * KTN / nslices;
    };
    k_first = __builtin_amdgcn_readfirstlane(start(slice));
    KTN = __builtin_amdgcn_readfirstlane(start(slice + 1)) - k_first;
    A += (long)k_first * BK;
    W += (long)k_first * BK;
  }
  const int per_group = GM * tiles_n;
  const int group = tile / per_group;
  const int first_m = group * GM;
  const int gsz = (tiles_m - first_m) < GM ? (tiles_m - first_m) : GM;
  const int in_group = tile - group * per_group;
  // Within a group the tiles that run together on one XCD share operands in its L2. Normally they are taken row tile
  // fastest (8 row tiles x 4 column tiles at a time). When the activation rows are long and the weight matrix is only
  // a few tiles wide, column tile fastest is better: all column tiles of a row tile run together, so every activation
  // panel, the operand too big for any cache, leaves HBM once.
  const bool n_fastest = tiles_n <= 8 && K >= 4096;
  const int tm_idx = n_fastest ? first_m + in_group / tiles_n : first_m + in_group % gsz;
  const int tn_idx = n_fastest ? in_group % tiles_n : in_group / gsz;
  const long m0 = (long)tm_idx * BM;
  const int n0 = tn_idx * BN;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int lj = lane & 15, lg = lane >> 4;

  // ---- loader: load i of half h covers 8 of the tile's rows from WTM h + 4 WBM wave + 8 i on (of W: WTN h + 4 WBN wave + 8
  // i); lane -> (row, position). One lane offset per load serves every step: the step's place in the rows is a scalar, and
  // rows past the matrix's end are past the descriptor's too (such loads fetch nothing; their results are never stored).
  const int lr = lane >> 3, lp = lane & 7;
  constexpr int LA = WBM / 2, LB = WBN / 2;  // loads of a half step
  // (the arrays that the lambdas below capture have the large tile's size for either tile: a bound that depends on
  // the template parameter loses the kernel's host-side stub)
  int oa[8], ob[8];
  const int rows_a = M - m0 < BM ? (int)(M - m0) : BM, rows_b = N - n0 < BN ? N - n0 : BN;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int i = 0; i < LA; ++i) {
      const int r = WTM * h + 4 * WBM * wave + 8 * i + lr;
      const int at = (lp ^ ((r >> 1) & 7)) * 16;  // the global chunk that belongs at position lp
      oa[LA * h + i] = FAR ? (r < rows_a ? r : rows_a - 1) : r * (2 * K) + at;
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      const int r = WTN * h + 4 * WBN * wave + 8 * i + lr;
      const int at = (lp ^ ((r >> 1) & 7)) * 16;
      ob[LB * h + i] = FAR ? (r < rows_b ? r : rows_b - 1) : r * (2 * K) + at;
    }
  }
  void* const base_a = uniform_address(A + m0 * K);
  void* const base_b = uniform_address(W + (long)n0 * K);
  const int bytes_a = __builtin_amdgcn_readfirstlane(FAR ? 0 : (rows_a * K - k_first * BK) * 2);
  const int bytes_b = __builtin_amdgcn_readfirstlane(FAR ? 0 : (rows_b * K - k_first * BK) * 2);
  // load t (A's first, then W's) of half step hs (half hs % 2 of the rows of step hs / 2), into the ring at slot
  auto issue = [&](int hs, int h, int slot, int t) {
    const bool of_w = t >= LA;
    const int i = of_w ? t - LA : t, kt = hs >> 1;
    __attribute__((address_space(3))) void* const dst =
        (__attribute__((address_space(3))) void*)(smem + (of_w ? C * HA + slot * HB + (4 * WBN * wave + 8 * i) * BK
                                                                : slot * HA + (4 * WBM * wave + 8 * i) * BK));
    if constexpr (FAR) {
      const int r = of_w ? ob[LB * h + i] : oa[LA * h + i];
      const int row = (of_w ? WTN * h + 4 * WBN * wave : WTM * h + 4 * WBM * wave) + 8 * i + lr;
      const uint16_t* src = reinterpret_cast<const uint16_t*>(of_w ? base_b : base_a) + (long)r * K +
                            (long)(kt < KTN ? kt : KTN - 1) * BK + (lp ^ ((row >> 1) & 7)) * 8;
      __builtin_amdgcn_global_load_lds(src, dst, 16, 0, 0);
    } else {
      // past the last step an empty descriptor: the loads keep their place in the count and fetch nothing
      const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(of_w ? base_b : base_a, 0, kt < KTN ? (of_w ? bytes_b : bytes_a) : 0, 0x00027000);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, dst, 16, of_w ? ob[LB * h + i] : oa[LA * h + i], kt * (2 * BK), 0, 0);
    }
  };

  // ---- fragment read offsets (elements): row l % 16 of a 16-row block, 16-byte chunk 4 h + l / 16, swizzled by the row
  const int sw = (lj >> 1) & 7;
  int koff[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) koff[h] = ((4 * h + lg) ^ sw) * 8 + lj * BK;

  f32x4 acc[8][8];  // [n block][m block]; the WBN x WBM corner is used
#pragma unroll
  for (int nb = 0; nb < WBN; ++nb)
#pragma unroll
    for (int mb = 0; mb < WBM; ++mb) acc[nb][mb] = f32x4{0.f, 0.f, 0.f, 0.f};

  bf16x8 af[2][8], bfr[2][8];
  // fragment f of a half-step: 0 .. WBM-1 the activation blocks (m), then the WBN weight blocks (n); sa, sb: where the wave's
  // rows of the step start
  auto read_frag = [&](int sa, int sb, int h, int set, int f) {
    if (f < WBM)
      af[set][f] = *reinterpret_cast<const bf16x8*>(smem + sa + koff[h] + f * 16 * BK);
    else
      bfr[set][f - WBM] = *reinterpret_cast<const bf16x8*>(smem + sb + koff[h] + (f - WBM) * 16 * BK);
  };
  // MFMAs g0 .. g1-1 of the WBM * WBN of a half-step, weight block major: g = WBM nb + mb. In place on the accumulator
  // registers (left to itself the register allocator gives every result a new home and pays with hundreds of
  // accumulator moves per k-step); being volatile they also keep their place between the loads written around them.
  auto mfmas = [&](int set, int g0, int g1) {
#pragma unroll
    for (int g = g0; g < g1; ++g)
      asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[g / WBM][g % WBM]) : "v"(bfr[set][g / WBM]), "v"(af[set][g % WBM]));
  };
  // order in which the fragments of a half-step are fetched: what its first MFMAs need comes first (the first weight
  // block, the activation blocks, the other weight blocks)
  auto frag_order = [](int i) { return i == 0 ? WBM : (i <= WBM ? i - 1 : i); };

  // Schedule of one k-step (square tiles, WB = WBM = WBN: 2 WB^2 MFMAs a wave in 4 WB slots of WB / 2, 128 MFMAs in 32
  // slots of four for the large tile). Either half-step issues the loads of one half step further on, one every other slot.
  // The barrier sits between the two half-steps. In the first half a wave fetches its fragments of the second half (same
  // step); at the barrier every wave holds all its fragments of the current step in registers, so that the step's two
  // places in the ring are free behind it, and the whole next step is in LDS: what was requested behind that step, C - 4
  // half steps, stays in flight. The second half fetches the next step's first fragments. Fragment reads are
  // packed into the first kReadSlots slots of a half so that the last of them has returned when the half ends. With one
  // wave per SIMD nothing else feeds the matrix pipe while this wave issues something that is not an MFMA, so reads and
  // loads stand one at a time between single MFMAs, where they issue in the shadow of the MFMA in front of them, and
  // the wave index is kept in a scalar register so that the LDS address of a load costs no vector instruction.
  // A rectangular tile has no whole number of MFMAs per slot: its reads stand behind MFMAs spread evenly over the first
  // three quarters of a half, its loads over all of it.
  constexpr int NS = WBM + WBN;            // slots of a half-step = fragments of a half-step
  constexpr int NH = NS / 2;               // loads of a half step
  constexpr int G = WBM * WBN;             // MFMAs of a half-step
  constexpr int MPS = WBM / 2;             // MFMAs of a slot
  constexpr int kReadSlots = 3 * WBM / 2;  // 12 of 16 (6 of 8, 3 of 4)
  // reads of slot f: one fragment, two in the first NS - kReadSlots slots (which = 0: the first, 1: the second)
  auto read_of_slot = [&](int sa, int sb, int h, int set, int f, int which) {
    constexpr int kDouble = NS - kReadSlots;
    if (f < kDouble)
      read_frag(sa, sb, h, set, frag_order(2 * f + which));
    else if (f < kReadSlots && which == 0)
      read_frag(sa, sb, h, set, frag_order(f + kDouble));
  };
  // half-step h: its MFMAs, the fragments of the half-step behind it from sa, sb, the loads of half step hs into slot
  auto half_step = [&](int h, int sa, int sb, int hs, int slot) {
    if constexpr (WBM == WBN) {
#pragma unroll
      for (int f = 0; f < NS; ++f) {
        mfmas(h, MPS * f, MPS * f + 1);
        __builtin_amdgcn_sched_barrier(0);
        read_of_slot(sa, sb, 1 - h, 1 - h, f, 0);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (MPS > 1) mfmas(h, MPS * f + 1, MPS * f + 2);
        __builtin_amdgcn_sched_barrier(0);
        read_of_slot(sa, sb, 1 - h, 1 - h, f, 1);
        __builtin_amdgcn_sched_barrier(0);
        mfmas(h, MPS * f + 2, MPS * f + MPS - 1);  // (none for the small tiles)
        __builtin_amdgcn_sched_barrier(0);
        if (f & 1) issue(hs, (C - 1 + h) & 1, slot, f >> 1);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (MPS > 2) mfmas(h, MPS * f + MPS - 1, MPS * f + MPS);
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        mfmas(h, g, g + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < NS; ++i)
          if (i * 3 * G / (4 * NS) == g) read_frag(sa, sb, 1 - h, 1 - h, frag_order(i));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < NH; ++i)
          if ((2 * i + 1) * G / (2 * NH) == g) issue(hs, (C - 1 + h) & 1, slot, i);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  auto wrap = [](int slot) { return slot >= C ? slot - C : slot; };

#pragma unroll
  for (int hs = 0; hs < C - 1; ++hs)
#pragma unroll
    for (int t = 0; t < NH; ++t) issue(hs, hs & 1, hs, t);
  // the first step's pieces are in LDS, the later ones may be in flight (the barrier alone: a fence would wait for them)
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(NH * (C - 3)) : "memory");
  __builtin_amdgcn_sched_barrier(0);
  int first = 0;  // slot of the first half of step kt
  int sa = wm * HA, sb = C * HA + wn * HB;
#pragma unroll
  for (int f = 0; f < NS; ++f) read_frag(sa, sb, 0, 0, frag_order(f));
  __builtin_amdgcn_sched_barrier(0);

  for (int kt = 0; kt < KTN; ++kt) {
    const int next = wrap(first + 2);
    const int san = wrap(next + wm) * HA, sbn = C * HA + wrap(next + wn) * HB;
    half_step(0, sa, sb, 2 * kt + C - 1, wrap(first + C - 1));
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(NH * (C - 4)) : "memory");
    __builtin_amdgcn_sched_barrier(0);
    half_step(1, san, sbn, 2 * kt + C, first);
    first = next;
    sa = san;
    sb = sbn;
  }

  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));  // no direct load may land in the staging regions of the epilogue
  // The compiler does not know the assembly above for MFMAs and so keeps no distance between the last of them and the
  // first instruction that reads an accumulator: cover the longest such distance explicitly. The wait is tied to the
  // accumulators of the last four MFMAs (operands of the statement), so that no copy or spill of one of them can be
  // placed in front of it; every other accumulator was written at least four MFMAs earlier.
  asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15"
               : "+a"(acc[WBN - 1][WBM - 1]), "+a"(acc[WBN - 1][WBM - 2]), "+a"(acc[WBM > 2 ? WBN - 1 : 0][WBM > 2 ? WBM - 3 : 1]),
                 "+a"(acc[WBM > 2 ? WBN - 1 : 0][WBM > 2 ? WBM - 4 : 0]));
  lds_barrier();  // the staging regions of the epilogue overlay the operands
  if constexpr (SECOND::kChain) {
    static_assert(EPI == CHORUS_EPI_RESID, "slices of the gated residual");
    uint32_t* const count = twin.count + tile;
    if (slice > 0) {
      if (tid == 0)
        while ((__hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & Chain::kAdded) != (uint32_t)slice) __builtin_amdgcn_s_sleep(1);
      __syncthreads();
      asm volatile("" ::: "memory");  // the residual is read behind the count
      ep.bias = nullptr;              // went in with the first slice
    }
    gemm16_epilogue_resid<WBM, WBN, true>(acc, ep, reinterpret_cast<float*>(smem_raw) + wave * e16_f32_wave<WBN>(), m0 + wm * WTM,
                                          n0 + wn * WTN, M, N, lane);
    if (slice + 1 < nslices) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the wave's stores have completed, past the L2
      __syncthreads();
      if (tid == 0) __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return;
  }
  if constexpr (EPI == CHORUS_EPI_RESID) {
    if (slice + 1 < nslices) {
      const EpiArgs plain{parts.of(slice, M, N), nullptr, nullptr, nullptr, 1.f};
      gemm16_finish<CHORUS_EPI_F32, WBM, WBN>(acc, plain, smem_raw, wave, wm, wn, m0, n0, M, N, lane);
      return;
    }
  }
  gemm16_finish<EPI, WBM, WBN>(acc, ep, smem_raw, wave, wm, wn, m0, n0, M, N, lane);
#endif
}

template <int WBM, int WBN, int C, bool FAR = false>
int32_t launch_gemm_w16(const uint16_t* A, const uint16_t* W, long M, int N, int K, int epi, EpiArgs ep, hipStream_t s,
                        int slices, const PartPtrs& parts) {
  constexpr int BM = 32 * WBM, BN = 32 * WBN;
  long tm = (M + BM - 1) / BM;
  int tn = (N + BN - 1) / BN;
  if (tm * tn * slices > 0x7fffffffL) return CHORUS_E_SHAPE;
  dim3 grid((unsigned)(tm * tn), (unsigned)slices), block(256);
  const size_t smem = (size_t)C * (BM + BN) / 2 * BK * sizeof(uint16_t);
#define GEMM_W16(E)                                                                           \
  {                                                                                           \
    auto kern = gemm_w16_kernel<E, WBM, WBN, C, FAR, Alone>;                                  \
    static DynLdsOnce once;                                                                   \
    CHK_STATUS(once.ensure(reinterpret_cast<const void*>(kern), (int)smem));                  \
    hipLaunchKernelGGL(kern, grid, block, smem, s, A, W, M, N, K, ep, parts, (int)tm, tn, Alone{});   \
  }
  switch (epi) {
    case CHORUS_EPI_BF16: GEMM_W16(CHORUS_EPI_BF16); break;
    case CHORUS_EPI_GELU_BF16: GEMM_W16(CHORUS_EPI_GELU_BF16); break;
    case CHORUS_EPI_F32: GEMM_W16(CHORUS_EPI_F32); break;
    case CHORUS_EPI_RESID: GEMM_W16(CHORUS_EPI_RESID); break;
    default: return CHORUS_E_ARG;
  }
#undef GEMM_W16
  CHORUS_LAUNCH_CHECK();
  return CHORUS_OK;
}

// What the last slice of K left out: out[m][n] += gate[n] scale sum_s part_s[m][n], P parts in ascending order (the bias
// went in with the last slice).
template <int P>
__global__ __launch_bounds__(256) void gemm_add_parts_kernel(PartPtrs parts, long M, int N, EpiArgs ep) {
  const long n4 = N / 4, i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= M * n4) return;
  const int n = (int)(i % n4) * 4;
  f32x4 p[P];
#pragma unroll
  for (int k = 0; k < P; ++k) p[k] = *reinterpret_cast<const f32x4*>(parts.of(k, M, N) + i * 4);
  f32x4* o = reinterpret_cast<f32x4*>(reinterpret_cast<float*>(ep.out) + i * 4);
  const f32x4 cur = *o;
  f32x4 gate = {1.f, 1.f, 1.f, 1.f};
  if (ep.gate0 || ep.gate1) {
    gate = f32x4{0.f, 0.f, 0.f, 0.f};
    if (ep.gate0) gate += *reinterpret_cast<const f32x4*>(ep.gate0 + n);
    if (ep.gate1) gate += *reinterpret_cast<const f32x4*>(ep.gate1 + n);
  }
  gate *= ep.scale;
#pragma unroll
  for (int k = 1; k < P; ++k) p[0] += p[k];
  *o = cur + gate * p[0];
}

int32_t launch_add_parts(const PartPtrs& parts, int slices, long M, int N, const EpiArgs& ep, hipStream_t s) {
  const dim3 grid((unsigned)((M * (N / 4) + 255) / 256));
  switch (slices) {
    case 2: hipLaunchKernelGGL(gemm_add_parts_kernel<1>, grid, dim3(256), 0, s, parts, M, N, ep); break;
    case 3: hipLaunchKernelGGL(gemm_add_parts_kernel<2>, grid, dim3(256), 0, s, parts, M, N, ep); break;
    case 4: hipLaunchKernelGGL(gemm_add_parts_kernel<3>, grid, dim3(256), 0, s, parts, M, N, ep); break;
    default: return CHORUS_E_ARG;
  }
  CHORUS_LAUNCH_CHECK();
  return CHORUS_OK;
}

// ---------------------------------------------------------------------------
// Which tile, and in how many slices of K. The estimated time of each tile in microseconds, fitted to 3600 measurements
// on this chip with activations in the last-level cache and weights cold, as a request finds them (K from 256 to 13824, N
// from 256 to 15360, M from 64 to 13104; figures in brackets: gated residual, K = 1536 / K = 8960 where N = 1536). What is fitted is the
// choice: over those products the tile and slices taken cost 0.7 % more than the fastest (geometric mean).
// What bounds a launch that does not fill the chip is the rate at which ONE compute unit gets operands: its L1 holds
// 256 lines in flight, 32 KB, so a unit takes in about 60 KB per microsecond whatever the kernel does, and the launch
// that spreads the same problem over more units wins: smaller tiles, or slices of K.
//   256 x 256  one workgroup per unit, rounds of 256; a partly filled round is up to a quarter faster [38 / 161 us, full 54 / 215]
//   128 x 256  one workgroup per unit: up to 256 tiles [23 / 116 few, 32 / 128 all units busy], then a second round
//   128 x 128  two workgroups per unit: one round of up to 256 tiles [18 / 96], then rounds of 512 [31 / 135]
//   128 x 128  three steps and a half in LDS, one workgroup per unit: up to 256 tiles [14 / 75 few, 19 / 82 all units busy]
//   64 x 64    two workgroups per unit: up to 256 tiles [8.2 / 36], growing with the tiles up to 512 [14 / 69]
// ---------------------------------------------------------------------------
// a tile's bytes, 256 rows of 2 K, within the 32-bit offsets of its loads; longer rows are 64 x 64 tiles' alone
constexpr int kMaxOffsetK = (1 << 22) - 64;

enum Tile { kTile256, kTileWide, kTile128, kTile128Deep, kTile64, kTiles };
constexpr int kTileNumber[kTiles] = {3, 2, 4, 5, 1};  // as chorus_gemm_bf16_kernel names them
constexpr int kTileRows[kTiles] = {256, 128, 128, 128, 64};
constexpr int kTileCols[kTiles] = {256, 256, 128, 128, 64};
constexpr int kMaxSlices = 4;  // more slices than this were never the fastest

long tile_count(int tile, long m, int N) {
  const long rows = kTileRows[tile], cols = kTileCols[tile];
  return ((m + rows - 1) / rows) * ((N + cols - 1) / cols);
}

double tiles_time(int tile, long tiles, int K, int epi, int slices) {
  const double steps = (double)((K / BK + slices - 1) / slices);
  const double w = (double)(tiles * slices), fill = w / 256.0;
  const bool gelu = epi == CHORUS_EPI_GELU_BF16, f32 = slices == 1 && (epi == CHORUS_EPI_F32 || epi == CHORUS_EPI_RESID);
  auto by_epilogue = [&](double bf16, double with_gelu, double resid) { return f32 ? resid : gelu ? with_gelu : bf16; };
  switch (tile) {
    case kTile256: {
      const double full = by_epilogue(2.2, 3.59, 10.87) + 1.583 * steps;
      const double rounds = floor(fill), rest = fill - rounds;
      return full * (rounds + (rest > 0.0 ? 0.76 + 0.253 * rest * rest : 0.0));
    }
    case kTileWide: {
      if (w > 512.0) return INFINITY;
      const double c = by_epilogue(3.58, 3.83, 9.17);
      if (w <= 256.0) return c + (0.72 + 0.141 * fill * fill * fill) * steps;
      return (c + 0.861 * steps) * (1.6 + 0.4 * (fill - 1.0));
    }
    case kTile128: {
      const double one = by_epilogue(1.71, 3.67, 4.97) + 0.74 * steps, round512 = by_epilogue(0.48, 0.57, 5.67) + 1.001 * steps;
      if (w <= 256.0) return one;
      // With bf16 outputs half as many second workgroups cost the whole of it: over 115 products of 257 to 512 tiles (N 768 to 15360,
      // K 256 to 5120) the choice is 0.7 % slower than the fastest tile, 1.5 % with a straight line (1210 x 4608 x 1536, 360 tiles: 27.5
      // us, 128 x 256 24.8; 1956 x 2560 x 2560, 320 tiles: 41.2 and 36.8; the other way 746 x 6144 x 3072, 288 tiles: 40.7 and 45.6).
      const double second = f32 || epi == CHORUS_EPI_RESID ? fill - 1.0 : fmin(2.0 * (fill - 1.0), 1.0);
      if (w <= 512.0) return one + second * fmax(round512 - one, 0.0);
      return (0.784 * ceil(w / 512.0) + 0.216 * w / 512.0) * round512;
    }
    case kTile128Deep: {
      if (w > 256.0) return INFINITY;
      return by_epilogue(5.36, 3.64, 5.4) + (0.45 + 0.081 * fill * fill) * steps;
    }
    default:
      // Two workgroups a unit: a third one waits for their place (700 x 3072 x 8960, 528 tiles: 92 us, 69 with 480; the deep tile 66).
      // In none of 837 products was this tile the fastest with more.
      if (w > 512.0) return INFINITY;
      return (w <= 256.0 ? 1.0 : 1.141 + 0.677 * (fill - 1.0)) * (by_epilogue(3.62, 2.26, 3.14) + 0.246 * steps);
  }
}

double tile_time(int tile, long m, int N, int K, int epi, int slices) {
  if (K > kMaxOffsetK && tile != kTile64) return INFINITY;
  return tiles_time(tile, tile_count(tile, m, N), K, epi, slices);
}

constexpr GemmParts kNoParts{nullptr, 0, nullptr, 0, nullptr};

struct GemmPlan {
  int tile;
  int slices;
  double time;
  bool chain = false;  // the slices add to the residual one behind the other
};

// Chained slices: steps that a slice is longer than the one in front of it (about what an update of the residual takes), and the time.
// Every slice needs a compute unit from the start. Fitted to 16 products: microseconds a step and what does not depend on K (the last
// update of the residual among it). Measured, best plan without / with a chain, us: 3271 x 1536 x 8960 114 to 118 / 84 to 92 (256 x 256,
// three slices), 4500 115 / 107 (two), 2352 72 / 71 (128 x 256, two), 2000 78 / 70, 1350 68 / 56 (three), 1100 50 / 46 (128 x 128, two), 480 31
// / 34; 1200 x 5120 x 13824 179 / 152 (256 x 256, two), 960 173 / 125 (three), 544 101 / 96 (128 x 256, two).
// 300 x 5120 x 5120 45 / 30 (128 x 128, two), 200 38 / 28 (three), 960 72 / 64 (256 x 256, three). With fewer steps a slice the updates are the
// larger part: 1200 x 1536 x 1536 14 to 16.5 / 17, 4500 28 / 39. (With slices by workgroup number; a ticket adds about 1.)
constexpr int kMaxChain = 4, kChainTiles = 256, kChainSteps = 16;
constexpr int chain_update(int tile) { return tile == kTile256 || tile == kTileWide ? 5 : 8; }
int chain_stagger(int tile, int K, int slices) {
  const int want = chain_update(tile), most = K / BK / slices;
  return want * (slices - 1) < most ? want : most / slices;  // the first slice keeps half of its steps
}
double chain_time(int tile, long m, int N, int K, int slices) {
  const long tiles = tile_count(tile, m, N);
  if (tile == kTile128 || K > kMaxOffsetK || N > 1 << 20 || tiles * slices > kChainTiles || K / BK / slices < kChainSteps) return INFINITY;
  const double fill = (double)(tiles * slices) / 256.0;
  // The whole update also where the slices are too short to be that far apart: it is waited for there (65 to 128 rows x 5120 x 5120,
  // four slices of 20 steps: a block with two of them 285 us at 78 rows, 273 with whole tiles).
  const double steps = (double)(K / BK) / slices + 0.5 * (slices - 1) * chain_update(tile);
  switch (tile) {
    case kTile256: return 16.3 + 5.0 * (slices - 2) + (1.17 + fmax(fill - 0.8, 0.0)) * steps;
    case kTileWide: return 15.0 + 2.0 * (slices - 2) + 0.72 * steps;
    case kTile128Deep: return 5.4 + 1.7 * (slices - 2) + (0.45 + 0.081 * fill * fill) * steps;
    default: return 6.0 + 2.5 * (slices - 2) + 0.246 * steps;
  }
}

// The fastest tile by the estimates. With scratch a gated-residual product may also be cut into slices of K: every slice
// but the last writes its fp32 result and a second launch adds them (about 6 TB/s from the caches, and the launch itself).
// Measured where N = 1536, K = 8960, slices against the best whole tile: 128 rows 17 / 41 us, 480 rows 31 / 37, 1200
// rows 46 / 66, 2000 and 2300 rows (two slices of 128 x 256 tiles) 75 / 72 and 77 / 79; beyond that a whole tile fills the chip.
GemmPlan plan_slices(long m, int N, int K, int epi, const GemmParts& parts) {
  GemmPlan best{kTile64, 1, INFINITY};
  for (int t = 0; t < kTiles; ++t) {
    const double v = tile_time(t, m, N, K, epi, 1);
    if (v < best.time) best = GemmPlan{t, 1, v};
  }
  if (epi != CHORUS_EPI_RESID || !parts.first || !aligned16(parts.first) || !aligned16(parts.rest)) return best;
  const double whole = best.time;
  const size_t one = (size_t)m * (size_t)N * sizeof(float);
  if (one > parts.first_bytes) return best;
  for (int sl = 2; sl <= kMaxSlices && sl <= K / BK; ++sl) {
    if (sl > 2 && (!parts.rest || (size_t)(sl - 2) * one > parts.rest_bytes)) break;
    const double add = 3.0 + (double)(2 * sl) * 4.0 * (double)m * N / 6.0e6;
    for (int t = 0; t < kTiles; ++t) {
      const double v = tile_time(t, m, N, K, epi, sl) + add;
      if (v < 0.95 * whole && v < best.time) best = GemmPlan{t, sl, v};
    }
  }
  return best;
}

// The same, or a chain where one may be taken and is estimated to be faster.
GemmPlan plan_gemm(long m, int N, int K, int epi, const GemmParts& parts) {
  GemmPlan best = plan_slices(m, N, K, epi, parts);
  if (!parts.counts || epi != CHORUS_EPI_RESID) return best;
  const double without = best.time;
  for (int sl = 2; sl <= kMaxChain && sl <= K / BK; ++sl)
    for (int t = 0; t < kTiles; ++t) {
      const double v = chain_time(t, m, N, K, sl);
      if (v < 0.97 * without && v < best.time) best = GemmPlan{t, sl, v, true};
    }
  return best;
}

constexpr int kHalvesDeep = 7, kHalves64 = 9;

// The groups of a chain: an XCD each, or two, four or all of them where their units would be fewer than their workgroups that way (three slices
// of 81 to 84 tiles: four groups; 880 x 1536 x 8960, 84 tiles: in one group a block 200.3 us, so 196.8).
int chain_groups(int tiles, int slices) {
  for (int groups = 8; groups > 1; groups /= 2)
    if ((tiles + groups - 1) / groups * groups * slices <= kChainTiles) return groups;
  return 1;
}

template <int WBM, int WBN, int C>
int32_t launch_chain(const uint16_t* A, const uint16_t* W, long M, int N, int K, const EpiArgs& ep, int slices, uint32_t* count,
                     int stagger, hipStream_t s) {
  constexpr int BM = 32 * WBM, BN = 32 * WBN;
  const long tm = (M + BM - 1) / BM;
  const int tn = (N + BN - 1) / BN;
  const size_t smem = (size_t)C * (BM + BN) / 2 * BK * sizeof(uint16_t);
  auto kern = gemm_w16_kernel<CHORUS_EPI_RESID, WBM, WBN, C, false, Chain>;
  static DynLdsOnce once;
  CHK_STATUS(once.ensure(reinterpret_cast<const void*>(kern), (int)smem));
  const int tiles = (int)(tm * tn), groups = chain_groups(tiles, slices);
  hipLaunchKernelGGL(kern, dim3((unsigned)align_up(tiles, groups), (unsigned)slices), dim3(256), smem, s, A, W, M, N, K, ep,
                     PartPtrs{nullptr, nullptr}, (int)tm, tn, Chain{count, stagger, tiles, groups});
  CHORUS_LAUNCH_CHECK();
  return CHORUS_OK;
}

int32_t launch_chain_tile(int tile, const uint16_t* A, const uint16_t* W, long M, int N, int K, const EpiArgs& ep, int slices,
                          uint32_t* counts, hipStream_t s) {
  const int stagger = chain_stagger(tile, K, slices);
  switch (tile) {
    case kTile256: return launch_chain<8, 8, 5>(A, W, M, N, K, ep, slices, counts, stagger, s);
    case kTileWide: return launch_chain<4, 8, 6>(A, W, M, N, K, ep, slices, counts, stagger, s);
    case kTile128Deep: return launch_chain<4, 4, kHalvesDeep>(A, W, M, N, K, ep, slices, counts, stagger, s);
    case kTile64: return launch_chain<2, 2, kHalves64>(A, W, M, N, K, ep, slices, counts, stagger, s);
    default: return CHORUS_E_ARG;
  }
}

int32_t launch_tile(int tile, const uint16_t* A, const uint16_t* W, long M, int N, int K, int epi, const EpiArgs& ep,
                    hipStream_t s, int slices = 1, const PartPtrs& parts = PartPtrs{nullptr, nullptr}) {
  if (K > kMaxOffsetK) return launch_gemm_w16<2, 2, kHalves64, true>(A, W, M, N, K, epi, ep, s, slices, parts);
  switch (tile) {
    case kTile256: return launch_gemm_w16<8, 8, 5>(A, W, M, N, K, epi, ep, s, slices, parts);
    case kTileWide: return launch_gemm_w16<4, 8, 6>(A, W, M, N, K, epi, ep, s, slices, parts);
    case kTile128: return launch_gemm_w16<4, 4, 5>(A, W, M, N, K, epi, ep, s, slices, parts);
    case kTile128Deep: return launch_gemm_w16<4, 4, kHalvesDeep>(A, W, M, N, K, epi, ep, s, slices, parts);
    default: return launch_gemm_w16<2, 2, kHalves64>(A, W, M, N, K, epi, ep, s, slices, parts);
  }
}

int32_t launch_plan(const GemmPlan& p, const uint16_t* A, const uint16_t* W, long M, int N, int K, int epi, const EpiArgs& ep,
                    const GemmParts& parts, hipStream_t s) {
  if (p.chain) return launch_chain_tile(p.tile, A, W, M, N, K, ep, p.slices, parts.counts, s);
  const PartPtrs pp{static_cast<float*>(parts.first), static_cast<float*>(parts.rest)};
  CHK_STATUS(launch_tile(p.tile, A, W, M, N, K, epi, ep, s, p.slices, pp));
  return p.slices > 1 ? launch_add_parts(pp, p.slices, M, N, ep, s) : CHORUS_OK;
}

// two products with bf16 outputs and the same K in one launch
template <int WBM, int WBN, int C>
int32_t launch_two(const uint16_t* A, const uint16_t* W, long M, int N, int K, const EpiArgs& ep, Twin twin, hipStream_t s) {
  constexpr int BM = 32 * WBM, BN = 32 * WBN;
  const long tm = (M + BM - 1) / BM, tm2 = (twin.M + BM - 1) / BM;
  const int tn = (N + BN - 1) / BN;
  twin.tiles_m = (int)tm2;
  twin.tiles_n = (twin.N + BN - 1) / BN;
  const long first = tm * tn, all = first + tm2 * twin.tiles_n;
  if (all > 0x7fffffffL) return CHORUS_E_SHAPE;
  twin.first = (int)first;
  const size_t smem = (size_t)C * (BM + BN) / 2 * BK * sizeof(uint16_t);
  auto kern = gemm_w16_kernel<CHORUS_EPI_BF16, WBM, WBN, C, false, Twin>;
  static DynLdsOnce once;
  CHK_STATUS(once.ensure(reinterpret_cast<const void*>(kern), (int)smem));
  hipLaunchKernelGGL(kern, dim3((unsigned)all), dim3(256), smem, s, A, W, M, N, K, ep, PartPtrs{nullptr, nullptr}, (int)tm, tn, twin);
  CHORUS_LAUNCH_CHECK();
  return CHORUS_OK;
}

int32_t check_gemm(const uint16_t* A, const uint16_t* W, int64_t M, int32_t N, int32_t K, const void* out, const float* bias,
                   const float* gate0, const float* gate1) {
  if (M < 0 || N <= 0 || K <= 0) return CHORUS_E_ARG;
  if (M == 0) return CHORUS_OK;
  if (!A || !W || !out) return CHORUS_E_ARG;
  if (K % BK || N % 8) return CHORUS_E_SHAPE;
  if (!aligned16(A) || !aligned16(W) || !aligned16(out) || !aligned16(bias) || !aligned16(gate0) || !aligned16(gate1))
    return CHORUS_E_ARG;
  return CHORUS_OK;
}

// The whole choice: the first head_rows rows in whole rounds of 256 x 256 tiles (0: no cut), the others by `rest`. A last
// round of 256 x 256 tiles that fills a small part of the chip costs most of a whole round. The rows can be cut instead:
// the row tiles that make up whole rounds go to the 256 x 256 kernel, the rows left over to whichever kernel suits that many
// rows, in a second launch behind the first. Taken when the estimate is better by 5 %; with up to three k-steps it was slower
// wherever it was taken (gated residual, 22 products with K = 64 and 128: 1.06 to 1.16 times; 4500 x 4608 x 128 36 us, whole 31).
struct GemmCut {
  long head_rows;
  GemmPlan rest;
  double time;  // of both launches
};
GemmCut plan_rows(long M, int N, int K, int epi, const GemmParts& parts) {
  const GemmPlan whole = plan_gemm(M, N, K, epi, parts);
  const long tiles_n256 = (N + 255) / 256, tiles256 = ((M + 255) / 256) * tiles_n256;
  const long head_rows = tiles256 > 256 && K >= 4 * BK ? (tiles256 / 256 * 256 / tiles_n256) * 256 : 0;
  if (head_rows > 0 && head_rows < M) {
    const GemmPlan tail = plan_gemm(M - head_rows, N, K, epi, GemmParts{nullptr, 0, nullptr, 0, parts.counts});
    const double time = tile_time(kTile256, head_rows, N, K, epi, 1) + tail.time;
    if (time < 0.95 * whole.time) return GemmCut{head_rows, tail, time};
  }
  return GemmCut{0, whole, whole.time};
}

// The tile on which two products with bf16 outputs and the same K run in one launch, kTiles: each in a launch of its own,
// whichever is the fastest by the estimates for the tiles of both together. 64 x 64 tiles up to one round of two workgroups a
// unit, the deep 128 x 128 ones up to two rounds of one; beyond that the larger product's own best tile is another one. Measured
// (tokens and text tokens, QKV and the text's keys and values; 64 x 64 / deep / apart, us): width 256, 128 and 16 4.8 / 5.7 / 7.8; width 1536, 100 and 16 9.9 / 18.2 / 17.9, 480 and 512 29.2 / 19.9 / 33.7, 800
// and 16 30.2 / 28.1 / 24.5, 900 and 512 40.9 / 33.3 / 39.4; width 5120, 100 and 512 160 / 113 / 129, 200 and 16 99 / 89 / 77, 200 and 512
// 179 / 152 / 129. Over 91 such pairs the choice is 1.2 % slower than the best (geometric mean), and never slower than apart.
int plan_two(long M, int N, long M2, int N2, int K) {
  if (K > kMaxOffsetK) return kTiles;
  const long small = tile_count(kTile64, M, N) + tile_count(kTile64, M2, N2);
  const long deep = tile_count(kTile128Deep, M, N) + tile_count(kTile128Deep, M2, N2);
  double best = plan_rows(M, N, K, CHORUS_EPI_BF16, kNoParts).time + plan_rows(M2, N2, K, CHORUS_EPI_BF16, kNoParts).time;
  int tile = kTiles;
  auto consider = [&](int t, double time) {
    if (time < best) {
      best = time;
      tile = t;
    }
  };
  consider(kTile64, tiles_time(kTile64, small, K, CHORUS_EPI_BF16, 1));
  if (deep <= 512)
    consider(kTile128Deep, tiles_time(kTile128Deep, deep < 256 ? deep : 256, K, CHORUS_EPI_BF16, 1) +
                               (deep > 256 ? tiles_time(kTile128Deep, deep - 256, K, CHORUS_EPI_BF16, 1) : 0.0));
  return tile;
}

}  // namespace

// One launch where plan_two says so (a block of 128 tokens of width 256 with 16 text tokens, its text keys and values prepared
// beside the tokens' in the same way: 62.9 -> 56.8 us).
int32_t gemm_bf16_two(const uint16_t* A, const uint16_t* W, int64_t M, int32_t N, int32_t K, uint16_t* out, const float* bias,
                      const uint16_t* A2, const uint16_t* W2, int64_t M2, int32_t N2, uint16_t* out2, const float* bias2,
                      void* stream) {
  CHK_STATUS(check_gemm(A, W, M, N, K, out, bias, nullptr, nullptr));
  CHK_STATUS(check_gemm(A2, W2, M2, N2, K, out2, bias2, nullptr, nullptr));
  if (M > 0 && M2 > 0) {
    const EpiArgs ep{out, bias, nullptr, nullptr, 1.f};
    const Twin twin{A2, W2, out2, bias2, (long)M2, N2, 0, 0, 0};
    switch (plan_two((long)M, N, (long)M2, N2, K)) {
      case kTile64: return launch_two<2, 2, kHalves64>(A, W, (long)M, N, K, ep, twin, (hipStream_t)stream);
      case kTile128Deep: return launch_two<4, 4, kHalvesDeep>(A, W, (long)M, N, K, ep, twin, (hipStream_t)stream);
      default: break;
    }
  }
  CHK_STATUS(gemm_bf16_parts(A, W, M, N, K, CHORUS_EPI_BF16, out, bias, nullptr, nullptr, 1.f, kNoParts, stream));
  return gemm_bf16_parts(A2, W2, M2, N2, K, CHORUS_EPI_BF16, out2, bias2, nullptr, nullptr, 1.f, kNoParts, stream);
}

bool gemm_bf16_chained(int64_t M, int32_t N, int32_t K, const GemmParts& parts) {
  return parts.counts && K / BK >= 2 * kChainSteps && plan_rows((long)M, N, K, CHORUS_EPI_RESID, parts).rest.chain;
}

int32_t gemm_bf16_parts(const uint16_t* A, const uint16_t* W, int64_t M, int32_t N, int32_t K, int32_t epilogue, void* out,
                        const float* bias, const float* gate0, const float* gate1, float scale, const GemmParts& parts,
                        void* stream) {
  CHK_STATUS(check_gemm(A, W, M, N, K, out, bias, gate0, gate1));
  if (M == 0) return CHORUS_OK;
  if (epilogue < CHORUS_EPI_BF16 || epilogue > CHORUS_EPI_RESID) return CHORUS_E_ARG;
  const EpiArgs ep{out, bias, gate0, gate1, scale};
  hipStream_t s = (hipStream_t)stream;
  const GemmCut cut = plan_rows((long)M, N, K, epilogue, parts);
  if (cut.head_rows == 0) return launch_plan(cut.rest, A, W, (long)M, N, K, epilogue, ep, parts, s);
  CHK_STATUS(launch_tile(kTile256, A, W, cut.head_rows, N, K, epilogue, ep, s));
  const size_t out_elt = (epilogue == CHORUS_EPI_F32 || epilogue == CHORUS_EPI_RESID) ? 4 : 2;
  EpiArgs ep_rest = ep;
  ep_rest.out = static_cast<uint8_t*>(out) + (size_t)cut.head_rows * (size_t)N * out_elt;
  return launch_plan(cut.rest, A + (size_t)cut.head_rows * (size_t)K, W, (long)M - cut.head_rows, N, K, epilogue, ep_rest,
                     GemmParts{nullptr, 0, nullptr, 0, parts.counts}, s);
}

}  // namespace chorus

using namespace chorus;

// tile of a kernel number, -1 for none
static int tile_of_number(int32_t kernel) {
  for (int t = 0; t < kTiles; ++t)
    if (kTileNumber[t] == kernel) return t;
  return -1;
}

extern "C" int32_t chorus_gemm_bf16_kernel(const uint16_t* A, const uint16_t* W, int64_t M, int32_t N, int32_t K,
                                           int32_t epilogue, void* out, const float* bias, const float* gate0,
                                           const float* gate1, float scale, int32_t kernel, void* stream) {
  if (kernel == 0) return gemm_bf16_parts(A, W, M, N, K, epilogue, out, bias, gate0, gate1, scale, kNoParts, stream);
  const int tile = tile_of_number(kernel);
  if (tile < 0) return CHORUS_E_ARG;
  CHK_STATUS(check_gemm(A, W, M, N, K, out, bias, gate0, gate1));
  if (M == 0) return CHORUS_OK;
  return launch_tile(tile, A, W, (long)M, N, K, epilogue, EpiArgs{out, bias, gate0, gate1, scale}, (hipStream_t)stream);
}

extern "C" int32_t chorus_gemm_bf16_slices(const uint16_t* A, const uint16_t* W, int64_t M, int32_t N, int32_t K, float* out,
                                           const float* bias, const float* gate0, const float* gate1, float scale,
                                           int32_t kernel, int32_t slices, float* parts, size_t parts_bytes, void* stream) {
  const int tile = tile_of_number(kernel);
  if (tile < 0 || slices < 1 || slices > kMaxSlices) return CHORUS_E_ARG;
  CHK_STATUS(check_gemm(A, W, M, N, K, out, bias, gate0, gate1));
  if (slices > K / BK) return CHORUS_E_SHAPE;
  if (M == 0) return CHORUS_OK;
  const size_t one = (size_t)M * (size_t)N * sizeof(float);
  if (slices > 1 && (!parts || !aligned16(parts) || parts_bytes < (size_t)(slices - 1) * one)) return CHORUS_E_WORKSPACE;
  const GemmParts two{parts, one, parts + (slices > 1 ? (size_t)M * N : 0), slices > 2 ? (size_t)(slices - 2) * one : 0, nullptr};
  return launch_plan(GemmPlan{tile, slices, 0.0}, A, W, (long)M, N, K, CHORUS_EPI_RESID, EpiArgs{out, bias, gate0, gate1, scale},
                     two, (hipStream_t)stream);
}

extern "C" int32_t chorus_gemm_bf16_plan(int64_t M, int32_t N, int32_t K, int32_t epilogue, size_t first_bytes, size_t rest_bytes,
                                         chorus_gemm_plan* out) {
  if (!out || M < 1 || N <= 0 || K <= 0 || epilogue < CHORUS_EPI_BF16 || epilogue > CHORUS_EPI_RESID) return CHORUS_E_ARG;
  if (K % BK || N % 8) return CHORUS_E_SHAPE;
  void* some = reinterpret_cast<void*>(uintptr_t{16});  // where the scratch lies does not matter
  const GemmCut cut = plan_rows((long)M, N, K, epilogue,
                                GemmParts{first_bytes ? some : nullptr, first_bytes, rest_bytes ? some : nullptr, rest_bytes, nullptr});
  *out = chorus_gemm_plan{cut.head_rows, kTileNumber[cut.rest.tile], cut.rest.slices};
  return CHORUS_OK;
}

extern "C" int32_t chorus_gemm_bf16_two_plan(int64_t M, int32_t N, int64_t M2, int32_t N2, int32_t K, int32_t* kernel) {
  if (!kernel || M < 1 || M2 < 1 || N <= 0 || N2 <= 0 || K <= 0) return CHORUS_E_ARG;
  if (K % BK || N % 8 || N2 % 8) return CHORUS_E_SHAPE;
  const int tile = plan_two((long)M, N, (long)M2, N2, K);
  *kernel = tile == kTiles ? 0 : kTileNumber[tile];
  return CHORUS_OK;
}

extern "C" int32_t chorus_gemm_bf16(const uint16_t* A, const uint16_t* W, int64_t M, int32_t N, int32_t K,
                                    int32_t epilogue, void* out, const float* bias, const float* gate0,
                                    const float* gate1, float scale, void* stream) {
  return gemm_bf16_parts(A, W, M, N, K, epilogue, out, bias, gate0, gate1, scale, kNoParts, stream);
}

__global__ __launch_bounds__(256) void clear_counts_kernel(uint32_t* p, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0;
}

extern "C" int32_t chorus_gemm_bf16_chain(const uint16_t* A, const uint16_t* W, int64_t M, int32_t N, int32_t K, float* out,
                                          const float* bias, const float* gate0, const float* gate1, float scale, int32_t kernel,
                                          int32_t slices, uint32_t* counts, int32_t n_counts, void* stream) {
  const int tile = tile_of_number(kernel);
  if (tile < 0 || tile == kTile128 || slices < 1 || slices > kMaxChain) return CHORUS_E_ARG;
  CHK_STATUS(check_gemm(A, W, M, N, K, out, bias, gate0, gate1));
  if (slices > K / BK || K > kMaxOffsetK || N > 1 << 20) return CHORUS_E_SHAPE;
  if (M == 0) return CHORUS_OK;
  const long tiles = tile_count(tile, (long)M, N);
  if (tiles * slices > 0x7fffffffL / 256) return CHORUS_E_SHAPE;
  if (!counts || n_counts < tiles) return CHORUS_E_WORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  hipLaunchKernelGGL(clear_counts_kernel, dim3((unsigned)((tiles + 255) / 256)), dim3(256), 0, s, counts, (int)tiles);
  CHORUS_LAUNCH_CHECK();
  return launch_chain_tile(tile, A, W, (long)M, N, K, EpiArgs{out, bias, gate0, gate1, scale}, slices, counts, s);
}

extern "C" int32_t chorus_gemm_bf16_chain_plan(int64_t M, int32_t N, int32_t K, size_t first_bytes, size_t rest_bytes, chorus_gemm_plan* out,
                                               int32_t* chained) {
  if (!out || !chained || M < 1 || N <= 0 || K <= 0) return CHORUS_E_ARG;
  if (K % BK || N % 8) return CHORUS_E_SHAPE;
  void* some = reinterpret_cast<void*>(uintptr_t{16});  // where the scratch lies does not matter
  const GemmCut cut = plan_rows((long)M, N, K, CHORUS_EPI_RESID, GemmParts{first_bytes ? some : nullptr, first_bytes,
                                rest_bytes ? some : nullptr, rest_bytes, static_cast<uint32_t*>(some)});
  *out = chorus_gemm_plan{cut.head_rows, kTileNumber[cut.rest.tile], cut.rest.slices};
  *chained = cut.rest.chain;
  return CHORUS_OK;
}
