// Flash-style attention for gfx950: O = softmax(g_j * (Q K^T) / sqrt(dh)) V, bf16
// operands on the matrix pipe, fp32 online softmax, logits never leave registers.
// Used for the block's 3-D self-attention (g = 1) and for the text cross-attention
// with TGAA key amplification (Eq. 2: scaling key j by gamma_k scales logit column j).
// Two kernels of one design: attention_pp_kernel on v_mfma_f32_32x32x16_bf16 (64-key
// tiles: keys padded to 64 only, and many queries on few keys), described first, and
// attention_pp16_kernel on v_mfma_f32_16x16x32_bf16 (128-key tiles: the rest, see
// attention_variant), whose differences are described in front of it.
// Both take the optional per-key logit factor.
//
// Work split: a workgroup of 8 waves owns 256 query rows of one head (32 per wave, held in
// registers) and sweeps all keys in tiles of 64 (128 in the second kernel). K tiles [keys][dh] and V^T tiles
// [dh][keys] are staged through LDS (double-buffered, rows padded by 16 bytes against bank
// conflicts) and shared by the 8 waves.
//
// The wave computes S^T = K Q^T, so a lane's 16 accumulator registers of a 32x32
// block all belong to ONE query row (column l%32) and 16 different keys
// (4*(l/32) + 8*j + i): the softmax row reductions are in-lane plus one exchange
// with lane l^32, and the probabilities are already laid out as the B operand of
// O^T = V^T P^T. The keys a lane holds for one 16-key MFMA step are
// {4c..4c+3, 8+4c..8+4c+3}; V^T is stored with that permutation (see
// chorus_v_transpose) so the matching A operand is a single 16-byte LDS read.
//
// The running maximum is only refreshed when a tile exceeds it by more than 8
// (in log2 units), which keeps exp2 arguments <= 8 and makes the accumulator
// rescale rare; the final division by the row sum makes the result exact either way.
#include "attention.h"
#include "chorus_ops.h"
#include "common.h"

namespace chorus {
namespace {

constexpr int KT = 64;  // granularity of the key padding (the smaller of the two tile sizes)

// ---------------------------------------------------------------------------
// Ping-pong phases: 8 waves, one block of 32 query rows each, two groups of four
// waves (one wave of each group per SIMD). A wave alternates between a VALU phase
// (softmax of tile j) and an MFMA phase (O += V(j) P(j), then S(j+1) = K(j+1) Q^T),
// separated by workgroup barriers; group 1 runs one phase behind group 0, so on
// every SIMD one wave feeds the matrix pipe while the other runs the softmax.
//
// LDS holds two K and two V^T tiles. In its MFMA phase of tile j a wave first
// stores the registers it prefetched one iteration earlier (K(j+2) into the
// buffer S(j) was read from, V(j+1) into the buffer of V(j-1)), then issues the
// global loads for K(j+3) and V(j+2). Both groups have finished reading a buffer
// at least one barrier before either group overwrites it.
// ---------------------------------------------------------------------------
template <int DH, int KTL, bool COLSCALE>
__global__ __launch_bounds__(512, 2) void attention_pp_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ Vt,
    uint16_t* __restrict__ O, const float* __restrict__ col_scale, long Lq, long Lk, long LqPad, long LkPad, int H,
    int n_qtiles, float scale_log2) {
  constexpr int NT = 512;
  constexpr int KS = DH + 8, VS = KTL + 8;  // padded LDS row strides (elements)
  constexpr int KB = KTL / 32;                // 32-key blocks of S^T per tile
  constexpr int NKS = KTL / 16;               // 16-key MFMA steps of P V per tile
  constexpr int K_LD = KTL * (DH / 8) / NT;
  constexpr int V_LD = DH * (KTL / 8) / NT;
  constexpr int SK = DH / 16;
  constexpr int TD = DH / 32;
  constexpr int QROWS = 8 * 32;

  extern __shared__ __attribute__((aligned(16))) uint8_t smem_raw[];
  uint16_t* smk = reinterpret_cast<uint16_t*>(smem_raw);   // [2][KTL][KS]
  uint16_t* smv = smk + 2 * KTL * KS;                      // [2][DH][VS]

  const int tile_id = xcd_remap(blockIdx.x, H * n_qtiles);
  const int head = tile_id / n_qtiles;
  const int qt = tile_id - head * n_qtiles;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int group = wave >> 2;
  const int lrow = lane & 31, c = lane >> 5, lk = c * 8;
  const long q_wave0 = (long)qt * QROWS + wave * 32;

  const uint16_t* Kh = K + (long)head * LkPad * DH;
  const uint16_t* Vh = Vt + (long)head * DH * LkPad;

  bf16x8 qf[SK];
  {
    long q = q_wave0 + lrow;
    if (q > Lq - 1) q = Lq - 1;
    const uint16_t* qp = Q + ((long)head * LqPad + q) * DH + lk;
#pragma unroll
    for (int s = 0; s < SK; ++s) qf[s] = *reinterpret_cast<const bf16x8*>(qp + 16 * s);
  }

  f32x16 o[TD];
#pragma unroll
  for (int t = 0; t < TD; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[t][r] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;

  const int ntiles = (int)((Lk + KTL - 1) / KTL);
  u32x4 rk[K_LD], rv[V_LD];

  auto load_k = [&](int kt) {
#pragma unroll
    for (int i = 0; i < K_LD; ++i)
      rk[i] = *reinterpret_cast<const u32x4*>(Kh + (long)kt * KTL * DH + (tid + NT * i) * 8);
  };
  auto load_v = [&](int kt) {
#pragma unroll
    for (int i = 0; i < V_LD; ++i) {
      int id = tid + NT * i, row = id / (KTL / 8), ch = id % (KTL / 8);
      rv[i] = *reinterpret_cast<const u32x4*>(Vh + (long)row * LkPad + (long)kt * KTL + ch * 8);
    }
  };
  auto store_k = [&](int buf) {
#pragma unroll
    for (int i = 0; i < K_LD; ++i) {
      int id = tid + NT * i, row = id / (DH / 8), ch = id % (DH / 8);
      *reinterpret_cast<u32x4*>(&smk[(buf * KTL + row) * KS + ch * 8]) = rk[i];
    }
  };
  auto store_v = [&](int buf) {
#pragma unroll
    for (int i = 0; i < V_LD; ++i) {
      int id = tid + NT * i, row = id / (KTL / 8), ch = id % (KTL / 8);
      *reinterpret_cast<u32x4*>(&smv[(buf * DH + row) * VS + ch * 8]) = rv[i];
    }
  };
  f32x16 s[KB];
  auto compute_s = [&](int buf) {
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) s[kb][r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < SK; ++ks) {
      bf16x8 kf[KB];
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
        kf[kb] = *reinterpret_cast<const bf16x8*>(&smk[(buf * KTL + 32 * kb + lrow) * KS + 16 * ks + lk]);
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kb], qf[ks], s[kb], 0, 0, 0);
    }
  };

  // prologue: K(0), V(0), K(1) into LDS; K(2), V(1) into the prefetch registers
  load_k(0);
  load_v(0);
  store_k(0);
  store_v(0);
  if (ntiles > 1) {
    load_k(1);
    store_k(1);
    load_v(1);
  }
  if (ntiles > 2) load_k(2);
#pragma unroll
  for (int sI = 0; sI < SK; ++sI) asm volatile("" : "+v"(qf[sI]));  // Q fragments resident before the loop
  __syncthreads();
  compute_s(0);
  __syncthreads();
  if (group == 1) lds_barrier();  // run one phase behind group 0

  for (int j = 0; j < ntiles; ++j) {
    // ================= VALU phase: softmax of tile j =================
    __builtin_amdgcn_sched_barrier(0);
    const long key0 = (long)j * KTL + 4 * c;
    if (COLSCALE) {
      // a lane's keys come in runs of four: one 16-byte load per run (the runs that cross the end one key at a time)
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const long key = key0 + 32 * kb + 8 * q4;
          f32x4 cf;
          if (key + 3 < Lk) {
            cf = *reinterpret_cast<const f32x4*>(col_scale + key);
          } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) cf[i] = key + i < Lk ? col_scale[key + i] : 1.0f;
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) s[kb][4 * q4 + i] *= cf[i] * scale_log2;
        }
    }
    if (j == ntiles - 1 && (Lk % KTL) != 0) {
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          long key = key0 + 32 * kb + 8 * (r >> 2) + (r & 3);
          if (key >= Lk) s[kb][r] = -INFINITY;
        }
    }
    float mx = s[0][0];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[kb][r]);
    mx = fmaxf(mx, swap_halves(mx));
    const float mxs = COLSCALE ? mx : mx * scale_log2;
    if (__any(mxs > m_run + 8.0f)) {
      const float m_new = fmaxf(m_run, mxs);
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int t = 0; t < TD; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[t][r] *= alpha;
    }
    bf16x8 pf[NKS];
    {
      const float mref = m_run;
      float lsum = 0.f;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        float p[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float a = COLSCALE ? (s[kb][r] - mref) : __builtin_fmaf(s[kb][r], scale_log2, -mref);
          p[r] = __builtin_amdgcn_exp2f(a);
          lsum += p[r];
        }
#pragma unroll
        for (int h2 = 0; h2 < 2; ++h2)
#pragma unroll
          for (int e = 0; e < 8; ++e) pf[2 * kb + h2][e] = (bf16_t)p[8 * h2 + e];
      }
      l_run += lsum;
    }
    // the probabilities must exist before the barrier (otherwise the compiler sinks the
    // exponentials into the MFMA phase, which defeats the phase split)
#pragma unroll
    for (int i = 0; i < NKS; ++i) asm volatile("" : "+v"(pf[i]));
    __builtin_amdgcn_sched_barrier(0);
    lds_barrier();
    __builtin_amdgcn_sched_barrier(0);

    // ================= MFMA phase: O += V(j) P(j); S(j+1) = K(j+1) Q^T =================
    // Branch-free on purpose (one basic block the scheduler can pipeline): past the last
    // tiles the prefetch re-reads the final tile and the extra stores / S tile are never used.
    __builtin_amdgcn_s_setprio(1);
    store_k(j & 1);
    store_v((j + 1) & 1);
    load_k(j + 3 < ntiles ? j + 3 : ntiles - 1);
    load_v(j + 2 < ntiles ? j + 2 : ntiles - 1);
    {
      const int vb = j & 1;
#pragma unroll
      for (int t = 0; t < TD; ++t) {
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
          const bf16x8 vf = *reinterpret_cast<const bf16x8*>(&smv[(vb * DH + 32 * t + lrow) * VS + 16 * ks + lk]);
          o[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[ks], o[t], 0, 0, 0);
        }
      }
    }
    compute_s((j + 1) & 1);
    // issue order: LDS stores, global prefetch, then LDS operand reads kept 6 ahead of the MFMAs
    __builtin_amdgcn_sched_group_barrier(0x200, K_LD + V_LD, 0);
    __builtin_amdgcn_sched_group_barrier(0x020, K_LD + V_LD, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
#pragma unroll
    for (int i = 0; i < NKS * TD + KB * SK - 6; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 6, 0);
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    lds_barrier();  // this wave's LDS stores are done; the global prefetch stays in flight
    __builtin_amdgcn_sched_barrier(0);
  }
  if (group == 0) lds_barrier();  // every wave executes the same number of barriers

  const int D = H * DH;
  const float l = l_run + __shfl_xor(l_run, 32, 64);
  const float inv = 1.0f / l;
  const long q = q_wave0 + lrow;
  if (q < Lq) {
    uint16_t* op = O + q * (long)D + head * DH + 4 * c;
#pragma unroll
    for (int t = 0; t < TD; ++t)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        uint2 w;
        w.x = pack_bf16x2(o[t][4 * jj + 0] * inv, o[t][4 * jj + 1] * inv);
        w.y = pack_bf16x2(o[t][4 * jj + 2] * inv, o[t][4 * jj + 3] * inv);
        *reinterpret_cast<uint2*>(op + 32 * t + 8 * jj) = w;
      }
  }
}

// Slices of the keys. A last round of tiles that leaves half of the compute units idle or more runs `slices` workgroups a tile, each over
// its share of the 128-key tiles (`units`) and from a reference of its own; the last of a tile's workgroups to end puts it together:
//   every workgroup takes a number (`ticket`); all but the last leave their unnormalised fp32 result, row sums and references in
//   a slab and report it (`done`); the last keeps its own in registers, waits until the others have reported, and adds all of them
//   in the order of their keys, so that the result does not depend on who was last.
// The wait ends: it is for workgroups that have taken their number, which run and have nothing to wait for but their own stores.
// Slabs and counts are agent-scope accesses past the L2s (the workgroups of a tile run on different XCDs); a slab is reported when its
// stores have completed. ticket and done start at zero (attn_prepare clears them).
struct KeySlices {
  uint32_t* words;  // ticket [tiles], done [tiles], which slice a slab holds [tiles][slices - 1]; then slabs
  float* slab1;     // the slabs that do not fit there
  int tiles, slices, units;
  int slab0, n0;    // where the first slab stands behind `words`, in 32-bit words, and how many stand there
  static constexpr bool kSliced = true, kRun = false;
};
struct WholeKeys {
  static constexpr bool kSliced = false, kRun = false;
};
// A workgroup that walks over its share of `tiles` tiles. The loop over a tile's keys runs on into the next tile's: the next queries
// are requested in the last softmax phase, when this tile's are no longer needed, the next first keys in their usual place, and the finished
// tile leaves in the next first softmax phase, under the other group's MFMAs. A workgroup that ends instead leaves its unit to one
// that starts cold: 3 to 4 us a tile (32760 x 512, 12 heads, six tiles a unit 152 -> 127 us; 75600 x 512, 40 heads, 47 tiles 1002 -> 866).
struct TileRun {
  const uint16_t *Q, *K, *Vt;
  uint16_t* O;
  long Lq, LqPad, LkPad;
  int H, n_qtiles, tiles, stride;
  static constexpr bool kSliced = false, kRun = true;
};
// 8-byte words of one lane in a slab: the results in halves of four, then (reference, row sum) per block of rows
constexpr int slab_words(int dh, int rb) { return (dh / 16 * 2 + 1) * rb; }

__device__ __forceinline__ void store_pair(float* p, float a, float b) {
  const uint64_t v = ((uint64_t)__float_as_uint(b) << 32) | __float_as_uint(a);
  __hip_atomic_store(reinterpret_cast<uint64_t*>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 load_pair(const float* p) {
  const uint64_t v = __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_float2(__uint_as_float((uint32_t)v), __uint_as_float((uint32_t)(v >> 32)));
}

// ---------------------------------------------------------------------------
// The same ping-pong kernel on v_mfma_f32_16x16x32_bf16, 128-key tiles, no column scale. Per flop this shape writes
// half the accumulator registers of the 32x32x16 one and a result block is accumulated by four MFMAs in a row (the
// whole head dimension or the whole key tile), which is what the power-managed part rewards.
//
// A wave still owns 32 query rows, as two blocks of 16 (rb). Lane l: query row l % 16 of each block, and of every
// 16 x 16 result block the four rows 4 g .. 4 g + 3, g = l / 16.
//   S^T block kb (16 keys x 16 query rows, kb = 0..7 of a 128-key tile): the K fragment's row r is key
//   32 (kb / 2) + 16 (r / 8) + 8 (kb % 2) + r % 8 of the tile, so the lane holds keys 32 (kb / 2) + 16 (g / 2) +
//   8 (kb % 2) + 4 (g % 2) + i. For a 32-key step of O^T += V^T P^T (blocks kb = 2 c, 2 c + 1) these eight keys are
//   {4 (g % 2) .. + 3, 8 + 4 (g % 2) .. + 3} of the 16-key group 2 c + g / 2: exactly the eight consecutive
//   positions 8 g .. 8 g + 7 of the step in the stored V^T order (see chorus_v_transpose), so the V operand is one
//   16-byte LDS read and the lane's probabilities are its B operand as they stand.
// LDS rows are padded by 32 bytes: with 16 rows x 4 chunks per fragment read that stride is free of bank conflicts.
// Two things leave the vector pipe, which in this kernel is as loaded as the matrix pipe: the softmax row sums are
// taken by the matrix pipe (one more result block per 16 query rows whose V operand is all ones, so the sum is over
// the same bf16-rounded probabilities that weight V and the weights of a row add up to exactly one), and the global
// prefetch of the next tiles is issued at the start of the softmax phase instead of the MFMA phase.
// ---------------------------------------------------------------------------
// KIND 0 and 1 are the same code: 1 gives launches with a key sequence other than the query sequence (the text
// cross-attention) a kernel name of their own, so that a kernel profile lists self- and cross-attention separately.
// KIND 2 multiplies the logit of key j by col_scale[j] (TGAA's key amplification, Eq. 2, applied to the logit): the
// S^T accumulators then start at zero and one multiply-add per logit applies the factor and, with PRE, the reference.
// The factors of a tile come through LDS like its keys: read from memory where they are used, in pairs for want of
// registers, they cost four memory latencies per tile (480 x 512 24.3 -> 15.5 us, 13104 x 512 73.6 -> 69.2).
// KIND 3 and 4 are 1 and 2 for fewer than 512 keys: the row sums are taken by the vector pipe, in fp32 over the
// probabilities before they are rounded, as attention_pp_kernel takes them. Over a few tiles that costs next to nothing, and a
// call has the same denominator whichever of the two kernels runs it.
template <int DH, bool PRE, int RB, int KIND, class KEYS>
__global__ __launch_bounds__(512, 2) void attention_pp16_kernel(
    KEYS keys_arg, const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ Vt,
    uint16_t* __restrict__ O, const float* __restrict__ col_scale, long Lq, long Lk, long LqPad, long LkPad, int H,
    int n_qtiles, int tile_base, float scale_log2) {
  constexpr bool CS = KIND == 2 || KIND == 4, SUM32 = KIND >= 3;
  constexpr int NT = 512;
  constexpr int KTL = 128;
  constexpr int KS = DH + 16, VS = KTL + 16;  // padded LDS row strides (elements)
  constexpr int KB = KTL / 16;                 // 16-key blocks of S^T per tile
  constexpr int NC = KTL / 32;                 // 32-key MFMA steps of P V per tile
  constexpr int KC = DH / 32;                  // 32-wide steps over the head dimension
  constexpr int DB = DH / 16;                  // 16-row blocks of O^T
  constexpr int K_LD = KTL * (DH / 8) / NT;
  constexpr int V_LD = DH * (KTL / 8) / NT;
  constexpr int QROWS = 8 * 16 * RB;  // RB blocks of 16 query rows per wave

  extern __shared__ __attribute__((aligned(16))) uint8_t smem_raw[];
  uint16_t* smk = reinterpret_cast<uint16_t*>(smem_raw);   // [2][KTL][KS]
  uint16_t* smv = smk + 2 * KTL * KS;                      // [2][DH][VS]
  float* smc = reinterpret_cast<float*>(smv + 2 * DH * VS);  // [2][KTL]: the key factors of two tiles (CS)

  // this launch covers the tiles tile_base .. tile_base + gridDim.x - 1 of the H * n_qtiles of its tile size, or in slices a
  // keys.slices-th as many
  int tile_id = tile_base + xcd_remap(blockIdx.x, gridDim.x), first_kt = 0;
  int stride = 1, runs = 1;  // TileRun: the workgroups of an XCD take its range of tiles in turn, neighbours at a time
  if constexpr (KEYS::kRun) {
    const int xcd = blockIdx.x % 8, q = keys_arg.tiles / 8, r = keys_arg.tiles % 8, mine = q + (xcd < r), local = blockIdx.x / 8;
    stride = keys_arg.stride;
    runs = (mine - local + stride - 1) / stride;
    if (runs <= 0) return;
    tile_id = tile_base + xcd * q + (xcd < r ? xcd : r) + local;
  }
  if constexpr (KEYS::kSliced) {
    const KeySlices& keys = keys_arg;
    const int at = tile_id - tile_base, t = at / keys.slices, slice = at - t * keys.slices;
    tile_id = tile_base + t;
    first_kt = first_of_slice(slice, keys.units, keys.slices);
    const long end = (long)first_of_slice(slice + 1, keys.units, keys.slices) * KTL;
    Lk = (Lk < end ? Lk : end) - (long)first_kt * KTL;
  }
  const int head = tile_id / n_qtiles;
  const int qt = tile_id - head * n_qtiles;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int group = wave >> 2;
  const int lq = lane & 15, g = lane >> 4;

  const uint16_t* Kh = K + ((long)head * LkPad + (long)first_kt * KTL) * DH;
  const uint16_t* Vh = Vt + (long)head * DH * LkPad + (long)first_kt * KTL;

  bf16x8 qf[RB][KC];
  auto load_q = [&](const uint16_t* Q, long Lq, long LqPad, int of_head, int of_qt) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      int t = tid;
      if constexpr (CS && KEYS::kRun) asm volatile("" : "+v"(t));  // as fresh_tid below
      long q = (long)of_qt * QROWS + (t >> 6) * 16 * RB + 16 * rb + (t & 15);
      if (q > Lq - 1) q = Lq - 1;
      const uint16_t* qp = Q + ((long)of_head * LqPad + q) * DH + 8 * ((t & 63) >> 4);
#pragma unroll
      for (int kc = 0; kc < KC; ++kc) qf[rb][kc] = *reinterpret_cast<const bf16x8*>(qp + 32 * kc);
    }
  };
  load_q(Q, Lq, LqPad, head, qt);

  f32x4 o[DB][RB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) o[db][rb] = f32x4{0.f, 0.f, 0.f, 0.f};
  // PRE: Q arrives multiplied by log2(e) / sqrt(dh) and the S^T accumulators start at minus the running reference, so
  // a logit leaves the MFMA as the exponent of its probability; the reference starts at 0 and the first tile sets it.
  float m_run[RB];
  f32x4 lacc[RB];   // row sums (a row's sum in every element), unless SUM32:
  float l_run[RB];  // this lane's part of them
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    m_run[rb] = PRE ? 0.f : -INFINITY;
    lacc[rb] = f32x4{0.f, 0.f, 0.f, 0.f};
    l_run[rb] = 0.f;
  }
  bf16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = (bf16_t)1.0f;

  const int ntiles = (int)((Lk + KTL - 1) / KTL);
  u32x4 rk[K_LD], rv[V_LD];

  auto load_k_of = [&](const uint16_t* base, int kt) {
#pragma unroll
    for (int i = 0; i < K_LD; ++i)
      rk[i] = *reinterpret_cast<const u32x4*>(base + (long)kt * KTL * DH + (uint32_t)((tid + NT * i) * 8));
  };
  auto load_v_of = [&](const uint16_t* base, int kt) {
#pragma unroll
    for (int i = 0; i < V_LD; ++i) {
      int id = tid + NT * i, row = id / (KTL / 8), ch = id % (KTL / 8);
      if constexpr (KEYS::kRun)  // a scalar base and a 32-bit offset: 128 rows of at most 2^23 keys
        rv[i] = *reinterpret_cast<const u32x4*>(base + (long)kt * KTL + (uint32_t)(row * (int)LkPad + ch * 8));
      else
        rv[i] = *reinterpret_cast<const u32x4*>(base + (long)row * LkPad + (long)kt * KTL + ch * 8);
    }
  };
  auto load_k = [&](int kt) { load_k_of(Kh, kt); };
  auto load_v = [&](int kt) { load_v_of(Vh, kt); };
  auto store_k = [&](int buf) {
#pragma unroll
    for (int i = 0; i < K_LD; ++i) {
      int id = tid + NT * i, row = id / (DH / 8), ch = id % (DH / 8);
      *reinterpret_cast<u32x4*>(&smk[(buf * KTL + row) * KS + ch * 8]) = rk[i];
    }
  };
  auto store_v = [&](int buf) {
#pragma unroll
    for (int i = 0; i < V_LD; ++i) {
      int id = tid + NT * i, row = id / (KTL / 8), ch = id % (KTL / 8);
      *reinterpret_cast<u32x4*>(&smv[(buf * DH + row) * VS + ch * 8]) = rv[i];
    }
  };
  // Key factors of a tile: a thread of the first two waves fetches one with the tile before and stores it in its MFMA
  // phase, one barrier ahead of the softmax phase that reads it (the other group, half an iteration behind, then still
  // reads the other buffer). Keys past the end get 1.
  // With factors and 256 rows the kernel is at the register limit, and what a few instructions make again from the thread
  // id must not be kept across the loop: this hides the id from the compiler, which would keep it and spill six registers.
  // That is the factors' addresses and the output's (scaled queries, 32760 x 512, 12 heads 141.3 -> 137.3 us, 13104 x 512, 40 heads
  // 209 -> 202, 13104 x 226, 40 heads 173 -> 165). The V rows' addresses stay: made again for every tile they cost 10 % of the launch.
  auto fresh_tid = [&]() {
    int t = tid;
    if constexpr (CS) asm volatile("" : "+v"(t));
    return t;
  };
  float rc = 1.f;
  auto load_c = [&](int kt) {
    const int key = kt * KTL + fresh_tid();
    if (tid < KTL) rc = key < (int)Lk ? col_scale[key] : 1.0f;
  };
  auto store_c = [&](int buf) {
    if (tid < KTL) smc[buf * KTL + fresh_tid()] = rc;
  };
  // LDS row of the K tile that fragment row lane % 16 of block kb stands for
  const int krow0 = 16 * (lq >> 3) + (lq & 7);
  f32x4 s[KB][RB];
  auto compute_s = [&](int buf) {
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      bf16x8 kf[KC];
      const int row = 32 * (kb >> 1) + 8 * (kb & 1) + krow0;
#pragma unroll
      for (int kc = 0; kc < KC; ++kc)
        kf[kc] = *reinterpret_cast<const bf16x8*>(&smk[(buf * KTL + row) * KS + 32 * kc + 8 * g]);
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        const float a0 = (PRE && !CS) ? -m_run[rb] : 0.f;
        f32x4 acc = {a0, a0, a0, a0};
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[kc], qf[rb][kc], acc, 0, 0, 0);
        s[kb][rb] = acc;
      }
    }
  };

  // Prologue: K(0), V(0), K(1) into LDS. Half tiles and short keys request all three before the first is stored. In the
  // long launches that costs more than it saves (75600 x 75600, 40 heads: 90.0 ms against 88.7): the workgroups of an XCD
  // then no longer read the same keys closely enough one behind the other.
  if constexpr (RB == 2 && !CS) {
    load_k(0);
    load_v(0);
    store_k(0);
    store_v(0);
    if (ntiles > 1) {
      load_k(1);
      store_k(1);
    }
  } else {
    load_k(0);
    load_v(0);
    if constexpr (CS) load_c(0);
    u32x4 r0[K_LD];
#pragma unroll
    for (int i = 0; i < K_LD; ++i) r0[i] = rk[i];
    load_k(ntiles > 1 ? 1 : 0);
#pragma unroll
    for (int i = 0; i < K_LD; ++i) {
      const int id = tid + NT * i, row = id / (DH / 8), ch = id % (DH / 8);
      *reinterpret_cast<u32x4*>(&smk[row * KS + ch * 8]) = r0[i];
    }
    store_v(0);
    if constexpr (CS) store_c(0);
    store_k(1);
  }
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) asm volatile("" : "+v"(qf[rb][kc]));  // Q fragments resident before the loop
  __syncthreads();
  compute_s(0);
  __syncthreads();
  if (group == 1) lds_barrier();  // run one phase behind group 0

  // TileRun: the arguments again, read where they are needed instead of kept in scalar registers across the loop
  typedef const __attribute__((address_space(4))) KEYS* ArgPtr;
  auto args = [&]() {
    ArgPtr a = (ArgPtr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(a));
    return a;
  };
  // the rows of a tile leave
  auto finish = [&](uint16_t* O, long Lq, int D, int head, int qt) {
    const long q_wave0 = (long)qt * QROWS + wave * 16 * RB;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      float l = lacc[rb][0];
      if constexpr (SUM32) {  // the four lanes that share a query row
        l = l_run[rb] + swap_rows16(l_run[rb]);
        l += swap_halves(l);
      }
      const float inv = 1.0f / l;
      const int t = fresh_tid();
      const long q = CS ? (long)qt * QROWS + (t >> 6) * 16 * RB + 16 * rb + (t & 15) : q_wave0 + 16 * rb + lq;
      if (q < Lq) {
        uint16_t* op = O + q * (long)D + head * DH + 4 * (CS ? (t & 63) >> 4 : g);
#pragma unroll
        for (int db = 0; db < DB; ++db) {
          uint2 w;
          w.x = pack_bf16x2(o[db][rb][0] * inv, o[db][rb][1] * inv);
          w.y = pack_bf16x2(o[db][rb][2] * inv, o[db][rb][3] * inv);
          *reinterpret_cast<uint2*>(op + 16 * db) = w;
        }
      }
    }
  };
  bool started = false;  // a tile is waiting to leave
  int parity = 0;        // of all key tiles so far
  for (int j = 0; KEYS::kRun || j < ntiles;) {  // j: which tile of keys
    const int buf = KEYS::kRun ? parity : j & 1;  // where in LDS it is
    // ================= VALU phase: softmax of tile j =================
    __builtin_amdgcn_sched_barrier(0);
    const bool last_kt = j == ntiles - 1;
    const bool on = KEYS::kRun && runs > 1;  // another tile of queries behind this one
    const uint16_t *Kn = Kh, *Vn = Vh;       // its keys and values
    if constexpr (KEYS::kRun) {
      if (j == 0 && started) {
        const ArgPtr a = args();
        const int t = tile_id - a->stride, nq = a->n_qtiles, of_head = t / nq;
        finish(a->O, a->Lq, a->H * DH, of_head, t - of_head * nq);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          lacc[rb] = f32x4{0.f, 0.f, 0.f, 0.f};
          l_run[rb] = 0.f;
#pragma unroll
          for (int db = 0; db < DB; ++db) o[db][rb] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (on && j + 2 >= ntiles) {
        const ArgPtr a = args();
        const int t = tile_id + a->stride, nq = a->n_qtiles, of_head = t / nq;
        Kn = a->K + (long)of_head * a->LkPad * DH;
        Vn = a->Vt + (long)of_head * DH * a->LkPad;
        if (last_kt) load_q(a->Q, a->Lq, a->LqPad, of_head, t - of_head * nq);
      }
    }
    if constexpr (CS) {
      const float* cfs = smc + buf * KTL + 16 * (g >> 1) + 4 * (g & 1);
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        const f32x4 cf = *reinterpret_cast<const f32x4*>(cfs + 32 * (kb >> 1) + 8 * (kb & 1));
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            s[kb][rb][i] = PRE ? __builtin_fmaf(s[kb][rb][i], cf[i], -m_run[rb]) : s[kb][rb][i] * cf[i];
        if (kb % 2 == 1) __builtin_amdgcn_sched_barrier(0);  // two factors in flight at a time: there are no registers for eight
      }
      load_c(!last_kt ? j + 1 : on ? 0 : ntiles - 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    // the global prefetch of the tiles that the next MFMA phase stores: K(j+2), V(j+1) (past the end the next tile's first, or the last again)
    load_k_of(j + 2 < ntiles ? Kh : Kn, j + 2 < ntiles ? j + 2 : on ? j + 2 - ntiles : ntiles - 1);
    load_v_of(last_kt ? Vn : Vh, !last_kt ? j + 1 : on ? 0 : ntiles - 1);
    if (last_kt && (Lk % KTL) != 0) {
      // Long keys: compared here. Hoisted out of the loop the 32 results take 64 scalar registers, and what that displaces costs the LDS
      // reads of the MFMA phase their lead where registers are short (with factors, and where workgroups walk over tiles). Over a few
      // tiles of keys the comparisons themselves cost more (13104 x 226 with factors, 40 heads 165 -> 173 us).
      const int gg = CS && !SUM32 ? (fresh_tid() & 63) >> 4 : g;
      int rest = (int)(Lk - (long)j * KTL) - (16 * (gg >> 1) + 4 * (gg & 1));
      if constexpr (!SUM32) asm volatile("" : "+v"(rest));
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const bool past = SUM32 ? (long)j * KTL + 16 * (g >> 1) + 4 * (g & 1) + 32 * (kb >> 1) + 8 * (kb & 1) + i >= Lk
                                  : 32 * (kb >> 1) + 8 * (kb & 1) + i >= rest;
          if (past) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) s[kb][rb][i] = -INFINITY;
          }
        }
    }
    float mxs[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      float mx = s[0][rb][0];
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int i = 0; i < 4; ++i) mx = fmaxf(mx, s[kb][rb][i]);
      mx = fmaxf(mx, swap_rows16(mx));
      mx = fmaxf(mx, swap_halves(mx));
      mxs[rb] = PRE ? mx : mx * scale_log2;
    }
    if constexpr (PRE) {
      // logits are relative to the reference already: move it when a row exceeds it by more than 8, and on the first tile
      bool move = false;
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) move = move || mxs[rb] > 8.0f;
      if (__any(move) || j == 0) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          const float delta = j == 0 ? mxs[rb] : fmaxf(mxs[rb], 0.f);
          const float alpha = j == 0 ? 1.0f : __builtin_amdgcn_exp2f(-delta);  // nothing is accumulated before the first tile
          m_run[rb] += delta;
          lacc[rb] *= alpha;
          l_run[rb] *= alpha;
#pragma unroll
          for (int db = 0; db < DB; ++db) o[db][rb] *= alpha;
#pragma unroll
          for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int i = 0; i < 4; ++i) s[kb][rb][i] -= delta;
        }
      }
    } else {
      bool move = false;
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) move = move || mxs[rb] > m_run[rb] + 8.0f;
      if (__any(move)) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        const float m_new = fmaxf(m_run[rb], mxs[rb]);
        const float alpha = __builtin_amdgcn_exp2f(m_run[rb] - m_new);
        m_run[rb] = m_new;
        lacc[rb] *= alpha;
        l_run[rb] *= alpha;
#pragma unroll
        for (int db = 0; db < DB; ++db) o[db][rb] *= alpha;
      }
      }
    }
    bf16x8 pf[NC][RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const float mref = m_run[rb];
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float p = PRE ? __builtin_amdgcn_exp2f(s[2 * c + b][rb][i])
                                : __builtin_amdgcn_exp2f(__builtin_fmaf(s[2 * c + b][rb][i], scale_log2, -mref));
            if constexpr (SUM32) l_run[rb] += p;
            pf[c][rb][4 * b + i] = (bf16_t)p;
          }
    }
    // the probabilities must exist before the barrier (otherwise the compiler sinks the
    // exponentials into the MFMA phase, which defeats the phase split)
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) asm volatile("" : "+v"(pf[c][rb]));
    __builtin_amdgcn_sched_barrier(0);
    lds_barrier();
    __builtin_amdgcn_sched_barrier(0);

    // ================= MFMA phase: O += V(j) P(j); S(j+1) = K(j+1) Q^T =================
    __builtin_amdgcn_s_setprio(1);
    store_k(buf);
    store_v(buf ^ 1);
    if constexpr (CS) store_c(buf ^ 1);
    {
      const int vb = buf;
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        bf16x8 vf[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c)
          vf[c] = *reinterpret_cast<const bf16x8*>(&smv[(vb * DH + 16 * db + lq) * VS + 32 * c + 8 * g]);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int c = 0; c < NC; ++c) o[db][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[c], pf[c][rb], o[db][rb], 0, 0, 0);
      }
      if constexpr (!SUM32)
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int c = 0; c < NC; ++c) lacc[rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pf[c][rb], lacc[rb], 0, 0, 0);
    }
    if constexpr (KEYS::kRun) {
      // the next tile's references start where the first one's did: plain queries move theirs only past a logit that exceeds it by 8, and
      // from zero a row of logits below about -126 (in log2 units) would lose all of its keys
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) m_run[rb] = last_kt ? (PRE ? 0.f : -INFINITY) : m_run[rb];
    }
    compute_s(buf ^ 1);
    // issue order: LDS stores, then LDS operand reads kept ahead of the MFMAs (one read feeds two)
    constexpr int kAhead = 6;  // more reads in flight cost the registers the schedule needs; fewer expose LDS latency
    __builtin_amdgcn_sched_group_barrier(0x200, K_LD + V_LD, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, kAhead, 0);
#pragma unroll
    for (int i = 0; i < DB * NC + KB * KC - kAhead; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, RB, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, RB * kAhead + (SUM32 ? 0 : RB * NC), 0);
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    lds_barrier();  // this wave's LDS stores are done
    __builtin_amdgcn_sched_barrier(0);
    ++j;
    if constexpr (KEYS::kRun) {
      parity ^= 1;
      if (last_kt) {
        if (!on) break;
        j = 0;
        --runs;
        tile_id += args()->stride;
        Kh = Kn;
        Vh = Vn;
        started = true;
      }
    }
  }
  if (group == 0) lds_barrier();  // every wave executes the same number of barriers

  if constexpr (KEYS::kSliced) {
    static_assert(PRE && !SUM32, "the references are those of scaled queries, the row sums the matrix pipe's");
    constexpr int W = slab_words(DH, RB);
    // What the thread's and the workgroup's ids give is made again here, and the arguments are read again, instead of kept across the
    // loop: with a register more alive there its LDS reads lose their lead over the MFMAs (112 tiles of 13104 keys in halves 294 us, so
    // about 150).
    int tid = threadIdx.x, block = blockIdx.x;
    typedef const __attribute__((address_space(4))) KeySlices* ArgPtr;
    ArgPtr arg = (ArgPtr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+v"(tid), "+s"(block), "+s"(arg));
    const KeySlices keys{arg->words, arg->slab1, arg->tiles, arg->slices, arg->units, arg->slab0, arg->n0};
    tid &= NT - 1;
    const int lane = tid & 63, wave = tid >> 6;
    const int place = xcd_remap(block, gridDim.x), slot = place / keys.slices, slice = place - slot * keys.slices;
    uint32_t *const ticket = keys.words + slot, *const done = ticket + keys.tiles, *const slice_of = keys.words + 2 * keys.tiles;
    const int others = keys.slices - 1, slab_first = slot * others;
    uint32_t* flag = reinterpret_cast<uint32_t*>(smem_raw);
    if (tid == 0) flag[0] = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int number = __builtin_amdgcn_readfirstlane((int)flag[0]);
    auto slab = [&](int i) {
      const int at = slab_first + i;
      return (at < keys.n0 ? reinterpret_cast<float*>(keys.words + keys.slab0) + (size_t)at * W * 1024 : keys.slab1 + (size_t)(at - keys.n0) * W * 1024) +
             ((size_t)wave * W * 64 + lane) * 2;
    };
    if (number < others) {
      float* p = slab(number);
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
        for (int db = 0; db < DB; ++db) {
          store_pair(p + 128 * (2 * (DB * rb + db)), o[db][rb][0], o[db][rb][1]);
          store_pair(p + 128 * (2 * (DB * rb + db) + 1), o[db][rb][2], o[db][rb][3]);
        }
        store_pair(p + 128 * (2 * DB * RB + rb), m_run[rb], lacc[rb][0]);
      }
      if (tid == 0) __hip_atomic_store(&slice_of[slab_first + number], (uint32_t)slice, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the wave's stores have completed, past the L2
      __syncthreads();
      if (tid == 0) __hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return;
    }
    if (tid == 0)
      while (__hip_atomic_load(done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != (uint32_t)others) __builtin_amdgcn_s_sleep(2);
    __syncthreads();
    asm volatile("" ::: "memory");  // the slabs are read behind the count
    // the largest reference, then the slices in the order of their keys, half of the results at a time
    float m_all[RB], own_l[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      m_all[rb] = m_run[rb];
      own_l[rb] = lacc[rb][0];
    }
#pragma unroll 1
    for (int i = 0; i < others; ++i)
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) m_all[rb] = fmaxf(m_all[rb], load_pair(slab(i) + 128 * (2 * DB * RB + rb)).x);
    constexpr int HB = DB / 2;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      f32x4 sum[HB][RB];
      float l[RB];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        l[rb] = 0.f;
#pragma unroll
        for (int db = 0; db < HB; ++db) sum[db][rb] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll 1
      for (int sl = 0; sl <= others; ++sl) {
        // fused multiply-adds by name: both branches round alike
        if (sl == slice) {
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) {
            const float f = __builtin_amdgcn_exp2f(m_run[rb] - m_all[rb]);
            l[rb] = __builtin_fmaf(f, own_l[rb], l[rb]);
#pragma unroll
            for (int db = 0; db < HB; ++db)
#pragma unroll
              for (int e = 0; e < 4; ++e) sum[db][rb][e] = __builtin_fmaf(f, o[HB * half + db][rb][e], sum[db][rb][e]);
          }
          continue;
        }
        int i = 0;
        while (i + 1 < others &&
               __hip_atomic_load(&slice_of[slab_first + i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != (uint32_t)sl)
          ++i;
        const float* p = slab(__builtin_amdgcn_readfirstlane(i));
        float2 ml[RB], v[2 * HB * RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          ml[rb] = load_pair(p + 128 * (2 * DB * RB + rb));
#pragma unroll
          for (int k = 0; k < 2 * HB; ++k) v[2 * HB * rb + k] = load_pair(p + 128 * (2 * (DB * rb + HB * half) + k));
        }
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          const float f = __builtin_amdgcn_exp2f(ml[rb].x - m_all[rb]);
          l[rb] = __builtin_fmaf(f, ml[rb].y, l[rb]);
#pragma unroll
          for (int db = 0; db < HB; ++db) {
            const float2 a = v[2 * (HB * rb + db)], b = v[2 * (HB * rb + db) + 1];
            const f32x4 w = {a.x, a.y, b.x, b.y};
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[db][rb][e] = __builtin_fmaf(f, w[e], sum[db][rb][e]);
          }
        }
      }
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        lacc[rb][0] = l[rb];
#pragma unroll
        for (int db = 0; db < HB; ++db) o[HB * half + db][rb] = sum[db][rb];
      }
    }
  }

  if constexpr (KEYS::kRun) {
    const ArgPtr a = args();
    const int nq = a->n_qtiles, of_head = tile_id / nq;
    finish(a->O, a->Lq, a->H * DH, of_head, tile_id - of_head * nq);
  } else {
    finish(O, Lq, H * DH, head, qt);
  }
}

// One launch of the 16x16x32 kernel with RB blocks of 16 query rows per wave over the tiles from tile_base on, a workgroup a tile or a slice of one.
template <int DH, bool PRE, int RB, int KIND, class KEYS = WholeKeys>
int32_t launch_attn_pp16_tiles(const uint16_t* Q, const uint16_t* K, const uint16_t* Vt, uint16_t* O, const float* cs,
                               long Lq, long Lk, long LqPad, long LkPad, int H, long nqt, long tile_base, long groups,
                               hipStream_t s, KEYS keys = KEYS{}) {
  size_t smem = 2 * ((size_t)128 * (DH + 16) + (size_t)DH * (128 + 16)) * sizeof(uint16_t) + (KIND == 2 || KIND == 4 ? 2 * 128 * sizeof(float) : 0);
  auto kern = attention_pp16_kernel<DH, PRE, RB, KIND, KEYS>;
  static DynLdsOnce once;  // the raised dynamic-LDS limit is a per-device property of the kernel
  CHK_STATUS(once.ensure(reinterpret_cast<const void*>(kern), (int)smem));
  const float scale_log2 = 1.4426950408889634f / sqrtf((float)DH);
  hipLaunchKernelGGL(kern, dim3((unsigned)groups), dim3(512), smem, s, keys, Q, K, Vt, O, cs, Lq, Lk, LqPad, LkPad, H,
                     (int)nqt, (int)tile_base, scale_log2);
  CHORUS_LAUNCH_CHECK();
  return CHORUS_OK;
}

// More tiles than CUs: workgroups that stay and walk over tiles (TileRun), over 512 to 2048 keys, where the walk fits the registers
// (not plain queries with factors).
// A share is four tiles of queries at most, and 32 tiles of keys in all: what it costs a stream whose neighbour holds a few units is
// the wait for the last share, which no other unit can take over. us alone / with eight units held by another stream: 32760 x 512, 12 heads
// without a walk 152 / 179, one share of six tiles a unit 127 / 218, two of three 131 / 178; 75600 x 512, 40 heads 1002 / 1282, one share of
// 47 866 / 1387, of eight 883 / 1063, of four 905 / 1102, of two 953 / 1174; 32000 x 1536, 12 heads 264 without, 240 with. Over long
// keys a walk gains nothing that shows: 13104 tokens, 12 heads 844 / 1151 without, 846 / 1285 with; 32760 tokens 4636 / 5600 and 4620 / 5430.
// Its offsets into the values have 32 bits.
constexpr int kMostTiles = 4, kMostKeyTiles = 32;
template <bool PRE, int KIND> constexpr bool kWalks = KIND <= 2 && (PRE || KIND != 2);
// how many tiles a workgroup walks over on average at most; 1: no walk
template <bool PRE, int KIND>
int walk_share(long tiles, long Lk, long LkPad, int cus) {
  const long most = kMostKeyTiles / ((Lk + 127) / 128);
  if (!kWalks<PRE, KIND> || tiles <= cus || cus % 8 || LkPad > 1 << 23 || most < 2) return 1;
  return (int)(most < kMostTiles ? most : kMostTiles);
}

// the first `tiles` tiles of 256 rows
template <int DH, bool PRE, int KIND>
int32_t launch_attn_full(const uint16_t* Q, const uint16_t* K, const uint16_t* Vt, uint16_t* O, const float* cs, long Lq, long Lk,
                         long LqPad, long LkPad, int H, long tiles, int cus, hipStream_t s) {
  const long nqt = (Lq + 255) / 256;
  if constexpr (kWalks<PRE, KIND>) {
    const int share = walk_share<PRE, KIND>(tiles, Lk, LkPad, cus);
    if (share > 1) {
      const long rounds = (tiles + cus - 1) / cus, groups = cus * ((rounds + share - 1) / share);
      return launch_attn_pp16_tiles<DH, PRE, 2, KIND, TileRun>(Q, K, Vt, O, cs, Lq, Lk, LqPad, LkPad, H, nqt, 0, groups, s,
                                                               TileRun{Q, K, Vt, O, Lq, LqPad, LkPad, H, (int)nqt, (int)tiles, (int)(groups / 8)});
    }
  }
  return launch_attn_pp16_tiles<DH, PRE, 2, KIND>(Q, K, Vt, O, cs, Lq, Lk, LqPad, LkPad, H, nqt, 0, tiles, s);
}

// Launches of at most half as many 256-row tiles as CUs run as workgroups of 128 rows throughout (1200 tokens, 12 heads:
// 36.2 -> 24.8 us). Else 256 query rows per workgroup. One workgroup fits a CU, so a launch runs in rounds of as many workgroups as the device
// has CUs. When the last round would be at most half full, its tiles run as workgroups of 128 rows instead (one block
// of 16 rows per wave: the same K / V stream for half the arithmetic, 0.63-0.67 of a full workgroup's time), twice as
// many of them, in a second launch behind the first: the partly filled round then takes two thirds of a full one. Also behind a walk,
// whose next tile costs less than a workgroup's: 512 keys, 12 heads, the tail in the walk / in half tiles, us: 280 tiles (40 heads) 41.7 /
// 39.6, 320 (40 heads) 38.1 / 36.8, 624 54.3 / 54.1, with factors 56.7 / 56.9; 1536 keys, 624 tiles 120 / 115. (With scratch, as a block
// has it, and long keys the last round runs in slices instead: attention_slices.)
template <int DH, bool PRE, int KIND>
int32_t launch_attn_pp16_kind(const uint16_t* Q, const uint16_t* K, const uint16_t* Vt, uint16_t* O, const float* cs, long Lq,
                              long Lk, long LqPad, long LkPad, int H, hipStream_t s) {
  const long nqt = (Lq + 255) / 256;
  const long tiles = nqt * H;
  if (2 * tiles > 0x7fffffffL) return CHORUS_E_SHAPE;
  const int cus = device_cus();
  if (cus < 0) return cus;
  if (2 * tiles <= cus)
    return launch_attn_pp16_tiles<DH, PRE, 1, KIND>(Q, K, Vt, O, cs, Lq, Lk, LqPad, LkPad, H, 2 * nqt, 0, 2 * tiles, s);
  const long tail = cus > 0 ? tiles % cus : 0;
  const bool halves = tiles > cus && tail > 0 && 2 * tail <= cus;
  CHK_STATUS((launch_attn_full<DH, PRE, KIND>(Q, K, Vt, O, cs, Lq, Lk, LqPad, LkPad, H, halves ? tiles - tail : tiles, cus, s)));
  if (!halves) return CHORUS_OK;
  return launch_attn_pp16_tiles<DH, PRE, 1, KIND>(Q, K, Vt, O, cs, Lq, Lk, LqPad, LkPad, H, 2 * nqt, 2 * (tiles - tail), 2 * tail, s);
}

template <int DH, bool PRE>
int32_t launch_attn_pp16(const uint16_t* Q, const uint16_t* K, const uint16_t* Vt, uint16_t* O, const float* cs, long Lq,
                         long Lk, long LqPad, long LkPad, int H, hipStream_t s) {
  if (!CHORUS_ATTENTION_LONG_KEYS(Lk, LkPad))
    return cs ? launch_attn_pp16_kind<DH, PRE, 4>(Q, K, Vt, O, cs, Lq, Lk, LqPad, LkPad, H, s)
              : launch_attn_pp16_kind<DH, PRE, 3>(Q, K, Vt, O, cs, Lq, Lk, LqPad, LkPad, H, s);
  if (cs) return launch_attn_pp16_kind<DH, PRE, 2>(Q, K, Vt, O, cs, Lq, Lk, LqPad, LkPad, H, s);
  return Lq == Lk ? launch_attn_pp16_kind<DH, PRE, 0>(Q, K, Vt, O, cs, Lq, Lk, LqPad, LkPad, H, s)
                  : launch_attn_pp16_kind<DH, PRE, 1>(Q, K, Vt, O, cs, Lq, Lk, LqPad, LkPad, H, s);
}

// ---------------------------------------------------------------------------
// Few keys (at most 128) for few queries, heads of 64: nothing to stream, so nothing to stage. A wave takes 16 queries of one head and all
// keys: it requests its queries, the keys, the values and the factors at once, as MFMA operands straight from memory, and is through after
// one latency, where the kernels above go through LDS, barriers and two phases (128 queries, 4 heads: 16 keys with factors 7.9 us
// behind 3.0 of normalisation, here 6.9 with it; 128 keys 6.4 in either). What is left is the wave's own instructions. Operand layout,
// logits, sums and their order are those of attention_pp16_kernel over one tile of keys on plain queries, so its bits too. Every wave reads
// all keys: with many queries the L1s would be the bound.
// NORM: the queries come as their projection's rows [Lq, H * 64]: the wave normalises its 16 rows itself, as qk_norm_rope_kernel does it (the
// same order of additions), H * 64 <= 512.
// ---------------------------------------------------------------------------
struct NormalisedQ {
  static constexpr bool kNorm = false;
};
struct RawQ {
  const float* gain;
  static constexpr bool kNorm = true;
};
template <int NC, class QUERIES>
__global__ __launch_bounds__(256) void attention_few_kernel(const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
                                                            const uint16_t* __restrict__ Vt, uint16_t* __restrict__ O,
                                                            const float* __restrict__ col_scale, long Lq, int Lk, long LqPad,
                                                            long LkPad, int H, float scale_log2, QUERIES queries) {
  constexpr int DH = 64, KB = 2 * NC, KC = DH / 32, DB = DH / 16;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lq = lane & 15, g = lane >> 4;
  const int head = blockIdx.y, D = H * DH;
  const long q0 = (long)blockIdx.x * 64 + wave * 16;
  if (q0 >= Lq) return;
  const long q = q0 + lq < Lq ? q0 + lq : Lq - 1;
  const uint16_t* Kh = K + (long)head * LkPad * DH;
  const uint16_t* Vh = Vt + (long)head * DH * LkPad;
  bf16x8 qf[KC], kf[KB][KC], vf[DB][NC];
  u32x4 rows[QUERIES::kNorm ? 16 : 1];
  if constexpr (QUERIES::kNorm) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const long row = q0 + r < Lq ? q0 + r : Lq - 1;
      rows[r] = u32x4{0u, 0u, 0u, 0u};
      if (8 * lane < D) rows[r] = *reinterpret_cast<const u32x4*>(Q + row * D + 8 * lane);
    }
  }
#pragma unroll
  for (int kc = 0; kc < KC; ++kc)
    qf[kc] = *reinterpret_cast<const bf16x8*>(QUERIES::kNorm ? Q + q * D + head * DH + 32 * kc + 8 * g
                                                              : Q + ((long)head * LqPad + q) * DH + 32 * kc + 8 * g);
#pragma unroll
  for (int kb = 0; kb < KB; ++kb)
#pragma unroll
    for (int kc = 0; kc < KC; ++kc)
      kf[kb][kc] = *reinterpret_cast<const bf16x8*>(Kh + (32 * (kb >> 1) + 16 * (lq >> 3) + 8 * (kb & 1) + (lq & 7)) * DH + 32 * kc + 8 * g);
  // the four keys of a lane in block kb
  auto key = [&](int kb) { return 32 * (kb >> 1) + 16 * (g >> 1) + 8 * (kb & 1) + 4 * (g & 1); };
  f32x4 cf[KB];
  if (col_scale) {
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int i = 0; i < 4; ++i) cf[kb][i] = key(kb) + i < Lk ? col_scale[key(kb) + i] : 1.0f;
  }
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int c = 0; c < NC; ++c) vf[db][c] = *reinterpret_cast<const bf16x8*>(Vh + (long)(16 * db + lq) * LkPad + 32 * c + 8 * g);
  if constexpr (QUERIES::kNorm) {
    float mine = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float ss = 0.f;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float a = __uint_as_float(rows[r][k] << 16), b = __uint_as_float(rows[r][k] & 0xffff0000u);
        ss += a * a + b * b;
      }
      const float rstd = rsqrtf(wave_sum(ss) / (float)D + 1e-6f);
      if (lq == r) mine = rstd;
    }
    const u32x4* raw = reinterpret_cast<const u32x4*>(qf);
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) {
      const f32x4* gain = reinterpret_cast<const f32x4*>(queries.gain + head * DH + 32 * kc + 8 * g);
      const f32x4 ga = gain[0], gb = gain[1];
      const float gv[8] = {ga[0], ga[1], ga[2], ga[3], gb[0], gb[1], gb[2], gb[3]};
      const u32x4 w = raw[kc];
      u32x4 o;
#pragma unroll
      for (int k = 0; k < 4; ++k)
        o[k] = pack_bf16x2(__uint_as_float(w[k] << 16) * mine * gv[2 * k], __uint_as_float(w[k] & 0xffff0000u) * mine * gv[2 * k + 1]);
      qf[kc] = __builtin_bit_cast(bf16x8, o);
    }
  }
  f32x4 s[KB];
  float mx = -INFINITY;
#pragma unroll
  for (int kb = 0; kb < KB; ++kb) {
    s[kb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) s[kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[kb][kc], qf[kc], s[kb], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (col_scale) s[kb][i] *= cf[kb][i];
      if (key(kb) + i >= Lk) s[kb][i] = -INFINITY;
      mx = fmaxf(mx, s[kb][i]);
    }
  }
  mx = fmaxf(mx, swap_rows16(mx));
  mx = fmaxf(mx, swap_halves(mx));
  const float mref = mx * scale_log2;
  bf16x8 pf[NC];
  float l = 0.f;
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[2 * c + b][i], scale_log2, -mref));
        l += p;
        pf[c][4 * b + i] = (bf16_t)p;
      }
  l += swap_rows16(l);
  l += swap_halves(l);
  const float inv = 1.0f / l;
  uint16_t* op = O + q * (long)D + head * DH + 4 * g;
#pragma unroll
  for (int db = 0; db < DB; ++db) {
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < NC; ++c) o = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[db][c], pf[c], o, 0, 0, 0);
    if (q0 + lq < Lq) *reinterpret_cast<uint2*>(op + 16 * db) = make_uint2(pack_bf16x2(o[0] * inv, o[1] * inv), pack_bf16x2(o[2] * inv, o[3] * inv));
  }
}

constexpr int kFewKeys = 128;
template <class QUERIES>
int32_t launch_attn_few(const uint16_t* Q, const uint16_t* K, const uint16_t* Vt, uint16_t* O, const float* cs, long Lq, long Lk,
                        long LqPad, long LkPad, int H, const QUERIES& queries, hipStream_t s) {
  if (H > 65535 || Lq > 0x7fffffffL) return CHORUS_E_SHAPE;
  const dim3 grid((unsigned)((Lq + 63) / 64), (unsigned)H);
  const float scale_log2 = 1.4426950408889634f / sqrtf(64.f);
#define ATTN_FEW(NC) \
  hipLaunchKernelGGL((attention_few_kernel<NC, QUERIES>), grid, dim3(256), 0, s, Q, K, Vt, O, cs, Lq, (int)Lk, LqPad, LkPad, H, scale_log2, queries)
  switch ((Lk + 31) / 32) {
    case 1: ATTN_FEW(1); break;
    case 2: ATTN_FEW(2); break;
    case 3: ATTN_FEW(3); break;
    case 4: ATTN_FEW(4); break;
    default: return CHORUS_E_SHAPE;
  }
#undef ATTN_FEW
  CHORUS_LAUNCH_CHECK();
  return CHORUS_OK;
}

template <int DH, int KTL, bool CS>
int32_t launch_attn_pp(const uint16_t* Q, const uint16_t* K, const uint16_t* Vt, uint16_t* O, const float* cs, long Lq,
                       long Lk, long LqPad, long LkPad, int H, hipStream_t s) {
  long nqt = (Lq + 255) / 256;
  if (nqt * H > 0x7fffffffL) return CHORUS_E_SHAPE;
  size_t smem = 2 * ((size_t)KTL * (DH + 8) + (size_t)DH * (KTL + 8)) * sizeof(uint16_t);
  auto kern = attention_pp_kernel<DH, KTL, CS>;
  static DynLdsOnce once;  // the raised dynamic-LDS limit is a per-device property of the kernel
  CHK_STATUS(once.ensure(reinterpret_cast<const void*>(kern), (int)smem));
  const float scale_log2 = 1.4426950408889634f / sqrtf((float)DH);
  hipLaunchKernelGGL(kern, dim3((unsigned)(nqt * H)), dim3(512), smem, s, Q, K, Vt, O, cs, Lq, Lk, LqPad, LkPad, H,
                     (int)nqt, scale_log2);
  CHORUS_LAUNCH_CHECK();
  return CHORUS_OK;
}

// Under 512 keys. Launches of half tiles: the 64-key kernel has none (12 heads of 128, microseconds, 64-key kernel / 128-key
// kernel: 480 x 480 20.4 / 13.7, 1200 x 77 12.6 / 9.6, 128 x 128 9.7 / 9.0). Launches of full tiles, time of the 128-key
// kernel over that of the 64-key kernel on 288 to 2080 tiles:
//   key factors, heads of 64: 0.6 to 0.9 from 70 to 511 keys: the factors come from LDS
//   where half of the last 128-key tile or more is padding: 180 keys 0.95 to 1.14, 300 keys 0.91 to 1.12, 400 keys 0.95 to
//   1.07 without factors, 0.85 to 1.07, mostly under 1, with them
//   key factors, heads of 128: 70 to 90 keys 0.85 to 1.03, 100 keys 0.88 to 1.05, 110 and 128 keys (few or none masked)
//   0.88 to 1.07, mostly over 1; 200, 226, 480 keys 0.81 to 0.99
//   without: 70 to 128 keys 0.95 to 1.08, mostly over 1; 200 to 511 keys 0.88 to 1.03, but 1.00 to 1.05 on 156 to 240
//   tiles, where one round does not fill the chip
int attention_variant(long Lq, long Lk, long LkPad, int H, int dh, bool factor, int cus) {
  const long tiles = (Lq + 255) / 256 * H;
  if (dh == 64 && Lk <= kFewKeys && 2 * tiles <= cus) return 7;
  if (LkPad % 128) return 3;
  if (CHORUS_ATTENTION_LONG_KEYS(Lk, LkPad)) return 5;
  if (Lk <= 64) return 3;
  if (2 * tiles <= cus || (factor && dh == 64)) return 5;
  if ((Lk + 63) / 64 % 2 && !(factor && Lk > 384)) return 3;
  return (factor ? Lk <= 96 || Lk > 128 : Lk > 128 && tiles > cus) ? 5 : 3;
}

// Counts, slice numbers, then a slab for every slice of a tile but one.
struct SliceScratch {
  size_t counts, slab;
  long slabs;
};
SliceScratch slice_scratch(int dh, int sliced, int slices) {
  const long slabs = (long)sliced * (slices - 1);
  return SliceScratch{align_up((size_t)(2L * sliced + slabs) * 4, 256), (size_t)slab_words(dh, 2) * 512 * 8, slabs};
}
bool slices_fit(const SliceScratch& r, const AttnScratch& sc) {
  if (!sc.first || !aligned16(sc.first) || !aligned16(sc.rest) || sc.first_bytes < r.counts) return false;
  return (long)((sc.first_bytes - r.counts) / r.slab + (sc.rest ? sc.rest_bytes / r.slab : 0)) >= r.slabs;
}

template <int DH>
int32_t launch_attn_sliced(const uint16_t* Q, const uint16_t* K, const uint16_t* Vt, uint16_t* O, long L, long LPad, int H,
                           const AttnSlices& p, const AttnScratch& sc, hipStream_t s) {
  const long nqt = (L + 255) / 256;
  const SliceScratch r = slice_scratch(DH, p.sliced, p.slices);
  if (!slices_fit(r, sc)) return CHORUS_E_WORKSPACE;
  if (p.whole > 0) {
    const int cus = device_cus();
    if (cus < 0) return cus;
    CHK_STATUS((launch_attn_full<DH, true, 0>(Q, K, Vt, O, nullptr, L, L, LPad, LPad, H, p.whole, cus, s)));
  }
  const KeySlices keys{static_cast<uint32_t*>(sc.first), static_cast<float*>(sc.rest), p.sliced, p.slices, (int)((L + 127) / 128),
                       (int)(r.counts / 4), (int)((sc.first_bytes - r.counts) / r.slab)};
  return launch_attn_pp16_tiles<DH, true, 2, 0, KeySlices>(Q, K, Vt, O, nullptr, L, L, LPad, LPad, H, nqt, p.whole,
                                                           (long)p.sliced * p.slices, s, keys);
}

__global__ __launch_bounds__(256) void clear_words_kernel(uint32_t* p, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0;
}

// Five slices and more were never faster by more than 1 us.
constexpr int kMaxKeySlices = 4;

}  // namespace

int device_cus() {
  int dev = 0, cus = 0;
  CHORUS_HIP(hipGetDevice(&dev));
  CHORUS_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  return cus;
}

// The tiles of a last round that fills two thirds of the chip or less: in as many slices as there are units for, four at most, where the sweep
// over the keys is long enough for what a slice costs beside it, about 20 us of chip time (its first loads, the ping-pong's start
// and end, and 139 KB a slab out and in). Whole call, halves of 128 rows as before / slices, us: 13104 tokens, 12 heads (112 tiles, two
// slices) 853 / 786; 8100 (128, two) 329 / 311; 5632 (8, four; 44 key tiles) 216 / 190, in two slices 208; 6000 (32, four) 230 / 202; 40
// heads: 7168 tokens (96, two) 802 / 793, 3300 (8, four; 26 key tiles) 221 / 212, 2000 (64, three; 16) 91 / 90; 4 heads of 64, 3584 tokens
// (56, four; 28) 30.6 / 28. Up to two thirds of the chip, three slices a tile in two rounds: 8840 tokens, 12 heads (164; 70 key tiles)
// whole tiles 410 / slices 392, 3271 (156; 26) 75 / 84. Slower: 2560 tokens, 12 heads (120, two; 20 key tiles) 44 / 43 to 45, 1792, 40 heads
// (24, four; 14) 82 / 84.
AttnSlices attention_slices(long L, int H, int dh, int cus, const AttnScratch& scratch) {
  const AttnSlices none{0, 0, 0};
  const long tiles = (L + 255) / 256 * H, units = (L + 127) / 128;
  if (cus <= 0 || tiles > 0x7fffffffL / 2) return none;
  const long sliced = tiles % cus;
  if (sliced == 0) return none;
  if (2 * sliced > cus) {
    if (3 * sliced > 2L * cus || units < 60 || !slices_fit(slice_scratch(dh, (int)sliced, 3), scratch)) return none;
    return AttnSlices{tiles - sliced, (int)sliced, 3};
  }
  for (int slices = (int)(cus / sliced < kMaxKeySlices ? cus / sliced : kMaxKeySlices); slices >= 2; --slices)
    if (slices_fit(slice_scratch(dh, (int)sliced, slices), scratch))
      return units < (slices == 2 ? 40 : 24) ? none : AttnSlices{tiles - sliced, (int)sliced, slices};
  return none;
}

bool attention_raw_queries(long Lq, long Lk, long LkPad, int H, int dh, bool factor, int cus) {
  return H * dh <= 512 && attention_variant(Lq, Lk, LkPad, H, dh, factor, cus) == 7;
}

int32_t attention_raw(const uint16_t* q, const float* gain, const uint16_t* K, const uint16_t* Vt, uint16_t* O, const float* col_scale, long Lq,
                      long Lk, long LkPad, int H, void* stream) {
  if (!gain || !aligned16(gain) || !aligned16(q)) return CHORUS_E_ARG;
  return launch_attn_few(q, K, Vt, O, col_scale, Lq, Lk, 0, LkPad, H, RawQ{gain}, (hipStream_t)stream);
}

int32_t attention_sliced(const uint16_t* Q, const uint16_t* K, const uint16_t* Vt, uint16_t* O, long L, long LPad, int H, int dh,
                         const AttnSlices& plan, const AttnScratch& scratch, void* stream) {
  return dh == 128 ? launch_attn_sliced<128>(Q, K, Vt, O, L, LPad, H, plan, scratch, (hipStream_t)stream)
                   : launch_attn_sliced<64>(Q, K, Vt, O, L, LPad, H, plan, scratch, (hipStream_t)stream);
}

}  // namespace chorus

using namespace chorus;

extern "C" int32_t chorus_attention_slices(const uint16_t* Q, const uint16_t* K, const uint16_t* Vt, uint16_t* O, int64_t L,
                                           int64_t LPad, int32_t H, int32_t dh, int64_t whole, int32_t slices, void* scratch,
                                           size_t scratch_bytes, void* stream) {
  if (L < 0 || H <= 0 || whole < 0 || slices < 2) return CHORUS_E_ARG;
  if (L == 0) return CHORUS_OK;
  if (!Q || !K || !Vt || !O) return CHORUS_E_ARG;
  if ((dh != 64 && dh != 128) || LPad < L || LPad % 128 || LPad > 0x7fffffffL) return CHORUS_E_SHAPE;
  if (!aligned16(Q) || !aligned16(K) || !aligned16(Vt) || !aligned16(O)) return CHORUS_E_ARG;
  const long tiles = ((long)L + 255) / 256 * H, units = ((long)L + 127) / 128;
  if (whole >= tiles || slices > units || (tiles - whole) * slices > 65536) return CHORUS_E_SHAPE;
  if (!scratch || !aligned16(scratch)) return CHORUS_E_WORKSPACE;
  const AttnScratch sc{scratch, scratch_bytes, nullptr, 0};
  const AttnSlices plan{(long)whole, (int)(tiles - whole), slices};
  if (!slices_fit(slice_scratch(dh, plan.sliced, slices), sc)) return CHORUS_E_WORKSPACE;
  const int words = attention_slices_words(plan);
  hipLaunchKernelGGL(clear_words_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                     static_cast<uint32_t*>(scratch), words);
  CHORUS_LAUNCH_CHECK();
  return attention_sliced(Q, K, Vt, O, (long)L, (long)LPad, H, dh, plan, sc, stream);
}

extern "C" int32_t chorus_attention_slices_plan(int64_t L, int32_t H, int32_t dh, int32_t cus, size_t first_bytes, size_t rest_bytes,
                                                int64_t* whole, int32_t* slices) {
  if (L < 1 || H <= 0 || cus <= 0 || !whole || !slices) return CHORUS_E_ARG;
  if (dh != 64 && dh != 128) return CHORUS_E_SHAPE;
  void* some = reinterpret_cast<void*>(uintptr_t{16});  // where the scratch lies does not matter
  const AttnSlices p = attention_slices((long)L, H, dh, cus, AttnScratch{first_bytes ? some : nullptr, first_bytes,
                                                                         rest_bytes ? some : nullptr, rest_bytes});
  *whole = p.whole;
  *slices = p.slices;
  return CHORUS_OK;
}

extern "C" int32_t chorus_attention_variant(int64_t Lq, int64_t Lk, int64_t LkPad, int32_t H, int32_t dh, int32_t factor, int32_t cus) {
  if (Lq < 1 || Lk < 1 || LkPad < Lk || H <= 0 || cus <= 0) return CHORUS_E_ARG;
  if ((dh != 64 && dh != 128) || LkPad % KT) return CHORUS_E_SHAPE;
  return attention_variant((long)Lq, (long)Lk, (long)LkPad, H, dh, factor != 0, cus);
}

// variant: 0 = default choice; 3 = 64-key tiles on 32x32x16 MFMAs; 5 = 128-key tiles on 16x16x32 MFMAs
// (LkPad % 128 == 0); 6 = the same on pre-scaled queries
extern "C" int32_t chorus_attention(const uint16_t* Q, const uint16_t* K, const uint16_t* Vt, uint16_t* O,
                                    const float* col_scale, int64_t Lq, int64_t Lk, int64_t LqPad, int64_t LkPad,
                                    int32_t H, int32_t dh, int32_t variant, void* stream) {
  if (Lq < 0 || Lk < 0 || H <= 0) return CHORUS_E_ARG;
  if (variant != 0 && variant != 3 && variant != 5 && variant != 6 && variant != 7) return CHORUS_E_ARG;
  if (Lq == 0) return CHORUS_OK;
  if (Lk < 1) return CHORUS_E_SHAPE;
  if (!Q || !K || !Vt || !O) return CHORUS_E_ARG;
  if ((dh != 64 && dh != 128) || LkPad % KT || LkPad < Lk || LqPad < Lq || LkPad > 0x7fffffffL) return CHORUS_E_SHAPE;
  if (!aligned16(Q) || !aligned16(K) || !aligned16(Vt) || !aligned16(O) || !aligned16(col_scale)) return CHORUS_E_ARG;
  hipStream_t s = (hipStream_t)stream;
  const bool cs = col_scale != nullptr;
  if (variant == 0) {
    const int cus = device_cus();
    if (cus < 0) return cus;
    variant = attention_variant((long)Lq, (long)Lk, (long)LkPad, H, dh, cs, cus);
  }
  if (variant == 7) {
    if (dh != 64 || Lk > kFewKeys) return CHORUS_E_SHAPE;
    return launch_attn_few(Q, K, Vt, O, col_scale, Lq, Lk, LqPad, LkPad, H, NormalisedQ{}, s);
  }
  if (variant == 5 || variant == 6) {
    if (LkPad % 128) return CHORUS_E_SHAPE;
    if (variant == 6)
      return dh == 128 ? launch_attn_pp16<128, true>(Q, K, Vt, O, col_scale, Lq, Lk, LqPad, LkPad, H, s)
                       : launch_attn_pp16<64, true>(Q, K, Vt, O, col_scale, Lq, Lk, LqPad, LkPad, H, s);
    return dh == 128 ? launch_attn_pp16<128, false>(Q, K, Vt, O, col_scale, Lq, Lk, LqPad, LkPad, H, s)
                     : launch_attn_pp16<64, false>(Q, K, Vt, O, col_scale, Lq, Lk, LqPad, LkPad, H, s);
  }
  if (dh == 128)
    return cs ? launch_attn_pp<128, 64, true>(Q, K, Vt, O, col_scale, Lq, Lk, LqPad, LkPad, H, s)
              : launch_attn_pp<128, 64, false>(Q, K, Vt, O, col_scale, Lq, Lk, LqPad, LkPad, H, s);
  return cs ? launch_attn_pp<64, 64, true>(Q, K, Vt, O, col_scale, Lq, Lk, LqPad, LkPad, H, s)
            : launch_attn_pp<64, 64, false>(Q, K, Vt, O, col_scale, Lq, Lk, LqPad, LkPad, H, s);
}
