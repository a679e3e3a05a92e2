// Stage-1 retrieval over a low-precision copy of the prompt-embedding cache (cache maintenance around
// Sec. 3.1 "Full Reuse"): the scan reads bf16 (half the bytes) or FP8 E4M3 rows (a quarter), and the rows whose
// approximate score lies within a proven margin of the best one are re-scored from the fp32 rows, so the result
// is the fp32 lookup's. HBM-bound like the fp32 scan.
//
// Why the margin suffices: replacing a row c by its low-precision copy c^ turns it by at most
// asin(|c^ - c| / |c|), and a cosine moves by at most that angle. bf16 keeps 8 significant bits (every element
// within 2^-8 of itself); FP8 E4M3 keeps 4 down to 2^-6 and steps of 2^-9 below, on a row scaled so that its
// largest magnitude is 448. With eps that bound, the true best row's approximate score is within 2 eps of the
// best approximate score.
#include <cmath>

#include "chorus_ops.h"
#include "common.h"
#include "lookup_row.h"

namespace chorus {
namespace {

constexpr int kWaves = 4;            // waves per workgroup of the scan and of the re-rank
constexpr int kMaxBlocks = 1024;     // workgroups of either: four on every compute unit; beyond that a wave takes several rows
// workgroups of the scan over several rows a wave of 2 KB and more, see lp_scan_blocks
constexpr int kScanBlocks = 512;
constexpr int kMaxScanBlocks = 4096; // the workspace has room for this many: its size stays what callers hold

inline long lp_blocks(long N) {
  long g = (N + kWaves - 1) / kWaves;
  return g < kMaxBlocks ? g : kMaxBlocks;
}
// Of the scan: a wave a row as far as that goes. Beyond it rows of 2 KB and more go to half as many waves, each with two rows
// in flight: a wave's fp32 query is 16 KB through the L1 at d = 4096, as much as four of its FP8 rows (65536 x 4096 FP8 51.7
// -> 48.9 us the call, 8192 x 4096 bf16 20.9 -> 19.4, 5000 x 4096 FP8 16.8 -> 14.6). Shorter rows want the loads in flight of
// all waves (65536 x 768 FP8 23.3, with half as many 26.0).
inline long lp_scan_blocks(long N, long row_bytes) { return N <= (long)kMaxBlocks * kWaves || row_bytes < 2048 ? lp_blocks(N) : kScanBlocks; }

// Where the re-rank's workgroups leave what they found; the first workgroup of the scan resets it. A line each: when
// every row is a candidate a thousand workgroups arrive, and atomics on one line are served one at a time (10 ns).
constexpr int kSlots = 64;
struct alignas(128) LpSlot {
  unsigned long long best;  // best exact r with its row (pack_best), 0 = none
  int32_t count;            // rows re-scored
};
struct LpWs {
  float* qnorm2;
  LpSlot* slots;           // [kSlots]
  float* partial_max;      // [lp_blocks]
  float* scores;           // [N] approximate r_j = <q, c^_j> / |c^_j|
  size_t bytes;
};
static_assert(kSlots * sizeof(LpSlot) <= (size_t)kMaxScanBlocks * 16, "the slots' place in the workspace");
LpWs carve_lp(long N, void* base) {
  const BytePtr p(base);
  LpWs w;
  size_t off = 0;
  w.qnorm2 = (float*)(p + off);
  off += 256;
  w.partial_max = (float*)(p + off);
  off += align_up((size_t)kMaxScanBlocks * sizeof(float), 256);
  w.slots = (LpSlot*)(p + off);
  off += (size_t)kMaxScanBlocks * 16;
  w.scores = (float*)(p + off);
  off += align_up((size_t)(N > 0 ? N : 1) * sizeof(float), 256);
  w.bytes = off;
  return w;
}

// r > -inf and its row as one integer that orders by r and, between equal r (0 and -0 are equal), by the lower row
__device__ __forceinline__ unsigned long long pack_best(float r, uint32_t row) {
  const uint32_t u = __float_as_uint(r + 0.0f);
  const uint32_t ord = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return ((unsigned long long)ord << 32) | (uint32_t)~row;
}
__device__ __forceinline__ float unpack_r(unsigned long long k) {
  const uint32_t ord = (uint32_t)(k >> 32);
  return __uint_as_float((ord & 0x80000000u) ? (ord & 0x7fffffffu) : ~ord);
}

// ---- decoding 16 bytes of a row into floats ------------------------------------------------
template <int FMT>
struct Codes;
template <>
struct Codes<CHORUS_LP_BF16> {
  static constexpr int kPer16 = 8;  // elements per 16-byte load
  __device__ static __forceinline__ void decode(const u32x4& v, float (&f)[8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f[2 * i] = __uint_as_float(v[i] << 16);
      f[2 * i + 1] = __uint_as_float(v[i] & 0xffff0000u);
    }
  }
};
template <>
struct Codes<CHORUS_LP_FP8> {
  static constexpr int kPer16 = 16;
  __device__ static __forceinline__ void decode(const u32x4& v, float (&f)[16]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const auto lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)v[i], false);  // bytes 0, 1
      const auto hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)v[i], true);   // bytes 2, 3
      f[4 * i] = lo[0];
      f[4 * i + 1] = lo[1];
      f[4 * i + 2] = hi[0];
      f[4 * i + 3] = hi[1];
    }
  }
};

// ---- store: fp32 rows -> low-precision rows ---------------------------------------------------
// One wave per row. bf16: round to nearest even. FP8: y = c * (448 / max|c|), both single fp32 operations,
// clamped to [-448, 448] (a product may land one fp32 step above 448), then rounded to nearest even.
template <int FMT>
__global__ __launch_bounds__(256) void lowprec_store_kernel(const float* __restrict__ emb, long n_rows, int d,
                                                            void* __restrict__ out) {
  const int lane = threadIdx.x & 63;
  const long row = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= n_rows) return;
  const float4* c4 = reinterpret_cast<const float4*>(emb + row * (long)d);
  const int n4 = d >> 2;
  if (FMT == CHORUS_LP_BF16) {
    uint2* o = reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(out) + row * (long)d);
    for (int i = lane; i < n4; i += 64) {
      const float4 c = c4[i];
      uint2 w;
      w.x = pack_bf16x2(c.x, c.y);
      w.y = pack_bf16x2(c.z, c.w);
      o[i] = w;
    }
  } else {
    float amax = 0.f;
    for (int i = lane; i < n4; i += 64) {
      const float4 c = c4[i];
      amax = fmaxf(fmaxf(amax, fmaxf(fabsf(c.x), fabsf(c.y))), fmaxf(fabsf(c.z), fabsf(c.w)));
    }
    amax = wave_max(amax);
    const float inv = amax > 0.f ? __fdiv_rn(448.0f, amax) : 0.f;
    uint32_t* o = reinterpret_cast<uint32_t*>(reinterpret_cast<uint8_t*>(out) + row * (long)d);
    for (int i = lane; i < n4; i += 64) {
      const float4 c = c4[i];
      const float y0 = fminf(fmaxf(__fmul_rn(c.x, inv), -448.f), 448.f), y1 = fminf(fmaxf(__fmul_rn(c.y, inv), -448.f), 448.f);
      const float y2 = fminf(fmaxf(__fmul_rn(c.z, inv), -448.f), 448.f), y3 = fminf(fmaxf(__fmul_rn(c.w, inv), -448.f), 448.f);
      int w = __builtin_amdgcn_cvt_pk_fp8_f32(y0, y1, 0, false);
      w = __builtin_amdgcn_cvt_pk_fp8_f32(y2, y3, w, true);
      o[i] = (uint32_t)w;
    }
  }
}

// ---- scan of the low-precision rows -------------------------------------------------------------
// One 16-byte chunk of codes against its query values: dot += <f, q>, cc += <f, f>, four elements at a time in
// ascending order (the order of additions depends on d only, so equal rows score equal)
template <int FMT>
__device__ __forceinline__ void add_chunk(const u32x4& v, const float4* q, float& dot, float& cc) {
  constexpr int E = Codes<FMT>::kPer16;
  float f[E];
  Codes<FMT>::decode(v, f);
#pragma unroll
  for (int e4 = 0; e4 < E / 4; ++e4) {
    dot += f[4 * e4] * q[e4].x + f[4 * e4 + 1] * q[e4].y + f[4 * e4 + 2] * q[e4].z + f[4 * e4 + 3] * q[e4].w;
    cc += f[4 * e4] * f[4 * e4] + f[4 * e4 + 1] * f[4 * e4 + 1] + f[4 * e4 + 2] * f[4 * e4 + 2] + f[4 * e4 + 3] * f[4 * e4 + 3];
  }
}

// One wave per row at a time. NC > 0: a row has at most 64 NC chunks of 16 bytes, and a lane keeps the query values of
// its NC chunks (64 registers at d = 4096) for all its rows and has the next two rows' chunks in flight while it sums
// this one. Read again for every row, the fp32 query is four times the bytes of an FP8 row, all through the L1, which is
// what bound this kernel: 16384 x 4096 FP8 (67 MB) 23.8 us that way. NC = 0: any d, the query is read for every row; also the choice where a wave has only one.
template <int FMT, int NC>
__global__ __launch_bounds__(kWaves * 64) void lowprec_scan_kernel(const void* __restrict__ cache_lp,
                                                                   const float* __restrict__ query, long N, int d,
                                                                   float* __restrict__ scores,
                                                                   float* __restrict__ partial_max,
                                                                   float* __restrict__ qnorm2, LpSlot* __restrict__ slots) {
  constexpr int E = Codes<FMT>::kPer16;
  __shared__ float sv[kWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n16 = d / E;  // 16-byte chunks per row
  const long row_bytes = (long)d * (16 / E);
  const uint8_t* base = reinterpret_cast<const uint8_t*>(cache_lp);
  float best = -INFINITY;
  const long stride = (long)gridDim.x * kWaves;
  long row = (long)blockIdx.x * kWaves + wave;
  auto finish = [&](long r, float dot, float cc) {
    const float v = row_ratio(wave_sum(dot), wave_sum(cc));
    if (lane == 0) scores[r] = v;
    best = fmaxf(best, v);
  };
  if constexpr (NC > 0) {
    float4 q[NC][E / 4];
    u32x4 v[3][NC];
    auto fetch = [&](u32x4 (&dst)[NC], long r) {
      const u32x4* c16 = reinterpret_cast<const u32x4*>(base + r * row_bytes);
#pragma unroll
      for (int c = 0; c < NC; ++c)
        dst[c] = __builtin_nontemporal_load(&c16[lane + 64 * c < n16 ? lane + 64 * c : n16 - 1]);
    };
    auto sum = [&](const u32x4 (&src)[NC], long r) {
      float dot = 0.f, cc = 0.f;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const u32x4 w = lane + 64 * c < n16 ? src[c] : u32x4{0u, 0u, 0u, 0u};  // code 0 is 0.0 in both formats
        add_chunk<FMT>(w, q[c], dot, cc);
      }
      finish(r, dot, cc);
    };
    if (row < N) fetch(v[0], row);
    if (row + stride < N) fetch(v[1], row + stride);
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int e = 0; e < E / 4; ++e)
        q[c][e] = reinterpret_cast<const float4*>(query)[(lane + 64 * c < n16 ? lane + 64 * c : n16 - 1) * (E / 4) + e];
    for (; row < N; row += 3 * stride) {  // three rows a turn: the buffers are named, not indexed
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        if (row + u * stride >= N) break;
        if (row + (u + 2) * stride < N) fetch(v[(u + 2) % 3], row + (u + 2) * stride);
        sum(v[u], row + u * stride);
      }
    }
  } else {
    for (; row < N; row += stride) {
      const u32x4* c16 = reinterpret_cast<const u32x4*>(base + row * row_bytes);
      constexpr int U = 4;  // 16-byte loads in flight per lane
      float dot = 0.f, cc = 0.f;
      int i = lane;
      for (; i + (U - 1) * 64 < n16; i += U * 64) {
        u32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = __builtin_nontemporal_load(&c16[i + u * 64]);
#pragma unroll
        for (int u = 0; u < U; ++u) add_chunk<FMT>(v[u], reinterpret_cast<const float4*>(query + (long)(i + u * 64) * E), dot, cc);
      }
      for (; i < n16; i += 64)
        add_chunk<FMT>(__builtin_nontemporal_load(&c16[i]), reinterpret_cast<const float4*>(query + (long)i * E), dot, cc);
      finish(row, dot, cc);
    }
  }
  if (blockIdx.x == 0 && wave == 0) {  // |q|^2 exactly as the fp32 lookup sums it
    float qq = 0.f;
    const float4* q4 = reinterpret_cast<const float4*>(query);
    const int n4 = d >> 2;
    int i = lane;
    for (; i + 7 * 64 < n4; i += 8 * 64) {
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float4 q = q4[i + u * 64];
        qq += q.x * q.x + q.y * q.y + q.z * q.z + q.w * q.w;
      }
    }
    for (; i < n4; i += 64) {
      const float4 q = q4[i];
      qq += q.x * q.x + q.y * q.y + q.z * q.z + q.w * q.w;
    }
    qq = wave_sum(qq);
    if (lane == 0) *qnorm2 = qq;
    static_assert(kSlots == 64, "one slot per lane");
    slots[lane].best = 0;
    slots[lane].count = 0;
  }
  if (lane == 0) sv[wave] = best;
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 1; w < kWaves; ++w) best = fmaxf(best, sv[w]);
    partial_max[blockIdx.x] = best;
  }
}

// ---- candidates and exact re-rank ---------------------------------------------------------------
// threshold = best approximate r - margin * |q| (r = cosine * |q|); every row at or above it is re-scored from its
// fp32 row by a whole wave with the fp32 lookup's own row pass. A wave owns every nwaves-th row and looks at the scores of
// 64 of them at once. Candidates tend to stand side by side (variants of a prompt are stored one after the other): dealt
// out singly they go to different waves, in runs of consecutive rows one wave would re-score them all in series (262144 x
// 1024 FP8, 256 neighbours among the candidates: the call 194 us, dealt out 72). So even when every row is a candidate
// (FP8 on a query far from every entry) the re-rank costs one fp32 scan. From 16 rows a wave on, neighbouring waves run on
// one XCD, so that a line of scores is read into one L2 (1048576 x 64: 228.4 us without, 224.4 with); below, most waves
// find the scores in the L2 of the XCD that wrote them (4100 x 1024 FP8: 9.8 us, 10.4 elsewhere). Each workgroup reduces
// the scan's partial maxima itself (at most 1024, four per thread). Usually a handful of waves have a row at all, so the
// winners meet in atomic maxima in memory. (With every wave of 4096 workgroups reducing 4096 maxima, and a partial result
// per workgroup, the re-rank of one row among 16384 took 35.9 us and its final reduction 7.5.)
__global__ __launch_bounds__(kWaves * 64) void lowprec_rerank_kernel(const float* __restrict__ cache_emb,
                                                                     const float* __restrict__ query, long N, int d,
                                                                     const float* __restrict__ scores,
                                                                     const float* __restrict__ partial_max, int nparts,
                                                                     const float* __restrict__ qnorm2, float margin,
                                                                     LpSlot* __restrict__ slots) {
  __shared__ float sm[kWaves];
  __shared__ float sv[kWaves];
  __shared__ int32_t si[kWaves];
  __shared__ int32_t sc[kWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long nwaves = (long)gridDim.x * kWaves;
  const long w_id = (long)(N >= 16 * nwaves ? xcd_remap(blockIdx.x, gridDim.x) : blockIdx.x) * kWaves + wave;
  const long step = 64 * nwaves;  // rows that the chip looks at in one turn
  auto score = [&](long r0) { return r0 + lane * nwaves < N ? scores[r0 + lane * nwaves] : -INFINITY; };
  float own = score(w_id);  // in flight beside the maxima
  const float nq = sqrtf(*qnorm2);
  float mx = -INFINITY;
  for (int j = threadIdx.x; j < nparts; j += kWaves * 64) mx = fmaxf(mx, partial_max[j]);
  mx = wave_max(mx);
  if (lane == 0) sm[wave] = mx;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kWaves; ++w) mx = fmaxf(mx, sm[w]);
  // no finite score (all rows zero) or a zero query: every exact score is -inf as well, nothing is re-scored
  const float thr = nq > 0.f ? mx - margin * nq : -INFINITY;
  const float4* q4 = reinterpret_cast<const float4*>(query);
  const int n4 = d >> 2;
  float best = -INFINITY;
  int32_t bi = 0x7fffffff, count = 0;
  if (thr > -INFINITY) {
    for (long r0 = w_id; r0 < N; r0 += step) {
      if (r0 != w_id) own = score(r0);
      unsigned long long todo = __ballot(own >= thr);
      count += __popcll(todo);
      while (todo) {  // ascending rows
        const long row = r0 + __builtin_ctzll(todo) * nwaves;
        todo &= todo - 1;
        float dot, cc, qq;
        fp32_row_products(reinterpret_cast<const float4*>(cache_emb + row * (long)d), q4, n4, lane, dot, cc, qq);
        const float r = row_ratio(dot, cc);
        if (r > best) {
          best = r;
          bi = (int32_t)row;
        }
      }
    }
  }
  if (lane == 0) {
    sv[wave] = best;
    si[wave] = bi;
    sc[wave] = count;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 1; w < kWaves; ++w) {
      if (sv[w] > best || (sv[w] == best && si[w] < bi)) {
        best = sv[w];
        bi = si[w];
      }
      count += sc[w];
    }
    LpSlot& slot = slots[blockIdx.x % kSlots];
    if (count > 0) atomicAdd(&slot.count, count);
    if (best > -INFINITY) atomicMax(&slot.best, pack_best(best, (uint32_t)bi));
  }
}

// One wave: the best of the slots, the division by |q| and the threshold test, as in the fp32 lookup.
__global__ __launch_bounds__(64) void lowprec_final_kernel(const LpSlot* __restrict__ slots, const float* __restrict__ qnorm2,
                                                           long N, float tau, chorus_lookup_result* __restrict__ out,
                                                           int32_t* __restrict__ n_rescored) {
  unsigned long long key = N > 0 ? slots[threadIdx.x].best : 0;
  int32_t count = N > 0 ? slots[threadIdx.x].count : 0;
  const float nq = N > 0 ? sqrtf(*qnorm2) : 0.f;
  key = wave_max_key(key);
  count = wave_sum_i32(count);
  if (threadIdx.x != 0) return;
  chorus_lookup_result r;
  if (N <= 0) {
    r.index = -1;
    r.score = -INFINITY;
    r.hit = 0;
  } else {
    const float best = key ? unpack_r(key) : -INFINITY;
    float mm = (nq > 0.f && best > -INFINITY) ? best / nq : -INFINITY;
    if (!(mm == mm)) mm = -INFINITY;
    r.index = mm == -INFINITY ? 0 : (int32_t)~(uint32_t)key;
    r.score = mm;
    r.hit = mm >= tau ? 1 : 0;
  }
  *out = r;
  if (n_rescored) *n_rescored = count;
}

template <int FMT>
void launch_lp_scan(const void* cache_lp, const float* query, long N, int d, const LpWs& w, unsigned grid, hipStream_t s) {
  const int nc = (d / Codes<FMT>::kPer16 + 63) / 64, most = 64 / Codes<FMT>::kPer16;  // 64 query values per lane
#define LP_SCAN(NC) \
  hipLaunchKernelGGL((lowprec_scan_kernel<FMT, NC>), dim3(grid), dim3(kWaves * 64), 0, s, cache_lp, query, N, d, w.scores, w.partial_max, w.qnorm2, w.slots)
  // one row a wave: nothing to reuse, and the query's registers only delay the row's loads (4096 x 4096 FP8 15.9 us that
  // way, 14.2 without; 4096 x 3072 15.0 / 12.7; up to 1024 values the same). 4100 rows, the first with two: 16.1
  if (nc > most || N <= (long)grid * kWaves) LP_SCAN(0);
  else if (nc > most / 2) LP_SCAN(64 / Codes<FMT>::kPer16);
  else if (nc > most / 4) LP_SCAN(32 / Codes<FMT>::kPer16);
  else LP_SCAN(16 / Codes<FMT>::kPer16);
#undef LP_SCAN
}

inline double lowprec_margin(int format, int d) {
  const double delta = format == CHORUS_LP_BF16 ? std::ldexp(1.0, -8)
                                                 : std::ldexp(1.0, -4) + std::sqrt((double)d) * std::ldexp(1.0, -10) / 448.0;
  // twice the bound, plus room for the fp32 summation of the approximate scores themselves
  return 2.0 * std::asin(delta) + 4.0e-6 * std::sqrt((double)d);
}

}  // namespace
}  // namespace chorus

using namespace chorus;

extern "C" {

size_t chorus_cache_lowprec_bytes(int64_t N, int32_t d, int32_t format) {
  if (N < 0 || d <= 0 || (format != CHORUS_LP_BF16 && format != CHORUS_LP_FP8)) return 0;
  return (size_t)N * (size_t)d * (format == CHORUS_LP_BF16 ? 2 : 1);
}

int32_t chorus_cache_lowprec_store(const float* emb, int64_t n_rows, int32_t d, int32_t format, void* out, void* stream) {
  if (n_rows < 0 || d <= 0) return CHORUS_E_ARG;
  if (format != CHORUS_LP_BF16 && format != CHORUS_LP_FP8) return CHORUS_E_ARG;
  if (n_rows == 0) return CHORUS_OK;
  if (!emb || !out) return CHORUS_E_ARG;
  if (d % 16) return CHORUS_E_SHAPE;
  if (!aligned16(emb) || !aligned16(out)) return CHORUS_E_ARG;
  if ((n_rows + 3) / 4 > 0x7fffffffLL) return CHORUS_E_SHAPE;
  const unsigned grid = (unsigned)((n_rows + 3) / 4);
  hipStream_t s = (hipStream_t)stream;
  if (format == CHORUS_LP_BF16)
    hipLaunchKernelGGL(lowprec_store_kernel<CHORUS_LP_BF16>, dim3(grid), dim3(256), 0, s, emb, (long)n_rows, d, out);
  else
    hipLaunchKernelGGL(lowprec_store_kernel<CHORUS_LP_FP8>, dim3(grid), dim3(256), 0, s, emb, (long)n_rows, d, out);
  CHORUS_LAUNCH_CHECK();
  return CHORUS_OK;
}

size_t chorus_cache_lookup_lowprec_workspace_bytes(int64_t N) { return carve_lp(N > 0 ? (long)N : 0, nullptr).bytes; }

int32_t chorus_cache_lookup_lowprec(const float* cache_emb, const void* cache_lp, int32_t format, int64_t N, int32_t d,
                                    const float* query, float tau, chorus_lookup_result* out, int32_t* n_rescored, void* ws,
                                    size_t ws_bytes, void* stream) {
  if (N < 0 || d <= 0 || !out || !query) return CHORUS_E_ARG;
  if (format != CHORUS_LP_BF16 && format != CHORUS_LP_FP8) return CHORUS_E_ARG;
  if (N > 0 && (!cache_emb || !cache_lp)) return CHORUS_E_ARG;
  if (d % 16) return CHORUS_E_SHAPE;
  if (N > 0x7fffffffLL - 1) return CHORUS_E_SHAPE;
  if (!aligned16(cache_emb) || !aligned16(cache_lp) || !aligned16(query) || !aligned16(ws)) return CHORUS_E_ARG;
  if (!ws || ws_bytes < chorus_cache_lookup_lowprec_workspace_bytes(N)) return CHORUS_E_WORKSPACE;
  LpWs w = carve_lp((long)N, ws);
  hipStream_t s = (hipStream_t)stream;
  if (N > 0) {
    const unsigned grid = (unsigned)lp_blocks((long)N), scan_grid = (unsigned)lp_scan_blocks((long)N, (long)d * (format == CHORUS_LP_BF16 ? 2 : 1));
    if (format == CHORUS_LP_BF16)
      launch_lp_scan<CHORUS_LP_BF16>(cache_lp, query, (long)N, d, w, scan_grid, s);
    else
      launch_lp_scan<CHORUS_LP_FP8>(cache_lp, query, (long)N, d, w, scan_grid, s);
    CHORUS_LAUNCH_CHECK();
    hipLaunchKernelGGL(lowprec_rerank_kernel, dim3(grid), dim3(kWaves * 64), 0, s, cache_emb, query, (long)N, d, w.scores,
                       w.partial_max, (int)scan_grid, w.qnorm2, (float)lowprec_margin(format, d), w.slots);
    CHORUS_LAUNCH_CHECK();
  }
  hipLaunchKernelGGL(lowprec_final_kernel, dim3(1), dim3(64), 0, s, w.slots, w.qnorm2, (long)N, tau, out, n_rescored);
  CHORUS_LAUNCH_CHECK();
  return CHORUS_OK;
}

}  // extern "C"
