// Batched top-k retrieval (Sec. 3.1 "Full Reuse" for a queue of requests): the k best cache
// entries by cosine similarity for each of Q prompt embeddings, with ONE pass over the
// [N, d] fp32 cache per 32 queries instead of one per query. The scan is a [N, d] x [d, Q]
// contraction in fp32, so it runs on the fp32 matrix pipe (16x16x4), which at 16-32 queries
// needs about the cycles that HBM needs to deliver the cache rows; row norms are accumulated
// from the same registers.
#include "common.h"
#include "lookup_row.h"

namespace chorus {
namespace {

constexpr int kRB = 1;        // 16-row blocks per wave
constexpr int kBR = 64 * kRB;  // cache rows per workgroup, 16 kRB per wave
constexpr int kBK = 64;       // floats of every row per step (256 bytes: two full cache lines)
constexpr int kLS = kBK + 4;  // LDS row stride in floats (16-byte aligned, staggers the banks)

struct BatchPlan {
  int tiles;             // row tiles
  int KS;                // slices along d
  int chunks_per_slice;  // kBK-float steps per slice
};

inline BatchPlan plan_batch(long N, int d) {
  BatchPlan p;
  p.tiles = (int)((N + kBR - 1) / kBR);
  const int nchunks = (d + kBK - 1) / kBK;
  // As many workgroups as fit the chip at once, four on each of 256 CUs, and no more: a few beyond that are a second round
  // (20000 x 4096, 32 queries: 1252 workgroups 130 us the call, 939 108). Partial sums of the slices are added in a fixed order
  // afterwards.
  int want = p.tiles > 0 ? 1024 / p.tiles : 1;
  if (want < 1) want = 1;
  if (want > nchunks) want = nchunks;
  if (want > 16) want = 16;  // every slice writes and re-reads its own partial sums
  p.chunks_per_slice = (nchunks + want - 1) / want;
  p.KS = (nchunks + p.chunks_per_slice - 1) / p.chunks_per_slice;
  return p;
}

// part_dot [KS][Qp][Npad] (row fastest, Npad = N rounded up to 128), part_cc [KS][Npad]; Qp = 16 * QB
template <int QB>
__global__ __launch_bounds__(256) void lookup_batch_scores_kernel(const float* __restrict__ cache,
                                                                  const float* __restrict__ queries,
                                                                  float* __restrict__ part_dot,
                                                                  float* __restrict__ part_cc, long N, int d, int Q,
                                                                  int chunks_per_slice, uint32_t* __restrict__ done) {
  constexpr int QP = 16 * QB;
  __shared__ __attribute__((aligned(16))) float sA[kBR * kLS];
  __shared__ __attribute__((aligned(16))) float sB[QP * kLS];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (done && blockIdx.x == 0 && blockIdx.y == 0 && tid < QP) done[tid] = 0;  // arrivals of the selection's workgroups
  const long row0 = (long)blockIdx.x * kBR;
  const long Npad = (long)gridDim.x * kBR;
  const int ks = blockIdx.y;
  const int c0 = ks * chunks_per_slice;
  const int nchunks = (d + kBK - 1) / kBK;
  const int c1 = c0 + chunks_per_slice < nchunks ? c0 + chunks_per_slice : nchunks;

  // loader role: 16 threads per row segment of 256 bytes
  const int lcol = tid & 15, lrow = tid >> 4;
  f32x4 ra[2][4 * kRB], rb[2][QB];  // two chunks in flight
  auto load_chunk = [&](int st, int c) {
    const int k = c * kBK + 4 * lcol;
#pragma unroll
    for (int i = 0; i < 4 * kRB; ++i) {
      const long r = row0 + lrow + 16 * i;
      const bool ok = r < N && k < d;
      const float* p = cache + (ok ? r : 0) * (long)d + (ok ? k : 0);
      f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p));
      ra[st][i] = ok ? v : f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int i = 0; i < QB; ++i) {
      const int q = lrow + 16 * i;
      const bool ok = q < Q && k < d;
      const float* p = queries + (long)(ok ? q : 0) * d + (ok ? k : 0);
      f32x4 v = *reinterpret_cast<const f32x4*>(p);
      rb[st][i] = ok ? v : f32x4{0.f, 0.f, 0.f, 0.f};
    }
  };
  auto store_chunk = [&](int st) {
#pragma unroll
    for (int i = 0; i < 4 * kRB; ++i) *reinterpret_cast<f32x4*>(&sA[(lrow + 16 * i) * kLS + 4 * lcol]) = ra[st][i];
#pragma unroll
    for (int i = 0; i < QB; ++i) *reinterpret_cast<f32x4*>(&sB[(lrow + 16 * i) * kLS + 4 * lcol]) = rb[st][i];
  };

  // compute role: a wave owns 32 rows = two 16-row blocks; lane = (row or query l % 16, k quarter l / 16)
  const int l16 = lane & 15, kq = lane >> 4;
  f32x4 acc[kRB][QB];
#pragma unroll
  for (int r = 0; r < kRB; ++r)
#pragma unroll
    for (int q = 0; q < QB; ++q) acc[r][q] = f32x4{0.f, 0.f, 0.f, 0.f};
  float cc[kRB] = {};

  // chunk c + 1 is already in flight when chunk c is stored, and chunk c + 2 is requested right after: two chunks
  // (64 KB per workgroup) are on their way during the MFMAs. Past the slice the loads are masked to zeros.
  auto step = [&](int st, int c) {
    __syncthreads();  // the previous step's reads are done
    store_chunk(st);
    __syncthreads();
    if (c + 2 < c1) load_chunk(st, c + 2);
#pragma unroll
    for (int j = 0; j < kBK / 16; ++j) {
      f32x4 a[kRB], b[QB];
#pragma unroll
      for (int r = 0; r < kRB; ++r) a[r] = *reinterpret_cast<const f32x4*>(&sA[(16 * kRB * wave + 16 * r + l16) * kLS + 16 * j + 4 * kq]);
#pragma unroll
      for (int q = 0; q < QB; ++q) b[q] = *reinterpret_cast<const f32x4*>(&sB[(16 * q + l16) * kLS + 16 * j + 4 * kq]);
#pragma unroll
      for (int r = 0; r < kRB; ++r) {
        cc[r] += a[r][0] * a[r][0] + a[r][1] * a[r][1] + a[r][2] * a[r][2] + a[r][3] * a[r][3];
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int q = 0; q < QB; ++q) acc[r][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[r][e], b[q][e], acc[r][q], 0, 0, 0);
      }
    }
  };
  if (c0 < c1) load_chunk(0, c0);
  if (c0 + 1 < c1) load_chunk(1, c0 + 1);
  for (int c = c0; c < c1; c += 2) {
    step(0, c);
    if (c + 1 < c1) step(1, c + 1);
  }
  // row norms: the four k quarters of a row sit in lanes l16, l16 + 16, l16 + 32, l16 + 48
#pragma unroll
  for (int r = 0; r < kRB; ++r) {
    cc[r] += __shfl_xor(cc[r], 16, 64);
    cc[r] += __shfl_xor(cc[r], 32, 64);
    const long row = row0 + 16 * kRB * wave + 16 * r + l16;
    if (kq == 0) part_cc[(long)ks * Npad + row] = cc[r];
  }
  // accumulator elements 0..3 of lane (l16, kq): rows 4 kq .. 4 kq + 3 of the block, query l16 (rows past N hold zeros)
#pragma unroll
  for (int r = 0; r < kRB; ++r)
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      const long row = row0 + 16 * kRB * wave + 16 * r + 4 * kq;
      *reinterpret_cast<f32x4*>(&part_dot[((long)ks * QP + 16 * q + l16) * Npad + row]) = acc[r][q];
    }
}

// dot[u], cc[u] (u < RU) += the partial sums of entry j + STRIDE u over the KS slices, in ascending slice order
// whatever the grouping: G slices x RU entries x 2 loads are in flight at a time.
template <int RU, int G, int RMAX, int STRIDE>
__device__ __forceinline__ void sum_slices(const float* __restrict__ part_dot, const float* __restrict__ part_cc, int KS,
                                           int QP, int q, long Npad, long j, long N, float (&dot)[RMAX], float (&cc)[RMAX]) {
  for (int ks0 = 0; ks0 < KS; ks0 += G) {
    float pd[G][RU], pc[G][RU];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int ks = ks0 + g < KS ? ks0 + g : KS - 1;
#pragma unroll
      for (int u = 0; u < RU; ++u) {
        const long ju = j + (long)STRIDE * u;
        const long jj = ju < N ? ju : N - 1;
        pd[g][u] = part_dot[((long)ks * QP + q) * Npad + jj];
        pc[g][u] = part_cc[(long)ks * Npad + jj];
      }
    }
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int u = 0; u < RU; ++u) {
        const bool live = ks0 + g < KS;
        dot[u] += live ? pd[g][u] : 0.f;
        cc[u] += live ? pc[g][u] : 0.f;
      }
  }
}

// |q|, summed in one order by both kernels that divide by it, so that an entry has the same score whatever k is. The first
// 4096 values are requested by the constructor, ahead of the partial sums, and added behind them. d % 4 == 0, 256 threads.
struct QueryNorm {
  static constexpr int QU = 4;
  const f32x4* q4;
  int n4;
  f32x4 v[QU];
  __device__ __forceinline__ QueryNorm(const float* q, int d, int tid) : q4(reinterpret_cast<const f32x4*>(q)), n4(d >> 2) {
#pragma unroll
    for (int c = 0; c < QU; ++c) v[c] = tid + 256 * c < n4 ? q4[tid + 256 * c] : f32x4{0.f, 0.f, 0.f, 0.f};
  }
  __device__ __forceinline__ float get(float (&sq)[4], int tid) const {
    auto add = [](float s, const f32x4& w) {  // the roundings spelled out: not left to what each kernel's compilation contracts
#pragma clang fp contract(off)
      return s + (__builtin_fmaf(w[0], w[0], w[1] * w[1]) + __builtin_fmaf(w[2], w[2], w[3] * w[3]));
    };
    float qq = 0.f;
#pragma unroll
    for (int c = 0; c < QU; ++c) qq = add(qq, v[c]);
    for (int i = tid + 256 * QU; i < n4; i += 256) qq = add(qq, q4[i]);
    qq = wave_sum(qq);
    if ((tid & 63) == 0) sq[tid >> 6] = qq;
    __syncthreads();
    return sqrtf(sq[0] + sq[1] + sq[2] + sq[3]);
  }
};

// the score of an entry: -inf for zero norms and NaN
__device__ __forceinline__ float batch_score(float dot, float cc, float qn) {
  const float den = sqrtf(cc) * qn;
  const float v = den > 0.f ? dot / den : -INFINITY;
  return v == v ? v : -INFINITY;
}

constexpr int kWaveK = 64;  // up to this k a list is one key per lane

// ---- keys: a score and its row as one integer, larger = better (higher score, then lower row); 0 = no entry ----
__device__ __forceinline__ uint64_t make_key(float score, uint32_t row) {
  const uint32_t u = __float_as_uint(score + 0.0f);  // 0 and -0 are equal
  return ((uint64_t)((u & 0x80000000u) ? ~u : (u | 0x80000000u)) << 32) | (uint32_t)~row;
}
__device__ __forceinline__ float key_score(uint64_t k) {
  const uint32_t ord = (uint32_t)(k >> 32);
  return k == 0 ? -INFINITY : __uint_as_float((ord & 0x80000000u) ? (ord & 0x7fffffffu) : ~ord);
}
__device__ __forceinline__ int key_row(uint64_t k) { return k == 0 ? -1 : (int)~(uint32_t)k; }

// The k <= 64 largest of the wave's keys (four per lane, all different but for 0), best first, one per lane (0 behind the
// last). Few: a lane keeps its four sorted and offers its best, a round per position is one wave-wide maximum (two
// chains of six 32-bit steps). More than kRounds: a bitonic sort of all 256, whose cost does not depend on k (about 3000).
constexpr int kRounds = 8;
__device__ __forceinline__ uint64_t shfl_key(uint64_t k, int from) {
  return ((uint64_t)(uint32_t)__shfl((int)(uint32_t)(k >> 32), from, 64) << 32) | (uint32_t)__shfl((int)(uint32_t)k, from, 64);
}
__device__ __forceinline__ uint64_t wave_topk(uint64_t (&key)[4], int k, int lane) {
  auto order = [&](int i, int j, bool down) {  // down: the larger one to i
    const bool swap = (key[i] < key[j]) == down;
    const uint64_t a = swap ? key[j] : key[i], b = swap ? key[i] : key[j];
    key[i] = a;
    key[j] = b;
  };
  uint64_t mine = 0;
  if (k <= kRounds) {
    order(0, 1, true);
    order(2, 3, true);
    order(0, 2, true);
    order(1, 3, true);
    order(1, 2, true);
    for (int r = 0; r < k; ++r) {
      const uint64_t best = wave_max_key(key[0]);
      if (best == 0) break;
      if (lane == r) mine = best;
      if (key[0] == best) {
        key[0] = key[1];
        key[1] = key[2];
        key[2] = key[3];
        key[3] = 0;
      }
    }
    return mine;
  }
  // element i = 4 * lane + u; runs of `size` are sorted in alternating directions, the last one downwards
  order(0, 1, true);
  order(2, 3, false);
  for (int size = 4; size <= 256; size *= 2) {
    const bool down = ((4 * lane) & size) == 0;
    for (int dist = size / 2; dist >= 4; dist /= 2) {
      const int other = lane ^ (dist / 4);
      const bool keep_max = (((4 * lane) & dist) == 0) == down;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint64_t o = shfl_key(key[u], other);
        key[u] = (o > key[u]) == keep_max ? o : key[u];
      }
    }
    order(0, 2, down);
    order(1, 3, down);
    order(0, 1, down);
    order(2, 3, down);
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const uint64_t o = shfl_key(key[u], lane >> 2);
    if ((lane & 3) == u) mine = o;
  }
  return lane < k ? mine : 0;
}

// Final scores and selection for k <= 64: score[q][j] = (partial dots summed in slice order) / (|c_j| |q|), -inf for zero
// norms and NaN. Grid (row blocks of 1024, queries): spread over the chip, because one workgroup per query would pull its
// KS slices (half a megabyte at 4096 entries) through a single compute unit. A wave keeps its 256 scores in registers and
// lists the k best of them; the last workgroup of a query to arrive merges the lists. Lists and arrivals are
// agent-scope atomics, as the workgroups of a query run on different XCDs, whose L2s are not coherent otherwise. With
// the scores written out and one workgroup per query selecting from them (two launches): 23 us at 4096 x 32 queries,
// k = 8, in this kernel 9.5; 20000 entries, 48 queries, k = 50 the whole call 538 -> 109 us. ONE is k = 1 (8192 x 64, 32 queries
// 10.1 us the call, in two launches 12.0, through the lists 11.0).
template <bool ONE>
__global__ __launch_bounds__(256) void lookup_batch_select_kernel(const float* __restrict__ part_dot,
                                                                  const float* __restrict__ part_cc,
                                                                  const float* __restrict__ queries, uint64_t* lists,
                                                                  uint32_t* done, long N, long Npad, int d, int QP, int KS,
                                                                  int k, float tau, int32_t* __restrict__ out_idx,
                                                                  float* __restrict__ out_score,
                                                                  int32_t* __restrict__ out_hit) {
  constexpr int R = 4;
  __shared__ float sq[4];
  __shared__ uint64_t sl[4][kWaveK];
  __shared__ uint32_t s_arrived;
  const int q = blockIdx.y, nb = gridDim.x;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const long j0 = (long)blockIdx.x * (256 * R) + tid;
  float dot[R], cc[R];
#pragma unroll
  for (int u = 0; u < R; ++u) dot[u] = cc[u] = 0.f;
  const QueryNorm norm(queries + (long)q * d, d, tid);
  sum_slices<R, 8, R, 256>(part_dot, part_cc, KS, QP, q, Npad, j0, N, dot, cc);
  const float qn = norm.get(sq, tid);
  uint64_t key[4];
#pragma unroll
  for (int u = 0; u < R; ++u) {
    const long j = j0 + 256L * u;
    key[u] = j < N ? make_key(batch_score(dot[u], cc[u], qn), (uint32_t)j) : 0;
  }
  // ONE: the best entry alone is a maximum, of the thread's entries, the wave's, the workgroup's, the query's.
  if constexpr (ONE) {
    uint64_t best = key[0] > key[1] ? key[0] : key[1];
    best = key[2] > best ? key[2] : best;
    best = key[3] > best ? key[3] : best;
    best = wave_max_key(best);
    if (lane == 0) sl[0][wave] = best;
    __syncthreads();
    if (wave != 0) return;
    best = wave_max_key(sl[0][lane & 3]);
    uint64_t* all = lists + (long)q * nb;
    if (nb > 1) {
      uint32_t arrived = 0;
      if (lane == 0) {
        __hip_atomic_store(&all[blockIdx.x], best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // as below
        arrived = __hip_atomic_fetch_add(&done[q], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      if ((uint32_t)__builtin_amdgcn_readfirstlane((int)arrived) != (uint32_t)nb - 1) return;
      asm volatile("" ::: "memory");
      for (long i = lane; i < nb; i += 64) {
        const uint64_t o = __hip_atomic_load(&all[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        best = o > best ? o : best;
      }
      best = wave_max_key(best);
    }
    if (lane == 0) {
      const float sc = key_score(best);
      out_idx[q] = key_row(best);
      out_score[q] = sc;
      out_hit[q] = (best != 0 && sc >= tau) ? 1 : 0;
    }
    return;
  }
  // Every wave lists the k best of its 256 entries; with several row blocks the lists of a query meet in memory, one per
  // wave while the last workgroup can take them all in one go, else one per workgroup.
  uint64_t own = wave_topk(key, k, lane);
  const bool per_wave = (long)nb * 4 * k <= 256;
  if (nb > 1 && !per_wave) {
    if (lane < k) sl[wave][lane] = own;
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int w = 0; w < 4; ++w) key[w] = lane < k ? sl[w][lane] : 0;
      own = wave_topk(key, k, lane);
    }
  }
  const long total = (long)nb * (per_wave ? 4 : 1) * k;
  uint64_t* all = lists + (long)q * total;
  if (nb > 1) {
    const long at = per_wave ? (long)blockIdx.x * 4 + wave : (long)blockIdx.x;
    if (lane < k && (per_wave || wave == 0))
      __hip_atomic_store(&all[at * k + lane], own, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // Every wave waits for its own stores, the barrier joins them, one lane reports the arrival. The lists are agent-scope
    // atomics, written and read past the L2s, so that once they have completed there is nothing to release: the fence that stood
    // here wrote the XCD's whole L2 back (4096 entries, 32 queries, k = 8: this kernel 11.8 -> 9.5 us, the call 33.1 -> 30.7).
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) s_arrived = __hip_atomic_fetch_add(&done[q], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (s_arrived != (uint32_t)nb - 1) return;
    asm volatile("" ::: "memory");  // the lists are read behind the count
  } else {
    if (lane < k) sl[wave][lane] = own;
    __syncthreads();
  }
  uint64_t best = 0;  // wave 0, lane r: the r-th best
  if (nb == 1 || total <= 256) {  // four keys per lane are all there are
    if (wave != 0) return;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (nb == 1)
        key[u] = lane < k ? sl[u][lane] : 0;
      else
        key[u] = 64 * u + lane < total ? __hip_atomic_load(&all[64 * u + lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    }
    best = wave_topk(key, k, lane);
  } else {
    // every wave merges its share of the lists into its own k best, 192 new keys at a time beside the 64 it may hold
    uint64_t run = 0;
    for (long i0 = (long)wave * 192; i0 < total; i0 += 4 * 192) {
      key[0] = run;
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        const long i = i0 + 64 * u + lane;
        key[u + 1] = i < total ? __hip_atomic_load(&all[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
      }
      run = wave_topk(key, k, lane);
    }
    if (lane < k) sl[wave][lane] = run;
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int w = 0; w < 4; ++w) key[w] = lane < k ? sl[w][lane] : 0;
      best = wave_topk(key, k, lane);
    }
  }
  if (wave == 0 && lane < k) {
    const float sc = key_score(best);
    out_idx[(long)q * k + lane] = key_row(best);
    out_score[(long)q * k + lane] = sc;
    if (lane == 0) out_hit[q] = (best != 0 && sc >= tau) ? 1 : 0;
  }
}

// Final scores alone, where the selection is a pass of its own
__global__ __launch_bounds__(256) void lookup_batch_final_kernel(const float* __restrict__ part_dot,
                                                                 const float* __restrict__ part_cc,
                                                                 const float* __restrict__ queries,
                                                                 float* __restrict__ scores, long N, long Npad, int d,
                                                                 int QP, int KS) {
  constexpr int R = 4;
  __shared__ float sq[4];
  const int q = blockIdx.y;
  const int tid = threadIdx.x;
  const long j0 = (long)blockIdx.x * (256 * R) + tid;
  float dot[R], cc[R];
#pragma unroll
  for (int u = 0; u < R; ++u) dot[u] = cc[u] = 0.f;
  const QueryNorm norm(queries + (long)q * d, d, tid);
  sum_slices<R, 8, R, 256>(part_dot, part_cc, KS, QP, q, Npad, j0, N, dot, cc);
  const float qn = norm.get(sq, tid);
#pragma unroll
  for (int u = 0; u < R; ++u) {
    const long j = j0 + 256L * u;
    if (j < N) scores[(long)q * Npad + j] = batch_score(dot[u], cc[u], qn);
  }
}

// k > 64 or an empty cache. One workgroup per query: k rounds over its final scores, each picking the best entry that comes after the
// previous winner in the order (score descending, index ascending). REG: the scores of a thread live in registers
// (N <= kTopkRegs), else they are re-read from `scores`.
constexpr long kTopkRegs = 8 * 1024;
template <bool REG>
__global__ __launch_bounds__(1024) void lookup_topk_kernel(const float* __restrict__ scores, long N, long Npad, int k,
                                                           float tau, int32_t* __restrict__ out_idx,
                                                           float* __restrict__ out_score, int32_t* __restrict__ out_hit) {
  constexpr int R = 8;
  static_assert(R * 1024 == kTopkRegs, "the scores that 1024 threads hold");
  __shared__ uint64_t sk[2][16];
  const int q = blockIdx.x;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const float* sc = scores + (long)q * Npad;
  uint64_t mine[R];
#pragma unroll
  for (int u = 0; u < R; ++u) {
    const long j = tid + 1024L * u;
    mine[u] = (REG && j < N) ? make_key(sc[j], (uint32_t)j) : 0;
  }
  uint64_t prev = ~0ull;
  for (int r = 0; r < k; ++r) {
    uint64_t best = 0;
    if (REG) {
#pragma unroll
      for (int u = 0; u < R; ++u) {
        if (mine[u] == prev) mine[u] = 0;  // the previous winner
        best = mine[u] > best ? mine[u] : best;
      }
    } else {
      for (long j = tid; j < N; j += 1024) {
        const uint64_t key = make_key(sc[j], (uint32_t)j);
        best = key < prev && key > best ? key : best;
      }
    }
    best = wave_max_key(best);
    const int buf = r & 1;  // alternating buffers: one barrier per round
    if (lane == 0) sk[buf][wave] = best;
    __syncthreads();
    prev = wave_max_key(sk[buf][lane & 15]);  // every wave reduces the 16 candidates again
    if (tid == 0) {
      const float b = key_score(prev);
      out_idx[(long)q * k + r] = key_row(prev);
      out_score[(long)q * k + r] = b;
      if (r == 0) out_hit[q] = (prev != 0 && b >= tau) ? 1 : 0;
    }
    if (prev == 0) {  // the cache is exhausted: the remaining positions are empty
      for (int rr = r + 1 + tid; rr < k; rr += 1024) {
        out_idx[(long)q * k + rr] = -1;
        out_score[(long)q * k + rr] = -INFINITY;
      }
      break;
    }
  }
}

struct BatchWs {
  float* part_dot;
  float* part_cc;
  float* scores;
  size_t bytes;
};

BatchWs carve_batch(long N, int d, int Qc, void* base) {
  BatchWs w;
  const BatchPlan p = plan_batch(N, d);
  const int QP = Qc > 16 ? 32 : 16;
  const long rows = p.tiles > 0 ? (long)p.tiles * kBR : kBR;  // padded to whole row tiles
  const BytePtr b(base);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    void* r = b + off;
    off += align_up(bytes, 256);
    return r;
  };
  w.part_dot = (float*)take((size_t)p.KS * rows * QP * 4);
  w.part_cc = (float*)take((size_t)p.KS * rows * 4);
  w.scores = (float*)take((size_t)32 * rows * 4);
  w.bytes = off;
  return w;
}

}  // namespace
}  // namespace chorus

using namespace chorus;

extern "C" {

size_t chorus_cache_lookup_batch_workspace_bytes(int64_t N, int32_t d, int32_t Q) {
  if (N < 0 || d <= 0 || Q < 0) return 0;
  return carve_batch((long)N, d, Q > 32 ? 32 : Q, nullptr).bytes;
}

int32_t chorus_cache_lookup_batch(const float* cache_emb, int64_t N, int32_t d, const float* queries, int32_t Q, float tau,
                                  int32_t k, int32_t* out_index, float* out_score, int32_t* out_hit, void* ws,
                                  size_t ws_bytes, void* stream) {
  if (N < 0 || d <= 0 || Q < 0 || k < 1 || k > 1024) return CHORUS_E_ARG;
  if (Q == 0) return CHORUS_OK;
  if (!queries || !out_index || !out_score || !out_hit || (N > 0 && !cache_emb)) return CHORUS_E_ARG;
  if ((d & 3) != 0) return CHORUS_E_SHAPE;
  if (!aligned16(cache_emb) || !aligned16(queries)) return CHORUS_E_ARG;
  if (N > 0x7fffff00LL) return CHORUS_E_SHAPE;
  if (!ws || !aligned16(ws) || ws_bytes < chorus_cache_lookup_batch_workspace_bytes(N, d, Q)) return CHORUS_E_WORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  const BatchPlan p = plan_batch((long)N, d);
  for (int q0 = 0; q0 < Q; q0 += 32) {
    const int Qc = Q - q0 < 32 ? Q - q0 : 32;
    const int QP = Qc > 16 ? 32 : 16;
    BatchWs w = carve_batch((long)N, d, Q > 32 ? 32 : Q, ws);
    const float* qs = queries + (long)q0 * d;
    const long Npad = (long)p.tiles * kBR;
    const long nb = (N + 1023) / 1024;  // row blocks of the selection
    const bool lists_fit = k <= kWaveK;  // selected where the scores are made
    // the waves' lists take the place of the scores (128 bytes a row against at most 64 a row of a block), the arrival
    // counts stand behind them; a single row block needs neither
    uint64_t* lists = reinterpret_cast<uint64_t*>(w.scores);
    uint32_t* done = lists_fit && nb > 1 ? reinterpret_cast<uint32_t*>(lists + nb * 4 * 32 * kWaveK) : nullptr;
    if (N > 0) {
      const dim3 grid((unsigned)p.tiles, (unsigned)p.KS);
      if (QP == 32)
        hipLaunchKernelGGL(lookup_batch_scores_kernel<2>, grid, dim3(256), 0, s, cache_emb, qs, w.part_dot, w.part_cc,
                           (long)N, d, Qc, p.chunks_per_slice, done);
      else
        hipLaunchKernelGGL(lookup_batch_scores_kernel<1>, grid, dim3(256), 0, s, cache_emb, qs, w.part_dot, w.part_cc,
                           (long)N, d, Qc, p.chunks_per_slice, done);
      CHORUS_LAUNCH_CHECK();
      if (lists_fit) {
        const auto select = k == 1 ? lookup_batch_select_kernel<true> : lookup_batch_select_kernel<false>;
        hipLaunchKernelGGL(select, dim3((unsigned)nb, (unsigned)Qc), dim3(256), 0, s, w.part_dot, w.part_cc, qs, lists, done, (long)N,
                           Npad, d, QP, p.KS, k, tau, out_index + (long)q0 * k, out_score + (long)q0 * k, out_hit + q0);
        CHORUS_LAUNCH_CHECK();
        continue;
      }
      hipLaunchKernelGGL(lookup_batch_final_kernel, dim3((unsigned)nb, (unsigned)Qc), dim3(256), 0, s, w.part_dot, w.part_cc,
                         qs, w.scores, (long)N, Npad, d, QP, p.KS);
      CHORUS_LAUNCH_CHECK();
    }
    if (N <= kTopkRegs)
      hipLaunchKernelGGL(lookup_topk_kernel<true>, dim3(Qc), dim3(1024), 0, s, w.scores, (long)N, Npad, k, tau,
                         out_index + (long)q0 * k, out_score + (long)q0 * k, out_hit + q0);
    else
      hipLaunchKernelGGL(lookup_topk_kernel<false>, dim3(Qc), dim3(1024), 0, s, w.scores, (long)N, Npad, k, tau,
                         out_index + (long)q0 * k, out_score + (long)q0 * k, out_hit + q0);
    CHORUS_LAUNCH_CHECK();
  }
  return CHORUS_OK;
}

}  // extern "C"
