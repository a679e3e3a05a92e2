// Batched top-k retrieval (Sec. 3.1 "Full Reuse" for a queue of requests): the k best cache
// entries by cosine similarity for each of Q prompt embeddings, with ONE pass over the
// [N, d] fp32 cache per 32 queries instead of one per query. The scan is a [N, d] x [d, Q]
// contraction in fp32, so it runs on the fp32 matrix pipe (16x16x4), which with 32 queries
// needs about half the time that HBM needs to deliver the cache rows; row norms are accumulated
// from the same registers.
#include "common.h"
#include "lookup_row.h"

namespace chorus {
namespace {

constexpr int kBlock = 64;   // rows that partial sums are padded to
constexpr int kBK = 64;      // floats of every row per step (256 bytes: two full cache lines)
constexpr int kRing = 2;     // steps of cache rows a wave has in LDS or on their way there

struct BatchPlan {
  int waves;             // of a workgroup: 16 rows each
  int tiles;             // row tiles
  int KS;                // slices along d
  int chunks_per_slice;  // kBK-float steps per slice
  long Npad;             // rows of the partial sums
};

// Slices along d that the workspace has room for; their partial sums are added in a fixed order afterwards. (The workspace's size is
// what it always was: slices of equal length, as many of them as 1024 workgroups of 64 rows allow, at most 16.)
inline int max_slices(long N, int d) {
  const long blocks = (N + kBlock - 1) / kBlock;
  const int nchunks = (d + kBK - 1) / kBK;
  long want = blocks > 0 ? 1024 / blocks : 1;
  if (want > nchunks) want = nchunks;
  if (want > 16) want = 16;
  if (want < 1) want = 1;
  const int per = (nchunks + (int)want - 1) / (int)want;
  return (nchunks + per - 1) / per;
}

// The number of slices and the workgroup's size by an estimate of the two kernels' time in microseconds. What bounds the scan is what a
// compute unit takes in, about 25 KB a microsecond of its busiest share, the queries (from the L2) at a tenth of a row's cost; a second round
// of workgroups starts cold, and each slice's partial sums cost the selection 0.13 us. With up to 16 queries a unit holds two workgroups of eight
// waves or three of four, else one or two. Where the rows lie a multiple of 4 KB apart and the slices too, all workgroups read the same
// 256 bytes of every 4 KB at a time, and take a fifth longer (7700 x 4096, 16 queries: four slices 38.3 us, three 32.5). Fitted to 1434 calls: 0.6 % off
// the best choice. Measured (rows x d, queries: eight waves / four waves, slices), whole call, us: 4096 x 4096, 32: 25.9 (8) / 26.1 (8);
// 20000 x 4096, 32: 87 (3) / 91 (3); 20000 x 1024, 32: 40.0 (3) / 39.4 (2); 2000 x 4096, 32: 20.1 (16) / 19.6 (8); 500 x 4096, 32: 16.9
// (16) / 14.9 (16); 12000 x 512, 32: 22.0 (2) / 22.1 (2); 18061 x 472, 16: 23.5 (1) / 22.9 (2).
// The slices are those of the two query blocks: which of a call's groups a query is in, and how many queries stand beside it, must not
// change the order in which its sums are added. The workgroup's size may follow the group, it does not change that order.
inline BatchPlan plan_batch(long N, int d, int QP) {
  const int nchunks = (d + kBK - 1) / kBK, most = max_slices(N, d);
  auto estimate = [&](int waves, int per, int qp) {
    const long tiles = (N + 16 * waves - 1) / (16 * waves), slots = 256 * (waves == 8 ? (qp == 16 ? 2 : 1) : (qp == 16 ? 3 : 2));
    const long KS = (nchunks + per - 1) / per, groups = tiles * KS, later = (groups + slots - 1) / slots - 1;
    const double intake = (double)((groups + 255) / 256) * per * (4.0 * waves + 0.1 * qp) / 25.0;
    const bool same_place = KS > 1 && per % 16 == 0 && d % 1024 == 0;  // every slice of every row starts in the same 4 KB
    return intake * (same_place ? 1.2 : 1.0) + (double)later * (waves == 8 ? 5.5 : 1.7) + 0.13 * (double)KS;
  };
  int per = 0;
  double best = 0.0;
  for (int waves = 4; waves <= 8; waves += 4)
    for (int want = 1; want <= most; ++want) {
      const int p = (nchunks + want - 1) / want;
      const double time = estimate(waves, p, 32);
      if (per == 0 || time < best) {
        best = time;
        per = p;
      }
    }
  const int waves = estimate(8, per, QP) < estimate(4, per, QP) ? 8 : 4;
  return BatchPlan{waves, (int)((N + 16 * waves - 1) / (16 * waves)), (nchunks + per - 1) / per, per, (N + kBlock - 1) / kBlock * kBlock};
}

// part_dot [KS][Qp][Npad] (row fastest), part_cc [KS][Npad]; Qp = 16 QB.
// A wave owns 16 rows. Their next steps stream global -> LDS directly into a ring of its own, so that no wave waits for another's rows:
// only the queries' values, two steps of them at a time in two buffers, are shared, and only at their change stands a barrier. (With
// rows and queries staged through registers and two barriers a step the scan of 4096 x 4096 with 32 queries took 23.9 us, so 17.5 to 19;
// the fp32 matrix pipe needs 7 of them, HBM 12.)
// A direct load writes the 64 lanes' 16-byte pieces side by side (four rows of 256 bytes, or two of a query's 512); the 16-byte piece c
// of row r lives at position c ^ (r % 16), which spreads the 16 rows of a fragment read over all banks.
template <int QB, int NW>
__global__ __launch_bounds__(64 * NW, 4) void lookup_batch_scores_kernel(const float* __restrict__ cache,
                                                                         const float* __restrict__ queries,
                                                                         float* __restrict__ part_dot,
                                                                         float* __restrict__ part_cc, long N, long Npad, int d,
                                                                         int Q, int chunks_per_slice,
                                                                         uint32_t* __restrict__ done) {
  constexpr int QP = 16 * QB;
  constexpr int LB = 8 * QB / NW;       // a wave's loads of two steps of the queries
  constexpr int AW = kRing * 16 * kBK;  // floats of a wave's ring
  extern __shared__ __attribute__((aligned(1024))) float smem[];
  float* const sB = smem;  // [2][QP][2 kBK]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  float* const sA = smem + 2 * QP * 2 * kBK + wave * AW;  // [kRing][16][kBK]
  if (done && blockIdx.x == 0 && blockIdx.y == 0 && tid < QP) done[tid] = 0;  // arrivals of the selection's workgroups
  const long row0 = ((long)blockIdx.x * NW + wave) * 16;
  const int ks = blockIdx.y;
  const int c0 = ks * chunks_per_slice;
  const int nchunks = (d + kBK - 1) / kBK;
  const int n = __builtin_amdgcn_readfirstlane((c0 + chunks_per_slice < nchunks ? c0 + chunks_per_slice : nchunks) - c0);

  const float* rowp[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const long r = row0 + 4 * i + (lane >> 4);
    rowp[i] = cache + (r < N ? r : N - 1) * (long)d;  // rows past the end read the last one
  }
  typedef __attribute__((address_space(3))) void* Lds;
  auto issue_rows = [&](int c, int slot) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      int k = (c0 + c) * kBK + 4 * ((lane & 15) ^ (4 * i + (lane >> 4)));
      k = k < d ? k : d - 4;  // masked where it is used
      __builtin_amdgcn_global_load_lds(rowp[i] + k, (Lds)(sA + (slot * 16 + 4 * i) * kBK), 16, 0, 2);  // non-temporal
    }
  };
  auto issue_queries = [&](int s) {  // steps 2 s and 2 s + 1
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      const int q0 = 2 * (wave * LB + i), q = q0 + (lane >> 5);
      int k = (c0 + 2 * s) * kBK + 4 * ((lane & 31) ^ (q & 15));
      k = k < d ? k : d - 4;
      __builtin_amdgcn_global_load_lds(queries + (long)(q < Q ? q : Q - 1) * d + k, (Lds)(sB + ((s & 1) * QP + q0) * 2 * kBK), 16, 0, 0);
    }
  };

  const int l16 = lane & 15, kq = lane >> 4;
  // a sum per quarter of a step, added at the end: four short chains of additions in place of a long one (error of the scores against
  // 64 bits at 4096 x 4096 1.5e-7 with one, 0.8e-7 with four, 1.1e-7 with sixteen slices of one chain each as before)
  f32x4 acc[4][QB];
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int q = 0; q < QB; ++q) acc[j][q] = f32x4{0.f, 0.f, 0.f, 0.f};
  float cc4[4] = {0.f, 0.f, 0.f, 0.f};
  auto compute = [&](const f32x4 (&a)[4], int c, bool mask) {
    const float* b0 = sB + ((c >> 1) & 1) * QP * 2 * kBK;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      f32x4 av = a[j], b[QB];
#pragma unroll
      for (int q = 0; q < QB; ++q)
        b[q] = *reinterpret_cast<const f32x4*>(b0 + (16 * q + l16) * 2 * kBK + 4 * (((c & 1) * 16 + 4 * j + kq) ^ l16));
      if (mask && (c0 + c) * kBK + 16 * j + 4 * kq >= d) {
        av = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < QB; ++q) b[q] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      cc4[j] += av[0] * av[0] + av[1] * av[1] + av[2] * av[2] + av[3] * av[3];
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int q = 0; q < QB; ++q) acc[j][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[e], b[q][e], acc[j][q], 0, 0, 0);
    }
  };

  issue_queries(0);
  issue_rows(0, 0);
  if (1 < n) issue_rows(1, 1);
  int slot = 0;
  // Loads in flight at step c: rows c and c + 1, and from an even step on the queries of the next two, requested ahead of the rows of
  // step c + 2. Loads retire in order: at most as many as were requested behind what the step needs may be left.
  for (int c = 0; c < n; ++c) {
    const bool more = c + kRing <= n;  // rows c + 1 have been requested
    if ((c & 1) == 0) {
      if (more)
        asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)\n\ts_barrier" ::: "memory");
      else
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
      if (c + 2 < n) issue_queries((c >> 1) + 1);  // into the buffer that everyone has left behind the barrier
    } else if (more) {
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 + LB) : "memory");
    } else {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    f32x4 a[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      a[j] = *reinterpret_cast<const f32x4*>(sA + (slot * 16 + l16) * kBK + 4 * ((4 * j + kq) ^ l16));
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3])::"memory");
    if (c + kRing < n) issue_rows(c + kRing, slot);
    slot = slot == kRing - 1 ? 0 : slot + 1;
    if ((c0 + c + 1) * kBK <= d)
      compute(a, c, false);
    else
      compute(a, c, true);
  }
  if (row0 >= Npad) return;  // the second half of the last tile
  // row norms: the four k quarters of a row sit in lanes l16, l16 + 16, l16 + 32, l16 + 48
  float cc = (cc4[0] + cc4[1]) + (cc4[2] + cc4[3]);
  cc += __shfl_xor(cc, 16, 64);
  cc += __shfl_xor(cc, 32, 64);
  if (kq == 0) part_cc[(long)ks * Npad + row0 + l16] = cc;
  // accumulator elements 0..3 of lane (l16, kq): rows 4 kq .. 4 kq + 3 of the block, query l16
#pragma unroll
  for (int q = 0; q < QB; ++q)
    *reinterpret_cast<f32x4*>(&part_dot[((long)ks * QP + 16 * q + l16) * Npad + row0 + 4 * kq]) = (acc[0][q] + acc[1][q]) + (acc[2][q] + acc[3][q]);
}

template <int QB, int NW>
int32_t launch_scores(const float* cache, const float* queries, float* part_dot, float* part_cc, long N, int d, int Q,
                      const BatchPlan& p, uint32_t* done, hipStream_t s) {
  constexpr size_t smem = (size_t)(2 * 16 * QB * 2 * kBK + NW * kRing * 16 * kBK) * sizeof(float);
  auto kern = lookup_batch_scores_kernel<QB, NW>;
  static DynLdsOnce once;
  CHK_STATUS(once.ensure(reinterpret_cast<const void*>(kern), (int)smem));
  hipLaunchKernelGGL(kern, dim3((unsigned)p.tiles, (unsigned)p.KS), dim3(64 * NW), smem, s, cache, queries, part_dot, part_cc, N,
                     p.Npad, d, Q, p.chunks_per_slice, done);
  CHORUS_LAUNCH_CHECK();
  return CHORUS_OK;
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
  const int QP = Qc > 16 ? 32 : 16, slices = max_slices(N, d);
  const long rows = N > 0 ? (N + kBlock - 1) / kBlock * kBlock : kBlock;
  const BytePtr b(base);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    void* r = b + off;
    off += align_up(bytes, 256);
    return r;
  };
  w.part_dot = (float*)take((size_t)slices * rows * QP * 4);
  w.part_cc = (float*)take((size_t)slices * rows * 4);
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
  for (int q0 = 0; q0 < Q; q0 += 32) {
    const int Qc = Q - q0 < 32 ? Q - q0 : 32;
    const int QP = Qc > 16 ? 32 : 16;
    BatchWs w = carve_batch((long)N, d, Q > 32 ? 32 : Q, ws);
    const float* qs = queries + (long)q0 * d;
    const BatchPlan p = plan_batch((long)N, d, QP);
    const long Npad = p.Npad;
    const long nb = (N + 1023) / 1024;  // row blocks of the selection
    const bool lists_fit = k <= kWaveK;  // selected where the scores are made
    // the waves' lists take the place of the scores (128 bytes a row against at most 64 a row of a block), the arrival
    // counts stand behind them; a single row block needs neither
    uint64_t* lists = reinterpret_cast<uint64_t*>(w.scores);
    uint32_t* done = lists_fit && nb > 1 ? reinterpret_cast<uint32_t*>(lists + nb * 4 * 32 * kWaveK) : nullptr;
    if (N > 0) {
      auto scores = p.waves == 8 ? (QP == 32 ? launch_scores<2, 8> : launch_scores<1, 8>)
                                 : (QP == 32 ? launch_scores<2, 4> : launch_scores<1, 4>);
      CHK_STATUS(scores(cache_emb, qs, w.part_dot, w.part_cc, (long)N, d, Qc, p, done, s));
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
