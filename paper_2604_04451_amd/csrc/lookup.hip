// Stage-1 retrieval: top-1 cosine similarity over the prompt-embedding cache
// (Sec. 3.1 "Full Reuse"). HBM-bound: the [N, d] fp32 cache is streamed once.
#include "chorus_ops.h"
#include "common.h"
#include "lookup_row.h"
#include "tagged.h"

namespace chorus {

thread_local int32_t g_last_hip_error = 0;

namespace {

// A cache in one launch: waves per workgroup of the scan, one cache row per wave at a time; beyond kMaxScanBlocks workgroups a
// wave walks several rows. In two launches, where a workgroup's hand-over costs nothing: half as many waves, twice the workgroups
// (1024 x 4096 in a graph 7.5 us, with eight waves 8.3).
constexpr int kWaves = 8, kMaxScanBlocks = 2048;
constexpr int kWavesTwo = 4, kMaxScanBlocksTwo = 4096;
// Larger caches (16 GB) take two launches: the second one is 0.2 % of the scan there, and a last workgroup whose wait ran out
// would have the whole cache to itself, at 38 GB/s.
constexpr size_t kMaxWaitValues = (size_t)1 << 32;

// What one workgroup of the scan leaves behind: the best r_j = <q, c_j> / |c_j| among its rows and that row (the lowest one among
// equal values), as row_key orders them; in one launch as two tagged words.
struct LookupSlot {
  uint64_t r, row;
};
constexpr size_t kLookupHeaderBytes = 256;  // in front of them, unused: part of the size that callers hold

inline int scan_blocks(long N, int waves, int most) {
  const long g = (N + waves - 1) / waves;
  return (int)(g < most ? g : most);
}
// the size that callers hold: 8 bytes for every four rows, up to 4096 times; sixteen for every eight need no more
inline size_t lookup_scratch_bytes(long N) {
  return kLookupHeaderBytes + align_up((size_t)scan_blocks(N > 0 ? N : 1, kWavesTwo, kMaxScanBlocksTwo) * 8, 256);
}
static_assert(kMaxScanBlocks * sizeof(LookupSlot) <= (size_t)kMaxScanBlocksTwo * 8 && kWaves >= 2 * kWavesTwo, "the slots' place in the workspace");

// r and its row as one integer that orders by r and, between equal r (0 and -0 are equal), by the lower row; 0: no row
__device__ __forceinline__ uint64_t row_key(float r, uint32_t row) {
  const uint32_t u = __float_as_uint(r + 0.0f);
  return ((uint64_t)((u & 0x80000000u) ? ~u : (u | 0x80000000u)) << 32) | (uint32_t)~row;
}

__device__ __forceinline__ void write_result(chorus_lookup_result* out, uint64_t key, float qq, float tau) {
  const uint32_t ord = (uint32_t)(key >> 32);
  const float best = __uint_as_float((ord & 0x80000000u) ? (ord & 0x7fffffffu) : ~ord);
  const float nq = sqrtf(qq);
  float m = (nq > 0.f && best > -INFINITY) ? best / nq : -INFINITY;
  if (!(m == m)) m = -INFINITY;
  chorus_lookup_result res;
  res.index = m == -INFINITY ? 0 : (int32_t)~(uint32_t)key;  // every score -inf (zero-norm query or rows): like a first-maximum scan
  res.score = m;
  res.hit = m >= tau ? 1 : 0;
  *out = res;
}

// One wave per row: lanes stride over the row in float4, then a butterfly
// reduction. The order of additions depends only on d, never on the row index,
// so identical rows produce identical values. The scan compares r_j = <q, c_j> / |c_j|;
// the query norm is a positive constant for the whole scan and is applied once, at the
// end (score_j = r_j / |q|), which keeps this HBM-bound loop at 8 FMAs per
// 16 bytes read. |q|^2 falls out of the query values every wave loads anyway (the same
// additions in the same order in every wave); what collects sums it as a row of its own.
__device__ __forceinline__ void scan_rows(const float* __restrict__ cache, const float* __restrict__ query, long N, int d, int lane,
                                          long row, long stride, uint64_t& best, float& qq) {
  const float4* q4 = reinterpret_cast<const float4*>(query);
  const int n4 = d >> 2;
  for (; row < N; row += stride) {
    float dot, cc;
    fp32_row_products(reinterpret_cast<const float4*>(cache + row * (long)d), q4, n4, lane, dot, cc, qq);
    const uint64_t k = row_key(row_ratio(dot, cc), (uint32_t)row);
    best = k > best ? k : best;
  }
}
__device__ __forceinline__ float query_norm2(const float* __restrict__ query, int d, int lane) {
  const float4* q4 = reinterpret_cast<const float4*>(query);
  float dot, cc, qq;
  fp32_row_products(q4, q4, d >> 2, lane, dot, cc, qq);
  return qq;
}
// the best of the workgroup's waves, in every thread
template <int WAVES>
__device__ __forceinline__ uint64_t meet(uint64_t best) {
  __shared__ uint64_t sk[WAVES];
  if ((threadIdx.x & 63) == 0) sk[threadIdx.x >> 6] = best;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < WAVES; ++w) best = sk[w] > best ? sk[w] : best;
  return best;
}

// In one launch: the last workgroup scans nothing, it collects what the others leave, divides by |q| and tests the threshold. A
// second launch for that took 2.3 us (1000 x 768, the call 8.8 us, now 5.6) to 3.9 (4096 x 4096 from HBM 17.3, now 14.8; 1024 x
// 4096 8.9 and 7.5). What is behind the scan is a chain of latencies, so the values that meet are one integer each, whose
// maximum over a wave stays in registers (compared as pairs through the LDS crossbar the calls took 16.0 and 9.0 us).
__global__ __launch_bounds__(kWaves * 64) void lookup_scan_kernel(const float* __restrict__ cache, const float* __restrict__ query,
                                                             long N, int d, float tau, uint64_t number, int rounds,
                                                             LookupSlot* slots, chorus_lookup_result* __restrict__ out) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int last = gridDim.x - 1;  // scans nothing
  const uint32_t tag_r = (uint32_t)(number >> 32), tag_i = (uint32_t)number;
  uint64_t best = 0;
  float qq = 0.f;
  if ((int)blockIdx.x != last) {
    scan_rows(cache, query, N, d, lane, (long)blockIdx.x * kWaves + wave, (long)last * kWaves, best, qq);
    best = meet<kWaves>(best);
    if (tid == 0) {
      leave_word(&slots[blockIdx.x].r, tag_r, (uint32_t)(best >> 32));
      leave_word(&slots[blockIdx.x].row, tag_i, (uint32_t)best);
    }
    return;
  }
  constexpr int R = kMaxScanBlocks / (kWaves * 64);  // slots per thread
  qq = query_norm2(query, d, lane);
  bool here = rounds >= 0;
  if (here) {
    uint64_t wr[R], wi[R];
    for (int round = 0;; ++round) {
      here = true;
#pragma unroll
      for (int u = 0; u < R; ++u) {
        const int j = tid + u * (kWaves * 64);
        wr[u] = j < last ? read_word(&slots[j].r) : (uint64_t)tag_r << 32;
        wi[u] = j < last ? read_word(&slots[j].row) : (uint64_t)tag_i << 32;
      }
#pragma unroll
      for (int u = 0; u < R; ++u) here = here && (uint32_t)(wr[u] >> 32) == tag_r && (uint32_t)(wi[u] >> 32) == tag_i;
      if (__all(here) || round == rounds) break;
      __builtin_amdgcn_s_sleep(1);
    }
    here = __syncthreads_and(here);
    if (here) {
#pragma unroll
      for (int u = 0; u < R; ++u) {
        const uint64_t k = tid + u * (kWaves * 64) < last ? (wr[u] << 32) | (uint32_t)wi[u] : 0;
        best = k > best ? k : best;
      }
      best = wave_max_key(best);
    }
  }
  if (!here) scan_rows(cache, query, N, d, lane, wave, kWaves, best, qq);  // alone
  best = meet<kWaves>(best);
  if (tid == 0) write_result(out, best, qq, tau);
}

// In two launches, where nothing waits.
__global__ __launch_bounds__(kWavesTwo * 64) void lookup_rows_kernel(const float* __restrict__ cache,
                                                                     const float* __restrict__ query, long N, int d,
                                                                     uint64_t* __restrict__ keys) {
  uint64_t best = 0;
  float qq;
  scan_rows(cache, query, N, d, threadIdx.x & 63, (long)blockIdx.x * kWavesTwo + (threadIdx.x >> 6), (long)gridDim.x * kWavesTwo, best, qq);
  best = meet<kWavesTwo>(best);
  if (threadIdx.x == 0) keys[blockIdx.x] = best;
}
__global__ __launch_bounds__(kWaves * 64) void lookup_collect_kernel(const uint64_t* __restrict__ keys, int n,
                                                                     const float* __restrict__ query, int d, float tau,
                                                                     chorus_lookup_result* __restrict__ out) {
  uint64_t best = 0;
#pragma unroll
  for (int u = 0; u < kMaxScanBlocksTwo / (kWaves * 64); ++u) {
    const int j = threadIdx.x + u * (kWaves * 64);
    const uint64_t k = j < n ? keys[j] : 0;
    best = k > best ? k : best;
  }
  const float qq = query_norm2(query, d, threadIdx.x & 63);
  best = meet<kWaves>(wave_max_key(best));
  if (threadIdx.x == 0) write_result(out, best, qq, tau);
}

// an empty cache
__global__ void lookup_none_kernel(chorus_lookup_result* __restrict__ out) {
  chorus_lookup_result r;
  r.index = -1;
  r.score = -INFINITY;
  r.hit = 0;
  *out = r;
}

// Is the stream being captured? Where that cannot be told it is not, and the launch says what is wrong.
bool is_captured(hipStream_t s) {
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &status) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return status != hipStreamCaptureStatusNone;
}

// `scratch` holds the header and the slots (lookup_scratch_bytes(N)). One launch, but two for large caches and under capture:
// a captured launch has the same number every time it is replayed and could not tell what an earlier replay left.
int32_t launch_lookup(const float* cache_emb, long N, int d, const float* query, float tau, chorus_lookup_result* out,
                      void* scratch, int rounds, hipStream_t s) {
  uint8_t* slots = reinterpret_cast<uint8_t*>(scratch) + kLookupHeaderBytes;
  if (N <= 0) {
    hipLaunchKernelGGL(lookup_none_kernel, dim3(1), dim3(1), 0, s, out);
  } else if ((size_t)N * (size_t)d <= kMaxWaitValues && !is_captured(s)) {
    hipLaunchKernelGGL(lookup_scan_kernel, dim3((unsigned)scan_blocks(N, kWaves, kMaxScanBlocks) + 1), dim3(kWaves * 64), 0, s, cache_emb,
                       query, N, d, tau, launch_number(), rounds, reinterpret_cast<LookupSlot*>(slots), out);
  } else {
    const int n = scan_blocks(N, kWavesTwo, kMaxScanBlocksTwo);
    uint64_t* keys = reinterpret_cast<uint64_t*>(slots);
    hipLaunchKernelGGL(lookup_rows_kernel, dim3((unsigned)n), dim3(kWavesTwo * 64), 0, s, cache_emb, query, N, d, keys);
    CHORUS_LAUNCH_CHECK();
    hipLaunchKernelGGL(lookup_collect_kernel, dim3(1), dim3(kWaves * 64), 0, s, keys, n, query, d, tau, out);
  }
  CHORUS_LAUNCH_CHECK();
  return CHORUS_OK;
}

// Scratch of the entry point that allocates nothing: the header and the largest number of slots a scan uses
// (the scan caps its grid, so this serves every N). One copy per GPU, resident until the process ends.
constexpr size_t kStaticScratchBytes = kLookupHeaderBytes + (size_t)kMaxScanBlocksTwo * 8;
static __device__ __align__(256) uint8_t scratch[kStaticScratchBytes];

// Device address of `scratch` on each GPU. In host code the array's name is only a handle for
// hipGetSymbolAddress; the address it returns for the current device is what kernels are given.
constexpr int kMaxDevices = 64;
std::atomic<void*> g_scratch_ptr[kMaxDevices];

int32_t static_scratch(void** ptr) {
  int dev = -1;
  CHORUS_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return CHORUS_E_SHAPE;
  void* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (!p) {  // first call on this device (racing first calls resolve the same address)
    CHORUS_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return CHORUS_E_HIP;
    g_scratch_ptr[dev].store(p, std::memory_order_release);
  }
  *ptr = p;
  return CHORUS_OK;
}

int32_t check_lookup_args(const float* cache_emb, int64_t N, int32_t d, const float* query, const chorus_lookup_result* out) {
  if (N < 0 || d <= 0 || !out || !query) return CHORUS_E_ARG;
  if (N > 0 && !cache_emb) return CHORUS_E_ARG;
  if ((d & 3) != 0) return CHORUS_E_SHAPE;
  if (N > 0x7fffffffLL - 1) return CHORUS_E_SHAPE;  // the result index is an int32
  if (!aligned16(cache_emb) || !aligned16(query)) return CHORUS_E_ARG;
  return CHORUS_OK;
}

}  // namespace
}  // namespace chorus

using namespace chorus;

extern "C" {

int32_t chorus_version(void) { return 100; }
int32_t chorus_last_hip_error(void) { return g_last_hip_error; }

size_t chorus_cache_lookup_workspace_bytes(int64_t N) { return lookup_scratch_bytes(N > 0 ? (long)N : 0); }

int32_t chorus_cache_lookup(const float* cache_emb, int64_t N, int32_t d, const float* query, float tau,
                            chorus_lookup_result* out, void* ws, size_t ws_bytes, void* stream) {
  CHK_STATUS(check_lookup_args(cache_emb, N, d, query, out));
  if (!ws || ws_bytes < chorus_cache_lookup_workspace_bytes(N)) return CHORUS_E_WORKSPACE;
  if (!aligned16(ws)) return CHORUS_E_ARG;
  return launch_lookup(cache_emb, (long)N, d, query, tau, out, ws, kWaitRounds, (hipStream_t)stream);
}

int32_t chorus_cache_lookup_wait(const float* cache_emb, int64_t N, int32_t d, const float* query, float tau, int32_t rounds,
                                 chorus_lookup_result* out, void* ws, size_t ws_bytes, void* stream) {
  CHK_STATUS(check_lookup_args(cache_emb, N, d, query, out));
  if (rounds < -1 || rounds > kWaitRounds) return CHORUS_E_ARG;
  if (!ws || ws_bytes < chorus_cache_lookup_workspace_bytes(N)) return CHORUS_E_WORKSPACE;
  if (!aligned16(ws)) return CHORUS_E_ARG;
  return launch_lookup(cache_emb, (long)N, d, query, tau, out, ws, rounds, (hipStream_t)stream);
}

int32_t chorus_cache_lookup_static(const float* cache_emb, int64_t N, int32_t d, const float* query, float tau,
                                   chorus_lookup_result* out, void* stream) {
  CHK_STATUS(check_lookup_args(cache_emb, N, d, query, out));
  if (lookup_scratch_bytes(N > 0 ? (long)N : 0) > kStaticScratchBytes) return CHORUS_E_SHAPE;
  void* ptr = nullptr;
  CHK_STATUS(static_scratch(&ptr));
  // nothing in the scratch has to start at zero: what an earlier call left does not carry this launch's number, and in two
  // launches the first one writes all that the second one reads
  return launch_lookup(cache_emb, (long)N, d, query, tau, out, ptr, kWaitRounds, (hipStream_t)stream);
}

}  // extern "C"
