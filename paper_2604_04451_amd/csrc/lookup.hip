// Stage-1 retrieval: top-1 cosine similarity over the prompt-embedding cache
// (Sec. 3.1 "Full Reuse"). HBM-bound: the [N, d] fp32 cache is streamed once.
#include "chorus_ops.h"
#include "common.h"
#include "lookup_row.h"
#include "tagged.h"

namespace chorus {

thread_local int32_t g_last_hip_error = 0;

namespace {

constexpr int kWaves = 8;            // waves per workgroup of the scan, one cache row per wave at a time
constexpr int kMaxScanBlocks = 2048; // beyond this many workgroups a wave walks several rows

// What one workgroup of the scan leaves behind (tagged words): the best r_j = <q, c_j> / |c_j| among its rows and that row
// (the lowest one among equal values), as row_key orders them. In front of them the number of a launch that gave its wait up.
struct LookupSlot {
  uint64_t r, row;
};
constexpr size_t kLookupHeaderBytes = 256;

inline long scan_blocks(long N) {
  long g = (N + kWaves - 1) / kWaves;
  return g < kMaxScanBlocks ? g : kMaxScanBlocks;
}
// The size that callers hold: 8 bytes for every four rows, up to 4096 times. Sixteen for every eight need no more.
inline size_t lookup_scratch_bytes(long N) {
  long g = (N + 3) / 4;
  g = g < 1 ? 1 : g < 4096 ? g : 4096;
  return kLookupHeaderBytes + align_up((size_t)g * 8, 256);
}
static_assert(kMaxScanBlocks * sizeof(LookupSlot) <= 4096 * 8, "the slots' place in the workspace");

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
// additions in the same order in every wave).
// The last workgroup scans nothing: it sums |q|^2 as a row of its own, collects what the others leave, divides by |q| and
// tests the threshold. A second launch for that took 2.3 us (1000 x 768, the call 8.8 us, now 5.6) to 3.9 (4096 x 4096 from
// HBM 17.3, now 14.8; 1024 x 4096 8.9 and 7.5). What is behind the scan is a chain of latencies, so the values that meet are
// one integer each, whose maximum over a wave stays in registers (compared as pairs through the LDS crossbar the calls took
// 16.0 and 9.0 us).
__global__ __launch_bounds__(kWaves * 64) void lookup_scan_kernel(const float* __restrict__ cache,
                                                                  const float* __restrict__ query, long N, int d, float tau,
                                                                  uint64_t number, int rounds, uint64_t* gave_up,
                                                                  LookupSlot* slots,
                                                                  chorus_lookup_result* __restrict__ out) {
  __shared__ uint64_t sk[kWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float4* q4 = reinterpret_cast<const float4*>(query);
  const int n4 = d >> 2;
  uint64_t best = 0;
  float qq = 0.f;
  auto take = [&](uint64_t k) { best = k > best ? k : best; };
  auto scan = [&](long row, long stride) {
    for (; row < N; row += stride) {
      float dot, cc;
      fp32_row_products(reinterpret_cast<const float4*>(cache + row * (long)d), q4, n4, lane, dot, cc, qq);
      take(row_key(row_ratio(dot, cc), (uint32_t)row));
    }
  };
  auto meet = [&]() {  // the best of the workgroup's waves, in every thread
    if (lane == 0) sk[wave] = best;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWaves; ++w) take(sk[w]);
  };
  const int last = gridDim.x - 1;  // scans nothing
  const uint32_t tag_r = (uint32_t)(number >> 32), tag_i = (uint32_t)number;
  if ((int)blockIdx.x != last) {
    scan((long)blockIdx.x * kWaves + wave, (long)last * kWaves);
    meet();
    if (tid == 0) {
      leave_word(&slots[blockIdx.x].r, tag_r, (uint32_t)(best >> 32));
      leave_word(&slots[blockIdx.x].row, tag_i, (uint32_t)best);
    }
    return;
  }
  constexpr int R = kMaxScanBlocks / (kWaves * 64);  // slots per thread
  {
    float dot, cc;
    fp32_row_products(q4, q4, n4, lane, dot, cc, qq);
  }
  bool here = rounds >= 0 && read_word(gave_up) != number;
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
        const int j = tid + u * (kWaves * 64);
        if (j >= last) continue;
        take((wr[u] << 32) | (uint32_t)wi[u]);
        leave_word(&slots[j].r, 0, 0);
        leave_word(&slots[j].row, 0, 0);
      }
      best = wave_max_key(best);
    } else if (tid == 0) {
      __hip_atomic_store(gave_up, number, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  if (!here) scan(wave, kWaves);  // alone
  meet();
  if (tid == 0) write_result(out, best, qq, tau);
}

// an empty cache
__global__ void lookup_none_kernel(chorus_lookup_result* __restrict__ out) {
  chorus_lookup_result r;
  r.index = -1;
  r.score = -INFINITY;
  r.hit = 0;
  *out = r;
}

// one launch; `scratch` holds the header and the slots (lookup_scratch_bytes(N))
int32_t launch_lookup(const float* cache_emb, long N, int d, const float* query, float tau, chorus_lookup_result* out,
                      void* scratch, int rounds, hipStream_t s) {
  if (N > 0)
    hipLaunchKernelGGL(lookup_scan_kernel, dim3((unsigned)scan_blocks(N) + 1), dim3(kWaves * 64), 0, s, cache_emb, query, N, d, tau,
                       launch_number(), rounds, reinterpret_cast<uint64_t*>(scratch),
                       reinterpret_cast<LookupSlot*>(reinterpret_cast<uint8_t*>(scratch) + kLookupHeaderBytes), out);
  else
    hipLaunchKernelGGL(lookup_none_kernel, dim3(1), dim3(1), 0, s, out);
  CHORUS_LAUNCH_CHECK();
  return CHORUS_OK;
}

// Scratch of the entry point that allocates nothing: the header and the largest number of slots a scan uses
// (the scan caps its grid, so this serves every N). One copy per GPU, resident until the process ends.
constexpr size_t kStaticScratchBytes = kLookupHeaderBytes + (size_t)kMaxScanBlocks * sizeof(LookupSlot);
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
  // nothing in the scratch has to start at zero: what an earlier call left does not carry this launch's number
  return launch_lookup(cache_emb, (long)N, d, query, tau, out, ptr, kWaitRounds, (hipStream_t)stream);
}

}  // extern "C"
