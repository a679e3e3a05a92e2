// Results that the workgroups of one launch leave for its last workgroup, which picks among them: a second launch for that
// took 2.3 to 3.9 us, and a counter of arrivals needs memory that starts at zero, which a caller's workspace does not.
//
// Every word that is left carries 32 bits of a number that only this launch has; a word that does not is not there yet,
// whatever the workspace held before. Words are relaxed agent-scope atomics, which pass by the L2s of the XCDs, and carry
// their own proof of arrival, so that no fence (which writes an L2 back) stands between them. The last workgroup waits
// only for workgroups in front of it, which were dispatched before it or run elsewhere on the chip and wait for nothing;
// the wait is bounded all the same (two calls that share one workspace against the rules would wait for ever), and a
// launch that gives up makes its result alone. The number is the launch's own, so a launch that is captured, and would
// have the same one at every replay, must not be of this kind.
#pragma once
#include <atomic>
#include <chrono>

#include "common.h"

namespace chorus {

// never the same twice in a process, and unlike what memory may hold (a counter mixed by the steps of SplitMix64: Steele, Lea,
// Flood, "Fast splittable pseudorandom number generators", 2014); both halves are used and neither is zero
inline uint64_t launch_number() {
  static std::atomic<uint64_t> count{(uint64_t)std::chrono::steady_clock::now().time_since_epoch().count() * 0x9e3779b97f4a7c15ull};
  uint64_t z = count.fetch_add(0x9e3779b97f4a7c15ull, std::memory_order_relaxed);
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  z ^= z >> 31;
  return z | 0x0000000100000001ull;
}

__device__ __forceinline__ void leave_word(uint64_t* at, uint32_t tag, uint32_t value) {
  __hip_atomic_store(at, ((uint64_t)tag << 32) | value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t read_word(const uint64_t* at) {
  return __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Looks before the wait is given up. A look takes 0.22 us (512 slots) to 0.43 (2048) on an idle chip, so this is 57 to 112 ms:
// 20 times the scan of the largest cache, and long enough for workgroups that stand behind another stream's kernels.
constexpr int kWaitRounds = 1 << 18;

}  // namespace chorus
