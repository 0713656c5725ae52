// Workgroups of one launch that leave results for whichever of them ends last, which goes on with them in place of a second
// launch (2 to 3 us on the device and as much on the host; what replaces it is two trips to memory).
//
// Nobody waits for anybody and nothing has to be cleared first.  Every workgroup stores its results, and when they have
// arrived at memory a word with the launch's tag; when that has arrived too it looks at the words of all.  Whoever finds them
// complete goes on: the last to arrive does, and perhaps another that arrived at the same time.  Where what follows may be done
// twice, with the same results to the same places and nothing else in between, both do (hand_over: each workgroup leaves its words once);
// where more is left for others afterwards one of them claims it (all_arrived, claimed).  The words are taken away again, so that a
// captured launch, whose tag is the same every time, finds none of its own from the replay before.  A tag
// is 62 bits mixed from a count of the process's launches, so that whatever a workspace holds from before is not taken for one.
//
// All of it goes past the caches of the XCDs (relaxed atomics at device scope: each of the eight has an L2 of its own), so that
// no cache has to be written back or invalidated.
#pragma once
#include <atomic>
#include <chrono>
#include "common.h"

namespace tslt {

struct Tag { uint32_t lo, hi; };       // neither is ever 0

inline Tag next_tag() {
  static std::atomic<uint64_t> count{uint64_t(std::chrono::steady_clock::now().time_since_epoch().count())};
  uint64_t x = count.fetch_add(1, std::memory_order_relaxed) * 0x9E3779B97F4A7C15ull;      // (a permutation, and so is the rest)
  x ^= x >> 32;
  x *= 0xD6E8FEB86659FD93ull;
  x ^= x >> 32;
  return Tag{uint32_t(x) | 1u, uint32_t(x >> 32) | 1u};
}

__device__ __forceinline__ void store_through(uint64_t* p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t load_through(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// This wave's stores have arrived at memory (and what follows in the program is not moved before that).
__device__ __forceinline__ void stores_arrived() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ uint64_t tag_word(Tag t) { return uint64_t(t.hi) << 32 | t.lo; }

// What lanes of this wave have written to LDS is there for its other lanes.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// All threads of a workgroup, one of `n` (64 at most) that share something: everything that any of its waves stored with
// store_through is at memory, it says so in words[i], and returns whether all the others have too.  `told` is a word of LDS.  What they
// have left may be asked for then; which workgroup goes on with it claimed() says.
__device__ __forceinline__ bool all_arrived(uint64_t* words, int i, int n, Tag tag, int& told) {
  stores_arrived();
  __syncthreads();
  if (wave_id() == 0) {
    const int lane = lane_id();
    if (lane == 0) store_through(&words[i], tag_word(tag));
    stores_arrived();
    const bool missing = lane < n && load_through(&words[lane]) != tag_word(tag);
    if (ballot(missing) != 0) { if (lane == 0) told = 0; }
    else if (lane == 0) told = 1;
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(told) != 0;
}

// One wave of a workgroup that has found all words: whether it is the one that goes on; it takes them away.
__device__ __forceinline__ bool claimed(uint64_t* words, int n, Tag tag) {
  const int lane = lane_id();
  uint64_t word = tag_word(tag);
  bool mine = false;
  if (lane == 0) mine = __hip_atomic_compare_exchange_strong(&words[0], &word, 0ull, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  mine = ballot(mine) != 0;
  if (mine && lane > 0 && lane < n) store_through(&words[lane], 0);
  return mine;
}

// The same where what is left fits beside the tag, two words of 32 bits for each of `n`: one wave leaves its own, and returns
// whether it has found those of all, which are then in LDS at a and c.  (It does not wait for what the workgroup stored before:
// where whoever goes on writes to the same places, the caller does, stores_arrived.)
__device__ __forceinline__ bool hand_over(uint64_t* words, int i, int n, uint32_t mine_a, uint32_t mine_c, Tag tag, int* a, int* c) {
  const int lane = lane_id();
  if (lane == 0) {
    store_through(&words[2 * i], uint64_t(tag.lo) << 32 | mine_a);
    store_through(&words[2 * i + 1], uint64_t(tag.hi) << 32 | mine_c);
  }
  stores_arrived();
  for (int k0 = 0; k0 < n; k0 += 256) {
    uint64_t x[4], y[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (k0 + 64 * u < n) {
        const int k = k0 + 64 * u + lane < n ? k0 + 64 * u + lane : n - 1;
        x[u] = load_through(&words[2 * k]);
        y[u] = load_through(&words[2 * k + 1]);
      }
    bool missing = false;
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (k0 + 64 * u < n) {
        missing |= uint32_t(x[u] >> 32) != tag.lo || uint32_t(y[u] >> 32) != tag.hi;
        if (k0 + 64 * u + lane < n) {
          a[k0 + 64 * u + lane] = int(uint32_t(x[u]));
          c[k0 + 64 * u + lane] = int(uint32_t(y[u]));
        }
      }
    if (ballot(missing) != 0) return false;
  }
  for (int k = lane; k < 2 * n; k += 64) store_through(&words[k], 0);
  wave_sync();
  return true;
}

}  // namespace tslt
