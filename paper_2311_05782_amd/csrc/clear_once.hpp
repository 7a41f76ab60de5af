// Words that one wave of a launch clears for all of its waves, in the place of a launch in front.
//
// `word` holds, for a launch with the even number `done`, at least done - 1 from when a wave has taken the clearing upon itself and
// at least done from when it has finished; launches that share a word follow each other and have larger and larger numbers.
// Workgroup 0 takes it at once, and whoever has something to write and finds it not taken takes it then: a wave waits
// only for one that is running, so that every wait ends in whatever order the workgroups start, and however many of other
// launches, waiting as well, fill the chip.
#pragma once
#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#endif
#include <stdint.h>

namespace fi {

// By a whole wave, as all of these: whether it is the one to clear.
__device__ __forceinline__ bool take_clearing(uint32_t* word, uint32_t done, uint32_t lane) {
  uint32_t before = 0;
  if (lane == 0) before = __hip_atomic_fetch_max(word, done - 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)before) < done - 1u;
}

// By the wave that is to, or by its whole workgroup with a barrier in front of the second.
__device__ __forceinline__ void clear_words(uint32_t* words, uint32_t n, uint32_t lane, uint32_t lanes) {
#pragma unroll 1
  for (uint32_t i = lane; i < n; i += lanes) __hip_atomic_store(words + i, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __builtin_amdgcn_s_waitcnt(0x0F70);                     // vmcnt(0)
}
__device__ __forceinline__ void clearing_done(uint32_t* word, uint32_t done, uint32_t lane) {
  if (lane == 0) __hip_atomic_fetch_max(word, done, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// In front of every write into the words.  seen: what this wave has read of `word` before, or 0.
__device__ __forceinline__ void cleared(uint32_t* words, uint32_t n, uint32_t* word, uint32_t done, uint32_t& seen, uint32_t lane, uint32_t lanes) {
  while ((uint32_t)__builtin_amdgcn_readfirstlane((int)seen) < done) {
    seen = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (__builtin_expect((uint32_t)__builtin_amdgcn_readfirstlane((int)seen) < done - 1u, 0)) {
      if (take_clearing(word, done, lane)) {
        clear_words(words, n, lane, lanes);
        clearing_done(word, done, lane);
        seen = done;
        break;
      }
    }
    __builtin_amdgcn_s_sleep(1);
  }
  asm volatile("" ::: "memory");                          // nothing is read that another wave has written
}

}  // namespace fi
