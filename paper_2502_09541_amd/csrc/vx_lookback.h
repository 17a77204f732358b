// Decoupled look-back between the workgroups of one launch (Merrill and Garland, "Single-pass parallel
// prefix scan with decoupled look-back", 2016): each tile finds the running total of the tiles
// before it while they run.
#pragma once

#include <cstdlib>

#include "vx_internal.h"

namespace vx {

// A look-back word: a tag in the top byte (2 * pass + 1: the tile's own count; 2 * pass + 2: the
// position after this tile) and the value below.  Tags differ from pass to pass, so the passes of
// one sort share words cleared once.  A word is written and read whole (64 bits, device scope), and
// nothing else passes between workgroups through it, so no fence is needed.
constexpr uint32_t kTagShift = 56;
constexpr unsigned long long kTagValue = (1ull << kTagShift) - 1;
constexpr uint32_t kLookWindow = 8;        // tiles read ahead in one look-back step

// Where a workgroup whose wait does not end says so (a host-mapped word), and after how many polls: seconds,
// never in a sound run.  VX_LOOK_POLLS lowers the limit, so that tests reach it (0: no tile waits at all).
struct LookLimit {
  uint32_t* stall;
  uint32_t polls;
};
inline LookLimit look_limit(const vx_ctx* ctx) {
  const char* e = getenv("VX_LOOK_POLLS");
  return LookLimit{stall_word(ctx), e ? (uint32_t)strtoul(e, nullptr, 10) : 1u << 22};
}

// Reads the limit where a kernel starts, beside its other arguments: read in look_back, a digit pass over
// 16.0 M int64 keys took 67.1 us instead of 66.5.
__device__ __forceinline__ void look_ready(LookLimit& limit) { asm volatile("" : "+s"(limit.polls)); }

__device__ __forceinline__ unsigned long long look_load(const unsigned long long* w) {
  return __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void look_store(unsigned long long* w, uint32_t tag, unsigned long long v) {
  __hip_atomic_store(w, ((unsigned long long)tag << kTagShift) | v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Position of tile t's first element of a group: the counts of the tiles before t, back to the nearest
// one whose running position is known (tile 0 starts from the group's base).  The group's words are
// words[t * stride].  Tiles are taken in ticket order, so every tile waited for is running or done
// and publishes its count before it waits itself: the wait ends.  It is bounded all the same: a
// workgroup that gives up sets the stall word, by which the call fails, and returns the part it has
// added up, at most the true position.
__device__ __forceinline__ unsigned long long look_back(const unsigned long long* words, uint32_t stride, uint64_t t,
                                                        uint32_t pass, LookLimit limit) {
  const uint32_t own = 2 * pass + 1, known = 2 * pass + 2;
  unsigned long long sum = 0;
  int64_t look = (int64_t)t - 1;
  uint32_t waits = 0;   // polls that found nothing new
  auto give_up = [&]() { __hip_atomic_store(limit.stall, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM); };
  // the limit is tested outside the loop and where a poll found nothing only: tested on each poll, a sweep of
  // 16.0 M rows of 16 bytes into 256 partitions took 140.8 us instead of 139.0
  if (limit.polls == 0) {
    give_up();
    return 0;
  }
  for (;;) {
    unsigned long long w[kLookWindow];
#pragma unroll
    for (uint32_t i = 0; i < kLookWindow; ++i) {
      const int64_t at = look - (int64_t)i;
      w[i] = look_load(words + (uint64_t)(at > 0 ? at : 0) * stride);
    }
    uint32_t took = 0;
    bool done = false;
#pragma unroll
    for (uint32_t i = 0; i < kLookWindow; ++i) {
      const uint32_t tag = (uint32_t)(w[i] >> kTagShift);
      if (!done && took == i && (tag == own || tag == known)) {
        sum += w[i] & kTagValue;
        took = i + 1;
        done = tag == known;    // tile 0 is always known, so nothing past it is taken
      }
    }
    if (done) return sum;
    look -= (int64_t)took;
    if (took == 0 && ++waits >= limit.polls) {
      give_up();
      return sum;
    }
    if (took == 0 && (waits & 4095u) == 4095u &&
        __hip_atomic_load(limit.stall, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) != 0)
      return sum;   // another gave up
  }
}

}  // namespace vx
