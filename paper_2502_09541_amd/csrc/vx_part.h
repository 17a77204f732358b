// Stable multisplit: partition ids, counts, stable scatter.
//
// part_count counts the rows of every partition in one pass over the keys and turns the counts into
// each partition's first position.  part_sweep then writes the rows to their places in one pass:
// its workgroups take tiles of consecutive rows in order, rank a tile's rows by partition in input
// order (ballots), find where each partition's rows go by look-back over the tiles before, sort the
// tile by partition in LDS and write it in that order, so that a partition's rows of a tile are one
// run of consecutive addresses.  Payload columns follow the keys through the same LDS buffer.
#pragma once

#include "vx_internal.h"

namespace vx {

constexpr uint32_t kMaxParts = 1024;

enum PartFn : uint32_t {
  kPartHash = 0,      // top log2 P bits of the MurmurHash3 64-bit finalizer
  kPartBits = 1,      // raw key bits [shift, shift + log2 P)
  kPartRange = 2      // number of splitters <= key
};

struct PartSpec {
  uint32_t fn;
  uint32_t n_parts;
  uint32_t log2p;
  uint32_t shift;
  uint32_t n_split;
  const long long* splitters;   // device, ascending
};

struct PartIO {
  const void* key;               // keys of this launch (row 0 = first row)
  uint32_t key_size;
  uint32_t n_pay;
  const void* pay[4];
  uint32_t pay_size[4];
  uint64_t n;
  void* out_key;                 // clustered outputs (device or host-mapped); null for a count
  void* out_pay[4];
  uint64_t out_base;             // row offset added to every output position
};

// Partition id of key k: hash, raw bits, or the count of splitters <= k (split[] ascending,
// ps.n_split entries, usually staged in LDS by the caller).
__device__ __forceinline__ unsigned long long fmix64(unsigned long long h) {
  h ^= h >> 33;
  h *= 0xff51afd7ed558ccdull;
  h ^= h >> 33;
  h *= 0xc4ceb9fe1a85ec53ull;
  h ^= h >> 33;
  return h;
}

// The ids of N keys at once: the searches of the range splitters run side by side.
template <uint32_t N, typename K>
__device__ __forceinline__ void part_ids(const PartSpec& ps, const K (&k)[N], const long long* split, uint32_t (&id)[N]) {
  if (ps.fn == kPartRange) {
#pragma unroll
    for (uint32_t j = 0; j < N; ++j) id[j] = 0;
    for (uint32_t step = kMaxParts >> 1; step; step >>= 1) {
      if (step > ps.n_split) continue;   // uniform
#pragma unroll
      for (uint32_t j = 0; j < N; ++j)
        if (id[j] + step <= ps.n_split && split[id[j] + step - 1] <= (long long)k[j]) id[j] += step;
    }
    return;
  }
  if (ps.fn == kPartHash) {
#pragma unroll
    for (uint32_t j = 0; j < N; ++j)
      id[j] = ps.log2p ? (uint32_t)(fmix64((unsigned long long)(long long)k[j]) >> (64 - ps.log2p)) : 0u;
    return;
  }
#pragma unroll
  for (uint32_t j = 0; j < N; ++j)
    id[j] = (uint32_t)((unsigned long long)(long long)k[j] >> ps.shift) & (ps.n_parts - 1);
}

__device__ __forceinline__ uint32_t part_of(const PartSpec& ps, long long k, const long long* split) {
  if (ps.fn == kPartHash) {
    return ps.log2p ? (uint32_t)(fmix64((unsigned long long)k) >> (64 - ps.log2p)) : 0u;
  }
  if (ps.fn == kPartBits) {
    return (uint32_t)(((unsigned long long)k >> ps.shift) & (unsigned long long)(ps.n_parts - 1));
  }
  uint32_t lo = 0, hi = ps.n_split;
  while (lo < hi) {
    uint32_t mid = (lo + hi) >> 1;
    if (split[mid] <= k) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

constexpr uint32_t kMaxSumSlots = 64;

// Rows of one launch over device-resident columns: the look-back words (8 bytes per partition and tile)
// take 32 MiB for 1024 partitions, whatever the column's length.
constexpr uint64_t kPartLaunchRows = 1ull << 25;

// Device scratch of part_count and part_sweep over at most `rows` rows per launch, and of part_count
// alone (sweep == false: no look-back words).
uint64_t part_work_bytes(uint32_t n_parts, uint64_t rows, bool sweep = true);

// Count the rows of every partition.  totals (n_parts u64) receives the counts, or has them added
// when `accumulate`; base (n_parts + 1) the exclusive prefix of totals and its sum; host_totals
// (optional, host-mapped) a copy of totals.  sums (optional): for partitions with sum_slot[p] >= 0
// (a device int array of n_parts entries, slots < kMaxSumSlots), the row count and the SUM of
// payload 0 are added to sums[2*slot] and sums[2*slot+1].  With `sweep` it leaves `work` ready for one
// part_sweep over the same rows.
vx_status part_count(vx_ctx* ctx, const PartSpec& ps, const PartIO& io, uint8_t* work, unsigned long long* totals,
                     bool accumulate, unsigned long long* base, unsigned long long* host_totals, const int* sum_slot,
                     unsigned long long* sums, hipStream_t s, bool sweep = true);
// Write the rows of io to their places: partition p's from out_base + base[p] on, in input order.
// next (optional, n_parts; may be base) receives the position after each partition's rows, the
// base of the chunk that follows.  `work` comes from part_count over the same rows, or was made
// ready by part_ready.
vx_status part_sweep(vx_ctx* ctx, const PartSpec& ps, const PartIO& io, uint8_t* work, const unsigned long long* base,
                     unsigned long long* next, hipStream_t s);
vx_status part_ready(const PartSpec& ps, uint64_t rows, uint8_t* work, hipStream_t s);

// LSD radix sort of `rows` int64 keys (signed order) that differ in their low 8 * passes bits only,
// from a, with b as the second buffer; *sorted receives
// the one that holds the result.  scratch holds sort_scratch_bytes(rows).
uint64_t sort_scratch_bytes(uint64_t rows);
vx_status sort_keys_i64(vx_ctx* ctx, long long* a, long long* b, uint64_t rows, uint32_t passes, uint8_t* scratch,
                        long long** sorted, hipStream_t s);

}  // namespace vx
