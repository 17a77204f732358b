// Out-of-core sort of a key column larger than the device budget (Sec. 6.1).
//
// Pass 1 (the paper's SortExKernel): the column streams through the chunk pipeline in runs of
// chunk_rows keys.  Each run is sorted on the GPU by an LSD radix sort of 8-bit digits (the sign
// bit flipped so that signed order comes out) whose stable passes sort tiles of 2048 to 16384 keys in LDS
// and write each digit's keys of a tile as one run, and is stored to pinned host scratch by a
// kernel on a second stream: kernel stores to mapped host memory run beside the host-to-device
// copies.
// Pass 2 (the paper's MergeExKernel): every run is cut at the same global ranks (multiples of the
// run length), found by binary search over the runs on the host.  Output range i then holds one
// sorted segment of every run.  Its segments are copied in, merged in a tree of pairwise
// merge-path launches (two device buffers used in turn), and the result is stored to its final
// place in the key column.  Up to three ranges are in flight: one copies in, one merges, one is
// stored.
#include <algorithm>
#include <cstring>
#include <thread>
#include <type_traits>
#include <vector>

#include "vx_device.h"
#include "vx_lookback.h"
#include "vx_part.h"
#include "vx_pipeline.h"

namespace vx {

namespace {

constexpr int kMergeThreads = 256;
constexpr int kMergeItems = 8;
constexpr int kMergeTile = kMergeThreads * kMergeItems;   // outputs per workgroup tile
// Merge workgroups per compute unit.  8 fit, but the merges share the memory with the copies and stores
// beside them, which bound the sort: pass 2 of 2^31 int64 keys in 32 runs takes 414 / 396 / 401 / 402 /
// 400 ms with 1 / 2 / 3 / 4 / 8.
constexpr int kMergeGroups = 2;

// One round of pairwise merges: pair p merges keys [a0, a1) and [a1, b1) of the source into [a0, b1) of
// the destination; its tiles are tile0[p] .. tile0[p + 1] of the launch.
struct MergeRound {
  static constexpr uint32_t kMax = 32;
  uint32_t n;
  uint32_t tile0[kMax + 1];
  uint64_t a0[kMax], a1[kMax], b1[kMax];
};

// Number of the first d outputs of merge(a, b) that come from a (ties: a first), known to lie in
// [lo, hi]; found by a wave, each step of which cuts the range by 64.
template <typename K>
__device__ __forceinline__ uint64_t merge_split(const K* a, uint64_t na, const K* b, uint64_t nb, uint64_t d, uint64_t lo,
                                                uint64_t hi) {
  const uint32_t l = threadIdx.x & 63;
  lo = d > nb && d - nb > lo ? d - nb : lo;
  hi = min(hi, d < na ? d : na);
  while (lo < hi) {   // alike in every lane
    const uint64_t step = (hi - lo + 63) / 64, mid = lo + l * step;
    const bool low = mid < hi && a[mid] <= b[d - 1 - mid];   // monotone: true, then false
    const uint32_t c = (uint32_t)__popcll(__ballot(low));
    if (c == 0) {
      hi = lo;
    } else {
      const uint64_t next = lo + c * step;
      lo += (c - 1) * step + 1;
      hi = min(hi, next);
    }
  }
  return lo;
}

// One round: a workgroup takes consecutive tiles of 2048 outputs.  Its first wave finds where the tile
// ends on the merge path, among the 2049 places past the tile's start, which is the end of the tile
// before (or searched for, once); the tile's inputs are staged in LDS with coalesced loads, every lane
// merges 8 outputs from LDS (its own start found by a binary search in LDS), and they go back through
// the same LDS into coalesced writes.  One launch per round, not two per pair: beside a store
// to host memory a launch takes the host 70 us.  16,777,213 int64 keys in 8 runs sort in 11.4 ms instead
// of 12.2.
template <typename K>
__global__ void __launch_bounds__(kMergeThreads) k_merge(const K* src, K* dst, MergeRound round) {
  __shared__ K buf[kMergeTile];   // a's keys, then b's; then the outputs
  __shared__ unsigned long long ends[2];
  const uint32_t tiles = round.tile0[round.n], per = (tiles + gridDim.x - 1) / gridDim.x;
  const uint32_t first = min(tiles, blockIdx.x * per), last = min(tiles, first + per);
  uint64_t s1 = 0;   // where the tile before ended
  for (uint32_t t = first; t < last; ++t) {
    uint32_t p = 0;
    while (t >= round.tile0[p + 1]) ++p;
    const uint64_t na = round.a1[p] - round.a0[p], nb = round.b1[p] - round.a1[p], n = na + nb;
    const K* a = src + round.a0[p];
    const K* b = src + round.a1[p];
    const uint64_t d0 = (uint64_t)(t - round.tile0[p]) * kMergeTile;
    const uint64_t d1 = d0 + kMergeTile < n ? d0 + kMergeTile : n;
    if (threadIdx.x < 64) {
      uint64_t x = s1;
      if (t == first || d0 == 0) x = merge_split(a, na, b, nb, d0, 0, d0);
      const uint64_t y = merge_split(a, na, b, nb, d1, x, x + (d1 - d0));
      if (threadIdx.x == 0) {
        ends[0] = x;
        ends[1] = y;
      }
    }
    __syncthreads();
    const uint64_t s0 = ends[0];
    s1 = ends[1];
    const uint64_t ia = s0, ib = d0 - s0;
    const uint32_t ma = (uint32_t)(s1 - s0), mb = (uint32_t)((d1 - s1) - ib);
    K* const sb = buf + ma;
    for (uint32_t k = threadIdx.x; k < ma; k += kMergeThreads) buf[k] = a[ia + k];
    for (uint32_t k = threadIdx.x; k < mb; k += kMergeThreads) sb[k] = b[ib + k];
    __syncthreads();
    const uint32_t m = ma + mb, t0 = min(threadIdx.x * kMergeItems, m);
    uint32_t lo = t0 > mb ? t0 - mb : 0, hi = t0 < ma ? t0 : ma;
    while (lo < hi) {
      const uint32_t mid = (lo + hi) >> 1;
      if (buf[mid] <= sb[t0 - 1 - mid]) lo = mid + 1;
      else hi = mid;
    }
    uint32_t i = lo, j = t0 - lo;
    K o[kMergeItems];
#pragma unroll
    for (uint32_t e = 0; e < kMergeItems; ++e) {
      const K x = buf[min(i, (uint32_t)kMergeTile - 1)], y = buf[min(ma + j, (uint32_t)kMergeTile - 1)];
      const bool take_a = j >= mb || (i < ma && x <= y);
      o[e] = take_a ? x : y;
      i += take_a;
      j += !take_a;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t e = 0; e < kMergeItems; ++e)
      if (t0 + e < m) buf[t0 + e] = o[e];
    __syncthreads();
    K* out = dst + round.a0[p] + d0;
    for (uint32_t k = threadIdx.x; k < m; k += kMergeThreads) out[k] = buf[k];
    __syncthreads();
  }
}

// dst[0, bytes) = src[0, bytes) with 16-byte vector stores (dst may be mapped host memory); both
// 16-byte aligned, bytes a multiple of 4.
__global__ void __launch_bounds__(256) k_store(const uint8_t* src, uint8_t* dst, uint64_t bytes) {
  const uint64_t n16 = bytes / 16;
  const uint4* s = (const uint4*)src;
  uint4* d = (uint4*)dst;
  for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n16; i += (uint64_t)gridDim.x * blockDim.x)
    d[i] = s[i];
  for (uint64_t i = n16 * 4 + blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < bytes / 4;
       i += (uint64_t)gridDim.x * blockDim.x)
    ((uint32_t*)dst)[i] = ((const uint32_t*)src)[i];
}

// The same for any 4-byte-aligned pointers, element by element.
__global__ void __launch_bounds__(256) k_store4(const uint32_t* src, uint32_t* dst, uint64_t words) {
  for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < words; i += (uint64_t)gridDim.x * blockDim.x)
    dst[i] = src[i];
}

// ---------------------------------------------------------------- LSD radix digit passes
//
// Each 8-bit digit pass reads every key once and writes it once: bytes in all, 16 per int64 key and
// pass plus 8 for the digit counts of the whole sort.  A pass is one launch (k_digit_sweep) whose
// workgroups take tiles of consecutive keys in order, by a ticket.  A tile ranks its keys by digit
// in input order, publishes its count of every digit, and finds where each digit's keys go by
// adding up the counts of the tiles before it, back to one whose running total is known
// (decoupled look-back: Merrill and Garland, "Single-pass parallel prefix scan with decoupled
// look-back", 2016; for radix sorting: Adinets and Merrill, "Onesweep", 2022).  The counts of every
// digit of the whole run, which give each digit's first position, come from one pass before
// (k_sweep_count, k_sweep_base).  A tile is sorted by digit in LDS and written in LDS order, so
// each digit's keys of a tile are one run of consecutive addresses (64 keys on average at 16384).
//
// 16.0 M int64 keys in one run: 576 us of kernels (k_sweep_count 40 us, 3.2 TB/s; a sweep 66.4 us,
// 3.9 TB/s read and written, against 4.8 TB/s of a large copy), where a histogram launch per
// pass, a three-launch column scan and a scatter took 1185 us (44 + 36 + 68 us a pass).  What bounds
// a sweep is the ranking: with 11 vector instructions per digit bit instead of 4 (same_id) it took
// 94 us.  The look-back is hidden behind other tiles' work: with windows of 4, 8, 16 and 32 tiles a sweep
// takes 66.8, 66.4, 67.6 and 74.0 us (tiles of 16384 keys).
constexpr uint32_t kDigitThreads = 1024;
constexpr uint32_t kDigitWaves = kDigitThreads / 64;
constexpr uint32_t kLocalSortMax = 8192;                        // runs sorted by one workgroup in LDS
constexpr uint32_t kCountThreads = 1024;
constexpr uint32_t kCountGroups = 256;                          // workgroups of k_sweep_count, at most

// byte `pass` of the key's order-preserving unsigned image (sign bit flipped)
__device__ __forceinline__ uint32_t digit_of(int32_t k, uint32_t pass) {
  return (((uint32_t)k ^ 0x80000000u) >> (8 * pass)) & 255u;
}
__device__ __forceinline__ uint32_t digit_of(int64_t k, uint32_t pass) {
  const uint32_t w = pass < 4 ? (uint32_t)(uint64_t)k : (uint32_t)((uint64_t)k >> 32) ^ 0x80000000u;
  return (w >> (8 * (pass & 3))) & 255u;
}

// this lane's keys, 64 apart from `first` on (zero past n); a full tile loads unconditionally
template <bool FULL, typename K, uint32_t ITEMS>
__device__ __forceinline__ void digit_load(const K* in, uint64_t n, uint64_t first, K (&k)[ITEMS]) {
  if (FULL) {
#pragma unroll
    for (uint32_t j = 0; j < ITEMS; ++j) k[j] = __builtin_nontemporal_load(in + first + j * 64);
  } else {
#pragma unroll
    for (uint32_t j = 0; j < ITEMS; ++j) k[j] = first + j * 64 < n ? in[first + j * 64] : K(0);
  }
}

// rank[j] = number of this wave's earlier keys with key j's digit; cnt[d] ends as the wave's
// count of digit d (cnt is the wave's own row, zeroed by the caller)
template <bool FULL, typename K, uint32_t ITEMS>
__device__ __forceinline__ void digit_rank(const K (&k)[ITEMS], uint64_t n, uint64_t first, uint32_t pass,
                                           uint32_t* cnt, uint32_t (&rank)[ITEMS]) {
  const uint32_t lane = threadIdx.x & 63;
  const unsigned long long lower = (1ull << lane) - 1;
#pragma unroll
  for (uint32_t j = 0; j < ITEMS; ++j) {
    const bool valid = FULL || first + j * 64 < n;
    const uint32_t d = digit_of(k[j], pass);
    const unsigned long long peers = same_id(d, 8, FULL ? ~0ull : __ballot(valid));
    const uint32_t below = (uint32_t)__popcll(peers & lower);
    const uint32_t c = valid ? cnt[d] : 0u;
    rank[j] = c + below;
    // every lane has read cnt[] before the group's first lane advances it
    __builtin_amdgcn_wave_barrier();
    if (valid && below == 0) cnt[d] = c + (uint32_t)__popcll(peers);
    __builtin_amdgcn_wave_barrier();
  }
}

// For threads 0..255 (thread d: digit d), from the waves' counts cnt[w][d]: `tot` the tile's count
// of d, `x` the inclusive sum of the counts within the thread's wave; the waves' sums go to wsum,
// read after the caller's barrier.
template <uint32_t WAVES>
__device__ __forceinline__ void digit_totals(const uint32_t (*cnt)[256], uint32_t* wsum, uint32_t& tot, uint32_t& x) {
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  tot = 0;
  if (threadIdx.x < 256) {
#pragma unroll
    for (uint32_t w = 0; w < WAVES; ++w) tot += cnt[w][threadIdx.x];
  }
  x = tot;
#pragma unroll
  for (uint32_t o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (threadIdx.x < 256 && lane == 63) wsum[wave] = x;
}

// After the barrier, for the same threads: cnt[w][d] becomes the place in the sorted tile of wave
// w's first key of digit d; returns the place of the tile's first key of d.
template <uint32_t WAVES>
__device__ __forceinline__ uint32_t digit_places(uint32_t (*cnt)[256], const uint32_t* wsum, uint32_t tot, uint32_t x) {
  uint32_t e = x - tot;
  for (uint32_t w = 0; w < threadIdx.x >> 6; ++w) e += wsum[w];
  uint32_t at = e;
#pragma unroll
  for (uint32_t w = 0; w < WAVES; ++w) {
    const uint32_t c = cnt[w][threadIdx.x];
    cnt[w][threadIdx.x] = at;
    at += c;
  }
  return e;
}

// Counts of all the keys' digits, part[(b * sizeof(K) + p) * 256 + d] for workgroup b, pass p, digit
// d; also clears the look-back words and the tickets of the passes that follow.  A wave whose keys
// share a digit (the high digits of small keys) adds its count at once instead of 64 times.
template <typename K>
__global__ void __launch_bounds__(kCountThreads) k_sweep_count(const K* in, uint64_t n, uint32_t* part,
                                                     unsigned long long* status, uint64_t status_words,
                                                     uint32_t* tickets) {
  constexpr uint32_t P = sizeof(K), U = 8;
  __shared__ uint32_t cnt[P][256];
  for (uint32_t i = threadIdx.x; i < P * 256; i += kCountThreads) (&cnt[0][0])[i] = 0;
  if (blockIdx.x == 0 && threadIdx.x < P) tickets[threadIdx.x] = 0;
  for (uint64_t i = blockIdx.x * (uint64_t)kCountThreads + threadIdx.x; i < status_words; i += (uint64_t)gridDim.x * kCountThreads) status[i] = 0;
  __syncthreads();
  auto add = [&](K k) {
#pragma unroll
    for (uint32_t p = 0; p < P; ++p) {
      const uint32_t d = digit_of(k, p);
      const uint32_t d0 = __builtin_amdgcn_readfirstlane(d);
      const unsigned long long active = __ballot(true), same = __ballot(d == d0);
      if (same == active) {
        if ((threadIdx.x & 63) == (uint32_t)__builtin_ctzll(active)) atomicAdd(&cnt[p][d], (uint32_t)__popcll(active));
      } else {
        atomicAdd(&cnt[p][d], 1u);
      }
    }
  };
  const uint64_t step = (uint64_t)gridDim.x * kCountThreads * U;
  for (uint64_t base = blockIdx.x * (uint64_t)kCountThreads * U + threadIdx.x; base < n; base += step) {
    if (base - threadIdx.x + (uint64_t)kCountThreads * U <= n) {
      K k[U];
#pragma unroll
      for (uint32_t j = 0; j < U; ++j) k[j] = in[base + j * kCountThreads];
#pragma unroll
      for (uint32_t j = 0; j < U; ++j) add(k[j]);
    } else {
      for (uint32_t j = 0; j < U; ++j)
        if (base + j * kCountThreads < n) add(in[base + j * kCountThreads]);
    }
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < P * 256; i += kCountThreads) part[blockIdx.x * (P * 256) + i] = (&cnt[0][0])[i];
}

// Workgroup p: base[p * 256 + d] = keys of the run whose digit in pass p is below d.
__global__ void __launch_bounds__(1024) k_sweep_base(const uint32_t* part, uint32_t groups, unsigned long long* base) {
  __shared__ unsigned long long seg[4][256];
  __shared__ unsigned long long ws[4];
  const uint32_t d = threadIdx.x & 255, q = threadIdx.x >> 8, lane = threadIdx.x & 63;
  const uint32_t* col = part + blockIdx.x * 256 + d;
  const uint32_t stride = gridDim.x * 256;
  unsigned long long s = 0;
  uint32_t g = q;
  for (; g + 60 < groups; g += 64) {   // sixteen loads in flight
    uint32_t v[16];
#pragma unroll
    for (uint32_t u = 0; u < 16; ++u) v[u] = col[(uint64_t)(g + 4 * u) * stride];
#pragma unroll
    for (uint32_t u = 0; u < 16; ++u) s += v[u];
  }
  for (; g < groups; g += 4) s += col[(uint64_t)g * stride];
  seg[q][d] = s;
  __syncthreads();
  unsigned long long tot = 0, x = 0;
  if (q == 0) {
    tot = seg[0][d] + seg[1][d] + seg[2][d] + seg[3][d];
    x = tot;
#pragma unroll
    for (uint32_t o = 1; o < 64; o <<= 1) {
      const unsigned long long y = __shfl_up(x, o, 64);
      if (lane >= o) x += y;
    }
    if (lane == 63) ws[threadIdx.x >> 6] = x;
  }
  __syncthreads();
  if (q == 0) {
    unsigned long long b = x - tot;
    for (uint32_t w = 0; w < threadIdx.x >> 6; ++w) b += ws[w];
    base[blockIdx.x * 256 + d] = b;
  }
}

// One digit pass over the run; tiles of kDigitThreads * ITEMS keys.  Smaller tiles for short runs,
// so that they still fill the chip (digit_tile).
template <typename K, uint32_t ITEMS>
__global__ void __launch_bounds__(kDigitThreads) k_digit_sweep(const K* in, K* out, uint64_t n, uint32_t pass,
                                                              const unsigned long long* base,
                                                              unsigned long long* status, uint32_t* tickets,
                                                              LookLimit limit) {
  constexpr uint32_t TILE = kDigitThreads * ITEMS;
  __shared__ K stage[TILE];
  __shared__ uint32_t cnt[kDigitWaves][256];
  __shared__ uint32_t wsum[4];
  __shared__ unsigned long long gbase[256];
  __shared__ uint32_t ticket, lost;
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (threadIdx.x == 0) {
    ticket = atomicAdd(tickets + pass, 1u);
    lost = 0;
  }
  look_ready(limit);
  for (uint32_t i = threadIdx.x; i < kDigitWaves * 256; i += kDigitThreads) (&cnt[0][0])[i] = 0;
  __syncthreads();
  const uint64_t t = ticket;
  const uint64_t first = t * TILE + wave * (64 * ITEMS) + lane;
  auto tile = [&](auto whole) {
    constexpr bool FULL = decltype(whole)::value;
    K k[ITEMS];
    uint32_t rank[ITEMS];
    digit_load<FULL>(in, n, first, k);
    digit_rank<FULL>(k, n, first, pass, cnt[wave], rank);
    __syncthreads();
    uint32_t tot, x;
    digit_totals<kDigitWaves>(cnt, wsum, tot, x);
    unsigned long long pos = 0;
    if (threadIdx.x < 256) {
      unsigned long long* mine = status + t * 256 + threadIdx.x;
      if (t == 0) {
        pos = base[pass * 256 + threadIdx.x];
        look_store(mine, 2 * pass + 2, pos + tot);
      } else {
        look_store(mine, 2 * pass + 1, tot);
      }
    }
    __syncthreads();
    uint32_t e = 0;
    if (threadIdx.x < 256) e = digit_places<kDigitWaves>(cnt, wsum, tot, x);
    __syncthreads();
#pragma unroll
    for (uint32_t j = 0; j < ITEMS; ++j)
      if (FULL || first + j * 64 < n) stage[cnt[wave][digit_of(k[j], pass)] + rank[j]] = k[j];
    if (threadIdx.x < 256) {
      if (t != 0) {
        pos = look_back(status + threadIdx.x, 256, t, pass, limit);
        look_store(status + t * 256 + threadIdx.x, 2 * pass + 2, pos + tot);
      }
      gbase[threadIdx.x] = pos - e;
      // only where an earlier pass gave up a wait: the keys are then not those that the bases count
      if (pos + tot > n) lost = 1;
    }
    __syncthreads();
    if (lost) return;
    const uint32_t m = FULL ? TILE : (uint32_t)(n - t * TILE);
#pragma unroll
    for (uint32_t j = 0; j < ITEMS; ++j) {
      const uint32_t p = j * kDigitThreads + threadIdx.x;
      if (FULL || p < m) {
        const K v = stage[p];
        out[gbase[digit_of(v, pass)] + p] = v;
      }
    }
  };
  if ((t + 1) * TILE <= n) tile(std::true_type{});
  else tile(std::false_type{});
}

// A whole run of at most kLocalSortMax keys, sorted by one workgroup: every digit pass in LDS, one
// read and one write of memory and one launch (the launches bound such a run).  A pass whose keys
// all share the digit is left out.  in == out is fine: every key is read before one is written.
template <typename K>
__global__ void __launch_bounds__(1024) k_local_sort(const K* in, K* out, uint32_t n) {
  constexpr uint32_t T = 1024, ITEMS = kLocalSortMax / T, W = T / 64;
  __shared__ K stage[kLocalSortMax];
  __shared__ uint32_t cnt[W][256];
  __shared__ uint32_t wsum[4];
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t first = wave * (64 * ITEMS) + lane;
  K k[ITEMS];
  uint32_t rank[ITEMS];
  digit_load<false>(in, (uint64_t)n, (uint64_t)first, k);
  for (uint32_t pass = 0; pass < sizeof(K); ++pass) {
    for (uint32_t i = threadIdx.x; i < W * 256; i += T) (&cnt[0][0])[i] = 0;
    __syncthreads();
    digit_rank<false>(k, (uint64_t)n, (uint64_t)first, pass, cnt[wave], rank);
    __syncthreads();
    uint32_t tot, x;
    digit_totals<W>(cnt, wsum, tot, x);
    if (__syncthreads_or(threadIdx.x < 256 && tot == n)) continue;   // one digit value: the order stands
    if (threadIdx.x < 256) digit_places<W>(cnt, wsum, tot, x);
    __syncthreads();
#pragma unroll
    for (uint32_t j = 0; j < ITEMS; ++j)
      if (first + j * 64 < n) stage[cnt[wave][digit_of(k[j], pass)] + rank[j]] = k[j];
    __syncthreads();
#pragma unroll
    for (uint32_t j = 0; j < ITEMS; ++j)
      if (first + j * 64 < n) k[j] = stage[first + j * 64];
  }
#pragma unroll
  for (uint32_t j = 0; j < ITEMS; ++j)
    if (first + j * 64 < n) out[first + j * 64] = k[j];
}

// The order-preserving map of a signed key to an unsigned one.
inline uint64_t ord(int64_t v) { return (uint64_t)v ^ 0x8000000000000000ull; }
inline int64_t unord(uint64_t u) { return (int64_t)(u ^ 0x8000000000000000ull); }

// Per-run cut at global rank r: the r smallest elements of the union of the sorted runs, ties
// taken from lower-numbered runs first.  Finds the smallest value v with at least r elements
// <= v (binary search over the value range, each step a binary search in every run), takes
// every element below v, then the elements equal to v run by run.
template <typename K>
void merge_cuts_t(const K* const* runs, const uint64_t* len, uint32_t n_runs, uint64_t r, uint64_t* cut) {
  uint64_t total = 0;
  for (uint32_t j = 0; j < n_runs; ++j) total += len[j];
  if (r == 0 || r >= total) {
    for (uint32_t j = 0; j < n_runs; ++j) cut[j] = r == 0 ? 0 : len[j];
    return;
  }
  uint64_t lo = ~0ull, hi = 0;
  for (uint32_t j = 0; j < n_runs; ++j)
    if (len[j]) {
      lo = std::min(lo, ord((int64_t)runs[j][0]));
      hi = std::max(hi, ord((int64_t)runs[j][len[j] - 1]));
    }
  auto count_le = [&](uint64_t u) {
    const int64_t v = unord(u);
    uint64_t c = 0;
    for (uint32_t j = 0; j < n_runs; ++j)
      c += (uint64_t)(std::upper_bound(runs[j], runs[j] + len[j], v,
                                       [](int64_t x, const K& y) { return x < (int64_t)y; }) - runs[j]);
    return c;
  };
  while (lo < hi) {
    const uint64_t mid = lo + (hi - lo) / 2;
    if (count_le(mid) >= r) hi = mid;
    else lo = mid + 1;
  }
  const int64_t v = unord(lo);
  uint64_t need = r;
  std::vector<uint64_t> eq(n_runs);
  for (uint32_t j = 0; j < n_runs; ++j) {
    const K* b = runs[j];
    const K* e = runs[j] + len[j];
    const K* l = std::lower_bound(b, e, v, [](const K& x, int64_t y) { return (int64_t)x < y; });
    const K* u = std::upper_bound(b, e, v, [](int64_t x, const K& y) { return x < (int64_t)y; });
    cut[j] = (uint64_t)(l - b);
    eq[j] = (uint64_t)(u - l);
    need -= cut[j];
  }
  for (uint32_t j = 0; j < n_runs && need; ++j) {
    const uint64_t t = std::min(need, eq[j]);
    cut[j] += t;
    need -= t;
  }
}

// Device scratch of one run's radix sort: look-back words, digit bases, tickets (digit_tile's rule
// needs 2048 bytes of words per 2048 keys up to 2^16 keys, per 4096 up to 2^18, and per 8192 at least beyond).
uint64_t sweep_bytes(uint64_t rows) {
  return 3072 * std::max<uint64_t>(1, (rows + 8191) / 8192) + 262144;
}

// Keys per tile of a digit pass.  A short run in large tiles leaves compute units idle; a long one in
// small tiles writes shorter runs per digit and looks back over more tiles.  Sort kernels of one run,
// int64 keys, us at tiles of 2048 / 4096 / 8192 / 16384: 20,000 keys 58 / 64 / 77 / 111; 262,144
// keys - / 92 / 96 / 120; 1.0 M - / 141 / 130 / 148; 2.0 M - / 196 / 159 / 167; 4.0 M - / 299 / 249 /
// 191; 16.0 M - / 844 / 714 / 566.  A tile of 8192 int64 keys takes 83,992 bytes of LDS and 78 registers a
// lane, just past what two workgroups per compute unit may have, and so is measured at one, like the tile of
// 16384; the smaller ones run at two.
uint32_t digit_tile(uint64_t rows) {
  return rows <= (1ull << 16) ? 2048 : rows <= (1ull << 18) ? 4096 : rows <= (1ull << 21) ? 8192 : 16384;
}

struct SweepScratch {
  unsigned long long* base;     // 8 * 256
  uint32_t* tickets;            // 8
  unsigned long long* status;   // 256 per tile
  explicit SweepScratch(uint8_t* p)
      : base((unsigned long long*)p), tickets((uint32_t*)(p + 16384)), status((unsigned long long*)(p + 16640)) {}
};

// LSD radix sort of rows keys from src into dst, through alt: `passes` digit passes of 8 bits, from the
// low byte of the key's order-preserving image up (the keys agree in what is left out).  Passes
// alternate between dst and alt so that the last one writes dst.  With an even number the first
// writes alt, so src may be dst; with an odd number src may be alt.  The digit counts of
// k_sweep_count sit in the buffer that the first pass writes.  scratch holds sweep_bytes(rows);
// limit is the context's.
// *launches grows by the launches made.
template <typename K>
vx_status radix_sort_keys(const K* src, K* alt, K* dst, uint64_t rows, uint32_t passes, uint8_t* scratch,
                          LookLimit limit, uint64_t* launches, hipStream_t s) {
  VX_CHECK(rows < (1ull << 44), VX_EINVAL, "sort: run of %llu keys is too long", (unsigned long long)rows);
  if (rows <= kLocalSortMax) {
    hipLaunchKernelGGL(k_local_sort<K>, dim3(1), dim3(1024), 0, s, src, dst, (uint32_t)rows);
    VX_HIP(hipGetLastError());
    ++*launches;
    return VX_OK;
  }
  const uint32_t tile = digit_tile(rows);
  const uint64_t tiles = (rows + tile - 1) / tile;
  SweepScratch w(scratch);
  // 256 * sizeof(K) counts of 4 bytes per workgroup must fit a buffer: at most one workgroup per 2048 keys
  const unsigned groups = (unsigned)std::min<uint64_t>(kCountGroups, rows / 2048);
  uint32_t* part = (uint32_t*)(passes % 2 ? dst : alt);
  hipLaunchKernelGGL(k_sweep_count<K>, dim3(groups), dim3(kCountThreads), 0, s, src, rows, part, w.status, tiles * 256,
                     w.tickets);
  hipLaunchKernelGGL(k_sweep_base, dim3(sizeof(K)), dim3(1024), 0, s, part, groups, w.base);
  const K* in = src;
  for (uint32_t p = 0; p < passes; ++p) {
    K* out = ((passes - 1 - p) % 2 == 0) ? dst : alt;
    const dim3 grid((unsigned)tiles), block(kDigitThreads);
    switch (tile) {
      case 2048:
        hipLaunchKernelGGL((k_digit_sweep<K, 2>), grid, block, 0, s, in, out, rows, p, w.base, w.status, w.tickets, limit);
        break;
      case 4096:
        hipLaunchKernelGGL((k_digit_sweep<K, 4>), grid, block, 0, s, in, out, rows, p, w.base, w.status, w.tickets, limit);
        break;
      case 8192:
        hipLaunchKernelGGL((k_digit_sweep<K, 8>), grid, block, 0, s, in, out, rows, p, w.base, w.status, w.tickets, limit);
        break;
      default:
        hipLaunchKernelGGL((k_digit_sweep<K, 16>), grid, block, 0, s, in, out, rows, p, w.base, w.status, w.tickets, limit);
        break;
    }
    VX_HIP(hipGetLastError());
    in = out;
  }
  *launches += 2 + passes;
  return VX_OK;
}

vx_status radix_sort_run(const void* src, void* alt, void* dst, uint64_t rows, uint32_t ks, uint8_t* scratch,
                         LookLimit limit, uint64_t* launches, hipStream_t s) {
  if (ks == 8)
    return radix_sort_keys((const int64_t*)src, (int64_t*)alt, (int64_t*)dst, rows, 8, scratch, limit, launches, s);
  return radix_sort_keys((const int32_t*)src, (int32_t*)alt, (int32_t*)dst, rows, 4, scratch, limit, launches, s);
}

uint64_t align_to(uint64_t v, uint64_t a) { return (v + a - 1) / a * a; }

// Stores of a sorted run or merged range to its place (host or device memory), on a second stream
// beside the sort and merge kernels.  One workgroup per 16 compute units: the stores slow the
// kernels beside them (on the full-size sort, 256 workgroups took 1077 ms per sort, 64 took
// 1030, 16 took 1001 and 8 took 1041, where the stores themselves became the limit).
vx_status launch_store(const vx_ctx* ctx, const uint8_t* src, uint8_t* dst, uint64_t bytes, hipStream_t s) {
  const unsigned g = (unsigned)std::max(1, ctx->cu_count / 16);
  if ((((uintptr_t)src | (uintptr_t)dst) & 15) == 0)
    hipLaunchKernelGGL(k_store, dim3(g), dim3(256), 0, s, src, dst, bytes);
  else
    hipLaunchKernelGGL(k_store4, dim3(g), dim3(256), 0, s, (const uint32_t*)src, (uint32_t*)dst, bytes / 4);
  VX_HIP(hipGetLastError());
  return VX_OK;
}

vx_status sort_impl(vx_ctx* ctx, const vx_sort_desc* d, vx_stats* stats) {
  const double t0 = now_ms();
  VX_HIP(hipSetDevice(ctx->device));
  ColInfo kc;
  VX_TRY(classify(ctx, d->key, d->n, &kc, "sort key"));
  const uint64_t n = d->n;
  const uint32_t ks = (uint32_t)kc.elsize;
  vx_stats st;
  std::memset(&st, 0, sizeof st);
  st.rows = n;
  if (n < 2) {
    if (stats) *stats = st;
    return VX_OK;
  }
  // run length: the largest power of two whose pass-1 buffers (2 pipeline buffers, one radix
  // buffer, two staging runs) and sort scratch fit the free arena; pass 2 needs 4 runs' room
  const uint64_t free0 = ctx->arena.capacity() - ctx->arena.used();
  auto pass1_bytes = [&](uint64_t rows) { return 5 * align_to(rows * ks, 256) + sweep_bytes(rows) + (1ull << 20); };
  // a device column that is one run is sorted where it lies and needs one buffer beside it
  const uint64_t direct_bytes = align_to(n * ks, 256) + sweep_bytes(n) + 256;
  const LookLimit limit = look_limit(ctx);
  uint64_t C = d->chunk_rows;
  if (!C && kc.where == Where::Device && direct_bytes <= ctx->arena.largest_free()) C = n;
  if (!C) {
    C = 1024;
    while (C * 2 <= n && pass1_bytes(C * 2) <= free0) C *= 2;
    if (C < n && pass1_bytes(n) <= free0) C = n;
    if (C > n) C = n;
  }
  VX_CHECK(C >= 1, VX_EINVAL, "sort: chunk_rows is 0");
  const uint64_t runs = (n + C - 1) / C;
  const uint64_t run_bytes = align_to(std::min(C, n) * ks, 256);
  // host scratch for the sorted runs (several runs only)
  uint8_t* hs = nullptr;
  if (runs > 1) VX_TRY(host_scratch(ctx, n * ks + 256, &hs));
  void* hs_dev = nullptr;
  if (hs) VX_HIP(hipHostGetDevicePointer(&hs_dev, hs, 0));
  uint8_t* out_dev = (uint8_t*)kc.dev;   // the key column as a device address (sorted in place)

  // ---------------- pass 1: sorted runs
  const double tp0 = now_ms();
  double sort_k_ms = 0;
  uint64_t launches = 0, sdma = 0;
  uint32_t nbuf_used = 0;
  if (runs == 1 && kc.where == Where::Device) {
    // no staging and no store: the passes go from the column to the buffer and back (16.0 M int64
    // keys: the store of the staged run alone took 572 us, as it runs on few workgroups)
    nbuf_used = d->n_buffers ? d->n_buffers : (uint32_t)env_u64("VX_BUFFERS", 2);
    VX_CHECK(nbuf_used >= 2 && nbuf_used <= kMaxBuffers, VX_EINVAL, "pipeline: n_buffers %u outside 2..%u", nbuf_used,
             kMaxBuffers);
    ArenaBlock blk;
    blk.a = &ctx->arena;
    blk.p = ctx->arena.alloc(direct_bytes);
    VX_CHECK(blk.p, VX_EBUDGET, "sort: no room for a run of %llu keys (radix buffer)", (unsigned long long)n);
    hipEvent_t e0 = get_event(ctx), e1 = get_event(ctx);
    auto direct = [&]() -> vx_status {
      VX_CHECK(e0 && e1, VX_EHIP, "sort: no HIP event");
      VX_HIP(hipEventRecord(e0, ctx->compute));
      VX_TRY(radix_sort_run(out_dev, blk.p, out_dev, n, ks, blk.p + align_to(n * ks, 256), limit, &launches,
                            ctx->compute));
      VX_HIP(hipEventRecord(e1, ctx->compute));
      return VX_OK;
    };
    vx_status rs = direct();
    const hipError_t se = hipStreamSynchronize(ctx->compute);
    float ms = 0;
    if (rs == VX_OK && se == hipSuccess && hipEventElapsedTime(&ms, e0, e1) == hipSuccess) sort_k_ms = ms;
    put_event(ctx, e0);
    put_event(ctx, e1);
    VX_TRY(rs);
    VX_HIP(se);
  } else {
    ArenaBlock blk;
    blk.a = &ctx->arena;
    blk.p = ctx->arena.alloc(3 * run_bytes + sweep_bytes(std::min(C, n)) + 256);
    VX_CHECK(blk.p, VX_EBUDGET, "sort: no room for runs of %llu keys (radix and staging buffers)",
             (unsigned long long)C);
    uint8_t* alt = blk.p;
    uint8_t* stage[2] = {blk.p + run_bytes, blk.p + 2 * run_bytes};
    uint8_t* scratch = blk.p + 3 * run_bytes;
    std::vector<PipeCol> cols(1);
    cols[0].info = kc;
    cols[0].may_copy = cols[0].copy = true;
    Pipeline pipe;
    VX_TRY(pipe.plan(ctx, n, C, d->n_buffers, cols));
    nbuf_used = pipe.n_buffers();
    hipEvent_t sorted_ev[2] = {get_event(ctx), get_event(ctx)}, wrote[2] = {get_event(ctx), get_event(ctx)};
    std::vector<hipEvent_t> kev;
    bool pending[2] = {false, false};
    auto kernel = [&](const ChunkView& v) -> vx_status {
      for (int b = 0; b < 2; ++b) VX_CHECK(sorted_ev[b] && wrote[b], VX_EHIP, "sort: no HIP event");
      const uint32_t b = (uint32_t)(v.index % 2);
      if (pending[b]) VX_HIP(hipStreamWaitEvent(ctx->compute, wrote[b], 0));
      const uint8_t* src = (v.global_mask & 1u) ? (const uint8_t*)v.ptr[0] + v.row0 * ks : (const uint8_t*)v.ptr[0];
      hipEvent_t e0 = get_event(ctx), e1 = get_event(ctx);
      VX_CHECK(e0 && e1, VX_EHIP, "sort: no HIP event");
      kev.push_back(e0);
      kev.push_back(e1);
      VX_HIP(hipEventRecord(e0, ctx->compute));
      VX_TRY(radix_sort_run(src, alt, stage[b], v.rows, ks, scratch, limit, &launches, ctx->compute));
      VX_HIP(hipEventRecord(e1, ctx->compute));
      VX_HIP(hipEventRecord(sorted_ev[b], ctx->compute));
      // a single run is the result: store it in place; otherwise to its rows of the scratch
      uint8_t* dst = (runs > 1 ? (uint8_t*)hs_dev : out_dev) + v.row0 * ks;
      VX_HIP(hipStreamWaitEvent(ctx->d2h, sorted_ev[b], 0));
      VX_TRY(launch_store(ctx, stage[b], dst, v.rows * ks, ctx->d2h));
      ++launches;
      VX_HIP(hipEventRecord(wrote[b], ctx->d2h));
      pending[b] = true;
      return VX_OK;
    };
    vx_status rs = pipe.run(kernel);
    (void)hipStreamSynchronize(ctx->compute);
    (void)hipStreamSynchronize(ctx->d2h);
    for (size_t i = 0; i + 1 < kev.size(); i += 2) {
      float ms = 0;
      if (hipEventElapsedTime(&ms, kev[i], kev[i + 1]) == hipSuccess) sort_k_ms += ms;
    }
    for (auto e : kev) put_event(ctx, e);
    for (int b = 0; b < 2; ++b) {
      put_event(ctx, sorted_ev[b]);
      put_event(ctx, wrote[b]);
    }
    VX_TRY(rs);
    sdma = pipe.sdma_bytes();
  }
  const double pass1_ms = now_ms() - tp0;
  VX_TRY(check_stall(ctx, "sort"));

  // ---------------- pass 2: regroup and merge
  const double tm0 = now_ms();
  double merge_k_ms = 0;
  uint64_t max_part = 0;
  if (runs > 1) {
    // cuts of every run at ranks 0, C, 2C, ..., n (host binary search over the pinned runs)
    const uint64_t M = runs;
    std::vector<uint64_t> rank(M + 1), len(runs);
    for (uint64_t i = 0; i <= M; ++i) rank[i] = std::min(i * C, n);
    for (uint64_t j = 0; j < runs; ++j) len[j] = std::min(C, n - j * C);
    std::vector<uint64_t> cuts((M + 1) * runs);
    {
      const unsigned nt = std::max(1u, std::min({16u, std::thread::hardware_concurrency(), (unsigned)std::min<uint64_t>(M + 1, 16)}));
      std::vector<std::thread> th;
      for (unsigned t = 0; t < nt; ++t)
        th.emplace_back([&, t]() {
          if (ks == 8) {
            std::vector<const long long*> rp(runs);
            for (uint64_t j = 0; j < runs; ++j) rp[j] = (const long long*)hs + j * C;
            for (uint64_t i = t; i <= M; i += nt)
              merge_cuts_t<long long>(rp.data(), len.data(), (uint32_t)runs, rank[i], &cuts[i * runs]);
          } else {
            std::vector<const int*> rp(runs);
            for (uint64_t j = 0; j < runs; ++j) rp[j] = (const int*)hs + j * C;
            for (uint64_t i = t; i <= M; i += nt)
              merge_cuts_t<int>(rp.data(), len.data(), (uint32_t)runs, rank[i], &cuts[i * runs]);
          }
        });
      for (auto& x : th) x.join();
    }
    for (uint64_t i = 0; i < M; ++i) max_part = std::max(max_part, rank[i + 1] - rank[i]);
    // three sets of (input, alternate) buffers when they fit, else two: a range holds its set from
    // its copy in to the end of its store, so with three the copies of the next ranges run while
    // one range merges and another is stored
    const uint64_t pbytes = align_to(max_part * ks, 256);
    ArenaBlock blk;
    blk.a = &ctx->arena;
    uint32_t nset = 3;
    blk.p = ctx->arena.largest_free() >= 6 * pbytes + (1u << 20) ? ctx->arena.alloc(6 * pbytes) : nullptr;
    if (!blk.p) {
      nset = 2;
      blk.p = ctx->arena.alloc(4 * pbytes);
    }
    VX_CHECK(blk.p, VX_EBUDGET, "sort: no room for the merge buffers (4 x %llu B)", (unsigned long long)pbytes);
    uint8_t* X[3] = {blk.p, blk.p + pbytes, blk.p + 2 * pbytes};
    uint8_t* Y[3] = {blk.p + nset * pbytes, blk.p + (nset + 1) * pbytes, blk.p + (nset + 2) * pbytes};
    hipEvent_t copied[3] = {get_event(ctx), get_event(ctx), get_event(ctx)},
               merged[3] = {get_event(ctx), get_event(ctx), get_event(ctx)},
               stored[3] = {get_event(ctx), get_event(ctx), get_event(ctx)};
    std::vector<hipEvent_t> kev;
    // one output range; on an error the streams are still drained before the buffers go back
    auto range = [&](uint64_t i) -> vx_status {
      for (int b = 0; b < 3; ++b) VX_CHECK(copied[b] && merged[b] && stored[b], VX_EHIP, "sort: no HIP event");
      const uint32_t b = (uint32_t)(i % nset);
      if (i >= nset) VX_HIP(hipEventSynchronize(stored[b]));   // range i - nset has left these buffers
      // copy in the range's segment of every run, back to back
      std::vector<uint64_t> off(runs + 1, 0);
      for (uint64_t j = 0; j < runs; ++j) {
        const uint64_t a = cuts[i * runs + j], e = cuts[(i + 1) * runs + j];
        off[j + 1] = off[j] + (e - a);
        if (e > a) {
          VX_HIP(hipMemcpyAsync(X[b] + off[j] * ks, hs + (j * C + a) * ks, (e - a) * ks, hipMemcpyHostToDevice,
                                ctx->copy));
          sdma += (e - a) * ks;
        }
      }
      VX_HIP(hipEventRecord(copied[b], ctx->copy));
      VX_HIP(hipStreamWaitEvent(ctx->compute, copied[b], 0));
      // merge rounds: pairs of neighbouring segments, X and Y in turn
      std::vector<uint64_t> seg;
      for (uint64_t j = 0; j <= runs; ++j)
        if (seg.empty() || off[j] != seg.back()) seg.push_back(off[j]);   // no segment is empty: every pair has tiles
      uint8_t* src = X[b];
      uint8_t* dst = Y[b];
      hipEvent_t e0 = get_event(ctx), e1 = get_event(ctx);
      VX_CHECK(e0 && e1, VX_EHIP, "sort: no HIP event");
      kev.push_back(e0);
      kev.push_back(e1);
      VX_HIP(hipEventRecord(e0, ctx->compute));
      while (seg.size() > 2) {
        std::vector<uint64_t> next;
        MergeRound round;
        round.n = 0;
        round.tile0[0] = 0;
        auto flush = [&]() -> vx_status {
          const uint32_t tiles = round.tile0[round.n];
          const unsigned g = (unsigned)std::min<uint64_t>(tiles, (uint64_t)ctx->cu_count * kMergeGroups);
          if (ks == 8)
            hipLaunchKernelGGL(k_merge<long long>, dim3(g), dim3(kMergeThreads), 0, ctx->compute, (const long long*)src,
                               (long long*)dst, round);
          else
            hipLaunchKernelGGL(k_merge<int>, dim3(g), dim3(kMergeThreads), 0, ctx->compute, (const int*)src, (int*)dst,
                               round);
          VX_HIP(hipGetLastError());
          ++launches;
          round.n = 0;
          return VX_OK;
        };
        for (size_t k = 0; k + 1 < seg.size(); k += 2) {
          const uint64_t a0 = seg[k], a1 = seg[k + 1], b1 = k + 2 < seg.size() ? seg[k + 2] : a1;
          const uint64_t tiles = (b1 - a0 + kMergeTile - 1) / kMergeTile;
          // a launch counts its tiles in 32 bits
          if (round.n == MergeRound::kMax || (round.n && round.tile0[round.n] + tiles > 0x7fffffffull)) VX_TRY(flush());
          VX_CHECK(tiles <= 0x7fffffffull, VX_EINVAL, "sort: a merged range of %llu keys", (unsigned long long)(b1 - a0));
          round.a0[round.n] = a0;
          round.a1[round.n] = a1;
          round.b1[round.n] = b1;
          round.tile0[round.n + 1] = round.tile0[round.n] + (uint32_t)tiles;
          ++round.n;
          next.push_back(a0);
        }
        VX_TRY(flush());
        next.push_back(seg.back());
        seg.swap(next);
        std::swap(src, dst);
      }
      VX_HIP(hipEventRecord(e1, ctx->compute));
      VX_HIP(hipEventRecord(merged[b], ctx->compute));
      // store the merged range to its place in the key column
      VX_HIP(hipStreamWaitEvent(ctx->d2h, merged[b], 0));
      const uint64_t rows = rank[i + 1] - rank[i];
      VX_TRY(launch_store(ctx, src, out_dev + rank[i] * ks, rows * ks, ctx->d2h));
      ++launches;
      VX_HIP(hipEventRecord(stored[b], ctx->d2h));
      return VX_OK;
    };
    vx_status rs = VX_OK;
    for (uint64_t i = 0; i < M && rs == VX_OK; ++i) rs = range(i);
    (void)hipStreamSynchronize(ctx->copy);
    (void)hipStreamSynchronize(ctx->compute);
    (void)hipStreamSynchronize(ctx->d2h);
    for (size_t k = 0; k + 1 < kev.size(); k += 2) {
      float ms = 0;
      if (hipEventElapsedTime(&ms, kev[k], kev[k + 1]) == hipSuccess) merge_k_ms += ms;
    }
    for (auto e : kev) put_event(ctx, e);
    for (int b = 0; b < 3; ++b) {
      put_event(ctx, copied[b]);
      put_event(ctx, merged[b]);
      put_event(ctx, stored[b]);
    }
    VX_TRY(rs);
  }
  VX_HIP(hipGetLastError());
  st.chunks = runs;
  st.chunk_rows = C;
  st.n_buffers = nbuf_used;
  st.part_ms = pass1_ms;
  st.probe_ms = runs > 1 ? now_ms() - tm0 : 0;
  st.kernel_ms = sort_k_ms;
  st.build_ms = merge_k_ms;
  st.sdma_bytes = sdma;
  st.kernel_launches = launches;
  st.total_ms = now_ms() - t0;
  if (stats) *stats = st;
  return VX_OK;
}

}  // namespace

uint64_t sort_scratch_bytes(uint64_t rows) {
  if (rows <= kLocalSortMax) return 0;
  return 16640 + (rows + digit_tile(rows) - 1) / digit_tile(rows) * 2048;
}

vx_status sort_keys_i64(vx_ctx* ctx, long long* a, long long* b, uint64_t rows, uint32_t passes, uint8_t* scratch,
                        long long** sorted, hipStream_t s) {
  uint64_t launches = 0;
  int64_t *src = (int64_t*)a, *other = (int64_t*)b;
  int64_t* dst = passes % 2 ? other : src;
  *sorted = (long long*)dst;
  return radix_sort_keys(src, passes % 2 ? src : other, dst, rows, passes, scratch, look_limit(ctx), &launches, s);
}

}  // namespace vx

extern "C" vx_status vx_sort(vx_ctx* ctx, const vx_sort_desc* d, vx_stats* stats) {
  VX_CHECK(ctx && d, VX_EINVAL, "vx_sort: null argument");
  vx::release_cached(ctx);
  return vx::sort_impl(ctx, d, stats);
}

extern "C" vx_status vx_merge_cuts(const int64_t* const* runs, const uint64_t* run_len, uint32_t n_runs,
                                   uint64_t rank, uint64_t* cut) {
  VX_CHECK(n_runs == 0 || (runs && run_len && cut), VX_EINVAL, "vx_merge_cuts: null argument");
  uint64_t total = 0;
  for (uint32_t j = 0; j < n_runs; ++j) {
    VX_CHECK(run_len[j] == 0 || runs[j], VX_EINVAL, "vx_merge_cuts: run %u is NULL", j);
    total += run_len[j];
  }
  VX_CHECK(rank <= total, VX_EINVAL, "vx_merge_cuts: rank %llu exceeds the %llu elements",
           (unsigned long long)rank, (unsigned long long)total);
  vx::merge_cuts_t<int64_t>(runs, run_len, n_runs, rank, cut);
  return VX_OK;
}
