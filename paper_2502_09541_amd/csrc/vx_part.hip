// Partitioning: ids, counts, the stable scatter in one launch, and vx_partition.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <type_traits>
#include <vector>

#include "vx_cdf.h"
#include "vx_device.h"
#include "vx_lookback.h"
#include "vx_part.h"
#include "vx_pipeline.h"

namespace vx {

// ---------------------------------------------------------------- device side

// Counting: workgroups take rows grid-stride, kCountItems keys per lane in flight, and count in LDS;
// the counters are repeated over the lanes (as often as 4096 counters allow) so that a few large
// partitions do not serialize a wave's additions.  part[g * P + p] receives workgroup g's counts.
// Also clears the look-back words and the ticket of the sweep that follows.
// Bound: the keys' read and the LDS additions; 16.0 M int64 keys in 256 hash partitions take 47 us
// (2.7 TB/s; 147 us with one key per lane in flight and a ballot per id bit).
constexpr uint32_t kCountThreads = 1024;
constexpr uint32_t kCountItems = 8;
constexpr uint32_t kCountGroups = 256;
constexpr uint32_t kCountSlots = 4096;

template <typename K>
__global__ void __launch_bounds__(kCountThreads) k_part_count(PartSpec ps, PartIO io, uint32_t copies, uint32_t* part,
                                                              unsigned long long* status, uint64_t status_words,
                                                              uint32_t* ticket, const int* sum_slot,
                                                              unsigned long long* sums) {
  __shared__ long long split[kMaxParts];
  __shared__ uint32_t cnt[kCountSlots];
  __shared__ unsigned long long ssum[kMaxSumSlots][2];
  const uint32_t P = ps.n_parts;
  const uint64_t n = io.n;
  if (blockIdx.x == 0 && threadIdx.x == 0) *ticket = 0;
  for (uint64_t i = blockIdx.x * (uint64_t)kCountThreads + threadIdx.x; i < status_words;
       i += (uint64_t)gridDim.x * kCountThreads)
    status[i] = 0;
  if (ps.fn == kPartRange)
    for (uint32_t j = threadIdx.x; j < ps.n_split; j += kCountThreads) split[j] = ps.splitters[j];
  for (uint32_t j = threadIdx.x; j < kCountSlots; j += kCountThreads) cnt[j] = 0;
  if (threadIdx.x < 2 * kMaxSumSlots) (&ssum[0][0])[threadIdx.x] = 0;
  __syncthreads();
  const K* key = (const K*)io.key;
  uint32_t* mine = cnt + (threadIdx.x & (copies - 1)) * P;
  const uint64_t block_rows = (uint64_t)kCountThreads * kCountItems;
  for (uint64_t b0 = blockIdx.x * block_rows; b0 < n; b0 += gridDim.x * block_rows) {
    const uint64_t i0 = b0 + threadIdx.x;
    K k[kCountItems];
    uint32_t id[kCountItems];
    const bool whole = b0 + block_rows <= n;
#pragma unroll
    for (uint32_t j = 0; j < kCountItems; ++j)
      k[j] = whole || i0 + j * kCountThreads < n ? key[i0 + j * kCountThreads] : K(0);
    part_ids<kCountItems>(ps, k, split, id);
#pragma unroll
    for (uint32_t j = 0; j < kCountItems; ++j)
      if (whole || i0 + j * kCountThreads < n) atomicAdd(mine + id[j], 1u);
    if (sum_slot) {
#pragma unroll
      for (uint32_t j = 0; j < kCountItems; ++j) {
        const uint64_t i = i0 + j * kCountThreads;
        const int slot = i < n ? sum_slot[id[j]] : -1;
        if (slot >= 0) {
          atomicAdd(&ssum[slot][0], 1ull);
          if (io.n_pay) atomicAdd(&ssum[slot][1], (unsigned long long)load_signed(io.pay[0], i, io.pay_size[0]));
        }
      }
    }
  }
  __syncthreads();
  for (uint32_t p = threadIdx.x; p < P; p += kCountThreads) {
    uint32_t c = 0;
    for (uint32_t r = 0; r < copies; ++r) c += cnt[r * P + p];
    part[(uint64_t)blockIdx.x * P + p] = c;
  }
  if (sum_slot && threadIdx.x < 2 * kMaxSumSlots) {
    const unsigned long long v = (&ssum[0][0])[threadIdx.x];
    if (v) atomicAdd(sums + threadIdx.x, v);
  }
}

// One workgroup: totals[p] (+)= SUM over the counting workgroups of part[g * P + p], base = the
// exclusive prefix of totals, base[P] = their sum.  The threads split the workgroups' rows into
// 1024 / padded interleaved shares (padded: P rounded up to a power of two, at least 64).
__global__ void __launch_bounds__(1024) k_part_base(const uint32_t* part, uint32_t groups, uint32_t P, uint32_t log2pad,
                                                    unsigned long long* totals, uint32_t accumulate,
                                                    unsigned long long* base, unsigned long long* host_totals) {
  __shared__ unsigned long long sum[1024];
  __shared__ unsigned long long ws[16];
  const uint32_t pad = 1u << log2pad, p = threadIdx.x & (pad - 1), q = threadIdx.x >> log2pad, shares = 1024u >> log2pad;
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  unsigned long long s = 0;
  if (p < P) {
    uint32_t g = q;
    for (; g + 15 * shares < groups; g += 16 * shares) {   // sixteen loads in flight
      uint32_t v[16];
#pragma unroll
      for (uint32_t u = 0; u < 16; ++u) v[u] = part[(uint64_t)(g + u * shares) * P + p];
#pragma unroll
      for (uint32_t u = 0; u < 16; ++u) s += v[u];
    }
    for (; g < groups; g += shares) s += part[(uint64_t)g * P + p];
  }
  sum[threadIdx.x] = s;
  __syncthreads();
  unsigned long long tot = 0;
  if (threadIdx.x < P) {
    for (uint32_t r = 0; r < shares; ++r) tot += sum[r * pad + threadIdx.x];
    if (accumulate) tot += totals[threadIdx.x];
    totals[threadIdx.x] = tot;
    if (host_totals) host_totals[threadIdx.x] = tot;
  }
  unsigned long long x = tot;
#pragma unroll
  for (uint32_t o = 1; o < 64; o <<= 1) {
    const unsigned long long y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) ws[wave] = x;
  __syncthreads();
  unsigned long long b = x - tot;
  for (uint32_t w = 0; w < wave; ++w) b += ws[w];
  if (threadIdx.x < P) {
    base[threadIdx.x] = b;
    if (threadIdx.x == P - 1) base[P] = b + tot;
  }
}

// The scatter.  A tile's rows are ranked by partition within each wave (same_id over BITS id bits
// and a per-wave LDS counter), the waves' counts give every row its place in the sorted tile, and
// the keys, then each payload column, go through LDS to consecutive addresses per partition.  The
// splitters sit in the staging buffer until the ids are known.  E is the widest column's size.
// Bound: the rows' read and write, with the ranking close behind.  16.0 M rows of 16 bytes into 256
// partitions take 136 us (3.8 TB/s read and written; a large copy reaches 4.8): 425 us when each wave
// placed 64 rows at a time into up to 64 partitions.
constexpr uint32_t kSweepThreads = 1024;

template <typename K, uint32_t E, uint32_t ITEMS, uint32_t BITS>
__global__ void __launch_bounds__(kSweepThreads, 4) k_part_sweep(PartSpec ps, PartIO io, const unsigned long long* base,
                                                                 unsigned long long* next, unsigned long long* status,
                                                                 uint32_t* ticket, LookLimit limit) {
  constexpr uint32_t THREADS = kSweepThreads, MAXP = 1u << BITS, WAVES = THREADS / 64, TILE = THREADS * ITEMS,
                     WROWS = 64 * ITEMS;
  static_assert(THREADS >= MAXP && E >= sizeof(K) && TILE * E >= 8 * (MAXP - 1) && TILE <= (1u << 15), "tile shape");
  using Id = typename std::conditional<BITS <= 8, uint8_t, uint16_t>::type;
  __shared__ __align__(16) uint8_t stage[TILE * E];
  __shared__ __align__(4) uint16_t cnt[WAVES][MAXP];
  __shared__ Id id_at[TILE];
  __shared__ unsigned long long gbase[MAXP];
  __shared__ uint32_t wsum[MAXP / 64];
  __shared__ uint32_t tile_no;
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6, P = ps.n_parts;
  if (threadIdx.x == 0) tile_no = atomicAdd(ticket, 1u);
  look_ready(limit);
  if (ps.fn == kPartRange)
    for (uint32_t j = threadIdx.x; j < ps.n_split; j += THREADS) ((long long*)stage)[j] = ps.splitters[j];
  for (uint32_t i = threadIdx.x; i < WAVES * MAXP / 2; i += THREADS) ((uint32_t*)&cnt[0][0])[i] = 0;
  __syncthreads();
  const uint64_t t = tile_no, n = io.n;
  const uint64_t first = t * TILE + wave * WROWS + lane;
  auto tile = [&](auto whole_tile) {
    constexpr bool FULL = decltype(whole_tile)::value;
    K k[ITEMS];
    uint32_t id[ITEMS];   // low half: the partition; high half: the place in the tile
    const K* key = (const K*)io.key;
#pragma unroll
    for (uint32_t j = 0; j < ITEMS; ++j)
      k[j] = FULL || first + j * 64 < n ? __builtin_nontemporal_load(key + first + j * 64) : K(0);
    part_ids<ITEMS>(ps, k, (const long long*)stage, id);
    const unsigned long long lower = (1ull << lane) - 1;
#pragma unroll
    for (uint32_t j = 0; j < ITEMS; ++j) {
      const bool valid = FULL || first + j * 64 < n;
      const unsigned long long peers = same_id(id[j], BITS, FULL ? ~0ull : __ballot(valid));
      const uint32_t below = (uint32_t)__popcll(peers & lower);
      const uint32_t c = valid ? cnt[wave][id[j]] : 0u;
      // every lane has read cnt[] before the group's first lane advances it
      __builtin_amdgcn_wave_barrier();
      if (valid && below == 0) cnt[wave][id[j]] = (uint16_t)(c + (uint32_t)__popcll(peers));
      __builtin_amdgcn_wave_barrier();
      id[j] |= (c + below) << 16;
    }
    __syncthreads();
    // thread p: partition p's rows in the tile, published for the tiles that follow
    uint32_t tot = 0;
    unsigned long long pos = 0;
    if (threadIdx.x < P) {
#pragma unroll
      for (uint32_t w = 0; w < WAVES; ++w) tot += cnt[w][threadIdx.x];
      unsigned long long* word = status + t * P + threadIdx.x;
      if (t == 0) {
        pos = base[threadIdx.x];
        look_store(word, 2, pos + tot);
      } else {
        look_store(word, 1, tot);
      }
    }
    uint32_t x = tot;
    if (threadIdx.x < MAXP) {
#pragma unroll
      for (uint32_t o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
      }
      if (lane == 63) wsum[wave] = x;
    }
    __syncthreads();
    uint32_t e = 0;
    if (threadIdx.x < P) {   // the places of the waves' first rows of partition p
      e = x - tot;
      for (uint32_t w = 0; w < wave; ++w) e += wsum[w];
      uint32_t at = e;
#pragma unroll
      for (uint32_t w = 0; w < WAVES; ++w) {
        const uint32_t c = cnt[w][threadIdx.x];
        cnt[w][threadIdx.x] = (uint16_t)at;
        at += c;
      }
    }
    __syncthreads();
#pragma unroll
    for (uint32_t j = 0; j < ITEMS; ++j)
      if (FULL || first + j * 64 < n) {
        const uint32_t p = id[j] & 0xffffu;
        id[j] = (id[j] >> 16) + cnt[wave][p];   // now the place alone
        ((K*)stage)[id[j]] = k[j];
        id_at[id[j]] = (Id)p;
      }
    if (threadIdx.x < P) {
      if (t != 0) {
        pos = look_back(status + threadIdx.x, P, t, 0, limit);
        look_store(status + t * P + threadIdx.x, 2, pos + tot);
      }
      gbase[threadIdx.x] = io.out_base + pos - e;
      if (next && (t + 1) * TILE >= n) next[threadIdx.x] = pos + tot;
    }
    __syncthreads();
    const uint32_t m = FULL ? TILE : (uint32_t)(n - t * TILE);
#pragma unroll
    for (uint32_t j = 0; j < ITEMS; ++j) {
      const uint32_t q = j * THREADS + threadIdx.x;
      if (FULL || q < m) ((K*)io.out_key)[gbase[id_at[q]] + q] = ((const K*)stage)[q];
    }
    for (uint32_t c = 0; c < io.n_pay; ++c) {
      if (!io.out_pay[c]) continue;
      auto column = [&](auto zero) {
        using V = decltype(zero);
        V v[ITEMS];
        const V* src = (const V*)io.pay[c];
#pragma unroll
        for (uint32_t j = 0; j < ITEMS; ++j)
          v[j] = FULL || first + j * 64 < n ? __builtin_nontemporal_load(src + first + j * 64) : V(0);
        __syncthreads();   // the stage has been read
#pragma unroll
        for (uint32_t j = 0; j < ITEMS; ++j)
          if (FULL || first + j * 64 < n) ((V*)stage)[id[j]] = v[j];
        __syncthreads();
#pragma unroll
        for (uint32_t j = 0; j < ITEMS; ++j) {
          const uint32_t q = j * THREADS + threadIdx.x;
          if (FULL || q < m) ((V*)io.out_pay[c])[gbase[id_at[q]] + q] = ((const V*)stage)[q];
        }
      };
      if (io.pay_size[c] == 8) {
        if constexpr (E == 8) column((int64_t)0);
      } else {
        column((int32_t)0);
      }
    }
  };
  if ((t + 1) * TILE <= n) tile(std::true_type{});
  else tile(std::false_type{});
}

// ---------------------------------------------------------------- host wrappers

// Rows per tile of the sweep.  Short inputs in large tiles leave compute units idle, long ones in small
// tiles write shorter runs and look back further: whole calls over rows of 16 bytes, 256 partitions,
// us at tiles of 2048 / 8192: 30,000 rows 42 / 45; 300,000 47 / 49; 600,000 54 / 53; 1.0 M 66 / 61;
// 16.0 M 296 / 210.
static uint32_t sweep_tile(uint64_t rows) { return rows <= (1ull << 19) ? 2048 : 8192; }

// words first, so that every array is 8-byte aligned: the ticket, the look-back words, the counts
static uint64_t sweep_words(uint32_t P, uint64_t rows) {
  const uint32_t tile = sweep_tile(rows);
  return (rows + tile - 1) / tile * P;
}
static uint32_t count_groups(uint64_t rows) {
  return (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(kCountGroups, rows / 4096));
}

// sizes grow with the rows except where the tile does, so a launch over fewer rows than planned for
// is allowed the small tiles' words
uint64_t part_work_bytes(uint32_t n_parts, uint64_t rows, bool sweep) {
  const uint64_t words = !sweep ? 0 : std::max(sweep_words(n_parts, rows), sweep_words(n_parts, std::min<uint64_t>(rows, 1ull << 19)));
  return 64 + words * 8 + (uint64_t)count_groups(rows) * n_parts * 4 + 8;
}

vx_status part_ready(const PartSpec& ps, uint64_t rows, uint8_t* work, hipStream_t s) {
  fill_zero((uint64_t*)work, 8 + sweep_words(ps.n_parts, rows), s);
  VX_HIP(hipGetLastError());
  return VX_OK;
}

vx_status part_count(vx_ctx* ctx, const PartSpec& ps, const PartIO& io, uint8_t* work, unsigned long long* totals,
                     bool accumulate, unsigned long long* base, unsigned long long* host_totals, const int* sum_slot,
                     unsigned long long* sums, hipStream_t s, bool sweep) {
  (void)ctx;
  const uint32_t P = ps.n_parts, groups = count_groups(io.n);
  const uint64_t words = sweep ? sweep_words(P, io.n) : 0;
  uint32_t* ticket = (uint32_t*)work;
  unsigned long long* status = (unsigned long long*)(work + 64);
  uint32_t* part = (uint32_t*)(status + words);
  uint32_t copies = 32;
  while (copies > 1 && copies * P > kCountSlots) copies >>= 1;
  if (io.key_size == 8)
    hipLaunchKernelGGL(k_part_count<int64_t>, dim3(groups), dim3(kCountThreads), 0, s, ps, io, copies, part, status,
                       words, ticket, sum_slot, sums);
  else
    hipLaunchKernelGGL(k_part_count<int32_t>, dim3(groups), dim3(kCountThreads), 0, s, ps, io, copies, part, status,
                       words, ticket, sum_slot, sums);
  uint32_t log2pad = 6;
  while ((1u << log2pad) < P) ++log2pad;
  hipLaunchKernelGGL(k_part_base, dim3(1), dim3(1024), 0, s, part, groups, P, log2pad, totals, accumulate ? 1u : 0u,
                     base, host_totals);
  VX_HIP(hipGetLastError());
  return VX_OK;
}

template <typename K, uint32_t E>
static void launch_sweep(const PartSpec& ps, const PartIO& io, const unsigned long long* base, unsigned long long* next,
                         unsigned long long* status, uint32_t* ticket, LookLimit limit, hipStream_t s) {
  const uint32_t tile = sweep_tile(io.n);
  const dim3 grid((unsigned)((io.n + tile - 1) / tile));
  const dim3 block(kSweepThreads);
  // more than 256 partitions take wider ids, counters and ballots
  if (ps.n_parts <= 256) {
    if (tile == 2048)
      hipLaunchKernelGGL((k_part_sweep<K, E, 2, 8>), grid, block, 0, s, ps, io, base, next, status, ticket, limit);
    else
      hipLaunchKernelGGL((k_part_sweep<K, E, 8, 8>), grid, block, 0, s, ps, io, base, next, status, ticket, limit);
  } else {
    if (tile == 2048)
      hipLaunchKernelGGL((k_part_sweep<K, E, 2, 10>), grid, block, 0, s, ps, io, base, next, status, ticket, limit);
    else
      hipLaunchKernelGGL((k_part_sweep<K, E, 8, 10>), grid, block, 0, s, ps, io, base, next, status, ticket, limit);
  }
}

vx_status part_sweep(vx_ctx* ctx, const PartSpec& ps, const PartIO& io, uint8_t* work, const unsigned long long* base,
                     unsigned long long* next, hipStream_t s) {
  if (io.n == 0) {
    if (next && next != base) VX_HIP(hipMemcpyAsync(next, base, ps.n_parts * 8, hipMemcpyDeviceToDevice, s));
    return VX_OK;
  }
  VX_CHECK((io.n + 2047) / 2048 < (1ull << 31), VX_EINVAL, "partition: %llu rows in one launch", (unsigned long long)io.n);
  uint32_t* ticket = (uint32_t*)work;
  unsigned long long* status = (unsigned long long*)(work + 64);
  const LookLimit limit = look_limit(ctx);
  bool wide = io.key_size == 8;
  for (uint32_t c = 0; c < io.n_pay; ++c) wide |= io.out_pay[c] && io.pay_size[c] == 8;
  if (io.key_size == 8) launch_sweep<int64_t, 8>(ps, io, base, next, status, ticket, limit, s);
  else if (wide) launch_sweep<int32_t, 8>(ps, io, base, next, status, ticket, limit, s);
  else launch_sweep<int32_t, 4>(ps, io, base, next, status, ticket, limit, s);
  VX_HIP(hipGetLastError());
  return VX_OK;
}

// ---------------------------------------------------------------- vx_partition

static uint32_t log2_ceil(uint64_t v) {
  uint32_t r = 0;
  while ((1ull << r) < v) ++r;
  return r;
}

vx_status make_spec(vx_ctx* ctx, const vx_part_opts& o, uint32_t n_parts, const int64_t* host_split,
                    uint32_t n_split, ArenaBlock& split_mem, PartSpec* ps) {
  std::memset(ps, 0, sizeof *ps);
  if (o.method == VX_PART_RADIX_HASH || o.method == VX_PART_RADIX_BITS) {
    uint32_t l = log2_ceil(std::max<uint32_t>(n_parts, 1));
    ps->fn = o.method == VX_PART_RADIX_HASH ? kPartHash : kPartBits;
    ps->n_parts = 1u << l;
    ps->log2p = l;
    ps->shift = o.shift;
    VX_CHECK(o.method == VX_PART_RADIX_HASH || o.shift + l <= 64, VX_EINVAL,
             "partition: shift %u + %u bits exceeds 64", o.shift, l);
  } else {
    ps->fn = kPartRange;
    ps->n_parts = n_split + 1;
    ps->n_split = n_split;
    for (uint32_t i = 1; i < n_split; ++i)
      VX_CHECK(host_split[i - 1] < host_split[i], VX_EINVAL, "partition: splitters not strictly ascending");
    if (n_split) {
      split_mem.a = &ctx->arena;
      split_mem.p = ctx->arena.alloc(n_split * 8);
      VX_CHECK(split_mem.p, VX_EBUDGET, "partition: no room for splitters");
      VX_HIP(hipMemcpyAsync(split_mem.p, host_split, n_split * 8, hipMemcpyHostToDevice, ctx->compute));
      ps->splitters = (const long long*)split_mem.p;
    }
  }
  VX_CHECK(ps->n_parts >= 1 && ps->n_parts <= kMaxParts, VX_EINVAL, "partition: %u partitions (1..%u)",
           ps->n_parts, kMaxParts);
  return VX_OK;
}

static vx_status partition_impl(vx_ctx* ctx, const vx_partition_desc* d, vx_partition_out* out) {
  VX_CHECK(d->n_pay <= 4, VX_EINVAL, "partition: at most 4 payload columns");
  VX_CHECK(d->n_pay == 0 || d->pay, VX_EINVAL, "partition: pay is NULL");
  VX_CHECK(out->hist && out->boundary, VX_EINVAL, "partition: hist and boundary are required");
  const vx_part_opts& o = d->opts;
  VX_CHECK(o.method <= VX_PART_RANGE, VX_EINVAL, "partition: method %u", o.method);
  VX_HIP(hipSetDevice(ctx->device));
  const uint64_t n = d->n;
  ColInfo kc;
  VX_TRY(classify(ctx, d->key, n, &kc, "partition key"));
  ColInfo pc[4];
  for (uint32_t c = 0; c < d->n_pay; ++c) VX_TRY(classify(ctx, d->pay[c], n, &pc[c], "partition payload"));
  uint32_t req = o.n_parts;
  if (req == 0) {
    // planned: a pre-aggregating table sized from each partition's rows fits half the free arena
    uint64_t free_b = ctx->arena.largest_free() / 2;
    uint64_t per = std::max<uint64_t>(free_b / 64, 1);   // 32-byte slots at load factor 0.5
    req = (uint32_t)std::min<uint64_t>(kMaxParts, std::max<uint64_t>(2, (n + per - 1) / per));
  }
  // splitters for range methods
  std::vector<int64_t> split;
  uint32_t method_used = o.method;
  CdfReport rep{};
  if (o.method == VX_PART_RANGE) {
    VX_CHECK(o.n_splitters == 0 || o.splitters, VX_EINVAL, "partition: splitters is NULL");
    split.assign(o.splitters, o.splitters + o.n_splitters);
  } else if (o.method == VX_PART_LEARNED || o.method == VX_PART_QUANTILE ||
             o.method == VX_PART_UNTRAINED || o.method == VX_PART_AUTO) {
    VX_TRY(cdf_splitters(ctx, kc, n, o, req, &split, &rep, out->model));
    method_used = o.method;
    if (o.method == VX_PART_AUTO)
      method_used = rep.imbalance_range < rep.imbalance_radix
                        ? (rep.auto_quantile ? VX_PART_QUANTILE : VX_PART_LEARNED)
                        : VX_PART_RADIX_HASH;
  }
  vx_part_opts eff = o;
  eff.method = method_used == VX_PART_LEARNED || method_used == VX_PART_QUANTILE ||
                       method_used == VX_PART_UNTRAINED
                   ? VX_PART_RANGE
                   : method_used;
  ArenaBlock split_mem;
  PartSpec ps;
  VX_TRY(make_spec(ctx, eff, req, split.data(), (uint32_t)split.size(), split_mem, &ps));
  const uint32_t P = ps.n_parts;
  VX_CHECK(out->n_parts_cap >= P, VX_ECAPACITY, "partition: %u partitions exceed n_parts_cap %u", P,
           out->n_parts_cap);

  // device scratch: totals, then the partitions' first positions
  ArenaBlock tot_mem;
  tot_mem.a = &ctx->arena;
  tot_mem.p = ctx->arena.alloc(2 * P * 8 + 8 * (P + 1));
  VX_CHECK(tot_mem.p, VX_EBUDGET, "partition: no room for histograms");
  unsigned long long* totals = (unsigned long long*)tot_mem.p;
  unsigned long long* bnd = totals + P;

  const bool scatter = d->out_key != nullptr;
  void* out_key = d->out_key;
  void* out_pay[4] = {};
  if (scatter) {
    // outputs may be device memory or pinned host memory (written by zero-copy stores)
    vx_col oc{d->out_key, d->key.type, 0};
    ColInfo oi;
    VX_TRY(classify(ctx, oc, n, &oi, "partition output key"));
    out_key = const_cast<void*>(oi.dev);
    for (uint32_t c = 0; c < d->n_pay; ++c) {
      VX_CHECK(d->out_pay && d->out_pay[c], VX_EINVAL, "partition: out_pay[%u] is NULL", c);
      vx_col pcol{d->out_pay[c], d->pay[c].type, 0};
      ColInfo pi;
      VX_TRY(classify(ctx, pcol, n, &pi, "partition output payload"));
      out_pay[c] = const_cast<void*>(pi.dev);
    }
  }

  // the counts land in host_acc (mapped), where the host reads them after the stream is drained
  const unsigned long long* h = (const unsigned long long*)ctx->host_acc;
  unsigned long long* h_dev = (unsigned long long*)ctx->host_acc_dev;
  for (uint32_t p = 0; p < P; ++p) ctx->host_acc[p] = 0;
  // Pass A counts every chunk; pass B scatters it from the running position of each partition.  A
  // single chunk needs no second look at its rows: its counts give the positions at once.
  bool counted_all = false;   // the first pass sweeps the only chunk too
  auto run_pass = [&](bool do_scatter) -> vx_status {
    std::vector<PipeCol> cols(1 + (scatter ? d->n_pay : 0));
    cols[0].info = kc;
    cols[0].may_copy = cols[0].copy = true;
    for (uint32_t c = 0; scatter && c < d->n_pay; ++c) {
      cols[1 + c].info = pc[c];
      cols[1 + c].may_copy = cols[1 + c].copy = do_scatter;
    }
    bool device = true;
    for (uint32_t c = 0; c < d->n_pay; ++c) device &= pc[c].where == Where::Device;
    const bool resident = kc.where == Where::Device && (device || !do_scatter);   // nothing to stream
    ArenaBlock wmem;
    wmem.a = &ctx->arena;
    std::unique_ptr<Pipeline> pipe;   // gone before wmem: it drains the streams
    for (uint64_t rows = resident ? std::min(n, kPartLaunchRows) : 0;; rows = pipe->chunk_rows() / 2) {
      pipe.reset(new Pipeline);
      VX_TRY(pipe->plan(ctx, n, rows, 0, cols));
      if (!do_scatter) counted_all = scatter && device && pipe->n_chunks() == 1 && !pipe->streamed();
      wmem.p = ctx->arena.alloc(part_work_bytes(P, pipe->chunk_rows(), do_scatter || counted_all));
      if (wmem.p) break;
      VX_CHECK(pipe->chunk_rows() > 1024, VX_EBUDGET, "partition: no room for the partition scratch");
    }
    auto kernel = [&](const ChunkView& v) -> vx_status {
      PartIO io{};
      io.key = (v.global_mask & 1u) ? (const uint8_t*)v.ptr[0] + v.row0 * kc.elsize : v.ptr[0];
      io.key_size = (uint32_t)kc.elsize;
      io.n = v.rows;
      if (!do_scatter)
        VX_TRY(part_count(ctx, ps, io, wmem.p, totals, v.index > 0, bnd, h_dev, nullptr, nullptr, ctx->compute,
                          counted_all));
      if (!do_scatter && !counted_all) return VX_OK;
      io.n_pay = d->n_pay;
      for (uint32_t c = 0; c < d->n_pay; ++c) {
        io.pay[c] = ((v.global_mask >> (1 + c)) & 1u) ? (const uint8_t*)v.ptr[1 + c] + v.row0 * pc[c].elsize
                                                      : v.ptr[1 + c];
        io.pay_size[c] = (uint32_t)pc[c].elsize;
        io.out_pay[c] = out_pay[c];
      }
      io.out_key = out_key;
      io.out_base = 0;
      if (do_scatter) VX_TRY(part_ready(ps, v.rows, wmem.p, ctx->compute));
      return part_sweep(ctx, ps, io, wmem.p, bnd, bnd, ctx->compute);
    };
    VX_TRY(pipe->run(kernel));
    VX_HIP(hipStreamSynchronize(ctx->compute));
    return VX_OK;
  };
  VX_TRY(run_pass(false));
  std::vector<unsigned long long> b(P + 1, 0);
  for (uint32_t p = 0; p < P; ++p) b[p + 1] = b[p] + h[p];
  if (scatter && !counted_all) VX_TRY(run_pass(true));
  VX_TRY(check_stall(ctx, "partition"));
  for (uint32_t p = 0; p < P; ++p) out->hist[p] = h[p];
  for (uint32_t p = 0; p <= P; ++p) out->boundary[p] = b[p];
  out->n_parts = P;
  out->method_used = method_used;
  out->n_splitters = (uint32_t)split.size();
  if (out->splitters && ps.fn == kPartRange)
    for (size_t i = 0; i < split.size() && i < out->n_parts_cap; ++i) out->splitters[i] = split[i];
  double mx = 0;
  for (uint32_t p = 0; p < P; ++p) mx = std::max(mx, (double)h[p]);
  out->imbalance = n ? mx / ((double)n / P) : 0.0;
  out->est_imbalance_radix = rep.imbalance_radix;
  out->est_imbalance_range = rep.imbalance_range;
  out->final_loss = rep.final_loss;
  return VX_OK;
}

}  // namespace vx

extern "C" vx_status vx_partition(vx_ctx* ctx, const vx_partition_desc* d, vx_partition_out* out) {
  VX_CHECK(ctx && d && out, VX_EINVAL, "vx_partition: null argument");
  vx::release_cached(ctx);
  return vx::partition_impl(ctx, d, out);
}
