// Star join with GROUP BY.
//
// The dimension tables are filtered and hashed on the GPU and stay resident; the fact table
// is streamed (the paper's star-schema plan).  Once the dimension tables are built, the
// fraction of rows that passed each filter is the selectivity estimate of the matching fact
// foreign key; dimensions are probed in ascending selectivity, so each later column is read
// only for rows still alive.  The first probed foreign key is streamed through the chunk
// pipeline; each other fact column is streamed too or read by zero-copy for the surviving
// rows only, chosen from the running selectivity before the scan starts (late
// materialization).  Survivors are aggregated into a device group table with 64-bit atomics.
#include <algorithm>
#include <cstring>
#include <numeric>

#include "vx_device.h"
#include "vx_pipeline.h"

namespace vx {


// ---------------------------------------------------------------- dimension build

// One dimension of the launch that builds them all.
struct DimArgs {
  TableView t;                // the filtered rows' table
  const void *key, *filt, *grp;
  uint32_t filt_size;
  long long lo, hi;
  uint64_t n;
  uint8_t* present;           // direct tables: a byte per key of the range, set for every row; or null
                              // (the keys have been checked by a table of their own)
  unsigned long long* passed;
  unsigned long long* filled; // the set bytes, counted by k_dims_count
};
struct DimList {
  DimArgs d[4];
};

// Dimension blockIdx.y: the rows that pass the filter go into its table, with plain stores in a direct
// one.  A repeated key (of any row) leaves a presence byte of a direct table's range unset, which
// k_dims_count finds; hashed dimensions are checked by an insert of every key beforehand.  The rows
// that pass are counted with one atomic per workgroup (one per wave took 54 of this build's 55 us for
// 300,000 rows: they all add to one word).
template <typename K>
__global__ void __launch_bounds__(256) k_build_dims(DimList list, unsigned int* flags) {
  using U = typename KeyTraits<K>::U;
  const U kEmpty = KeyTraits<K>::kEmpty;
  const DimArgs& a = list.d[blockIdx.y];
  const TableView& t = a.t;
  __shared__ uint32_t wpass[4];
  uint32_t passed = 0;
  for (uint64_t i = blockIdx.x * 256ull + threadIdx.x; i < a.n; i += gridDim.x * 256ull) {
    const long long f = load_signed(a.filt, i, a.filt_size);
    const bool pass = f >= a.lo && f <= a.hi;
    passed += pass;
    const K k = load_key<K>(a.key, i);
    const U kb = (U)k;
    if (kb == kEmpty) {
      if (pass) {
        atomicAdd(t.side, 1ull);
        if (a.grp) atomicAdd(t.side + 1, (unsigned long long)(long long)((const int*)a.grp)[i]);
      }
      continue;
    }
    uint64_t h;
    if (!first_slot(t, k, h)) {    // cannot happen: the range was measured over every dimension row
      atomicOr(flags, kFlagFull);
      continue;
    }
    if (t.direct) {
      if (a.present) a.present[h] = 1;
      if (pass) {
        uint8_t* slot = t.slots + (h << t.slot_shift);
        *(U*)slot = kb;
        if (a.grp) *(int*)(slot + t.pay_off[0]) = ((const int*)a.grp)[i];
      }
      continue;
    }
    if (!pass) continue;
    bool done = false;
    for (uint64_t step = 0; step <= t.mask; ++step) {
      uint8_t* slot = t.slots + (h << t.slot_shift);
      U prev = atomicCAS((U*)slot, kEmpty, kb);
      if (prev == kEmpty) {
        if (a.grp) *(int*)(slot + t.pay_off[0]) = ((const int*)a.grp)[i];
        done = true;
        break;
      }
      if (prev == kb) {
        atomicOr(flags, kFlagDup);
        done = true;
        break;
      }
      h = (h + 1) & t.mask;
    }
    if (!done) atomicOr(flags, kFlagFull);
  }
  for (int o = 32; o > 0; o >>= 1) passed += __shfl_xor(passed, o, 64);
  if ((threadIdx.x & 63) == 0) wpass[threadIdx.x >> 6] = passed;
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t c = wpass[0] + wpass[1] + wpass[2] + wpass[3];
    if (c) atomicAdd(a.passed, (unsigned long long)c);
  }
}

// The set presence bytes of dimension blockIdx.y (direct tables).
__global__ void __launch_bounds__(256) k_dims_count(DimList list) {
  const DimArgs& a = list.d[blockIdx.y];
  if (!a.present) return;   // uniform
  __shared__ uint32_t part[4];
  uint32_t c = 0;
  const uint64_t range = a.t.direct_range, words = range / 4;
  for (uint64_t w = blockIdx.x * 256ull + threadIdx.x; w < words; w += gridDim.x * 256ull)
    c += (uint32_t)__popc(((const uint32_t*)a.present)[w]);   // the bytes are 0 or 1
  for (uint64_t b = words * 4 + blockIdx.x * 256ull + threadIdx.x; b < range; b += gridDim.x * 256ull) c += a.present[b];
  for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    c = part[0] + part[1] + part[2] + part[3];
    if (c) atomicAdd(a.filled, (unsigned long long)c);
  }
}

// One wave: `words` device words and the flags after them, to where the host reads them.
__global__ void __launch_bounds__(64) k_star_publish(const unsigned long long* src, uint32_t words,
                                                     const unsigned int* flags, unsigned long long* host) {
  if (threadIdx.x < words) host[threadIdx.x] = src[threadIdx.x];
  else if (threadIdx.x == words) host[words] = *flags;
}

// ---------------------------------------------------------------- group table

// Slot: key (8), count (8), sums (4 x 8), padding -> 64 bytes.  Key = (u32)g0 << 32 | (u32)g1;
// all-ones marks an empty slot, so group (-1, -1) lives in the side record after the slots.
struct GroupTable {
  unsigned long long* slots;
  uint64_t mask;
  uint32_t log2cap;
  uint32_t n_meas;
};
constexpr unsigned long long kGroupEmpty = ~0ull;
constexpr int kGroupWords = 8;

// The groups with rows, to host memory: key, count, sums, in no particular order (the group of the side
// record gets its key); *n counts them, also those past `cap`.
__global__ void __launch_bounds__(256) k_star_groups(GroupTable g, unsigned long long* n, uint64_t cap,
                                                     unsigned long long* host) {
  for (uint64_t i = blockIdx.x * 256ull + threadIdx.x; i <= g.mask + 1; i += gridDim.x * 256ull) {
    const unsigned long long* w = g.slots + i * kGroupWords;
    if (w[1] == 0) continue;
    const unsigned long long at = atomicAdd(n, 1ull);
    if (at >= cap) continue;
    unsigned long long* o = host + at * kGroupWords;
    o[0] = i == g.mask + 1 ? kGroupEmpty : w[0];
#pragma unroll
    for (int k = 1; k < 6; ++k) o[k] = w[k];
  }
}

__device__ __forceinline__ void group_add(const GroupTable& g, unsigned long long key,
                                          const long long* meas, unsigned int* flags) {
  unsigned long long* w = nullptr;
  if (key == kGroupEmpty) {
    w = g.slots + (g.mask + 1) * kGroupWords;   // side record
  } else {
    uint64_t h = slot_of(key, g.log2cap);
    for (uint64_t step = 0; step <= g.mask; ++step) {
      unsigned long long* s = g.slots + h * kGroupWords;
      unsigned long long prev = atomicCAS(s, kGroupEmpty, key);
      if (prev == kGroupEmpty || prev == key) {
        w = s;
        break;
      }
      h = (h + 1) & g.mask;
    }
    if (!w) {
      atomicOr(flags, kFlagGroupOverflow);
      return;
    }
  }
  atomicAdd(w + 1, 1ull);
  for (uint32_t m = 0; m < g.n_meas; ++m) atomicAdd(w + 2 + m, (unsigned long long)meas[m]);
}

// ---------------------------------------------------------------- fact scan

struct StarArgs {
  uint32_t n_dims;
  uint32_t n_meas;
  TableView dim[4];            // probe order
  int gsel[4];                 // -1: no group; 0 / 1: writes g0 / g1
  const void* fk[4];           // probe order; chunk-local unless fk_global bit set
  uint32_t fk_global;
  const void* meas[4];
  uint32_t meas_size[4];
  uint32_t meas_global;
  uint64_t n, row0;
  GroupTable groups;
  unsigned int* flags;
  unsigned long long* survivors;   // [0] fact rows that pass every dimension, [1] zero-copy granules
  uint32_t fk_zc, meas_zc;         // bit set: the column is host memory read in place (count granules)
  uint32_t zc_shift;               // log2 of the zero-copy granule in bytes
};

// COUNT: count the zero-copy granules of the gathers (compiled in only when asked for).
template <typename K, int kStarItems, bool COUNT>
__global__ void __launch_bounds__(256) k_star(StarArgs a) {
  using U = typename KeyTraits<K>::U;
  const U kEmpty = KeyTraits<K>::kEmpty;
  unsigned long long alive_count = 0, granules = 0;
  const uint64_t tile = (uint64_t)blockDim.x * kStarItems;
  const uint64_t wave_row = threadIdx.x & ~63u;
  for (uint64_t base = blockIdx.x * tile; base < a.n; base += (uint64_t)gridDim.x * tile) {
    bool alive[kStarItems];
    int g[kStarItems][2];
#pragma unroll
    for (int j = 0; j < kStarItems; ++j) {
      alive[j] = base + (uint64_t)j * blockDim.x + threadIdx.x < a.n;
      g[j][0] = g[j][1] = 0;
    }
    for (uint32_t d = 0; d < a.n_dims; ++d) {
      const bool glob = (a.fk_global >> d) & 1u;
      K fk[kStarItems];
#pragma unroll
      for (int j = 0; j < kStarItems; ++j) {
        uint64_t i = base + (uint64_t)j * blockDim.x + threadIdx.x;
        fk[j] = 0;
        if (alive[j]) {
          if (d == 0 && !glob) fk[j] = __builtin_nontemporal_load(((const K*)a.fk[0]) + i);
          else fk[j] = load_key<K>(a.fk[d], glob ? a.row0 + i : i);
        }
      }
      if (COUNT && ((a.fk_zc >> d) & 1u)) {
#pragma unroll
        for (int j = 0; j < kStarItems; ++j) {
          const uint64_t r0 = a.row0 + base + (uint64_t)j * blockDim.x + wave_row;
          granules += wave_granules(alive[j], (uint64_t)(uintptr_t)a.fk[d] + r0 * sizeof(K), sizeof(K), a.zc_shift);
        }
      }
#pragma unroll
      for (int j = 0; j < kStarItems; ++j) {
        if (!alive[j]) continue;
        const TableView& t = a.dim[d];
        int grp = 0;
        bool found;
        if ((U)fk[j] == kEmpty) {
          found = t.side[0] != 0;
          grp = (int)t.side[1];
        } else {
          const uint8_t* s = find_slot<K>(t, fk[j]);
          found = s != nullptr;
          if (found && t.n_pay) grp = *(const int*)(s + t.pay_off[0]);
        }
        alive[j] = found;
        if (found && a.gsel[d] >= 0) g[j][a.gsel[d]] = grp;
      }
    }
    for (uint32_t c = 0; COUNT && c < a.n_meas; ++c) {
      if (!((a.meas_zc >> c) & 1u)) continue;
#pragma unroll
      for (int j = 0; j < kStarItems; ++j) {
        const uint64_t r0 = a.row0 + base + (uint64_t)j * blockDim.x + wave_row;
        granules += wave_granules(alive[j], (uint64_t)(uintptr_t)a.meas[c] + r0 * a.meas_size[c], a.meas_size[c],
                                  a.zc_shift);
      }
    }
#pragma unroll
    for (int j = 0; j < kStarItems; ++j) {
      if (!alive[j]) continue;
      uint64_t i = base + (uint64_t)j * blockDim.x + threadIdx.x;
      long long m[4] = {0, 0, 0, 0};
      for (uint32_t c = 0; c < a.n_meas; ++c)
        m[c] = load_signed(a.meas[c], ((a.meas_global >> c) & 1u) ? a.row0 + i : i, a.meas_size[c]);
      unsigned long long key = ((unsigned long long)(unsigned int)g[j][0] << 32) |
                               (unsigned long long)(unsigned int)g[j][1];
      group_add(a.groups, key, m, a.flags);
      ++alive_count;
    }
  }
  for (int o = 32; o > 0; o >>= 1) alive_count += __shfl_xor(alive_count, o, 64);
  if ((threadIdx.x & 63) == 0 && alive_count) atomicAdd(a.survivors, alive_count);
  // every lane holds its wave's granule count
  if (COUNT && (threadIdx.x & 63) == 0 && granules) atomicAdd(a.survivors + 1, granules);
}

// ---------------------------------------------------------------- host side

template <int ITEMS>
static void launch_star(bool k64, bool count, unsigned g, const StarArgs& a, hipStream_t s) {
  if (k64) {
    if (count) hipLaunchKernelGGL((k_star<int64_t, ITEMS, true>), dim3(g), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((k_star<int64_t, ITEMS, false>), dim3(g), dim3(256), 0, s, a);
  } else {
    if (count) hipLaunchKernelGGL((k_star<int32_t, ITEMS, true>), dim3(g), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((k_star<int32_t, ITEMS, false>), dim3(g), dim3(256), 0, s, a);
  }
}

// rows per lane in flight in the fact scan (VX_STAR_ITEMS = 4 or 8; default 8)
static int star_items() {
  const char* e = getenv("VX_STAR_ITEMS");
  return e && atoi(e) == 4 ? 4 : 8;
}

vx_status join_star(vx_ctx* ctx, const vx_star_join* d, vx_join_out* out) {
  double t0 = now_ms();
  VX_CHECK(d->n_dims >= 1 && d->n_dims <= 4, VX_EINVAL, "star: n_dims %u outside 1..4", d->n_dims);
  VX_CHECK(d->n_measures <= 4, VX_EINVAL, "star: n_measures %u > 4", d->n_measures);
  VX_CHECK(d->late_mat >= -1 && d->late_mat <= 2, VX_EINVAL, "star: late_mat %d", d->late_mat);
  VX_CHECK(d->groups != nullptr || d->groups_cap == 0, VX_EINVAL, "star: groups is NULL");
  VX_CHECK((d->flags & ~(uint32_t)VX_PROBE_COUNT_ZC) == 0, VX_EINVAL, "star: unknown flags %u", d->flags);
  const bool count_zc = (d->flags & VX_PROBE_COUNT_ZC) != 0;
  const int32_t ktype = d->dims[0].key.type;
  const uint32_t nd = d->n_dims;
  VX_HIP(hipSetDevice(ctx->device));
  for (uint32_t k = 0; k < nd; ++k) {
    VX_CHECK(d->dims[k].key.type == ktype && d->fact_fk[k].type == ktype, VX_EINVAL,
             "star: dimension keys and fact foreign keys must share one type");
    VX_CHECK(d->dims[k].group.data == nullptr || d->dims[k].group.type == VX_I32, VX_EINVAL,
             "star: group attributes must be VX_I32");
  }
  // group attribute slots: the first two dimensions (in dimension order) that carry one
  int gsel_dim[4] = {-1, -1, -1, -1};
  int ng = 0;
  for (uint32_t k = 0; k < nd; ++k)
    if (d->dims[k].group.data && ng < 2) gsel_dim[k] = ng++;

  // group table: 2 * groups_cap slots, as 64-byte records, and the side record
  const uint64_t want = std::max<uint64_t>(1024, 2 * std::max<uint64_t>(d->groups_cap, 1));
  uint64_t gcap = 1;
  while (gcap < want) gcap <<= 1;
  const uint64_t gwords = (gcap + 1) * kGroupWords;

  // dimension tables: uniqueness over all rows, and the filtered table
  struct Dim {
    vx_table* t = nullptr;
    double sel = 1.0;
    ColInfo key, filt, grp{};
    KeyRange range;
    ArenaBlock present;
  } dims[4];
  auto free_dims = [&]() {
    for (uint32_t k = 0; k < nd; ++k) {
      dims[k].present.reset();
      if (dims[k].t) {
        ctx->arena.release(dims[k].t->mem);
        delete dims[k].t;
        dims[k].t = nullptr;
      }
    }
  };
  vx_stats s{};
  // device words: [0] survivors, [1] granules, [2] groups; per dimension from kDimWords on: rows passed,
  // presence bytes set
  constexpr uint32_t kDimWords = 8, kDimCounters = 8;
  unsigned long long* words = (unsigned long long*)ctx->dev_acc;
  // Device-resident keys that fill a narrow range get direct tables (slot = key - min): the ranges of
  // all the dimensions are measured before one wait, and their tables and checks take one launch each
  // (a launch and a wait for every step of every dimension made a join of 12,000,007 host fact rows with
  // dimensions of 2,556, 20,000, 300,000 and 200,000 take 3.11 ms; it takes 2.56).
  bool measured = false;
  // Every row of dimension k into a table of its own that goes again: the uniqueness check without
  // presence bytes.
  auto check_unique = [&](uint32_t k) -> vx_status {
    vx_table* u = nullptr;
    VX_TRY(make_table(ctx, ktype, VX_UNIQUE, nullptr, 0, d->dims[k].n, 0.5f, &u, &dims[k].range));
    const vx_status st = table_insert(ctx, u, dims[k].key, nullptr, d->dims[k].n, ctx->compute, 1);
    ctx->arena.release(u->mem);   // whoever gets the memory next fills it on the same stream
    delete u;
    return st;
  };
  // Dimensions [k0, k1), their tables and presence bytes held together; `tight`: each checked before its
  // table is made, in no more memory than the larger of the two.
  auto build_dims = [&](uint32_t k0, uint32_t k1, bool tight) -> vx_status {
    for (uint32_t k = 0; k < nd && !measured; ++k) {
      const vx_star_dim& sd = d->dims[k];
      VX_TRY(classify(ctx, sd.key, sd.n, &dims[k].key, "star dimension key"));
      VX_TRY(classify(ctx, sd.filter, sd.n, &dims[k].filt, "star dimension filter"));
      if (sd.group.data) VX_TRY(classify(ctx, sd.group, sd.n, &dims[k].grp, "star dimension group"));
      if (dims[k].key.where != Where::Device || sd.n == 0) continue;
      VX_TRY(key_range_launch(ctx, ktype, dims[k].key.dev, sd.n, k));
    }
    if (!measured) {
      VX_HIP(hipStreamSynchronize(ctx->compute));
      for (uint32_t k = 0; k < nd; ++k)
        if (dims[k].key.where == Where::Device) key_range_collect(ctx, d->dims[k].n, k, &dims[k].range);
      measured = true;
    }
    FillList fills;
    fills.zero(words, (kDimWords + kDimCounters) * 8);
    if (tight) {
      fill_zero((uint64_t*)ctx->dev_flags, 1, ctx->compute);
      for (uint32_t k = k0; k < k1; ++k) VX_TRY(check_unique(k));
    } else {
      fills.zero(ctx->dev_flags, kFlagBytes);
    }
    DimList list{};
    uint64_t most = 0;
    for (uint32_t k = k0; k < k1; ++k) {
      const vx_star_dim& sd = d->dims[k];
      int32_t pt[1] = {VX_I32};
      // worst case every row passes; size the table for all rows
      VX_TRY(make_table(ctx, ktype, VX_UNIQUE, pt, sd.group.data ? 1 : 0, sd.n, 0.5f, &dims[k].t, &dims[k].range,
                        &fills));
      s.table_bytes += dims[k].t->bytes;
    }
    // the presence bytes after every table: they go again before the group table and the chunk buffers are
    // made, which may need the room in one piece
    for (uint32_t k = k0; k < k1; ++k) {
      const vx_star_dim& sd = d->dims[k];
      const TableView& v = dims[k].t->view;
      if (v.direct && !tight) {
        const uint64_t bytes = (v.direct_range + 255) / 256 * 256;
        dims[k].present.a = &ctx->arena;
        dims[k].present.p = ctx->arena.alloc(bytes);
        VX_CHECK(dims[k].present.p, VX_EBUDGET, "star: no room for the presence bytes of a dimension's keys");
        fills.zero(dims[k].present.p, bytes);
      }
      DimArgs& a = list.d[k - k0];
      a.t = v;
      a.key = dims[k].key.dev;
      a.filt = dims[k].filt.dev;
      a.grp = sd.group.data ? dims[k].grp.dev : nullptr;
      a.filt_size = (uint32_t)dims[k].filt.elsize;
      a.lo = (long long)sd.lo;
      a.hi = (long long)sd.hi;
      a.n = sd.n;
      a.present = dims[k].present.p;
      a.passed = words + kDimWords + 2 * k;
      a.filled = a.passed + 1;
      most = std::max(most, sd.n);
    }
    VX_TRY(fills.launch(ctx->compute));
    for (uint32_t k = k0; k < k1 && !tight; ++k)
      if (!dims[k].t->view.direct) VX_TRY(check_unique(k));
    if (most) {
      const dim3 g((unsigned)std::min<uint64_t>((most + 1023) / 1024, (uint64_t)ctx->cu_count * 4), k1 - k0);
      if (ktype == VX_I64) hipLaunchKernelGGL(k_build_dims<int64_t>, g, dim3(256), 0, ctx->compute, list, ctx->dev_flags);
      else hipLaunchKernelGGL(k_build_dims<int32_t>, g, dim3(256), 0, ctx->compute, list, ctx->dev_flags);
      const dim3 gc((unsigned)std::min<uint64_t>((most + 8191) / 8192, (uint64_t)ctx->cu_count), k1 - k0);
      if (!tight) hipLaunchKernelGGL(k_dims_count, gc, dim3(256), 0, ctx->compute, list);
    }
    unsigned long long* host = (unsigned long long*)ctx->host_small;
    hipLaunchKernelGGL(k_star_publish, dim3(1), dim3(64), 0, ctx->compute, words + kDimWords, kDimCounters,
                       ctx->dev_flags, (unsigned long long*)ctx->host_small_dev);
    VX_HIP(hipGetLastError());
    VX_HIP(hipStreamSynchronize(ctx->compute));
    unsigned int flags = (unsigned int)host[kDimCounters];
    for (uint32_t k = k0; k < k1; ++k) {
      const uint64_t n = d->dims[k].n;
      const bool counted = dims[k].present.p != nullptr;
      if (counted && host[2 * k + 1] + dims[k].range.empty_rows != n) flags |= kFlagDup;
      if (counted && dims[k].range.empty_rows > 1) flags |= kFlagDup;
      dims[k].t->n_rows = host[2 * k];
      dims[k].sel = n ? (double)host[2 * k] / (double)n : 0.0;
    }
    return flags_status(flags, "star dimension");
  };
  {
    vx_status st = build_dims(0, nd, false);
    if (st == VX_EBUDGET && measured) {
      (void)hipStreamSynchronize(ctx->compute);
      free_dims();
      s.table_bytes = 0;
      st = VX_OK;
      for (uint32_t k = 0; k < nd && st == VX_OK; ++k) st = build_dims(k, k + 1, true);
    }
    if (st != VX_OK) {
      (void)hipStreamSynchronize(ctx->compute);
      free_dims();
      return st;
    }
  }
  for (uint32_t k = 0; k < nd; ++k) dims[k].present.reset();
  s.build_ms = now_ms() - t0;

  // probe order: ascending estimated selectivity (stable)
  uint32_t order[4];
  std::iota(order, order + nd, 0u);
  std::stable_sort(order, order + nd, [&](uint32_t a, uint32_t b) { return dims[a].sel < dims[b].sel; });

  // pipeline columns: FKs in probe order, then measures
  std::vector<PipeCol> cols(nd + d->n_measures);
  std::vector<double> col_sel(cols.size());
  double run = 1.0;
  for (uint32_t k = 0; k < nd; ++k) {
    uint32_t dk = order[k];
    vx_status st = classify(ctx, d->fact_fk[dk], d->n_fact, &cols[k].info, "star fact key");
    if (st != VX_OK) {
      free_dims();
      return st;
    }
    col_sel[k] = run;
    run *= dims[dk].sel;
  }
  for (uint32_t c = 0; c < d->n_measures; ++c) {
    vx_status st = classify(ctx, d->measure[c], d->n_fact, &cols[nd + c].info, "star measure");
    if (st != VX_OK) {
      free_dims();
      return st;
    }
    col_sel[nd + c] = run;
  }
  for (size_t c = 0; c < cols.size(); ++c) {
    bool zc;
    int es = cols[c].info.elsize;
    if (c == 0) zc = false;                         // the first probed key is always streamed
    else if (d->late_mat == VX_LATE_SDMA) zc = false;
    else if (d->late_mat == VX_LATE_ZC) zc = true;
    else if (d->late_mat == VX_LATE_PAPER) zc = col_sel[c] < (double)es / (double)ctx->zc_line;
    else zc = zc_wire_bytes(1000000, (uint64_t)(col_sel[c] * 1e6), es, ctx->zc_line) / 1e6 < 0.95 * es;
    cols[c].copy = cols[c].may_copy = !zc;
  }

  // group table
  ArenaBlock gblock;
  gblock.a = &ctx->arena;
  gblock.p = ctx->arena.alloc(gwords * 8);
  if (!gblock.p) {
    free_dims();
    set_error("star: group table of %llu slots does not fit the arena", (unsigned long long)gcap);
    return VX_EBUDGET;
  }
  GroupTable gt{(unsigned long long*)gblock.p, gcap - 1, 0, d->n_measures};
  while ((1ull << gt.log2cap) < gcap) ++gt.log2cap;
  FillList ginit;
  ginit.pattern(gt.slots, gwords * 8, kGroupWords * 2, ~0u, ~0u);
  if (ginit.launch(ctx->compute) != VX_OK) {
    free_dims();
    return VX_EHIP;
  }
  unsigned long long* survivors = words;   // zero since the dimensions' build, as are the flags

  StarArgs base{};
  base.n_dims = nd;
  base.n_meas = d->n_measures;
  for (uint32_t k = 0; k < nd; ++k) {
    base.dim[k] = dims[order[k]].t->view;
    base.gsel[k] = gsel_dim[order[k]];
  }
  for (uint32_t c = 0; c < d->n_measures; ++c) base.meas_size[c] = (uint32_t)cols[nd + c].info.elsize;
  base.groups = gt;
  base.flags = ctx->dev_flags;
  base.survivors = survivors;
  while ((2u << base.zc_shift) <= ctx->zc_line) ++base.zc_shift;

  vx_status status;
  double tp0 = now_ms();
  uint64_t n_chunks = 0, chunk_rows = 0, sdma = 0, kl = 0;
  double kms = 0;
  uint32_t nbuf = 0;
  bool streamed = false;
  {
    Pipeline pipe;
    status = pipe.plan(ctx, d->n_fact, d->chunk_rows, 0, cols);
    if (status == VX_OK) {
      auto kernel = [&](const ChunkView& v) -> vx_status {
        StarArgs a = base;
        a.n = v.rows;
        a.row0 = v.row0;
        for (uint32_t k = 0; k < nd; ++k) {
          a.fk[k] = v.ptr[k];
          if ((v.global_mask >> k) & 1u) {
            a.fk_global |= 1u << k;
            if (cols[k].info.where == Where::Host) a.fk_zc |= 1u << k;
          }
        }
        for (uint32_t c = 0; c < d->n_measures; ++c) {
          a.meas[c] = v.ptr[nd + c];
          if ((v.global_mask >> (nd + c)) & 1u) {
            a.meas_global |= 1u << c;
            if (cols[nd + c].info.where == Where::Host) a.meas_zc |= 1u << c;
          }
        }
        if (a.n == 0) return VX_OK;
        const int items = star_items();
        unsigned g = (unsigned)std::min<uint64_t>((a.n + 256 * items - 1) / (256 * items),
                                                  (uint64_t)ctx->cu_count * 8);
        if (items == 8) launch_star<8>(ktype == VX_I64, count_zc, g, a, ctx->compute);
        else launch_star<4>(ktype == VX_I64, count_zc, g, a, ctx->compute);
        VX_HIP(hipGetLastError());
        return VX_OK;
      };
      status = pipe.run(kernel);
      if (status == VX_OK) {
        VX_HIP(hipStreamSynchronize(ctx->compute));
        n_chunks = pipe.n_chunks();
        chunk_rows = pipe.chunk_rows();
        sdma = pipe.sdma_bytes();
        kms = pipe.kernel_ms();
        kl = pipe.kernel_launches();
        nbuf = pipe.n_buffers();
        streamed = pipe.streamed();
      }
    }
  }
  // groups back to the host: compacted by the GPU, or (more than host_acc holds) the whole table
  const uint64_t host_cap = ctx->dev_acc_words / kGroupWords;
  if (status == VX_OK) {
    const unsigned g = (unsigned)std::min<uint64_t>((gcap + 256) / 256, (uint64_t)ctx->cu_count * 4);
    hipLaunchKernelGGL(k_star_groups, dim3(g), dim3(256), 0, ctx->compute, gt, words + 2, host_cap,
                       (unsigned long long*)ctx->host_acc_dev);
    hipLaunchKernelGGL(k_star_publish, dim3(1), dim3(64), 0, ctx->compute, words, 3u, ctx->dev_flags,
                       (unsigned long long*)ctx->host_small_dev);
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(ctx->compute) != hipSuccess) {
      set_error("star: reading the group table failed");
      status = VX_EHIP;
    }
  }
  if (status == VX_OK) status = flags_status((unsigned int)ctx->host_small[3], "star");
  if (status != VX_OK) {
    free_dims();
    return status;
  }
  const unsigned long long nsurv[2] = {ctx->host_small[0], ctx->host_small[1]};
  const uint64_t n_found = ctx->host_small[2];
  const unsigned long long* host = (const unsigned long long*)ctx->host_acc;
  std::vector<unsigned long long> whole;
  if (n_found > host_cap) {
    whole.resize(gwords);
    if (hipMemcpy(whole.data(), gt.slots, gwords * 8, hipMemcpyDeviceToHost) != hipSuccess) {
      free_dims();
      set_error("star: reading the group table failed");
      return VX_EHIP;
    }
    host = whole.data();
  }
  free_dims();
  std::vector<vx_group_row> rows;
  for (uint64_t i = 0; i < (whole.empty() ? n_found : gcap + 1); ++i) {
    const unsigned long long* w = host + i * kGroupWords;
    if (w[1] == 0) continue;
    unsigned long long key = !whole.empty() && i == gcap ? kGroupEmpty : w[0];
    vx_group_row r{};
    r.g0 = (int32_t)(uint32_t)(key >> 32);
    r.g1 = (int32_t)(uint32_t)(key & 0xffffffffull);
    r.count = w[1];
    for (uint32_t m = 0; m < 4; ++m) r.sum[m] = m < d->n_measures ? w[2 + m] : 0;
    rows.push_back(r);
  }
  std::sort(rows.begin(), rows.end(), [](const vx_group_row& a, const vx_group_row& b) {
    return a.g0 != b.g0 ? a.g0 < b.g0 : a.g1 < b.g1;
  });
  out->n_groups = rows.size();
  s.rows = d->n_fact;
  s.chunks = streamed ? n_chunks : 0;
  s.chunk_rows = chunk_rows;
  s.n_buffers = streamed ? nbuf : 0;
  s.sdma_bytes = sdma;
  s.kernel_ms = kms;
  s.kernel_launches = kl;
  for (size_t c = 0; c < cols.size(); ++c) {
    if (cols[c].info.where != Where::Host || cols[c].copy) continue;
    s.zc_mask |= 1u << c;
    if (!count_zc)   // not counted: the wire model's estimate from the estimated selectivities
      s.zc_bytes += (uint64_t)zc_wire_bytes(d->n_fact, (uint64_t)(col_sel[c] * d->n_fact), cols[c].info.elsize,
                                            ctx->zc_line);
  }
  if (count_zc) {
    s.zc_bytes = nsurv[1] << base.zc_shift;   // counted granules x granule
    s.zc_counted = s.zc_mask ? 1u : 0u;
  }
  s.probe_ms = now_ms() - tp0;
  s.total_ms = now_ms() - t0;
  s.survivors = nsurv[0];
  out->stats = s;
  VX_CHECK(rows.size() <= d->groups_cap, VX_ECAPACITY, "star: %zu groups exceed groups_cap %llu",
           rows.size(), (unsigned long long)d->groups_cap);
  std::copy(rows.begin(), rows.end(), d->groups);
  return VX_OK;
}

}  // namespace vx
