// Table lifecycle (Gleam Sec. 4.1.3: identified weight chunks stay in a shared cache
// across tasks, and LRU eviction keeps that cache bounded for long-lived multi-task
// serving; Sec. 4.1.2: the server ships the identifiers it holds at connect time).
//
//   touch   stamp present keys with max(stamp, epoch): the "use" of an entry
//   evict   keep the `keep` most recently used entries; order = (stamp, key) ascending
//   erase   remove the given keys
//   export  every entry, sorted by key (the identifier set, or a checkpoint)
//
// Both orders are of distinct keys, so they do not depend on where keys sit in the table.
// Evict looks for its victims by selection: a histogram over the range of (stamp, key)
// finds the bin that the last victim falls in, the entries up to that bin are gathered
// (about as many as are evicted) and only those are sorted, by the library's radix sort
// (radix_sort.h). Export sorts every entry (also by a partition, below). Every
// maintenance call enqueues kernels only (fills are kernels too), so each may be captured
// in a HIP graph.
//
// Erase and evict remove entries at a cost that follows the entries removed, and leave no
// tombstones: each removed entry's cluster (the run of occupied slots around it, bounded
// by empty slots; linear probing never crosses an empty slot) is repaired by one wave. It
// empties the removed slots and puts the cluster's other entries, in cluster order, each
// at the first free slot from its home, which is never past its old slot, so the cluster
// stays a valid probe sequence and other clusters are not touched. Clusters are found
// before any is repaired (a kernel boundary apart), and each is repaired by exactly one
// wave.
//
// The table header keeps the live-entry count (word 3): inserts add their new keys, erase
// subtracts what it removed, evict sets it, so erase can report the count without a scan.

#include "gleam_device.h"
#include "gleam_internal.h"
#include "radix_sort.h"

namespace gleam {
namespace {

constexpr int kThreads = 256;
constexpr uint32_t kMaxGrid = 8192;

// ---- workspace of evict and export ------------------------------------------------------
// Device words shared by the kernels of one call.
enum : int {
  kWCollected = 0,  // evict: entries collected; export: entries left to the radix sort
  kWDrop = 1,       // entries to evict
  kWLive = 2,       // live entries
  kWLeaders = 3,    // clusters to repair
  kWBits = 4,       // 4..7: the sort's AND/OR words
  kWBaseHi = 8,     // the histogram's origin
  kWBaseLo = 9,
  kWShift = 10,     // and log2 of its bins' width
};
constexpr size_t kCounterBytes = 256;

constexpr uint32_t kPickBins = 1024;        // evict's histogram
constexpr uint32_t kBinSlots = 4096;        // export: table slots per bin, up to kMaxBins bins
constexpr uint32_t kMaxBins = 16384;
constexpr uint32_t kSpreadGrid = 256;       // export: workgroups that spread the entries over the bins

struct Entry {  // an entry on its way to its place in the export
  uint64_t key, val, stamp, unused;  // (32 bytes: two 16-byte stores)
};

struct MaintLayout {
  uint64_t m;     // capacity + 1 (the last is the key kEmpty's header side slot)
  uint32_t bins, spread;
  size_t counters;
  size_t pick, leaders, hi, lo, idx, sort2;             // evict
  size_t share, starts, entries, xlo, xidx, sort1;      // export
  size_t total;
};

MaintLayout maint_layout(uint64_t capacity) {
  MaintLayout L;
  L.m = capacity + 1;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off = (off + bytes + 255) & ~(size_t)255;
    return o;
  };
  L.counters = take(kCounterBytes);
  L.leaders = take(4 * L.m);
  L.hi = take(8 * sort_capacity(L.m));  // the sort's keys and indices (its buffer a)
  L.lo = take(8 * sort_capacity(L.m));
  L.idx = take(4 * sort_capacity(L.m));
  L.sort2 = take(sort_layout(L.m, 2).total);
  L.pick = L.sort2;  // done with before the sort begins (its second buffer holds 8 KiB or more)
  const size_t evict_total = off;
  off = kCounterBytes;
  const uint64_t bins = capacity / kBinSlots;
  L.bins = (uint32_t)(bins < 1 ? 1 : bins < kMaxBins ? bins : kMaxBins);
  const uint64_t spread = (capacity + 4095) / 4096;
  L.spread = (uint32_t)(spread < kSpreadGrid ? spread : kSpreadGrid);
  L.share = take(4 * (size_t)L.bins * L.spread);
  L.starts = take(4 * ((size_t)L.bins + 1));
  L.entries = take(sizeof(Entry) * L.m);
  L.xlo = take(8 * sort_capacity(L.m));
  L.xidx = take(4 * sort_capacity(L.m));
  L.sort1 = take(sort_layout(L.m, 1).total);
  L.total = evict_total > off ? evict_total : off;
  return L;
}

template <typename T>
T* ws_at(void* ws, size_t off) {
  return reinterpret_cast<T*>(static_cast<uint8_t*>(ws) + off);
}

uint32_t grid_for(uint64_t n) {
  const uint64_t g = (n + kThreads - 1) / kThreads;
  return (uint32_t)(g == 0 ? 1 : (g < kMaxGrid ? g : kMaxGrid));
}

__device__ __forceinline__ unsigned long long* ull(uint64_t* p) { return reinterpret_cast<unsigned long long*>(p); }

// Slot of key k in the table, or -1 (k != kEmpty).
__device__ __forceinline__ int64_t find_slot(const TableRef& t, uint64_t k) {
  uint64_t pos = slot_hash(k, t.shift);
  for (uint64_t probe = 0; probe <= t.mask; ++probe) {
    const uint64_t key = t.slots[2 * pos];
    if (key == k) return (int64_t)pos;
    if (key == kEmpty) return -1;
    pos = (pos + 1) & t.mask;
  }
  return -1;
}

__device__ __forceinline__ uint64_t wave_sum(uint64_t x) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) x += shfl_xor64(x, o);
  return x;
}

// Touch. Copies of one key in a workgroup are folded first: an LDS table of lane numbers
// finds each key's lowest lane and takes the largest of the copies' epochs, and only that
// lane updates the stamp (at most one atomic per key per workgroup). A batch of one
// repeated key, as a zero-filled tensor gives, would otherwise queue one atomic per copy
// on one word (262,144 copies: 11.6 ms). A stamp only grows, so a lane whose stamp
// already reads at or past its epoch skips the atomic.
constexpr int kTouchSlots = 2 * kThreads;  // power of two, load at most 1/2

__global__ __launch_bounds__(kThreads) void touch_kernel(TableRef t, const uint64_t* keys, uint64_t n,
                                                         const uint64_t* epochs, uint64_t epoch,
                                                         uint64_t* n_touched) {
  __shared__ uint64_t bkeys[kThreads];
  __shared__ uint32_t bslot[kTouchSlots];  // lowest lane + 1 of the key in this slot (0 free)
  __shared__ uint64_t bmax[kTouchSlots];   // the largest epoch of that key's copies
  const uint32_t tid = threadIdx.x;
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + tid;
  const bool valid = i < n;
  const uint64_t k = valid ? keys[i] : 0;
  const uint64_t e = valid ? (epochs ? epochs[i] : epoch) : 0;
  bkeys[tid] = k;
  bslot[tid] = 0;
  bslot[tid + kThreads] = 0;
  bmax[tid] = 0;
  bmax[tid + kThreads] = 0;
  __syncthreads();
  uint32_t at = 0;
  if (valid) {
    static_assert(kTouchSlots == 512, "slot_hash shift");
    at = (uint32_t)slot_hash(k, 64 - 9);
    for (int probe = 0; probe < kTouchSlots; ++probe) {
      const uint32_t prev = atomicCAS(&bslot[at], 0u, tid + 1);
      if (prev == 0) break;
      if (bkeys[prev - 1] == k) {
        atomicMin(&bslot[at], tid + 1);
        break;
      }
      at = (at + 1) & (kTouchSlots - 1);
    }
    atomicMax(reinterpret_cast<unsigned long long*>(&bmax[at]), (unsigned long long)e);
  }
  __syncthreads();
  uint64_t hit = 0;
  if (valid) {
    const bool lead = bslot[at] == tid + 1;
    const uint64_t top = bmax[at];
    uint64_t* stamp = nullptr;
    if (k == kEmpty) {
      if (t.hdr[0]) stamp = &t.hdr[2];
    } else {
      const int64_t pos = find_slot(t, k);
      if (pos >= 0) stamp = &t.stamps[pos];
    }
    if (stamp) {
      hit = 1;
      if (lead && __hip_atomic_load(stamp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < top)
        atomicMax(ull(stamp), (unsigned long long)top);
    }
  }
  hit = wave_sum(hit);
  if (n_touched && (tid & 63) == 0 && hit) atomicAdd(ull(n_touched), (unsigned long long)hit);
}

// ---- selection over the range of (stamp, key) -----------------------------------------
typedef unsigned __int128 u128;
__device__ __forceinline__ u128 order_of(uint64_t stamp, uint64_t key) { return ((u128)stamp << 64) | key; }

// One workgroup: the counters of a call, and the origin and bin width of its histogram
// from the least and greatest of at most kSamples entries (every capacity / kSamples-th
// slot), with a margin of 1/1024 of their range on either side. An entry beyond takes the
// first or last bin: a bin number never decreases with the entry's order, which is all
// that the callers rely on.
constexpr uint32_t kInitThreads = 1024;
constexpr uint32_t kSamplesEach = 16;
constexpr uint64_t kSamples = (uint64_t)kInitThreads * kSamplesEach;

// kByStamp: the order is (stamp, key), else the key alone.
template <bool kByStamp>
__global__ __launch_bounds__(kInitThreads) void maint_init_kernel(TableRef t, uint64_t keep, uint32_t bins,
                                                                  uint64_t* counters, uint32_t* pick) {
  __shared__ uint64_t part[kInitThreads / 64][4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t capacity = t.mask + 1;
  if (pick)
    for (uint32_t i = threadIdx.x; i < bins; i += kInitThreads) pick[i] = 0;
  const uint64_t n = capacity < kSamples ? capacity : kSamples, step = capacity / n;
  uint64_t key[kSamplesEach], stamp[kSamplesEach];
#pragma unroll
  for (uint32_t r = 0; r < kSamplesEach; ++r) {  // unconditional (clamped) loads, issued together
    const uint64_t i = (uint64_t)r * kInitThreads + threadIdx.x;
    const uint64_t slot = (i < n ? i : 0) * step;
    key[r] = t.slots[2 * slot];
    stamp[r] = kByStamp ? t.stamps[slot] : 0;
  }
  u128 least = ~(u128)0, most = 0;
#pragma unroll
  for (uint32_t r = 0; r < kSamplesEach; ++r) {
    if (key[r] == kEmpty) continue;
    const u128 x = order_of(stamp[r], key[r]);
    least = x < least ? x : least;
    most = x > most ? x : most;
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const u128 a = order_of(shfl_xor64((uint64_t)(least >> 64), o), shfl_xor64((uint64_t)least, o));
    const u128 b = order_of(shfl_xor64((uint64_t)(most >> 64), o), shfl_xor64((uint64_t)most, o));
    least = a < least ? a : least;
    most = b > most ? b : most;
  }
  if (lane == 0) {
    part[wave][0] = (uint64_t)(least >> 64);
    part[wave][1] = (uint64_t)least;
    part[wave][2] = (uint64_t)(most >> 64);
    part[wave][3] = (uint64_t)most;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (uint32_t w = 1; w < kInitThreads / 64; ++w) {
    const u128 a = order_of(part[w][0], part[w][1]), b = order_of(part[w][2], part[w][3]);
    least = a < least ? a : least;
    most = b > most ? b : most;
  }
  if (least > most) least = most = 0;  // no entry among the samples
  const u128 margin = (most - least) >> 10;
  const u128 top = kByStamp ? ~(u128)0 : (u128)~0ull;
  const u128 base = least > margin ? least - margin : 0;
  const u128 end = most < top - margin ? most + margin : top;
  uint32_t shift = 0;
  while ((end - base) >> shift >= bins) ++shift;  // shift < 128: bins >= 1
  const uint64_t live = t.hdr[3];
  counters[kWCollected] = 0;
  counters[kWDrop] = live > keep ? live - keep : 0;
  counters[kWLive] = live;
  counters[kWLeaders] = 0;
  counters[kWBits + 0] = ~0ull;
  counters[kWBits + 1] = 0;
  counters[kWBits + 2] = ~0ull;
  counters[kWBits + 3] = 0;
  counters[kWBaseHi] = (uint64_t)(base >> 64);
  counters[kWBaseLo] = (uint64_t)base;
  counters[kWShift] = shift;
}

struct Bins {  // the histogram's geometry
  u128 base;
  uint32_t shift, last;
  __device__ Bins(const uint64_t* counters, uint32_t bins)
      : base(order_of(counters[kWBaseHi], counters[kWBaseLo])), shift((uint32_t)counters[kWShift]), last(bins - 1) {}
  __device__ __forceinline__ uint32_t of(u128 x) const {
    if (x < base) return 0;
    const u128 b = (x - base) >> shift;
    return b < last ? (uint32_t)b : last;
  }
};

// ---- evict ----------------------------------------------------------------------------
// Reads the table twice (the histogram, then the entries up to the bin of the last victim)
// and writes only what it evicts, so it is bound by two passes at HBM rate: 20 M entries in
// 2^25 slots, 20,000 evicted, 0.68 ms, against 5.9 ms for gathering, sorting and
// re-inserting every entry.
constexpr uint32_t kPickThreads = 1024;
constexpr uint32_t kPickGrid = 256;  // few enough that the final atomics on the bins stay few
constexpr uint32_t kPickItems = 4;

__global__ __launch_bounds__(kPickThreads) void evict_pick_kernel(TableRef t, const uint64_t* counters, uint32_t* pick) {
  __shared__ uint32_t h[kPickBins];
  if (counters[kWDrop] == 0) return;
  for (uint32_t i = threadIdx.x; i < kPickBins; i += kPickThreads) h[i] = 0;
  __syncthreads();
  const Bins bins(counters, kPickBins);
  const uint64_t capacity = t.mask + 1;
  for (uint64_t i0 = (uint64_t)blockIdx.x * kPickThreads * kPickItems; i0 < capacity;
       i0 += (uint64_t)gridDim.x * kPickThreads * kPickItems) {
    uint64_t key[kPickItems], stamp[kPickItems];
#pragma unroll
    for (uint32_t r = 0; r < kPickItems; ++r) {
      const uint64_t i = i0 + r * kPickThreads + threadIdx.x;
      const uint64_t at = i < capacity ? i : capacity - 1;
      key[r] = t.slots[2 * at];
      stamp[r] = t.stamps[at];
      if (i >= capacity) key[r] = kEmpty;
    }
#pragma unroll
    for (uint32_t r = 0; r < kPickItems; ++r)
      if (key[r] != kEmpty) atomicAdd(&h[bins.of(order_of(stamp[r], key[r]))], 1u);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0 && t.hdr[0]) atomicAdd(&h[bins.of(order_of(t.hdr[2], kEmpty))], 1u);
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < kPickBins; i += kPickThreads)
    if (h[i]) atomicAdd(&pick[i], h[i]);
}

// Collects the entries of the bins up to the one that the last victim falls in, as pairs
// (stamp, key) with their slot (the side slot: capacity). Each workgroup takes tiles of
// 4096 slots in turn, counts a tile's entries and claims that many positions with one
// atomic. It also folds the AND and OR of what it collects, once per workgroup at the
// end, from which the sort skips the digits every entry shares.
constexpr uint32_t kGatherItems = 16;
constexpr uint64_t kGatherTile = (uint64_t)kThreads * kGatherItems;
constexpr uint32_t kGatherMaxGrid = 1024;

__global__ __launch_bounds__(kThreads) void evict_collect_kernel(TableRef t, const uint32_t* pick, uint64_t* counters,
                                                                 SortBuf sb, uint64_t tiles) {
  static_assert(kPickBins == 4 * kThreads, "four bins per thread");
  __shared__ uint32_t wave_live[kThreads / 64];
  __shared__ uint64_t tile_base;
  __shared__ uint64_t fold[kThreads / 64][4];
  __shared__ uint32_t bin_limit;
  const uint64_t drop = counters[kWDrop];
  if (drop == 0) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
  {  // the first bin with which the running count reaches `drop`
    uint32_t c[4], sum = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      c[j] = pick[4 * threadIdx.x + j];
      sum += c[j];
    }
    uint32_t incl = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(incl, d, 64);
      if (lane >= d) incl += y;
    }
    if (lane == 63) wave_live[wave] = incl;
    if (threadIdx.x == 0) bin_limit = kPickBins - 1;
    __syncthreads();
    uint64_t run = incl - sum;
    for (int w = 0; w < wave; ++w) run += wave_live[w];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (run < drop && run + c[j] >= drop) bin_limit = 4 * threadIdx.x + j;
      run += c[j];
    }
    __syncthreads();
  }
  const uint32_t limit = bin_limit;
  const Bins bins(counters, kPickBins);
  const uint64_t capacity = t.mask + 1;
  uint64_t and_k = ~0ull, or_k = 0, and_s = ~0ull, or_s = 0;
  for (uint64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const uint64_t first = tile * kGatherTile + (uint64_t)wave * 64 * kGatherItems + lane;
    uint64_t key[kGatherItems], stamp[kGatherItems], mask[kGatherItems];
#pragma unroll
    for (uint32_t r = 0; r < kGatherItems; ++r) {  // unconditional (clamped) loads, issued together
      const uint64_t i = first + 64ull * r, at = i < capacity ? i : capacity - 1;
      key[r] = t.slots[2 * at];
      stamp[r] = t.stamps[at];
    }
    uint32_t live_n = 0;
#pragma unroll
    for (uint32_t r = 0; r < kGatherItems; ++r) {
      const uint64_t i = first + 64ull * r;
      bool live = i < capacity && key[r] != kEmpty;
      if (i == capacity && t.hdr[0]) {  // the side slot
        live = true;
        key[r] = kEmpty;
        stamp[r] = t.hdr[2];
      }
      mask[r] = __ballot(live && bins.of(order_of(stamp[r], key[r])) <= limit);
      live_n += (uint32_t)__popcll(mask[r]);
    }
    if (lane == 0) wave_live[wave] = live_n;
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t total = 0;
      for (int w = 0; w < kThreads / 64; ++w) total += wave_live[w];
      tile_base = total ? atomicAdd(ull(&counters[kWCollected]), (unsigned long long)total) : 0;
    }
    __syncthreads();
    uint64_t at = tile_base;
    for (int w = 0; w < wave; ++w) at += wave_live[w];
#pragma unroll
    for (uint32_t r = 0; r < kGatherItems; ++r) {
      if ((mask[r] >> lane) & 1ull) {
        const uint64_t p = at + (uint64_t)__popcll(mask[r] & lt);
        sb.hi[p] = stamp[r];
        sb.lo[p] = key[r];
        sb.idx[p] = (uint32_t)(first + 64ull * r);
        and_k &= key[r];
        or_k |= key[r];
        and_s &= stamp[r];
        or_s |= stamp[r];
      }
      at += (uint64_t)__popcll(mask[r]);
    }
    __syncthreads();  // wave_live and tile_base read before the next tile rewrites them
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    and_k &= shfl_xor64(and_k, o);
    or_k |= shfl_xor64(or_k, o);
    and_s &= shfl_xor64(and_s, o);
    or_s |= shfl_xor64(or_s, o);
  }
  if (lane == 0) {
    fold[wave][0] = and_k;
    fold[wave][1] = or_k;
    fold[wave][2] = and_s;
    fold[wave][3] = or_s;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kThreads / 64; ++w) {
      fold[0][0] &= fold[w][0];
      fold[0][1] |= fold[w][1];
      fold[0][2] &= fold[w][2];
      fold[0][3] |= fold[w][3];
    }
    if (fold[0][0] != ~0ull || fold[0][1] != 0) {  // some entry was collected (an all-ones key has OR != 0)
      atomicAnd(ull(&counters[kWBits + 0]), (unsigned long long)fold[0][0]);
      atomicOr(ull(&counters[kWBits + 1]), (unsigned long long)fold[0][1]);
      atomicAnd(ull(&counters[kWBits + 2]), (unsigned long long)fold[0][2]);
      atomicOr(ull(&counters[kWBits + 3]), (unsigned long long)fold[0][3]);
    }
  }
}

// (stamp, key) at or below those of the last victim: evicted.
struct UpTo {
  u128 last;
  __device__ bool operator()(uint64_t k, uint64_t stamp) const { return order_of(stamp, k) <= last; }
};

__device__ __forceinline__ UpTo last_victim(const SortBuf& sorted, uint64_t drop) {
  return UpTo{order_of(sorted.hi[drop - 1], sorted.lo[drop - 1])};
}

// The first `drop` of the sorted entries go: lists their keys, and finds the clusters to
// repair: the first victim of a cluster (no victim before it up to the cluster's start)
// lists the start. When every entry goes, the repair clears the table instead.
__global__ __launch_bounds__(kThreads) void evict_mark_kernel(TableRef t, SortBuf a, SortBuf b, uint64_t* counters,
                                                              uint32_t* leaders, uint64_t* evicted, uint64_t* counts) {
  const uint64_t drop = counters[kWDrop], live = counters[kWLive];
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  const uint64_t t0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t0 == 0) {
    counts[0] = drop;
    counts[1] = live - drop;
    t.hdr[3] = live - drop;
  }
  if (drop == 0) return;
  const SortBuf sorted = sort_result(a, b, counters + kWBits, 2);
  const UpTo gone = last_victim(sorted, drop);
  for (uint64_t i = t0; i < drop; i += stride) {
    if (evicted) evicted[i] = sorted.lo[i];
    const uint64_t p = sorted.idx[i];
    if (p > t.mask) {  // the side slot
      t.hdr[0] = t.hdr[1] = t.hdr[2] = 0;
      continue;
    }
    if (drop == live) continue;
    uint64_t c0 = p;
    bool first = true;
    for (uint64_t step = 0; step <= t.mask; ++step) {
      const uint64_t before = (c0 - 1) & t.mask;
      const uint64_t k = t.slots[2 * before];
      if (k == kEmpty) break;
      if (gone(k, t.stamps[before])) {
        first = false;
        break;
      }
      c0 = before;
    }
    if (first) leaders[atomicAdd(ull(&counters[kWLeaders]), 1ull)] = (uint32_t)c0;
  }
}

// ---- cluster repair -------------------------------------------------------------------
constexpr int kWaves = kThreads / 64;
constexpr uint32_t kRepairWords = 64;  // 64-slot windows of a cluster that a wave repairs (4,096 slots)

__device__ __forceinline__ uint32_t lane32(uint32_t x, int src) { return __builtin_amdgcn_readlane(x, src); }

// Repairs the cluster that starts at slot c0 (an occupied slot after an empty one), by one
// wave: removes the entries for which erased(key, stamp) and closes the gaps. Returns how
// many it removed. Lane i of a window holds slot 64 w + i of the cluster, so a cluster
// costs a few round trips of memory; one thread walking it slot by slot took 80 us for
// 5,167 keys of a table at load 0.5 (a chain of dependent reads as long as the longest
// cluster, each with its probe of the erased keys). `used` (kRepairWords words of LDS) has
// the final occupancy of the windows already done. Every lane of the wave calls it with
// the same c0. Only this wave touches the cluster and the empty slot after it is not
// written by any, so the end found here does not depend on other waves.
template <class Erased>
__device__ uint32_t wave_repair(const TableRef& t, uint64_t c0, const Erased& erased, uint64_t* used, int lane) {
  uint32_t len = 0;  // the cluster's slots
  for (uint32_t w = 0; len == 64 * w; ++w) {
    if (w == kRepairWords) break;
    const uint64_t k = t.slots[2 * ((c0 + len + lane) & t.mask)];
    const uint64_t free_slots = __ballot(k == kEmpty);
    len += free_slots ? (uint32_t)__builtin_ctzll(free_slots) : 64u;
    if (len > t.mask) break;  // a table has at least one free slot; bounded all the same
  }
  uint32_t removed = 0;
  if (len >= 64 * kRepairWords) {  // a longer cluster: one lane, slot by slot
    if (lane == 0) {
      uint64_t n = 0;
      for (uint64_t p = c0; n <= t.mask; p = (p + 1) & t.mask, ++n) {
        const uint64_t k = t.slots[2 * p];
        if (k == kEmpty) break;  // the cluster's end (slots emptied here lie behind)
        if (erased(k, t.stamps[p])) {
          t.slots[2 * p] = kEmpty;
          t.stamps[p] = 0;
          ++removed;
        }
      }
      for (uint64_t i = 0; removed && i < n; ++i) {
        const uint64_t p = (c0 + i) & t.mask;
        const uint64_t k = t.slots[2 * p];
        if (k == kEmpty) continue;
        uint64_t q = slot_hash(k, t.shift);
        while (q != p && t.slots[2 * q] != kEmpty) q = (q + 1) & t.mask;
        if (q == p) continue;  // no free slot before it: stays
        t.slots[2 * q] = k;
        t.slots[2 * q + 1] = t.slots[2 * p + 1];
        t.stamps[q] = t.stamps[p];
        t.slots[2 * p] = kEmpty;
        t.stamps[p] = 0;
      }
    }
    return lane32(removed, 0);
  }
  for (uint32_t w = 0; 64 * w < len; ++w) {
    const uint32_t i = 64 * w + (uint32_t)lane;
    const uint64_t p = (c0 + i) & t.mask;
    const uint4 e = *reinterpret_cast<const uint4*>(t.slots + 2 * p);
    const uint64_t stamp = t.stamps[p], k = lo64(e);
    const bool in = i < len;
    const bool gone = in && erased(k, stamp);
    const uint64_t keep = __ballot(in && !gone);
    removed += (uint32_t)__popcll(__ballot(gone));
    if (removed == 0) {  // nothing removed so far: every entry stays
      used[w] = keep;
      continue;
    }
    const uint32_t home = (uint32_t)((slot_hash(k, t.shift) - c0) & t.mask);  // from c0; below len for an entry here
    uint64_t now = 0;  // this window's final occupancy
    uint32_t to = i;
    for (uint64_t left = keep; left; left &= left - 1) {
      const int src = __builtin_ctzll(left);
      const uint32_t h = lane32(home, src);
      uint32_t q = ~0u;
      for (uint32_t x = h >> 6; x < w; ++x) {  // free slots of earlier windows
        uint64_t room = ~used[x];
        if (x == h >> 6) room &= ~0ull << (h & 63);
        if (room) {
          q = 64 * x + (uint32_t)__builtin_ctzll(room);
          used[x] |= room & (0 - room);
          break;
        }
      }
      if (q == ~0u) {  // the first free slot of this window from its home: at most its own
        const uint64_t room = ~now & (h >> 6 == w ? ~0ull << (h & 63) : ~0ull);
        q = 64 * w + (uint32_t)__builtin_ctzll(room);
        now |= room & (0 - room);
      }
      if (lane == src) to = q;
    }
    used[w] = now;
    if (in && !gone && to != i) {
      const uint64_t q = (c0 + to) & t.mask;
      *reinterpret_cast<uint4*>(t.slots + 2 * q) = e;
      t.stamps[q] = stamp;
    }
    if (in && !((now >> lane) & 1ull)) {  // a later window's entry may take it
      t.slots[2 * p] = kEmpty;
      t.stamps[p] = 0;
    }
  }
  return removed;
}

// ---- erase: O(keys erased) ------------------------------------------------------------
struct EraseWs {          // workspace of an erase of n keys
  uint64_t* hdr;          // [0] removed entries | arrived workgroups << 40, [1] clusters to repair
  uint64_t* keyset;       // cap slots: index + 1 of an erased key (0 free); keys read back
  uint64_t* starts;       // cap slots: cluster start + 1 (0 free)
  uint64_t* leaders;      // n cluster starts, one per cluster
  uint64_t mask;
  int shift;
};
constexpr int kArrivedShift = 40;  // n <= 2^36 entries, and a grid below 2^24 workgroups

__device__ __forceinline__ bool in_keyset(const EraseWs& w, const uint64_t* keys, uint64_t k) {
  uint64_t pos = slot_hash(k, w.shift);
  for (uint64_t probe = 0; probe <= w.mask; ++probe) {
    const uint64_t v = w.keyset[pos];
    if (v == 0) return false;
    if (keys[v - 1] == k) return true;
    pos = (pos + 1) & w.mask;
  }
  return false;
}

// Per erased key: into the key set; if the table holds it, the start of its cluster,
// claimed once. (The two do not depend on each other: one launch.)
__global__ __launch_bounds__(kThreads) void erase_find_kernel(TableRef t, const uint64_t* keys, uint64_t n, EraseWs w) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint64_t k = keys[i];
  if (k == kEmpty) {  // the header's side slot
    if (atomicExch(ull(&t.hdr[0]), 0ull) == 1ull) {
      t.hdr[2] = 0;
      atomicAdd(ull(&w.hdr[0]), 1ull);
    }
    return;
  }
  uint64_t pos = slot_hash(k, w.shift);
  for (uint64_t probe = 0; probe <= w.mask; ++probe) {
    const uint64_t prev = atomicCAS(ull(&w.keyset[pos]), 0ull, (unsigned long long)(i + 1));
    if (prev == 0) break;
    if (keys[prev - 1] == k) return;  // a repeat: the other one finds the cluster
    pos = (pos + 1) & w.mask;
  }
  const int64_t at = find_slot(t, k);
  if (at < 0) return;
  uint64_t c0 = (uint64_t)at;
  for (uint64_t step = 0; step <= t.mask; ++step) {
    const uint64_t before = (c0 - 1) & t.mask;
    if (t.slots[2 * before] == kEmpty) break;
    c0 = before;
  }
  pos = slot_hash(c0, w.shift);
  for (uint64_t probe = 0; probe <= w.mask; ++probe) {
    const uint64_t prev = atomicCAS(ull(&w.starts[pos]), 0ull, (unsigned long long)(c0 + 1));
    if (prev == 0) {
      w.leaders[atomicAdd(ull(&w.hdr[1]), 1ull)] = c0;
      return;
    }
    if (prev == c0 + 1) return;  // claimed by another key of this cluster
    pos = (pos + 1) & w.mask;
  }
}

struct InKeyset {
  const EraseWs& w;
  const uint64_t* keys;
  __device__ bool operator()(uint64_t k, uint64_t) const { return in_keyset(w, keys, k); }
};

// One wave per cluster; the last workgroup to arrive writes the counts.
__global__ __launch_bounds__(kThreads) void erase_repair_kernel(TableRef t, const uint64_t* keys, uint64_t n, EraseWs w,
                                                                uint64_t* counts) {
  __shared__ uint64_t used[kWaves][kRepairWords];
  __shared__ uint32_t removed[kWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t clusters = min(w.hdr[1], n);
  const InKeyset erased{w, keys};
  uint32_t mine = 0;
  for (uint64_t c = (uint64_t)blockIdx.x * kWaves + wave; c < clusters; c += (uint64_t)gridDim.x * kWaves)
    mine += wave_repair(t, w.leaders[c], erased, used[wave], lane);
  if (lane == 0) removed[wave] = mine;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t add = 1ull << kArrivedShift;
    for (int v = 0; v < kWaves; ++v) add += removed[v];
    const uint64_t now = atomicAdd(ull(&w.hdr[0]), (unsigned long long)add) + add;
    if (now >> kArrivedShift == gridDim.x) {
      const uint64_t total = now & ((1ull << kArrivedShift) - 1);
      const uint64_t live = t.hdr[3] - total;
      t.hdr[3] = live;
      counts[0] = total;
      counts[1] = live;
    }
  }
}

struct EraseLayout {
  uint64_t cap;
  size_t total;
};

EraseLayout erase_layout(uint64_t n) {
  EraseLayout L;
  L.cap = 64;
  while (L.cap < 2 * n) L.cap <<= 1;
  L.total = (kHeaderBytes + 16 * (size_t)L.cap + 8 * (size_t)n + 255) & ~(size_t)255;
  return L;
}

EraseWs erase_ws(void* ws, const EraseLayout& L) {
  uint8_t* b = static_cast<uint8_t*>(ws);
  EraseWs w;
  w.hdr = reinterpret_cast<uint64_t*>(b);
  w.keyset = reinterpret_cast<uint64_t*>(b + kHeaderBytes);
  w.starts = w.keyset + L.cap;
  w.leaders = w.starts + L.cap;
  w.mask = L.cap - 1;
  w.shift = 64 - log2_exact(L.cap);
  return w;
}

// One wave per cluster with victims.
__global__ __launch_bounds__(kThreads) void evict_repair_kernel(TableRef t, SortBuf a, SortBuf b,
                                                                const uint64_t* counters, const uint32_t* leaders) {
  __shared__ uint64_t used[kWaves][kRepairWords];
  const uint64_t drop = counters[kWDrop];
  if (drop == 0) return;
  if (drop == counters[kWLive]) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; p <= t.mask; p += stride) {
      t.slots[2 * p] = kEmpty;
      t.stamps[p] = 0;
    }
    return;
  }
  const UpTo gone = last_victim(sort_result(a, b, counters + kWBits, 2), drop);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t clusters = counters[kWLeaders];
  for (uint64_t c = (uint64_t)blockIdx.x * kWaves + wave; c < clusters; c += (uint64_t)gridDim.x * kWaves)
    wave_repair(t, leaders[c], gone, used[wave], lane);
}

// ---- export ---------------------------------------------------------------------------
// Every entry in key order by one partition: the key range is cut into bins (one per
// kBinSlots table slots), every entry is written once to its bin's place in the workspace,
// and one workgroup per bin sorts its few thousand entries in LDS and writes them out. Keys
// are digests, so the bins of an ordinary table are even; when one holds more than kBinMax
// entries (a skewed key set), all entries go through the radix sort instead, decided on
// the device. 20 M entries: 1.25 ms (the table read twice, the entries written and read
// once), against 3.0 ms for eight digit passes and a gather of the values.
constexpr uint32_t kSpreadThreads = 1024;
constexpr uint32_t kSpreadItems = 4;

// Entries of one spreading workgroup's share of the slots, by bin (share[g][bin]), or
// (kWrite) written to their places: the workgroup's place in a bin starts at
// starts[bin] + share[g][bin].
template <bool kWrite>
__global__ __launch_bounds__(kSpreadThreads) void export_spread_kernel(TableRef t, const uint64_t* counters,
                                                                       uint32_t n_bins, uint32_t* share,
                                                                       const uint32_t* starts, Entry* entries) {
  __shared__ uint32_t at[kMaxBins];
  uint32_t* row = share + (uint64_t)blockIdx.x * n_bins;
  for (uint32_t i = threadIdx.x; i < n_bins; i += kSpreadThreads) at[i] = kWrite ? starts[i] + row[i] : 0;
  __syncthreads();
  const Bins bins(counters, n_bins);
  const uint64_t capacity = t.mask + 1;
  const uint64_t each = (capacity + gridDim.x - 1) / gridDim.x;
  const uint64_t lo = blockIdx.x * each, hi = lo + each < capacity ? lo + each : capacity;
  auto put = [&](uint64_t key, uint64_t val, uint64_t stamp) {
    const uint32_t p = atomicAdd(&at[bins.of(key)], 1u);
    if (kWrite) {
      uint4* to = reinterpret_cast<uint4*>(&entries[p]);
      to[0] = make_uint4((uint32_t)key, (uint32_t)(key >> 32), (uint32_t)val, (uint32_t)(val >> 32));
      to[1] = make_uint4((uint32_t)stamp, (uint32_t)(stamp >> 32), 0, 0);
    }
  };
  for (uint64_t i0 = lo; i0 < hi; i0 += (uint64_t)kSpreadThreads * kSpreadItems) {
    uint4 slot[kSpreadItems];
    uint64_t stamp[kSpreadItems];
#pragma unroll
    for (uint32_t r = 0; r < kSpreadItems; ++r) {  // unconditional (clamped) loads, issued together
      const uint64_t i = i0 + r * kSpreadThreads + threadIdx.x, p = i < hi ? i : hi - 1;
      slot[r] = *reinterpret_cast<const uint4*>(t.slots + 2 * p);
      stamp[r] = kWrite ? t.stamps[p] : 0;
    }
#pragma unroll
    for (uint32_t r = 0; r < kSpreadItems; ++r) {
      const uint64_t i = i0 + r * kSpreadThreads + threadIdx.x;
      if (i < hi && lo64(slot[r]) != kEmpty) put(lo64(slot[r]), hi64(slot[r]), stamp[r]);
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0 && t.hdr[0]) put(kEmpty, t.hdr[1], t.hdr[2]);
  if (!kWrite) {
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < n_bins; i += kSpreadThreads) row[i] = at[i];
  }
}

// share[g][bin] becomes the count of the workgroups before g; starts[bin] the bin's total.
__global__ __launch_bounds__(64) void export_share_kernel(uint32_t n_bins, uint32_t groups, uint32_t* share,
                                                          uint32_t* starts) {
  const uint32_t bin = blockIdx.x * 64 + threadIdx.x;
  if (bin >= n_bins) return;
  constexpr uint32_t kAhead = 32;
  uint32_t sum = 0;
  for (uint32_t g0 = 0; g0 < groups; g0 += kAhead) {
    uint32_t c[kAhead];
#pragma unroll
    for (uint32_t k = 0; k < kAhead; ++k) {  // unconditional (clamped) loads, issued together
      const uint32_t g = g0 + k < groups ? g0 + k : groups - 1;
      c[k] = share[(uint64_t)g * n_bins + bin];
    }
#pragma unroll
    for (uint32_t k = 0; k < kAhead; ++k) {
      if (g0 + k >= groups) break;
      share[(uint64_t)(g0 + k) * n_bins + bin] = sum;
      sum += c[k];
    }
  }
  starts[bin] = sum;
}

constexpr uint32_t kBinMax = 6144;     // entries that a workgroup sorts in LDS
constexpr uint32_t kBinThreads = 512;
constexpr uint32_t kBinEach = kBinMax / kBinThreads;
constexpr uint32_t kSubBins = 4096;

// One workgroup: starts[bin] from totals to positions, starts[n_bins] = the entries; the
// count; and whether the radix sort takes over (counters[kWCollected]: its count, else 0).
__global__ __launch_bounds__(kInitThreads) void export_starts_kernel(uint32_t n_bins, uint32_t* starts,
                                                                     uint64_t* counters, uint64_t* count) {
  __shared__ uint32_t wave_sum[kInitThreads / 64], wave_most[kInitThreads / 64];
  constexpr uint32_t kEach = kMaxBins / kInitThreads;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t each = (n_bins + kInitThreads - 1) / kInitThreads;  // at most kEach
  const uint32_t first = threadIdx.x * each;
  uint32_t c[kEach], sum = 0, most = 0;
#pragma unroll
  for (uint32_t j = 0; j < kEach; ++j) c[j] = j < each && first + j < n_bins ? starts[first + j] : 0;
#pragma unroll
  for (uint32_t j = 0; j < kEach; ++j) {
    sum += c[j];
    most = c[j] > most ? c[j] : most;
  }
  uint32_t incl = sum;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = __shfl_up(incl, d, 64);
    if (lane >= d) incl += y;
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) most = max(most, (uint32_t)__shfl_xor((int)most, o, 64));
  if (lane == 63) wave_sum[wave] = incl;
  if (lane == 0) wave_most[wave] = most;
  __syncthreads();
  uint32_t run = incl - sum, total = 0;
  for (uint32_t w = 0; w < kInitThreads / 64; ++w) {
    if ((int)w < wave) run += wave_sum[w];
    total += wave_sum[w];
    most = max(most, wave_most[w]);
  }
#pragma unroll
  for (uint32_t j = 0; j < kEach; ++j) {
    if (j < each && first + j < n_bins) starts[first + j] = run;
    run += c[j];
  }
  if (threadIdx.x == 0) {
    starts[n_bins] = total;
    *count = total;
    counters[kWCollected] = most > kBinMax ? total : 0;
  }
}

// Sorts one bin. Its entries are counted over kSubBins cuts of the bin's range and placed
// cut by cut in LDS; within a cut (0.6 entries on average) an entry's rank is the number of
// smaller keys in it. When a cut holds more than kCutMax entries (keys crowded inside the
// bin's range) the workgroup sorts the bin with a comparison network instead.
constexpr uint32_t kCutMax = 32;

__global__ __launch_bounds__(kBinThreads) void export_bin_kernel(const uint64_t* counters, uint32_t n_bins,
                                                                 const uint32_t* starts, const Entry* entries,
                                                                 uint64_t* keys, uint64_t* vals, uint64_t* stamps) {
  __shared__ uint64_t skey[kBinMax];
  __shared__ uint16_t sidx[kBinMax];
  __shared__ uint32_t cut[kSubBins + 1];
  __shared__ uint32_t wave_sum[kBinThreads / 64];
  __shared__ uint32_t crowded;
  if (counters[kWCollected]) return;  // the radix sort takes over
  const uint32_t bin = blockIdx.x;
  const uint32_t s0 = starts[bin], n = starts[bin + 1] - s0;
  if (n == 0) return;
  const uint64_t base = counters[kWBaseLo];
  const uint32_t shift = (uint32_t)counters[kWShift];
  const uint64_t bin_lo = base + (shift < 64 ? (uint64_t)bin << shift : 0ull);
  const uint32_t cut_shift = shift > 12 ? shift - 12 : 0;
  static_assert(kSubBins == 1u << 12, "cut_shift");
  auto cut_of = [&](uint64_t k) -> uint32_t {  // never decreases with the key within the bin
    if (k < bin_lo) return 0;
    const uint64_t c = (k - bin_lo) >> cut_shift;
    return c < kSubBins ? (uint32_t)c : kSubBins - 1;
  };
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint64_t k[kBinEach];
#pragma unroll
  for (uint32_t r = 0; r < kBinEach; ++r) {
    const uint32_t i = r * kBinThreads + threadIdx.x;
    k[r] = i < n ? entries[s0 + i].key : 0;
  }
  for (uint32_t i = threadIdx.x; i < kSubBins + 1; i += kBinThreads) cut[i] = 0;
  if (threadIdx.x == 0) crowded = 0;
  __syncthreads();
  uint32_t ord[kBinEach];  // within its cut, in arrival order
#pragma unroll
  for (uint32_t r = 0; r < kBinEach; ++r) {
    const uint32_t i = r * kBinThreads + threadIdx.x;
    if (i >= n) continue;
    ord[r] = atomicAdd(&cut[cut_of(k[r])], 1u);
    if (ord[r] >= kCutMax) crowded = 1;
  }
  __syncthreads();
  {  // exclusive scan of the cuts' counts
    constexpr uint32_t kEach = kSubBins / kBinThreads;
    uint32_t c[kEach], sum = 0;
#pragma unroll
    for (uint32_t j = 0; j < kEach; ++j) {
      c[j] = cut[threadIdx.x * kEach + j];
      sum += c[j];
    }
    uint32_t incl = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(incl, d, 64);
      if (lane >= d) incl += y;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    uint32_t run = incl - sum;
    for (int w = 0; w < wave; ++w) run += wave_sum[w];
#pragma unroll
    for (uint32_t j = 0; j < kEach; ++j) {
      cut[threadIdx.x * kEach + j] = run;
      run += c[j];
    }
    if (threadIdx.x == kBinThreads - 1) cut[kSubBins] = run;
  }
  __syncthreads();
#pragma unroll
  for (uint32_t r = 0; r < kBinEach; ++r) {
    const uint32_t i = r * kBinThreads + threadIdx.x;
    if (i >= n) continue;
    const uint32_t p = cut[cut_of(k[r])] + ord[r];
    skey[p] = k[r];
    sidx[p] = (uint16_t)i;
  }
  __syncthreads();
  const bool network = crowded != 0;
  if (network) {  // ascending merges of runs of len / 2, the second run read backwards first
    for (uint32_t len = 2; len < 2 * n; len <<= 1) {
      for (uint32_t j = len / 2; j > 0; j >>= 1) {
        for (uint32_t q = threadIdx.x; q < kBinMax; q += kBinThreads) {
          const uint32_t at = q / j * 2 * j + q % j;
          const uint32_t other = j == len / 2 ? q / j * len + (len - 1 - q % j) : at + j;
          if (other < n && skey[at] > skey[other]) {
            const uint64_t tk = skey[at];
            skey[at] = skey[other];
            skey[other] = tk;
            const uint16_t ti = sidx[at];
            sidx[at] = sidx[other];
            sidx[other] = ti;
          }
        }
        __syncthreads();
      }
    }
  }
#pragma unroll
  for (uint32_t r = 0; r < kBinEach; ++r) {
    const uint32_t p = r * kBinThreads + threadIdx.x;
    if (p >= n) continue;
    const uint64_t key = skey[p];
    uint32_t rank = p;
    if (!network) {
      const uint32_t c = cut_of(key), from = cut[c], to = cut[c + 1];
      rank = from;
      for (uint32_t q = from; q < to; ++q) rank += skey[q] < key ? 1u : 0u;
    }
    const Entry* e = &entries[s0 + sidx[p]];
    keys[s0 + rank] = key;
    vals[s0 + rank] = e->val;
    if (stamps) stamps[s0 + rank] = e->stamp;
  }
}

// The radix sort's input: the keys with their entries' positions, and the AND/OR words.
__global__ __launch_bounds__(kThreads) void export_unpack_kernel(uint64_t* counters, const Entry* entries, SortBuf sb) {
  const uint64_t n = counters[kWCollected];
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  uint64_t and_k = ~0ull, or_k = 0;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const uint64_t k = entries[i].key;
    sb.lo[i] = k;
    sb.idx[i] = (uint32_t)i;
    and_k &= k;
    or_k |= k;
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    and_k &= shfl_xor64(and_k, o);
    or_k |= shfl_xor64(or_k, o);
  }
  if ((threadIdx.x & 63) == 0 && (and_k != ~0ull || or_k != 0)) {
    atomicAnd(ull(&counters[kWBits + 0]), (unsigned long long)and_k);
    atomicOr(ull(&counters[kWBits + 1]), (unsigned long long)or_k);
  }
}

__global__ __launch_bounds__(kThreads) void export_sorted_kernel(const uint64_t* counters, const Entry* entries,
                                                                 SortBuf a, SortBuf b, uint64_t* keys, uint64_t* vals,
                                                                 uint64_t* stamps) {
  const uint64_t n = counters[kWCollected];
  const SortBuf sorted = sort_result(a, b, counters + kWBits, 1);
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const Entry* e = &entries[sorted.idx[i]];
    keys[i] = sorted.lo[i];
    vals[i] = e->val;
    if (stamps) stamps[i] = e->stamp;
  }
}

gleam_status check_maint(const gleam_cache* c, void* ws, size_t ws_bytes, const char* who, MaintLayout* L) {
  if (!c) {
    set_error("%s: null table", who);
    return GLEAM_E_INVALID;
  }
  if (c->capacity > (1ull << 31)) {
    set_error("%s: tables above 2^31 slots are not supported", who);
    return GLEAM_E_UNSUPPORTED;
  }
  *L = maint_layout(c->capacity);
  if (!ws || !aligned256(ws)) {
    set_error("%s: workspace must be non-null and 256-byte aligned", who);
    return GLEAM_E_INVALID;
  }
  if (ws_bytes < L->total) {
    set_error("%s: workspace of %zu bytes, %zu needed", who, ws_bytes, L->total);
    return GLEAM_E_WORKSPACE;
  }
  return GLEAM_OK;
}

}  // namespace
// Loads this file's GPU code object on the current device (gleam_preload).
hipError_t preload_lifecycle() {
  hipFuncAttributes attr;
  return hipFuncGetAttributes(&attr, reinterpret_cast<const void*>(&erase_find_kernel));
}

}  // namespace gleam

extern "C" size_t gleam_cache_maint_bytes(const gleam_cache* c) {
  if (!c || c->capacity > (1ull << 31)) return 0;
  return gleam::maint_layout(c->capacity).total;
}

extern "C" gleam_status gleam_cache_touch(gleam_cache* c, const uint64_t* d_keys, uint64_t n,
                                          const uint64_t* d_epochs, uint64_t epoch, uint64_t* d_n_touched,
                                          void* stream) {
  using namespace gleam;
  clear_error();
  if (!c) {
    set_error("gleam_cache_touch: null table");
    return GLEAM_E_INVALID;
  }
  if (n > 0 && !d_keys) {
    set_error("gleam_cache_touch: null keys");
    return GLEAM_E_INVALID;
  }
  if (n > 0x7fffffffull * kThreads) {
    set_error("gleam_cache_touch: more than 2^31 workgroups of keys");
    return GLEAM_E_UNSUPPORTED;
  }
  hipStream_t s = (hipStream_t)stream;
  gleam_status st = GLEAM_OK;
  if (d_n_touched) st = fill_u64(d_n_touched, 1, 0, s);
  if (st != GLEAM_OK || n == 0) return st;
  hipLaunchKernelGGL(touch_kernel, dim3((uint32_t)((n + kThreads - 1) / kThreads)), dim3(kThreads), 0, s,
                     table_ref(c), d_keys, n, d_epochs, epoch, d_n_touched);
  return launch_status("touch_kernel");
}

extern "C" gleam_status gleam_cache_evict(gleam_cache* c, uint64_t keep, uint64_t* d_evicted, uint64_t* d_counts,
                                          void* d_ws, size_t ws_bytes, void* stream) {
  using namespace gleam;
  clear_error();
  MaintLayout L;
  gleam_status st = check_maint(c, d_ws, ws_bytes, "gleam_cache_evict", &L);
  if (st != GLEAM_OK) return st;
  if (!d_counts) {
    set_error("gleam_cache_evict: null counts");
    return GLEAM_E_INVALID;
  }
  hipStream_t s = (hipStream_t)stream;
  const TableRef t = table_ref(c);
  uint64_t* counters = ws_at<uint64_t>(d_ws, L.counters);
  uint32_t* pick = ws_at<uint32_t>(d_ws, L.pick);
  uint32_t* leaders = ws_at<uint32_t>(d_ws, L.leaders);
  const SortBuf sa{ws_at<uint64_t>(d_ws, L.hi), ws_at<uint64_t>(d_ws, L.lo), ws_at<uint32_t>(d_ws, L.idx)};
  const SortBuf sb = sort_other(ws_at<uint8_t>(d_ws, L.sort2), L.m, 2);
  hipLaunchKernelGGL(maint_init_kernel<true>, dim3(1), dim3(kInitThreads), 0, s, t, keep, kPickBins, counters, pick);
  if ((st = launch_status("maint_init_kernel")) != GLEAM_OK) return st;
  const uint64_t pick_want = (c->capacity + kPickThreads * kPickItems - 1) / (kPickThreads * kPickItems);
  hipLaunchKernelGGL(evict_pick_kernel, dim3((uint32_t)(pick_want < kPickGrid ? pick_want : kPickGrid)),
                     dim3(kPickThreads), 0, s, t, counters, pick);
  if ((st = launch_status("evict_pick_kernel")) != GLEAM_OK) return st;
  const uint64_t tiles = (L.m + kGatherTile - 1) / kGatherTile;
  hipLaunchKernelGGL(evict_collect_kernel, dim3((uint32_t)(tiles < kGatherMaxGrid ? tiles : kGatherMaxGrid)),
                     dim3(kThreads), 0, s, t, pick, counters, sa, tiles);
  if ((st = launch_status("evict_collect_kernel")) != GLEAM_OK) return st;
  st = radix_sort_pairs(sa, counters + kWCollected, counters + kWBits, L.m, 2, ws_at<uint8_t>(d_ws, L.sort2), s);
  if (st != GLEAM_OK) return st;
  const uint32_t grid = grid_for(L.m) < 2048 ? grid_for(L.m) : 2048;
  hipLaunchKernelGGL(evict_mark_kernel, dim3(grid), dim3(kThreads), 0, s, t, sa, sb, counters, leaders, d_evicted,
                     d_counts);
  if ((st = launch_status("evict_mark_kernel")) != GLEAM_OK) return st;
  hipLaunchKernelGGL(evict_repair_kernel, dim3(grid), dim3(kThreads), 0, s, t, sa, sb, counters, leaders);
  if ((st = launch_status("evict_repair_kernel")) != GLEAM_OK) return st;
  if (keep < c->key_bound) c->key_bound = keep;
  return GLEAM_OK;
}

extern "C" size_t gleam_cache_erase_bytes(uint64_t n) {
  if (n > (1ull << 36)) return 0;
  return gleam::erase_layout(n).total;
}

extern "C" gleam_status gleam_cache_erase(gleam_cache* c, const uint64_t* d_keys, uint64_t n, uint64_t* d_counts,
                                          void* d_ws, size_t ws_bytes, void* stream) {
  using namespace gleam;
  clear_error();
  if (!c || !d_counts || (n > 0 && !d_keys)) {
    set_error("gleam_cache_erase: null table, keys or counts");
    return GLEAM_E_INVALID;
  }
  if (n > (1ull << 36) || n > 0x7fffffffull * kThreads) {
    set_error("gleam_cache_erase: more than 2^36 keys");
    return GLEAM_E_UNSUPPORTED;
  }
  const EraseLayout L = erase_layout(n);
  if (!d_ws || !aligned256(d_ws)) {
    set_error("gleam_cache_erase: workspace must be non-null and 256-byte aligned");
    return GLEAM_E_INVALID;
  }
  if (ws_bytes < L.total) {
    set_error("gleam_cache_erase: workspace of %zu bytes, %zu needed", ws_bytes, L.total);
    return GLEAM_E_WORKSPACE;
  }
  hipStream_t s = (hipStream_t)stream;
  const EraseWs w = erase_ws(d_ws, L);
  const TableRef t = table_ref(c);
  // header and both sets to zero (a fill kernel, so the call can be captured in a graph)
  gleam_status st = fill_u64(w.hdr, (kHeaderBytes + 16 * L.cap) / 8, 0, s);
  if (st != GLEAM_OK) return st;
  const dim3 block(kThreads);
  if (n > 0) {
    hipLaunchKernelGGL(erase_find_kernel, dim3((uint32_t)((n + kThreads - 1) / kThreads)), block, 0, s, t, d_keys, n, w);
    if ((st = launch_status("erase_find_kernel")) != GLEAM_OK) return st;
  }
  const uint64_t want = (n + kWaves - 1) / kWaves;  // at most one cluster per key, one wave each
  hipLaunchKernelGGL(erase_repair_kernel, dim3((uint32_t)(want == 0 ? 1 : want < kMaxGrid ? want : kMaxGrid)), block, 0,
                     s, t, d_keys, n, w, d_counts);
  return launch_status("erase_repair_kernel");
}

extern "C" gleam_status gleam_cache_export(const gleam_cache* c, uint64_t* d_keys, uint64_t* d_vals,
                                           uint64_t* d_stamps, uint64_t* d_count, void* d_ws, size_t ws_bytes,
                                           void* stream) {
  using namespace gleam;
  clear_error();
  MaintLayout L;
  gleam_status st = check_maint(c, d_ws, ws_bytes, "gleam_cache_export", &L);
  if (st != GLEAM_OK) return st;
  if (!d_keys || !d_vals || !d_count) {
    set_error("gleam_cache_export: null output");
    return GLEAM_E_INVALID;
  }
  hipStream_t s = (hipStream_t)stream;
  const TableRef t = table_ref(c);
  uint64_t* counters = ws_at<uint64_t>(d_ws, L.counters);
  uint32_t* share = ws_at<uint32_t>(d_ws, L.share);
  uint32_t* starts = ws_at<uint32_t>(d_ws, L.starts);
  Entry* entries = ws_at<Entry>(d_ws, L.entries);
  hipLaunchKernelGGL(maint_init_kernel<false>, dim3(1), dim3(kInitThreads), 0, s, t, 0, L.bins, counters,
                     (uint32_t*)nullptr);
  if ((st = launch_status("maint_init_kernel")) != GLEAM_OK) return st;
  hipLaunchKernelGGL(export_spread_kernel<false>, dim3(L.spread), dim3(kSpreadThreads), 0, s, t, counters, L.bins, share,
                     starts, entries);
  if ((st = launch_status("export_spread_kernel")) != GLEAM_OK) return st;
  hipLaunchKernelGGL(export_share_kernel, dim3((L.bins + 63) / 64), dim3(64), 0, s, L.bins, L.spread, share, starts);
  if ((st = launch_status("export_share_kernel")) != GLEAM_OK) return st;
  hipLaunchKernelGGL(export_starts_kernel, dim3(1), dim3(kInitThreads), 0, s, L.bins, starts, counters, d_count);
  if ((st = launch_status("export_starts_kernel")) != GLEAM_OK) return st;
  hipLaunchKernelGGL(export_spread_kernel<true>, dim3(L.spread), dim3(kSpreadThreads), 0, s, t, counters, L.bins, share,
                     starts, entries);
  if ((st = launch_status("export_spread_kernel")) != GLEAM_OK) return st;
  hipLaunchKernelGGL(export_bin_kernel, dim3(L.bins), dim3(kBinThreads), 0, s, counters, L.bins, starts, entries, d_keys,
                     d_vals, d_stamps);
  if ((st = launch_status("export_bin_kernel")) != GLEAM_OK) return st;
  if (c->capacity <= kBinMax) return GLEAM_OK;  // no bin can hold more
  const SortBuf sa{nullptr, ws_at<uint64_t>(d_ws, L.xlo), ws_at<uint32_t>(d_ws, L.xidx)};
  const SortBuf sb = sort_other(ws_at<uint8_t>(d_ws, L.sort1), L.m, 1);
  const uint32_t grid = grid_for(L.m) < 1024 ? grid_for(L.m) : 1024;
  hipLaunchKernelGGL(export_unpack_kernel, dim3(grid), dim3(kThreads), 0, s, counters, entries, sa);
  if ((st = launch_status("export_unpack_kernel")) != GLEAM_OK) return st;
  st = radix_sort_pairs(sa, counters + kWCollected, counters + kWBits, L.m, 1, ws_at<uint8_t>(d_ws, L.sort1), s);
  if (st != GLEAM_OK) return st;
  hipLaunchKernelGGL(export_sorted_kernel, dim3(grid), dim3(kThreads), 0, s, counters, entries, sa, sb, d_keys, d_vals,
                     d_stamps);
  return launch_status("export_sorted_kernel");
}

extern "C" gleam_status gleam_cache_set_key_bound(gleam_cache* c, uint64_t n) {
  gleam::clear_error();
  if (!c || n > c->key_bound) {
    gleam::set_error("gleam_cache_set_key_bound: null table, or the bound would rise");
    return GLEAM_E_INVALID;
  }
  c->key_bound = n;
  return GLEAM_OK;
}
