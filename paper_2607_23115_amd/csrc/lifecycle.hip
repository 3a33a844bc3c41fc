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
// wave. Evict does not leave a long cluster to one wave: its entries are taken out and put
// back in parallel (see kLongFew).
//
// The table header keeps the live-entry count (word 3): inserts add their new keys, erase
// subtracts what it removed, evict sets it, so erase can report the count without a scan.

#include "gleam_device.h"
#include "gleam_internal.h"
#include "gleam_table.h"
#include "launch_shape.h"
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
  kWBits = 4,       // 4..7: the sort's AND/OR words
  kWBaseHi = 8,     // where the cells of the order start (see Cells)
  kWBaseLo = 9,
  kWWidthHi = 10,   // and their range
  kWWidthLo = 11,
  kWLimit = 12,     // evict: the last bin collected first
  kWLastHi = 13,    // evict: (stamp, key) of the last victim
  kWLastLo = 14,
  kWLong = 15,      // evict: a victim's cluster is long
  kWMoved = 16,     // evict: entries were taken out, to be put back
  kWFull = 17,      // evict: some kCollectTile slots in a row are all occupied
};
constexpr size_t kCounterBytes = 256;

constexpr uint32_t kPickBins = 1024;        // evict's histogram

// Export: bins of the key range, each of `parts` parts of kCuts cuts. A part covers
// kPartSlots table slots' share of the range, so a part of a digest table at load 0.7 has
// 5,734 entries, of the kPartMax that a workgroup sorts in LDS. Where the table may hold more
// than kPartFine entries a part (load 0.75, by the host's bound on its keys), there are twice
// as many bins: digests then fit at any load up to 2^27 slots, and up to load 0.75 in 2^28
// (kMaxAllParts). 2^20 slots at load 0.95: 109 us, against 304 when the parts overflow and
// the radix sort takes over, and 260 for gathering and sorting from the start. The entries are
// written to their bins only, so that a tile of 8,192 slots has several entries for each bin.
constexpr uint32_t kPartSlots = 8192;
constexpr uint32_t kPartMax = 7168;
constexpr uint32_t kPartFine = 6144;
constexpr uint32_t kCuts = 2048;
constexpr uint32_t kMaxParts = 8;
constexpr uint32_t kBinMax = 65535;         // entries of a bin (numbered in 16 bits)
constexpr uint32_t kMaxAllParts = 32768;
constexpr uint32_t kFewParts = 16384;       // up to these the kernels take half the LDS and registers
constexpr uint32_t kSpreadGrid = 256;       // workgroups that spread the entries over the bins

struct MaintLayout {
  uint64_t m;     // capacity + 1 (the last is the key kEmpty's header side slot)
  uint32_t bins, parts, spread;  // (bins: the fewer ones)
  size_t counters;
  size_t pick, occupied, leaders, hi, lo, idx, sort2;          // evict
  size_t share, starts, xkey, xpay, xidx, sort1;               // export
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
  L.occupied = take(8 * ((capacity + 63) / 64));
  L.leaders = take(4 * L.m);
  L.hi = take(8 * sort_capacity(L.m));  // the sort's keys and indices (its buffer a)
  L.lo = take(8 * sort_capacity(L.m));
  L.idx = take(4 * sort_capacity(L.m));
  L.sort2 = take(sort_layout(L.m, 2).total);
  L.pick = L.sort2;  // done with before the sort begins (its second buffer holds 8 KiB or more)
  const size_t evict_total = off;
  off = kCounterBytes;
  const uint64_t want = capacity / kPartSlots;
  const uint32_t all = (uint32_t)(want < 1 ? 1 : want < kMaxAllParts / 2 ? want : kMaxAllParts / 2);
  L.parts = all < kMaxParts ? all : kMaxParts;
  L.bins = all / L.parts;
  const uint64_t spread = (capacity + 4095) / 4096;
  L.spread = (uint32_t)(spread < kSpreadGrid ? spread : kSpreadGrid);
  L.share = take(4 * 2 * (size_t)all * L.spread);
  L.starts = take(4 * (2 * (size_t)all + 1));
  L.xkey = take(8 * sort_capacity(L.m));  // every entry's key by bin (the radix sort's buffer a)
  L.xpay = take(16 * L.m);                // and {value, stamp}
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

// Stamp word of key k (k != kEmpty) from slot pos of its probe sequence on, or null; *now
// gets the stamp, read along with the key.
__device__ __forceinline__ uint64_t* find_stamp(const TableRef& t, uint64_t k, uint64_t pos, uint64_t* now) {
  for (uint64_t probe = 0; probe <= t.mask; probe += kProbeAhead) {
    uint64_t key[kProbeAhead], stamp[kProbeAhead];
#pragma unroll
    for (int j = 0; j < kProbeAhead; ++j) {
      const uint64_t at = (pos + j) & t.mask;
      key[j] = t.slots[2 * at];
      stamp[j] = __hip_atomic_load(&t.stamps[at], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
#pragma unroll
    for (int j = 0; j < kProbeAhead; ++j) {
      if (key[j] == k) {
        *now = stamp[j];
        return &t.stamps[(pos + j) & t.mask];
      }
      if (key[j] == kEmpty) return nullptr;
    }
    pos = (pos + kProbeAhead) & t.mask;
  }
  return nullptr;
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
// already reads at or past its epoch skips the atomic. Bound by the round trips of the
// random reads.
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
  const uint64_t ki = keys[valid ? i : n - 1];  // n >= 1; clamped so the load is unconditional
  const uint64_t k = valid ? ki : 0;
  const uint64_t e = valid ? (epochs ? epochs[i] : epoch) : 0;
  // the home slot and its stamp are read before the workgroup's LDS pass, which hides
  // under them: most probes end there
  const uint64_t home = k != kEmpty ? slot_hash(k, t.shift) : 0;
  const uint64_t home_key = t.slots[2 * home];
  const uint64_t home_stamp = __hip_atomic_load(&t.stamps[home], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
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
    uint64_t now = home_stamp;
    if (k == kEmpty) {
      if (t.hdr[0]) {
        stamp = &t.hdr[2];
        now = 0;
      }
    } else if (home_key == k) {
      stamp = &t.stamps[home];
    } else if (home_key != kEmpty) {
      stamp = find_stamp(t, k, (home + 1) & t.mask, &now);
    }
    if (stamp) {
      hit = 1;
      if (lead && now < top) atomicMax(ull(stamp), (unsigned long long)top);
    }
  }
  hit = wave_sum(hit);
  __syncthreads();  // bkeys read by every thread
  if ((tid & 63) == 0) bkeys[tid >> 6] = hit;
  __syncthreads();
  if (n_touched && tid == 0) {
    for (int w = 1; w < kThreads / 64; ++w) hit += bkeys[w];
    if (hit) atomicAdd(ull(n_touched), (unsigned long long)hit);
  }
}

// ---- selection over the range of (stamp, key) -----------------------------------------
typedef unsigned __int128 u128;
__device__ __forceinline__ u128 order_of(uint64_t stamp, uint64_t key) { return ((u128)stamp << 64) | key; }

// The order cut into equal cells: cell(x) in [0, cells) never decreases with x, which is
// all that the callers rely on; entries outside the range take the first or the last
// cell. The 32 leading bits of x's distance from the base (leading: from the top bit of the
// range) times cells / range, so the cells are even for any range, not only powers of two.
struct Cells {
  u128 base, width;
  uint32_t lead;    // shift that brings the range's top bit to bit 127
  uint32_t factor;  // cells * 2^32 / (leading bits of the range + 1), at most 2 * cells
  __device__ Cells(const uint64_t* counters, uint32_t cells)
      : base(order_of(counters[kWBaseHi], counters[kWBaseLo])),
        width(order_of(counters[kWWidthHi], counters[kWWidthLo])) {
    const uint64_t hi = (uint64_t)(width >> 64), lo = (uint64_t)width;
    lead = hi ? (uint32_t)__builtin_clzll(hi) : lo ? 64u + (uint32_t)__builtin_clzll(lo) : 0u;
    const uint64_t top = (uint64_t)(uint32_t)((width << lead) >> 96) + 1;
    factor = width == 0 ? 0u : (uint32_t)(((uint64_t)cells << 32) / top);  // cells < 2^31
  }
  __device__ __forceinline__ uint32_t of(u128 x) const {
    if (x < base) return 0;
    u128 d = x - base;
    d = d < width ? d : width;
    return (uint32_t)(((uint64_t)(uint32_t)((d << lead) >> 96) * factor) >> 32);
  }
};

// The same for an order by key alone (the range below 2^64).
struct KeyCells {
  uint64_t base, width;
  uint32_t lead, factor;
  __device__ KeyCells(const uint64_t* counters, uint32_t cells) : base(counters[kWBaseLo]), width(counters[kWWidthLo]) {
    const Cells c(counters, cells);
    lead = width ? c.lead - 64 : 0;
    factor = c.factor;
  }
  __device__ __forceinline__ uint32_t of(uint64_t k) const {
    if (k < base) return 0;
    const uint64_t d = min(k - base, width);
    return (uint32_t)(((uint64_t)(uint32_t)((d << lead) >> 32) * factor) >> 32);
  }
};

// One workgroup: the counters of a call, and the range of its cells, from the least and
// greatest of at most kSamples entries (runs of 64 slots, evenly spaced: places in the
// table are hashes, so a run is as good a sample as scattered slots and an eighth of the
// lines), with a margin of 1/1024 of their range on either side. For eviction also the bin
// up to which to collect: the share of the victims among the samples, plus six standard
// deviations and a few, so that one pass over the table nearly always collects them all.
constexpr uint32_t kInitThreads = 1024;
constexpr uint32_t kSamplesEach = 16;
constexpr uint64_t kSamples = (uint64_t)kInitThreads * kSamplesEach;

// kByStamp: the order is (stamp, key), else the key alone.
template <bool kByStamp>
__global__ __launch_bounds__(kInitThreads) void maint_init_kernel(TableRef t, uint64_t keep, uint64_t* counters,
                                                                  uint32_t* pick) {
  static_assert(kPickBins == kInitThreads, "one bin per thread");
  __shared__ uint64_t part[kInitThreads / 64][4];
  __shared__ uint32_t h[kPickBins], wave_sum[kInitThreads / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t capacity = t.mask + 1;
  h[threadIdx.x] = 0;
  if (kByStamp) pick[threadIdx.x] = 0;
  const uint64_t n = capacity < kSamples ? capacity : kSamples, step = capacity / n;
  uint64_t key[kSamplesEach], stamp[kSamplesEach];
#pragma unroll
  for (uint32_t r = 0; r < kSamplesEach; ++r) {  // unconditional (clamped) loads, issued together
    const uint64_t i = (uint64_t)r * kInitThreads + threadIdx.x;
    const uint64_t slot = i < n ? (i - lane) * step + lane : 0;  // (capacity below 64: one run, step 1)
    key[r] = t.slots[2 * slot];
    stamp[r] = kByStamp ? t.stamps[slot] : 0;
    if (i >= n) key[r] = kEmpty;
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
  const uint64_t live = t.hdr[3];
  const uint64_t drop = live > keep ? live - keep : 0;
  if (threadIdx.x == 0) {
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
    counters[kWCollected] = 0;
    counters[kWDrop] = drop;
    counters[kWLive] = live;
    counters[kWBits + 0] = ~0ull;
    counters[kWBits + 1] = 0;
    counters[kWBits + 2] = ~0ull;
    counters[kWBits + 3] = 0;
    counters[kWBaseHi] = (uint64_t)(base >> 64);
    counters[kWBaseLo] = (uint64_t)base;
    counters[kWWidthHi] = (uint64_t)((end - base) >> 64);
    counters[kWWidthLo] = (uint64_t)(end - base);
    counters[kWLimit] = kPickBins - 1;
    counters[kWLong] = 0;
    counters[kWMoved] = 0;
    counters[kWFull] = 0;
  }
  if (!kByStamp) return;
  __syncthreads();  // the range, read back by every thread of this workgroup
  const Cells bins(counters, kPickBins);
#pragma unroll
  for (uint32_t r = 0; r < kSamplesEach; ++r)
    if (key[r] != kEmpty) atomicAdd(&h[bins.of(order_of(stamp[r], key[r]))], 1u);
  __syncthreads();
  const uint32_t c = h[threadIdx.x];
  uint32_t incl = c;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = __shfl_up(incl, d, 64);
    if (lane >= d) incl += y;
  }
  if (lane == 63) wave_sum[wave] = incl;
  __syncthreads();
  uint32_t run = incl - c, total = 0;
  for (int w = 0; w < (int)(kInitThreads / 64); ++w) {
    if (w < wave) run += wave_sum[w];
    total += wave_sum[w];
  }
  const float share = live ? (float)drop / (float)live * (float)total : 0.0f;
  const uint32_t want = (uint32_t)(share + 6.0f * sqrtf(share)) + 8;
  if (run < want && run + c >= want) counters[kWLimit] = threadIdx.x;
}

// Folds into a pair of AND/OR words. A word that would not change is only read: atomics on
// one address queue at about 10 ns each, and all but the first few change nothing.
__device__ __forceinline__ void fold_bits(uint64_t* bits, uint64_t and_w, uint64_t or_w) {
  const uint64_t a = __hip_atomic_load(&bits[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const uint64_t o = __hip_atomic_load(&bits[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if ((a & and_w) != a) atomicAnd(ull(&bits[0]), (unsigned long long)and_w);
  if ((o | or_w) != o) atomicOr(ull(&bits[1]), (unsigned long long)or_w);
}

// ---- evict ----------------------------------------------------------------------------
// Reads the table once (the entries up to a bin that the samples say holds the last
// victim) and writes only what it evicts. Should the samples have misled it, a histogram
// of the whole table finds the bin and a second pass collects what is missing. 20 M entries
// in 2^25 slots, 20,000 evicted: 0.38 ms (collecting 184 us, 4.4 TB/s; the sort's sixteen
// passes 136), against 5.9 ms for gathering, sorting and re-inserting every entry; half of
// them evicted 2.9 against 5.1 ms; all of them 4.6 against 4.5.
constexpr uint32_t kPickThreads = 1024;
constexpr uint32_t kPickGrid = 256;  // few enough that the final atomics on the bins stay few
constexpr uint32_t kPickItems = 4;

__global__ __launch_bounds__(kPickThreads) void evict_pick_kernel(TableRef t, const uint64_t* counters, uint32_t* pick) {
  __shared__ uint32_t h[kPickBins];
  if (counters[kWCollected] >= counters[kWDrop]) return;
  for (uint32_t i = threadIdx.x; i < kPickBins; i += kPickThreads) h[i] = 0;
  __syncthreads();
  const Cells bins(counters, kPickBins);
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

// Collects the entries up to the sampled bin (kAgain: those after it, up to the bin with
// which the histogram's running count reaches the victims) as pairs (stamp, key) with
// their slot (the side slot: capacity). A wave lists the slots that it takes in LDS and
// writes kListFlush or more of them at a time, claiming their positions with one atomic
// (the claims queue on one word: by 64, 20 M entries took 3 ms); it has no barrier on its
// way through the table. It also folds the AND and
// OR of what it collects, from which the sort skips the digits every entry shares, and
// notes which slots are occupied (a bit each), and whether a whole step of them is.
constexpr uint32_t kCollectItems = 8;
constexpr uint64_t kCollectTile = 64 * kCollectItems;  // slots per step of a wave
constexpr uint32_t kCollectGrid = 512;  // 2^25 slots: 512 workgroups 175 us, 1,024 190, 2,048 228
constexpr int kCollectWaves = kThreads / 64;
constexpr uint32_t kListFlush = 1536;  // listed slots that a wave writes out with one claim

template <bool kAgain>
__global__ __launch_bounds__(kThreads) void evict_collect_kernel(TableRef t, const uint32_t* pick, uint64_t* counters,
                                                                 SortBuf sb, uint64_t* occupied) {
  static_assert(kPickBins == 4 * kThreads, "four bins per thread");
  __shared__ uint32_t wave_sum[kCollectWaves];
  __shared__ uint32_t bin_limit;
  __shared__ uint64_t claimed;
  __shared__ uint32_t list[kCollectWaves][kListFlush + kCollectTile + 64];
  __shared__ uint64_t fold[kCollectWaves][4];
  const uint64_t drop = counters[kWDrop];
  if (drop == 0) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
  uint32_t after = 0, limit = (uint32_t)counters[kWLimit];  // bins [after, limit]
  if (kAgain) {
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
    if (lane == 63) wave_sum[wave] = incl;
    if (threadIdx.x == 0) bin_limit = 0;
    __syncthreads();
    uint64_t run = incl - sum;
    for (int w = 0; w < wave; ++w) run += wave_sum[w];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (run < drop && run + c[j] >= drop) bin_limit = 4 * threadIdx.x + j;
      run += c[j];
    }
    __syncthreads();
    after = limit + 1;
    limit = bin_limit;
    if (limit < after) return;  // the first pass collected them all (the histogram is all zero)
  }
  const Cells bins(counters, kPickBins);
  const uint64_t capacity = t.mask + 1;
  uint64_t and_k = ~0ull, or_k = 0, and_s = ~0ull, or_s = 0;
  uint32_t listed = 0;  // the same in every lane
  auto write = [&](uint64_t p, uint32_t from, uint32_t count) {  // list[from, from + count) to p on, count <= 64
    p += lane;
    if ((uint32_t)lane >= count) return;
    const uint32_t slot = list[wave][from + lane];
    const uint64_t key = slot < capacity ? t.slots[2 * (uint64_t)slot] : kEmpty;
    const uint64_t stamp = slot < capacity ? t.stamps[slot] : t.hdr[2];
    sb.hi[p] = stamp;
    sb.lo[p] = key;
    sb.idx[p] = slot;
    and_k &= key;
    or_k |= key;
    and_s &= stamp;
    or_s |= stamp;
  };
  auto in_range = [&](uint64_t key, uint64_t stamp) {
    const uint32_t b = bins.of(order_of(stamp, key));
    return b >= after && b <= limit;
  };
  const uint64_t waves = (uint64_t)gridDim.x * kCollectWaves;
  for (uint64_t i0 = ((uint64_t)blockIdx.x * kCollectWaves + wave) * kCollectTile; i0 < capacity;
       i0 += waves * kCollectTile) {
    uint64_t key[kCollectItems], stamp[kCollectItems];
#pragma unroll
    for (uint32_t r = 0; r < kCollectItems; ++r) {  // unconditional (clamped) loads, issued together
      const uint64_t i = i0 + 64 * r + lane, at = i < capacity ? i : capacity - 1;
      key[r] = t.slots[2 * at];
      stamp[r] = t.stamps[at];
    }
    uint64_t held_word = 0;
    bool full = true;
#pragma unroll
    for (uint32_t r = 0; r < kCollectItems; ++r) {
      const uint64_t i = i0 + 64 * r + lane;
      const bool held = i < capacity && key[r] != kEmpty;
      const uint64_t word = __ballot(held);
      if (lane == (int)r) held_word = word;
      full = full && word == ~0ull;
      const bool mine = held && in_range(key[r], stamp[r]);
      const uint64_t who = __ballot(mine);
      if (mine) list[wave][listed + (uint32_t)__popcll(who & lt)] = (uint32_t)i;
      listed += (uint32_t)__popcll(who);
    }
    if (!kAgain && lane < (int)kCollectItems && i0 + 64 * lane < capacity) occupied[i0 / 64 + lane] = held_word;
    if (!kAgain && full && lane == 0) counters[kWFull] = 1;
    wave_lds_sync();
    if (listed >= kListFlush) {  // all but a remainder, from the end of the list
      const uint32_t keep = listed % 64;
      uint64_t p = 0;
      if (lane == 0) p = atomicAdd(ull(&counters[kWCollected]), (unsigned long long)(listed - keep));
      p = shfl64(p, 0);
      for (uint32_t from = keep; from < listed; from += 64) write(p + from - keep, from, 64);
      listed = keep;
    }
    wave_lds_sync();  // the list read before the next step adds to it
  }
  if (blockIdx.x == 0 && wave == 0 && t.hdr[0] && in_range(kEmpty, t.hdr[2])) {
    if (lane == 0) list[0][listed] = (uint32_t)capacity;
    ++listed;
    wave_lds_sync();
  }
  // what is left in the lists: one claim per workgroup
  if (lane == 0) wave_sum[wave] = listed;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t total = 0;
    for (int w = 0; w < kCollectWaves; ++w) total += wave_sum[w];
    claimed = total ? atomicAdd(ull(&counters[kWCollected]), (unsigned long long)total) : 0;
  }
  __syncthreads();
  uint64_t p = claimed;
  for (int w = 0; w < wave; ++w) p += wave_sum[w];
  for (uint32_t from = 0; from < listed; from += 64) write(p + from, from, min(listed - from, 64u));
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
    for (int w = 1; w < kCollectWaves; ++w) {
      fold[0][0] &= fold[w][0];
      fold[0][1] |= fold[w][1];
      fold[0][2] &= fold[w][2];
      fold[0][3] |= fold[w][3];
    }
    fold_bits(counters + kWBits, fold[0][0], fold[0][1]);
    fold_bits(counters + kWBits + 2, fold[0][2], fold[0][3]);
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

// Eight lanes look along a table from one slot (128 bytes of slots): the cost of a probe or
// of a walk to a cluster's start is then a round trip or two of memory instead of one per
// slot.
constexpr int kSpan = 8;
constexpr uint64_t kFindGrid = 1u << 20;
__device__ __forceinline__ uint32_t span_ballot(bool x, int lane) {
  return (uint32_t)(__ballot(x) >> (lane & ~(kSpan - 1))) & ((1u << kSpan) - 1);
}

// The first `drop` of the sorted entries go: lists their keys, and finds the clusters to
// repair: starts[i] is the start of victim i's cluster if it is the cluster's first victim
// (no victim before it up to the start), else kNoStart. (One word per victim: a list of the
// starts needs an atomic per wave on one counter, 50 us for 20,000 victims.) Many victims
// are repaired in a pass over the whole table instead, which needs no starts.
constexpr uint32_t kNoStart = ~0u;

// A long cluster is a long chain for one wave, and the longest ones grow without bound as the
// load nears 1 (random keys in 2^20 slots: some of 4,096 slots from load 0.95 on, where one
// lane repaired them slot by slot: 1,000 victims 29 ms, 106 at load 0.97). So, where slots of
// a whole collecting step in a row are occupied (else no cluster has 1,024), the pass over the
// table takes the entries of long clusters out, each wave those of its 64 slots, and
// evict_put_back_kernel inserts them again, each by its own lane (1.0 and 1.8 ms). With few
// victims one in a cluster of kLongFew slots or more sends the call through that pass, and
// only such clusters are taken out (a wave repairs up to kLongFew slots, and there may be many
// clusters and no victim in most of them: 20 victims in 2^25 slots at load 0.95 took 0.48 ms
// so, 4.2 with 512 in the place of 4,096). With many victims nearly every cluster has some:
// from kLongMany slots on (half of 2^20 slots at load 0.95: 0.36 ms; 0.39 with 512).
constexpr uint32_t kLongFew = 4096, kLongMany = 256;

// From one victim in 64 slots on: in 2^25 slots a pass over the table takes about as long
// as finding and repairing the clusters of half a million victims one by one.
__device__ __forceinline__ bool many_victims(const TableRef& t, uint64_t drop) { return drop > (t.mask + 1) / 64; }
__global__ __launch_bounds__(kThreads) void evict_mark_kernel(TableRef t, SortBuf a, SortBuf b, uint64_t* counters,
                                                              const uint64_t* occupied, uint32_t* starts,
                                                              uint64_t* evicted, uint64_t* counts) {
  const uint64_t drop = counters[kWDrop], live = counters[kWLive];
  const uint64_t t0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t0 == 0) {
    counts[0] = drop;
    counts[1] = live - drop;
    t.hdr[3] = live - drop;
  }
  if (drop == 0) return;
  const SortBuf sorted = sort_result(a, b, counters + kWBits, 2);
  const UpTo gone = last_victim(sorted, drop);
  if (t0 == 0) {
    counters[kWLastHi] = (uint64_t)(gone.last >> 64);
    counters[kWLastLo] = (uint64_t)gone.last;
  }
  const int lane = threadIdx.x & 63, l = lane & (kSpan - 1);
  const bool full = counters[kWFull] != 0;
  if (many_victims(t, drop)) {
    for (uint64_t i = t0; i < drop; i += (uint64_t)gridDim.x * blockDim.x) {
      if (evicted) evicted[i] = sorted.lo[i];
      if (sorted.idx[i] > t.mask) t.hdr[0] = t.hdr[1] = t.hdr[2] = 0;  // the side slot
    }
    return;
  }
  const uint64_t spans = (uint64_t)gridDim.x * blockDim.x / kSpan;
  const uint64_t rounds = (drop + spans - 1) / spans;
  for (uint64_t r = 0; r < rounds; ++r) {  // the same number in every lane
    const uint64_t i = r * spans + t0 / kSpan;
    bool walking = i < drop;
    uint64_t c0 = 0;
    if (walking) {
      c0 = sorted.idx[i];
      if (evicted && l == 0) evicted[i] = sorted.lo[i];
      if (c0 > t.mask) {  // the side slot
        if (l == 0) t.hdr[0] = t.hdr[1] = t.hdr[2] = 0;
        walking = false;
      }
    }
    bool first = walking;
    // whole words of the cluster after the victim's, up to kLongFew slots
    const uint64_t v = walking ? c0 : 0, last_word = t.mask / 64;
    uint32_t after = 0;
    for (uint32_t at = 0; full && __any(walking && after == at) && at < kLongFew / 64 && at <= last_word; at += kSpan) {
      const uint32_t open = span_ballot(occupied[(v / 64 + 1 + at + l) & last_word] != ~0ull, lane);
      if (after == at) after += open ? __builtin_ctz(open) : kSpan;
    }
    uint32_t steps = 0;
    for (; __any(walking) && steps < kLongFew && steps <= t.mask; steps += kSpan) {
      const uint64_t p = (c0 - 1 - l) & t.mask;
      const uint64_t k = t.slots[2 * p], stamp = t.stamps[p];
      const uint32_t open = span_ballot(k == kEmpty, lane), hit = span_ballot(gone(k, stamp), lane);
      const int far = open ? __builtin_ctz(open) : kSpan;  // entries of the cluster before c0, up to here
      if (walking) {
        if (hit & ((1u << far) - 1)) {
          first = walking = false;
        } else {
          c0 = (c0 - far) & t.mask;
          walking = far == kSpan;
        }
      }
    }
    if (first && l == 0 && (walking || ((v - c0) & t.mask) + 64 * (uint64_t)after >= kLongFew)) counters[kWLong] = 1;
    if (i < drop && l == 0) starts[i] = first ? (uint32_t)c0 : kNoStart;
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
  const uint64_t p0 = (c0 + lane) & t.mask;
  const uint4 e0 = *reinterpret_cast<const uint4*>(t.slots + 2 * p0);
  const uint64_t stamp0 = t.stamps[p0];
  uint32_t len = 0;  // the cluster's slots
  {
    const uint64_t open = __ballot(lo64(e0) == kEmpty);
    len = open ? (uint32_t)__builtin_ctzll(open) : 64u;
    for (uint32_t w = 1; len == 64 * w && w < kRepairWords && len <= t.mask; ++w) {
      const uint64_t more = __ballot(t.slots[2 * ((c0 + len + lane) & t.mask)] == kEmpty);
      len += more ? (uint32_t)__builtin_ctzll(more) : 64u;
    }
  }
  uint32_t removed = 0;
  if (len >= 64 * kRepairWords) {  // a longer cluster (of an erased key): one lane, slot by slot
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
    uint4 e = e0;
    uint64_t stamp = stamp0;
    if (w) {
      e = *reinterpret_cast<const uint4*>(t.slots + 2 * p);
      stamp = t.stamps[p];
    }
    const uint64_t k = lo64(e);
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
  uint64_t* hdr;          // [0] removed entries | arrived workgroups << 40
  uint64_t* keyset;       // cap slots: the erased keys (kEmpty free; that key is never in it)
  uint64_t* starts;       // cap slots: cluster start + 1 (0 free)
  uint64_t* leaders;      // per key: the cluster start it claimed, or kNone
  uint64_t mask;
  int shift;
};
constexpr uint64_t kNone = ~0ull;
constexpr int kArrivedShift = 40;  // n <= 2^36 entries, and a grid below 2^24 workgroups

__global__ __launch_bounds__(kThreads) void erase_clear_kernel(EraseWs w) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  const uint64_t t0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t0 == 0) w.hdr[0] = 0;
  for (uint64_t i = t0; i <= w.mask; i += stride) {
    w.keyset[i] = kEmpty;
    w.starts[i] = 0;
  }
}

__device__ __forceinline__ bool in_keyset(const EraseWs& w, uint64_t k) {
  uint64_t pos = slot_hash(k, w.shift);
  for (uint64_t probe = 0; probe <= w.mask; ++probe) {
    const uint64_t v = w.keyset[pos];
    if (v == k) return true;
    if (v == kEmpty) return false;
    pos = (pos + 1) & w.mask;
  }
  return false;
}

// Per erased key, by kSpan lanes: into the key set; if the table holds it, the start of
// its cluster, claimed once. (The two do not depend on each other: one launch, the first
// probe of the table read before the key set's compare-and-swap.)
__global__ __launch_bounds__(kThreads) void erase_find_kernel(TableRef t, const uint64_t* keys, uint64_t n, EraseWs w) {
  const int lane = threadIdx.x & 63, l = lane & (kSpan - 1);
  const uint64_t spans = (uint64_t)gridDim.x * blockDim.x / kSpan;
  for (uint64_t base_i = (uint64_t)blockIdx.x * blockDim.x / kSpan; base_i < n; base_i += spans) {  // uniform
    const uint64_t i = base_i + threadIdx.x / kSpan;
    const uint64_t k = i < n ? keys[i] : kEmpty;
    bool looking = k != kEmpty;
    uint64_t at = slot_hash(k, t.shift);
    uint64_t seen = t.slots[2 * ((at + l) & t.mask)];
    uint32_t repeat = 0;
    if (l == 0 && i < n) {
      if (k == kEmpty) {  // the header's side slot
        if (atomicExch(ull(&t.hdr[0]), 0ull) == 1ull) {
          t.hdr[2] = 0;
          atomicAdd(ull(&w.hdr[0]), 1ull);
        }
      } else {
        uint64_t pos = slot_hash(k, w.shift);
        for (uint64_t probe = 0; probe <= w.mask; ++probe) {
          const uint64_t prev = atomicCAS(ull(&w.keyset[pos]), (unsigned long long)kEmpty, (unsigned long long)k);
          if (prev == kEmpty) break;
          if (prev == k) {  // a repeat: the other one finds the cluster
            repeat = 1;
            break;
          }
          pos = (pos + 1) & w.mask;
        }
      }
    }
    if (__shfl((int)repeat, lane & ~(kSpan - 1), 64)) looking = false;
    bool found = false;
    for (uint64_t step = 0; __any(looking) && step <= t.mask; step += kSpan) {
      const uint32_t same = span_ballot(seen == k, lane), open = span_ballot(seen == kEmpty, lane);
      if (looking) {
        if (same) {  // a key is held once, and before the first empty slot from its home
          const int j = __builtin_ctz(same);
          found = (open & ((1u << j) - 1)) == 0;
          at = (at + j) & t.mask;
          looking = false;
        } else if (open) {
          looking = false;
        } else {
          at = (at + kSpan) & t.mask;
        }
      }
      if (__any(looking)) seen = t.slots[2 * ((at + l) & t.mask)];
    }
    bool walking = found;
    uint64_t c0 = at;
    for (uint64_t step = 0; __any(walking) && step <= t.mask; step += kSpan) {
      const uint32_t open = span_ballot(t.slots[2 * ((c0 - 1 - l) & t.mask)] == kEmpty, lane);
      const int far = open ? __builtin_ctz(open) : kSpan;
      if (walking) {
        c0 = (c0 - far) & t.mask;
        walking = far == kSpan;
      }
    }
    bool first = false;
    if (found && l == 0) {
      uint64_t pos = slot_hash(c0, w.shift);
      for (uint64_t probe = 0; probe <= w.mask; ++probe) {
        const uint64_t prev = atomicCAS(ull(&w.starts[pos]), 0ull, (unsigned long long)(c0 + 1));
        if (prev == 0) first = true;
        if (prev == 0 || prev == c0 + 1) break;  // claimed here, or by another key of this cluster
        pos = (pos + 1) & w.mask;
      }
    }
    if (l == 0 && i < n) w.leaders[i] = first ? c0 : kNone;
  }
}

struct InKeyset {
  const EraseWs& w;
  __device__ bool operator()(uint64_t k, uint64_t) const { return in_keyset(w, k); }
};

// One wave per cluster; the last workgroup to arrive writes the counts. Sixteen waves per
// workgroup and a grid of at most kRepairGrid: the workgroups' arrivals queue on one word.
constexpr int kRepairThreads = 1024;
constexpr int kRepairWaves = kRepairThreads / 64;
constexpr uint64_t kRepairGrid = 512;
__global__ __launch_bounds__(kRepairThreads) void erase_repair_kernel(TableRef t, uint64_t n, EraseWs w,
                                                                      uint64_t* counts) {
  __shared__ uint64_t used[kRepairWaves][kRepairWords];
  __shared__ uint32_t removed[kRepairWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const InKeyset erased{w};
  uint32_t mine = 0;
  for (uint64_t c = (uint64_t)blockIdx.x * kRepairWaves + wave; c < n; c += (uint64_t)gridDim.x * kRepairWaves)
    if (w.leaders[c] != kNone) mine += wave_repair(t, w.leaders[c], erased, used[wave], lane);
  if (lane == 0) removed[wave] = mine;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t add = 1ull << kArrivedShift;
    for (int v = 0; v < kRepairWaves; ++v) add += removed[v];
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

// Entries of long clusters on their way out of the table and back: key, value and stamp by
// the slot that they come from, and a bit for each.
struct Moved {
  uint64_t *key, *val, *stamp, *bits;
};

// The slots of word w (occupied bits occ) that lie in clusters of `from` slots or more. A
// cluster gets that long only through a whole word, so most words need only their
// neighbours; else the wave reads the 64 words on either side. Every word of a cluster
// finds the same: its length, or that it reaches past those words. Every lane calls it.
__device__ __forceinline__ uint64_t long_slots(const uint64_t* occupied, uint64_t last_word, uint64_t w, uint64_t occ,
                                               uint32_t from, int lane) {
  static_assert(kLongMany >= 256 && kLongFew <= 4096, "seen from any of its words");
  const uint64_t prev = occupied[(w - 1) & last_word], next = occupied[(w + 1) & last_word];
  if (occ != ~0ull && prev != ~0ull && next != ~0ull) return 0;
  const uint64_t down = occupied[(w - 1 - lane) & last_word], up = occupied[(w + 1 + lane) & last_word];
  const uint64_t down_open = __ballot(down != ~0ull), up_open = __ballot(up != ~0ull);
  uint32_t before = 4096, after = 4096;  // occupied slots next to the word
  if (down_open) {
    const int j = __builtin_ctzll(down_open);
    before = 64 * j + (uint32_t)__builtin_clzll(~shfl64(down, j));
  }
  if (up_open) {
    const int j = __builtin_ctzll(up_open);
    after = 64 * j + (uint32_t)__builtin_ctzll(~shfl64(up, j));
  }
  if (occ == ~0ull) return before + 64 + after >= from ? ~0ull : 0;
  const uint32_t head = (uint32_t)__builtin_ctzll(~occ), tail = (uint32_t)__builtin_clzll(~occ);
  uint64_t slots = 0;
  if (head && before + head >= from) slots |= (1ull << head) - 1;
  if (tail && tail + after >= from) slots |= ~0ull << (64 - tail);
  return slots;
}

// The clusters that start in the 64 slots of word w, by one wave; `occupied` tells the
// clusters as they were before any repair (a neighbouring wave may already have emptied the
// slot before these). Those that end here too are done together: their entries are in the
// lanes, and empty slots, which stay empty, keep them apart. One that goes on past the word
// takes wave_repair. Of a long cluster the wave takes out the slots of this word only.
template <class Erased>
__device__ void wave_repair_word(const TableRef& t, const uint64_t* occupied, uint64_t w, const Erased& erased,
                                 uint64_t* used, const Moved& moved, uint64_t* any_moved, uint32_t long_from,
                                 int lane) {
  const uint64_t occ = occupied[w], before = (64 * w - 1) & t.mask;
  const uint32_t size = t.mask < 63 ? (uint32_t)t.mask + 1 : 64u;
  const uint64_t p = 64 * w + (uint64_t)lane < t.mask ? 64 * w + (uint64_t)lane : t.mask;
  const uint4 e = *reinterpret_cast<const uint4*>(t.slots + 2 * p);
  const uint64_t stamp = t.stamps[p], k = lo64(e);
  const uint64_t out = long_from ? long_slots(occupied, t.mask / 64, w, occ, long_from, lane) : 0;
  const uint64_t starts = occ & ~(occ << 1 | ((occupied[before / 64] >> (before & 63)) & 1)) & ~out;
  const bool mine_out = (out >> lane) & 1, back = mine_out && !erased(k, stamp);
  const uint64_t back_bits = __ballot(back);
  if (long_from && lane == 0) moved.bits[w] = back_bits;
  if (out) {  // uniform, as all the masks are
    if (lane == 0) *any_moved = 1;
    if (back) {
      moved.key[p] = k;
      moved.val[p] = hi64(e);
      moved.stamp[p] = stamp;
    }
    if (mine_out) {
      t.slots[2 * p] = kEmpty;
      t.stamps[p] = 0;
    }
  }
  if (starts == 0) return;
  // the slots of this word's own clusters: from the first start on
  uint64_t own = occ & ~out & (~0ull << __builtin_ctzll(starts));
  if ((own >> (size - 1)) & 1) {  // the last cluster reaches the word's end
    const int c = 63 - __builtin_clzll(starts);
    own &= (1ull << c) - 1;
    wave_repair(t, 64 * w + (uint64_t)c, erased, used, lane);
  }
  const uint64_t gone = __ballot(((own >> lane) & 1) && erased(k, stamp));
  if (gone == 0) return;
  // entries after a victim of their cluster: flood upwards through the occupied slots
  uint64_t flood = gone, run = own;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    flood |= run & (flood << d);
    run &= run << d;
  }
  uint64_t moves = flood & ~gone, now = own & ~flood;
  const uint32_t home = (uint32_t)(slot_hash(k, t.shift) - 64 * w) & 63;
  uint32_t to = (uint32_t)lane;
  for (uint64_t left = moves; left; left &= left - 1) {
    const int src = __builtin_ctzll(left);
    const uint64_t room = ~now & (~0ull << lane32(home, src));
    now |= room & (0 - room);
    if (lane == src) to = (uint32_t)__builtin_ctzll(room);
  }
  if (((moves >> lane) & 1) && to != (uint32_t)lane) {
    *reinterpret_cast<uint4*>(t.slots + 2 * (64 * w + to)) = e;
    t.stamps[64 * w + to] = stamp;
  }
  if (((own & ~now) >> lane) & 1) {
    t.slots[2 * p] = kEmpty;
    t.stamps[p] = 0;
  }
}

// One wave per cluster with victims, or, with many or in long clusters, one per 64 slots of
// the table; with nothing but victims, a clear. (`moved` lies where the sorted victims were.)
__global__ __launch_bounds__(kThreads) void evict_repair_kernel(TableRef t, uint64_t* counters, const uint32_t* starts,
                                                                const uint64_t* occupied, Moved moved) {
  __shared__ uint64_t used[kWaves][kRepairWords];
  const uint64_t drop = counters[kWDrop];
  if (drop == 0) return;
  if (drop == counters[kWLive]) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; p <= t.mask; p += stride) {
      *reinterpret_cast<uint4*>(t.slots + 2 * p) = make_uint4(~0u, ~0u, ~0u, ~0u);  // kEmpty, any value
      t.stamps[p] = 0;
    }
    return;
  }
  const UpTo gone{order_of(counters[kWLastHi], counters[kWLastLo])};
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t first = (uint64_t)blockIdx.x * kWaves + wave, stride = (uint64_t)gridDim.x * kWaves;
  const bool many = many_victims(t, drop);
  if (many || counters[kWLong]) {
    const uint32_t long_from = counters[kWFull] == 0 ? 0 : many ? kLongMany : kLongFew;
    const uint64_t words = (t.mask + 64) / 64;
    for (uint64_t w = first; w < words; w += stride)
      wave_repair_word(t, occupied, w, gone, used[wave], moved, &counters[kWMoved], long_from, lane);
  } else {
    for (uint64_t c = first; c < drop; c += stride)
      if (starts[c] != kNoStart) wave_repair(t, starts[c], gone, used[wave], lane);
  }
}

// Puts the entries of long clusters back: one lane each, at the first free slot from its
// home (the slots read kPutAhead at a time; only one that reads free costs a
// compare-and-swap). Any order of insertions leaves valid probe sequences.
constexpr int kPutAhead = 8;
__global__ __launch_bounds__(kThreads) void evict_put_back_kernel(TableRef t, const uint64_t* counters, Moved moved) {
  if (counters[kWMoved] == 0) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t words = (t.mask + 64) / 64;
  for (uint64_t w = (uint64_t)blockIdx.x * kWaves + wave; w < words; w += (uint64_t)gridDim.x * kWaves) {
    const uint64_t bits = moved.bits[w];
    if (!((bits >> lane) & 1)) continue;
    const uint64_t from = 64 * w + (uint64_t)lane;
    const uint64_t k = moved.key[from], val = moved.val[from], stamp = moved.stamp[from];
    uint64_t pos = slot_hash(k, t.shift);
    bool placed = false;
    for (uint64_t probe = 0; !placed && probe <= t.mask; probe += kPutAhead) {
      uint64_t seen[kPutAhead];
#pragma unroll
      for (int j = 0; j < kPutAhead; ++j) seen[j] = t.slots[2 * ((pos + j) & t.mask)];
#pragma unroll
      for (int j = 0; j < kPutAhead; ++j) {
        if (placed || seen[j] != kEmpty) continue;
        const uint64_t q = (pos + j) & t.mask;
        if (atomicCAS(ull(&t.slots[2 * q]), (unsigned long long)kEmpty, (unsigned long long)k) != kEmpty) continue;
        t.slots[2 * q + 1] = val;
        t.stamps[q] = stamp;
        placed = true;
      }
      pos = (pos + kPutAhead) & t.mask;
    }
  }
}

// ---- export ---------------------------------------------------------------------------
// Every entry in key order by one partition: each entry is written once to its bin of the
// key range, and one workgroup per part of a bin picks the part's entries out of the bin,
// sorts them in LDS and writes them out. Keys are digests, so the parts of an ordinary
// table are even; when one holds more than kPartMax entries or a bin more than kBinMax (a
// skewed key set, a table above 2^27 slots beyond the load that kMaxAllParts allows, a replayed
// graph whose table has outgrown the bound it was captured with), all entries go through the
// radix sort instead, decided on the device.
// 20 M entries of 2^25 slots: 1.0 ms (count 86 us, spread 398, parts 430), against 3.0 ms for
// eight digit passes and a gather of the values. Bound by the chains inside a workgroup: the
// table is read twice and the entries are written and read once, 0.3 ms at HBM rate.
constexpr uint32_t kSpreadThreads = 1024;
constexpr uint32_t kSpreadItems = 4;  // slots per thread and step when counting
constexpr uint32_t kSpreadEach = 8;   // slots per thread and tile when spreading

// Counts the entries of the (at most kMost) parts in this workgroup's share of the slots.
template <uint32_t kMost>
__global__ __launch_bounds__(kSpreadThreads) void export_count_kernel(TableRef t, const uint64_t* counters,
                                                                      uint32_t all, uint32_t* share) {
  __shared__ uint32_t h[kMost];
  for (uint32_t i = threadIdx.x; i < all; i += kSpreadThreads) h[i] = 0;
  __syncthreads();
  const KeyCells cells(counters, all * kCuts);
  const uint64_t capacity = t.mask + 1;
  const uint64_t each = (capacity + gridDim.x - 1) / gridDim.x;
  const uint64_t lo = blockIdx.x * each, hi = lo + each < capacity ? lo + each : capacity;
  for (uint64_t i0 = lo; i0 < hi; i0 += (uint64_t)kSpreadThreads * kSpreadItems) {
    uint64_t key[kSpreadItems];
#pragma unroll
    for (uint32_t r = 0; r < kSpreadItems; ++r) {  // unconditional (clamped) loads, issued together
      const uint64_t i = i0 + r * kSpreadThreads + threadIdx.x;
      key[r] = t.slots[2 * (i < hi ? i : hi - 1)];
      if (i >= hi) key[r] = kEmpty;
    }
#pragma unroll
    for (uint32_t r = 0; r < kSpreadItems; ++r)
      if (key[r] != kEmpty) atomicAdd(&h[cells.of(key[r]) / kCuts], 1u);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0 && t.hdr[0]) atomicAdd(&h[cells.of(kEmpty) / kCuts], 1u);
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < all; i += kSpreadThreads) share[(uint64_t)blockIdx.x * all + i] = h[i];
}

// share[g][part] becomes the count of the workgroups before g; starts[part] the part's total.
__global__ __launch_bounds__(64) void export_share_kernel(uint32_t all, uint32_t groups, uint32_t* share,
                                                          uint32_t* starts) {
  const uint32_t part = blockIdx.x * 64 + threadIdx.x;
  if (part >= all) return;
  constexpr uint32_t kAhead = 32;
  uint32_t sum = 0;
  for (uint32_t g0 = 0; g0 < groups; g0 += kAhead) {
    uint32_t c[kAhead];
#pragma unroll
    for (uint32_t k = 0; k < kAhead; ++k) {  // unconditional (clamped) loads, issued together
      const uint32_t g = g0 + k < groups ? g0 + k : groups - 1;
      c[k] = share[(uint64_t)g * all + part];
    }
#pragma unroll
    for (uint32_t k = 0; k < kAhead; ++k) {
      if (g0 + k >= groups) break;
      share[(uint64_t)(g0 + k) * all + part] = sum;
      sum += c[k];
    }
  }
  starts[part] = sum;
}

// One workgroup: starts[] from totals to positions, starts[all] = the entries; the count;
// and whether the radix sort takes over (counters[kWCollected]: its count, else 0).
template <uint32_t kMost>
__global__ __launch_bounds__(kInitThreads) void export_starts_kernel(uint32_t bins, uint32_t parts, uint32_t* starts,
                                                                     uint64_t* counters, uint64_t* count) {
  __shared__ uint32_t wave_sum[kInitThreads / 64];
  __shared__ uint32_t skewed;
  constexpr uint32_t kEach = kMost / kInitThreads;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t all = bins * parts;
  const uint32_t each = (all + kInitThreads - 1) / kInitThreads;  // at most kEach
  const uint32_t first = threadIdx.x * each;
  if (threadIdx.x == 0) skewed = 0;
  uint32_t c[kEach], sum = 0, most = 0;
#pragma unroll
  for (uint32_t j = 0; j < kEach; ++j) c[j] = j < each && first + j < all ? starts[first + j] : 0;
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
  if (lane == 63) wave_sum[wave] = incl;
  __syncthreads();
  uint32_t run = incl - sum, total = 0;
  for (int w = 0; w < (int)(kInitThreads / 64); ++w) {
    if (w < wave) run += wave_sum[w];
    total += wave_sum[w];
  }
#pragma unroll
  for (uint32_t j = 0; j < kEach; ++j) {
    if (j < each && first + j < all) starts[first + j] = run;
    run += c[j];
  }
  if (threadIdx.x == 0) starts[all] = total;
  __syncthreads();  // every start, read back by this workgroup
  bool bad = most > kPartMax;
  for (uint32_t b = threadIdx.x; b < bins; b += kInitThreads)
    bad = bad || starts[(b + 1) * parts] - starts[b * parts] > kBinMax;
  if (bad) skewed = 1;
  __syncthreads();
  if (threadIdx.x == 0) {
    *count = total;
    counters[kWCollected] = skewed ? total : 0;
  }
}

// Writes the entries of this workgroup's share of the slots to their bins: the workgroup's
// place in a bin starts after those of the workgroups before it. A tile of slots is put in
// bin order in LDS first, so that consecutive lanes write a bin's entries to consecutive
// addresses: written one by one, 20 M entries are 40 M small requests to the L2s (580 us).
constexpr uint32_t kTileSlots = kSpreadThreads * kSpreadEach;
template <uint32_t kMost>
__global__ __launch_bounds__(kSpreadThreads) void export_spread_kernel(TableRef t, const uint64_t* counters,
                                                                       uint32_t bins, uint32_t parts,
                                                                       const uint32_t* share, const uint32_t* starts,
                                                                       uint64_t* xkey, uint4* xpay) {
  constexpr uint32_t kMaxBins = kMost / kMaxParts;
  __shared__ uint32_t at[kMaxBins];     // the workgroup's next place in each bin
  __shared__ uint32_t count[kMaxBins];  // the tile's entries by bin, then their first places in the tile
  __shared__ uint16_t sbin[kTileSlots];
  __shared__ uint4 buf[kTileSlots / 2];  // the tile's keys, then one half and the other of the payloads
  __shared__ uint32_t wave_sum[kSpreadThreads / 64];
  const uint32_t all = bins * parts;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (uint32_t b = threadIdx.x; b < bins; b += kSpreadThreads) {
    uint32_t from = starts[b * parts];
    for (uint32_t j = 0; j < parts; ++j) from += share[(uint64_t)blockIdx.x * all + b * parts + j];
    at[b] = from;
  }
  const KeyCells cells(counters, all * kCuts);
  const uint32_t per_bin = parts * kCuts;
  const uint64_t capacity = t.mask + 1;
  const uint64_t each = (capacity + gridDim.x - 1) / gridDim.x;
  const uint64_t lo = blockIdx.x * each, hi = lo + each < capacity ? lo + each : capacity;
  uint64_t* skey = reinterpret_cast<uint64_t*>(buf);
  for (uint64_t i0 = lo; i0 < hi; i0 += kTileSlots) {
    uint4 slot[kSpreadEach];
    uint64_t stamp[kSpreadEach];
#pragma unroll
    for (uint32_t r = 0; r < kSpreadEach; ++r) {  // unconditional (clamped) loads, issued together
      const uint64_t i = i0 + r * kSpreadThreads + threadIdx.x, p = i < hi ? i : hi - 1;
      slot[r] = *reinterpret_cast<const uint4*>(t.slots + 2 * p);
      stamp[r] = t.stamps[p];
      if (i >= hi) slot[r].x = slot[r].y = ~0u;  // kEmpty
    }
    for (uint32_t b = threadIdx.x; b < bins; b += kSpreadThreads) count[b] = 0;
    __syncthreads();
    uint32_t bin[kSpreadEach], pos[kSpreadEach];
#pragma unroll
    for (uint32_t r = 0; r < kSpreadEach; ++r) {
      if (lo64(slot[r]) == kEmpty) continue;
      bin[r] = cells.of(lo64(slot[r])) / per_bin;
      pos[r] = atomicAdd(&count[bin[r]], 1u);
    }
    __syncthreads();
    {  // count becomes the bins' first places in the tile; at - count stays the shift to global places
      constexpr uint32_t kEach = kMaxBins / kSpreadThreads;
      uint32_t c[kEach], sum = 0;
#pragma unroll
      for (uint32_t j = 0; j < kEach; ++j) {
        const uint32_t b = threadIdx.x * kEach + j;
        c[j] = b < bins ? count[b] : 0;
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
        const uint32_t b = threadIdx.x * kEach + j;
        if (b < bins) count[b] = run;
        run += c[j];
      }
    }
    __syncthreads();
    uint32_t n = 0;  // the tile's entries
    for (int w = 0; w < (int)(kSpreadThreads / 64); ++w) n += wave_sum[w];
#pragma unroll
    for (uint32_t r = 0; r < kSpreadEach; ++r) {
      if (lo64(slot[r]) == kEmpty) continue;
      pos[r] += count[bin[r]];
      sbin[pos[r]] = (uint16_t)bin[r];
      skey[pos[r]] = lo64(slot[r]);
    }
    __syncthreads();
    uint32_t to[kSpreadEach];
#pragma unroll
    for (uint32_t r = 0; r < kSpreadEach; ++r) {
      const uint32_t j = r * kSpreadThreads + threadIdx.x;
      if (j >= n) continue;
      to[r] = at[sbin[j]] + j - count[sbin[j]];
      xkey[to[r]] = skey[j];
    }
#pragma unroll
    for (uint32_t half = 0; half < 2; ++half) {
      __syncthreads();  // buf read out
#pragma unroll
      for (uint32_t r = 0; r < kSpreadEach; ++r) {
        if (lo64(slot[r]) == kEmpty || pos[r] / (kTileSlots / 2) != half) continue;
        buf[pos[r] % (kTileSlots / 2)] =
            make_uint4(slot[r].z, slot[r].w, (uint32_t)stamp[r], (uint32_t)(stamp[r] >> 32));
      }
      __syncthreads();
#pragma unroll
      for (uint32_t r = half * kSpreadEach / 2; r < (half + 1) * kSpreadEach / 2; ++r) {
        const uint32_t j = r * kSpreadThreads + threadIdx.x;
        if (j < n) xpay[to[r]] = buf[j % (kTileSlots / 2)];
      }
    }
    for (uint32_t b = threadIdx.x; b < bins; b += kSpreadThreads)  // on to the next tile
      at[b] += (b + 1 < bins ? count[b + 1] : n) - count[b];
    __syncthreads();
  }
  if (blockIdx.x == 0 && threadIdx.x == 0 && t.hdr[0]) {
    const uint32_t p = at[cells.of(kEmpty) / per_bin];
    xkey[p] = kEmpty;
    xpay[p] = make_uint4((uint32_t)t.hdr[1], (uint32_t)(t.hdr[1] >> 32), (uint32_t)t.hdr[2], (uint32_t)(t.hdr[2] >> 32));
  }
}

// The least key of cell c (its cells start there: of(k) >= c exactly for the keys from it on),
// or 0 with *none set when no key reaches the cell.
__device__ __forceinline__ uint64_t first_key(const KeyCells& x, uint32_t c, bool* none) {
  *none = false;
  if (c == 0) return 0;
  *none = true;
  if (x.factor == 0) return 0;
  const uint64_t t = (((uint64_t)c << 32) + x.factor - 1) / x.factor;  // leading bits that reach c
  if (t >> 32) return 0;
  const uint64_t d = (t << 32) == 0 ? 0 : ((t << 32) - 1 >> x.lead) + 1;  // distances with those bits
  if (d > x.width) return 0;
  *none = false;
  return x.base + d;
}

// Sorts one part of a bin. It picks the part's keys out of the bin's, counts them over the
// part's kCuts cuts and places them cut by cut in LDS; within a cut (2.4 entries on
// average) an entry's rank is the number of smaller keys in it. When a cut holds more than
// kCutMax entries (keys crowded inside the part's range) the part is sorted by its keys'
// digits instead. The parts of a bin run on one XCD, one after another
// (workgroups go round the eight XCDs), so that XCD's L2 serves the bin's keys to them all.
constexpr uint32_t kPartThreads = 1024;
constexpr uint32_t kPartEach = kPartMax / kPartThreads;
constexpr uint32_t kCutMax = 48;
constexpr uint32_t kXcds = 8;

// Sorts skey[0, n) with sidx by all eight 8-bit digits, but those that every key shares, in
// place in LDS. `run` holds kPartWaves * 256 counts. Every thread of the workgroup calls it.
constexpr int kPartWaves = (int)kPartThreads / 64;
__device__ void part_radix_sort(uint64_t* skey, uint16_t* sidx, uint16_t* run, uint32_t* wave_sum, uint32_t n) {
  static_assert(kPartWaves * kDigits * sizeof(uint16_t) <= (kCuts + 1) * sizeof(uint32_t), "run fits in the cuts");
  static_assert(kPartThreads >= kDigits, "one thread per digit");
  __shared__ uint64_t fold[kPartWaves][2];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
  const uint32_t span0 = (uint32_t)wave * 64 * kPartEach;
  uint64_t and_k = ~0ull, or_k = 0;
  for (uint32_t i = threadIdx.x; i < n; i += kPartThreads) {
    and_k &= skey[i];
    or_k |= skey[i];
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    and_k &= shfl_xor64(and_k, o);
    or_k |= shfl_xor64(or_k, o);
  }
  if (lane == 0) {
    fold[wave][0] = and_k;
    fold[wave][1] = or_k;
  }
  __syncthreads();
  for (int w = 0; w < kPartWaves; ++w) {
    and_k &= fold[w][0];
    or_k |= fold[w][1];
  }
  const uint64_t differ = and_k ^ or_k;
  for (int sh = 0; sh < 64; sh += 8) {
    if (((differ >> sh) & 0xFFu) == 0) continue;  // uniform
    uint64_t k[kPartEach];
    uint32_t ix[kPartEach], at[kPartEach];
    for (int d = lane; d < kDigits; d += 64) run[wave * kDigits + d] = 0;
    wave_lds_sync();
#pragma unroll
    for (uint32_t r = 0; r < kPartEach; ++r) {
      const uint32_t i = span0 + 64 * r + lane;
      const bool valid = i < n;
      k[r] = valid ? skey[i] : 0;
      ix[r] = valid ? sidx[i] : 0;
      const uint32_t d = (uint32_t)(k[r] >> sh) & 0xFFu;
      uint64_t peers = __ballot(valid);
#pragma unroll
      for (int bit = 0; bit < 8; ++bit) {
        const uint64_t ones = __ballot(valid && ((d >> bit) & 1u));
        peers &= ((d >> bit) & 1u) ? ones : ~ones;
      }
      const uint32_t below = (uint32_t)__popcll(peers & lt), prior = run[wave * kDigits + d];
      at[r] = prior + below;
      if (valid && below == 0) run[wave * kDigits + d] = (uint16_t)(prior + (uint32_t)__popcll(peers));
      wave_lds_sync();  // this round's counts before the next round's reads
    }
    __syncthreads();
    uint32_t total = 0, incl = 0;
    if (threadIdx.x < kDigits) {
      for (int w = 0; w < kPartWaves; ++w) total += run[w * kDigits + threadIdx.x];
      incl = total;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
      }
      if (lane == 63) wave_sum[wave] = incl;
    }
    __syncthreads();
    if (threadIdx.x < kDigits) {
      uint32_t from = incl - total;
      for (int w = 0; w < wave; ++w) from += wave_sum[w];
      for (int w = 0; w < kPartWaves; ++w) {
        const uint32_t c = run[w * kDigits + threadIdx.x];
        run[w * kDigits + threadIdx.x] = (uint16_t)from;
        from += c;
      }
    }
    __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < kPartEach; ++r) {
      if (span0 + 64 * r + lane >= n) continue;
      const uint32_t p = at[r] + run[wave * kDigits + ((uint32_t)(k[r] >> sh) & 0xFFu)];
      skey[p] = k[r];
      sidx[p] = (uint16_t)ix[r];
    }
    __syncthreads();
  }
}

// kCrowded: the second launch, for the parts that the first left in left_over (their digit
// sort's registers would halve the first one's waves).
template <bool kCrowded>
__global__ __launch_bounds__(kPartThreads) void export_part_kernel(const uint64_t* counters, uint32_t bins,
                                                                   uint32_t parts, const uint32_t* starts,
                                                                   const uint64_t* xkey, const uint4* xpay,
                                                                   uint32_t* left_over, uint64_t* keys, uint64_t* vals,
                                                                   uint64_t* stamps) {
  __shared__ uint64_t skey[kPartMax];
  __shared__ uint16_t sidx[kPartMax];  // number within the bin
  __shared__ uint32_t cut[kCuts + 1];
  __shared__ uint32_t wave_sum[kPartThreads / 64];
  __shared__ uint32_t picked, crowded;
  if (counters[kWCollected]) return;  // the radix sort takes over
  uint32_t bin = blockIdx.x / parts, part = blockIdx.x % parts;
  if (bins % kXcds == 0) {
    const uint32_t y = blockIdx.x / kXcds;
    part = y % parts;
    bin = y / parts * kXcds + blockIdx.x % kXcds;
  }
  const uint32_t me = bin * parts + part;
  const uint32_t out0 = starts[me], n = starts[me + 1] - out0;
  if (kCrowded && !left_over[me]) return;
  if (n == 0) {
    if (!kCrowded && threadIdx.x == 0) left_over[me] = 0;
    return;
  }
  const uint32_t s0 = starts[bin * parts], n_bin = starts[(bin + 1) * parts] - s0;
  const KeyCells cells(counters, bins * parts * kCuts);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
  for (uint32_t i = threadIdx.x; i < kCuts + 1; i += kPartThreads) cut[i] = 0;
  if (threadIdx.x == 0) picked = crowded = 0;
  // the part's keys: [from, to), or from `from` on for the last part that any key reaches
  bool no_from, no_to;
  const uint64_t from = first_key(cells, me * kCuts, &no_from), to = first_key(cells, (me + 1) * kCuts, &no_to);
  __syncthreads();
  constexpr uint32_t kAhead = 8;
  for (uint32_t i0 = 0; i0 < n_bin; i0 += kAhead * kPartThreads) {
    uint64_t k[kAhead];
#pragma unroll
    for (uint32_t r = 0; r < kAhead; ++r) {  // unconditional (clamped) loads, issued together
      const uint32_t i = i0 + r * kPartThreads + threadIdx.x;
      k[r] = xkey[s0 + (i < n_bin ? i : n_bin - 1)];
    }
#pragma unroll
    for (uint32_t r = 0; r < kAhead; ++r) {
      const uint32_t i = i0 + r * kPartThreads + threadIdx.x;
      const bool mine = i < n_bin && k[r] >= from && (k[r] < to || no_to);
      const uint64_t who = __ballot(mine);
      if (who == 0) continue;
      uint32_t p = 0;
      if (lane == 0) p = atomicAdd(&picked, (uint32_t)__popcll(who));
      p = __builtin_amdgcn_readfirstlane(p) + (uint32_t)__popcll(who & lt);
      if (mine && p < kPartMax) {
        skey[p] = k[r];
        sidx[p] = (uint16_t)i;
      }
    }
  }
  __syncthreads();
  if (kCrowded) {
    part_radix_sort(skey, sidx, reinterpret_cast<uint16_t*>(cut), wave_sum, n);
    for (uint32_t p = threadIdx.x; p < n; p += kPartThreads) {
      const uint4 pay = xpay[s0 + sidx[p]];
      keys[out0 + p] = skey[p];
      vals[out0 + p] = lo64(pay);
      if (stamps) stamps[out0 + p] = hi64(pay);
    }
    return;
  }
  uint64_t k[kPartEach];
  uint32_t ord[kPartEach], ix[kPartEach];  // place within its cut, in arrival order; number within the bin
#pragma unroll
  for (uint32_t r = 0; r < kPartEach; ++r) {
    const uint32_t i = r * kPartThreads + threadIdx.x;
    if (i >= n) continue;
    k[r] = skey[i];
    ix[r] = sidx[i];
    ord[r] = atomicAdd(&cut[cells.of(k[r]) % kCuts], 1u);
    if (ord[r] >= kCutMax) crowded = 1;
  }
  __syncthreads();
  if (threadIdx.x == 0) left_over[me] = crowded;
  if (crowded) return;
  {  // exclusive scan of the cuts' counts
    constexpr uint32_t kEach = kCuts / kPartThreads;
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
    if (threadIdx.x == kPartThreads - 1) cut[kCuts] = run;
  }
  __syncthreads();
#pragma unroll
  for (uint32_t r = 0; r < kPartEach; ++r) {
    if (r * kPartThreads + threadIdx.x >= n) continue;
    const uint32_t p = cut[cells.of(k[r]) % kCuts] + ord[r];
    skey[p] = k[r];
    sidx[p] = (uint16_t)ix[r];
  }
  __syncthreads();
#pragma unroll
  for (uint32_t r = 0; r < kPartEach; ++r) {
    const uint32_t p = r * kPartThreads + threadIdx.x;
    if (p >= n) continue;
    const uint64_t key = skey[p];
    const uint4 pay = xpay[s0 + sidx[p]];
    const uint32_t c = cells.of(key) % kCuts, end = cut[c + 1];
    uint32_t rank = cut[c];
    for (uint32_t q = rank; q < end; ++q) rank += skey[q] < key ? 1u : 0u;
    keys[out0 + rank] = key;
    vals[out0 + rank] = lo64(pay);
    if (stamps) stamps[out0 + rank] = hi64(pay);
  }
}

// The radix sort's other input: the entries' numbers, and the AND/OR words. (One fold per
// workgroup, and few of them: those that start together all find the words to change and queue
// on them. A million entries: 61 us with a fold per wave of 1,024 workgroups.)
constexpr uint32_t kUnpackGrid = 512;
__global__ __launch_bounds__(kThreads) void export_unpack_kernel(uint64_t* counters, SortBuf sb) {
  __shared__ uint64_t fold[kWaves][2];
  const uint64_t n = counters[kWCollected];
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  uint64_t and_k = ~0ull, or_k = 0;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const uint64_t k = sb.lo[i];
    sb.idx[i] = (uint32_t)i;
    and_k &= k;
    or_k |= k;
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    and_k &= shfl_xor64(and_k, o);
    or_k |= shfl_xor64(or_k, o);
  }
  if ((threadIdx.x & 63) == 0) {
    fold[threadIdx.x >> 6][0] = and_k;
    fold[threadIdx.x >> 6][1] = or_k;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (int w = 1; w < kWaves; ++w) {
    and_k &= fold[w][0];
    or_k |= fold[w][1];
  }
  fold_bits(counters + kWBits, and_k, or_k);
}

__global__ __launch_bounds__(kThreads) void export_sorted_kernel(const uint64_t* counters, const uint4* xpay, SortBuf a,
                                                                 SortBuf b, uint64_t* keys, uint64_t* vals,
                                                                 uint64_t* stamps) {
  const uint64_t n = counters[kWCollected];
  const SortBuf sorted = sort_result(a, b, counters + kWBits, 1);
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const uint4 pay = xpay[sorted.idx[i]];
    keys[i] = sorted.lo[i];
    vals[i] = lo64(pay);
    if (stamps) stamps[i] = hi64(pay);
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
  if (n > max_workgroups(kThreads) * kThreads) {
    set_error("gleam_cache_touch: more keys than one launch has threads (2^32)");
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
  uint64_t* occupied = ws_at<uint64_t>(d_ws, L.occupied);
  const SortBuf sa{ws_at<uint64_t>(d_ws, L.hi), ws_at<uint64_t>(d_ws, L.lo), ws_at<uint32_t>(d_ws, L.idx)};
  const SortBuf sb = sort_other(ws_at<uint8_t>(d_ws, L.sort2), L.m, 2);
  hipLaunchKernelGGL(maint_init_kernel<true>, dim3(1), dim3(kInitThreads), 0, s, t, keep, counters, pick);
  if ((st = launch_status("maint_init_kernel")) != GLEAM_OK) return st;
  const uint64_t collect_want = (c->capacity + kCollectTile * kCollectWaves - 1) / (kCollectTile * kCollectWaves);
  const dim3 collect_grid((uint32_t)(collect_want < kCollectGrid ? collect_want : kCollectGrid));
  hipLaunchKernelGGL(evict_collect_kernel<false>, collect_grid, dim3(kThreads), 0, s, t, pick, counters, sa,
                     occupied);
  if ((st = launch_status("evict_collect_kernel")) != GLEAM_OK) return st;
  if (c->capacity > kSamples) {  // below, the samples are the whole table (but for the side slot, see there)
    const uint64_t pick_want = (c->capacity + kPickThreads * kPickItems - 1) / (kPickThreads * kPickItems);
    hipLaunchKernelGGL(evict_pick_kernel, dim3((uint32_t)(pick_want < kPickGrid ? pick_want : kPickGrid)),
                       dim3(kPickThreads), 0, s, t, counters, pick);
    if ((st = launch_status("evict_pick_kernel")) != GLEAM_OK) return st;
    hipLaunchKernelGGL(evict_collect_kernel<true>, collect_grid, dim3(kThreads), 0, s, t, pick, counters, sa,
                     occupied);
    if ((st = launch_status("evict_collect_kernel")) != GLEAM_OK) return st;
  }
  st = radix_sort_pairs(sa, counters + kWCollected, counters + kWBits, L.m, 2, ws_at<uint8_t>(d_ws, L.sort2), s);
  if (st != GLEAM_OK) return st;
  const uint32_t grid = grid_for(L.m) < 2048 ? grid_for(L.m) : 2048;
  hipLaunchKernelGGL(evict_mark_kernel, dim3(grid), dim3(kThreads), 0, s, t, sa, sb, counters, occupied, leaders,
                     d_evicted, d_counts);
  if ((st = launch_status("evict_mark_kernel")) != GLEAM_OK) return st;
  const Moved moved{sa.hi, sa.lo, sb.hi, reinterpret_cast<uint64_t*>(sa.idx)};
  hipLaunchKernelGGL(evict_repair_kernel, dim3(grid), dim3(kThreads), 0, s, t, counters, leaders, occupied, moved);
  if ((st = launch_status("evict_repair_kernel")) != GLEAM_OK) return st;
  if (c->capacity > kCollectTile) {  // else no step of slots is full
    hipLaunchKernelGGL(evict_put_back_kernel, dim3(grid), dim3(kThreads), 0, s, t, counters, moved);
    if ((st = launch_status("evict_put_back_kernel")) != GLEAM_OK) return st;
  }
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
  if (n > (1ull << 36)) {
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
  const dim3 block(kThreads);
  hipLaunchKernelGGL(erase_clear_kernel, dim3(grid_for(L.cap)), block, 0, s, w);
  gleam_status st = launch_status("erase_clear_kernel");
  if (st != GLEAM_OK) return st;
  if (n > 0) {
    const uint64_t groups = (n + kThreads / kSpan - 1) / (kThreads / kSpan);
    hipLaunchKernelGGL(erase_find_kernel, dim3((uint32_t)(groups < kFindGrid ? groups : kFindGrid)), block, 0, s, t,
                       d_keys, n, w);
    if ((st = launch_status("erase_find_kernel")) != GLEAM_OK) return st;
  }
  const uint64_t want = (n + kRepairWaves - 1) / kRepairWaves;  // at most one cluster per key, one wave each
  hipLaunchKernelGGL(erase_repair_kernel, dim3((uint32_t)(want == 0 ? 1 : want < kRepairGrid ? want : kRepairGrid)),
                     dim3(kRepairThreads), 0, s, t, n, w, d_counts);
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
  uint64_t* xkey = ws_at<uint64_t>(d_ws, L.xkey);
  uint4* xpay = ws_at<uint4>(d_ws, L.xpay);
  const uint32_t fewer = L.bins * L.parts;
  const uint32_t bins = c->key_bound > (uint64_t)fewer * kPartFine ? 2 * L.bins : L.bins, all = bins * L.parts;
  const bool few = all <= kFewParts;
  hipLaunchKernelGGL(maint_init_kernel<false>, dim3(1), dim3(kInitThreads), 0, s, t, 0, counters, (uint32_t*)nullptr);
  if ((st = launch_status("maint_init_kernel")) != GLEAM_OK) return st;
  hipLaunchKernelGGL(few ? export_count_kernel<kFewParts> : export_count_kernel<kMaxAllParts>, dim3(L.spread),
                     dim3(kSpreadThreads), 0, s, t, counters, all, share);
  if ((st = launch_status("export_count_kernel")) != GLEAM_OK) return st;
  hipLaunchKernelGGL(export_share_kernel, dim3((all + 63) / 64), dim3(64), 0, s, all, L.spread, share, starts);
  if ((st = launch_status("export_share_kernel")) != GLEAM_OK) return st;
  hipLaunchKernelGGL(few ? export_starts_kernel<kFewParts> : export_starts_kernel<kMaxAllParts>, dim3(1),
                     dim3(kInitThreads), 0, s, bins, L.parts, starts, counters, d_count);
  if ((st = launch_status("export_starts_kernel")) != GLEAM_OK) return st;
  hipLaunchKernelGGL(few ? export_spread_kernel<kFewParts> : export_spread_kernel<kMaxAllParts>, dim3(L.spread),
                     dim3(kSpreadThreads), 0, s, t, counters, bins, L.parts, share, starts, xkey, xpay);
  if ((st = launch_status("export_spread_kernel")) != GLEAM_OK) return st;
  // (the shares are done with: their first words tell the parts left to the second launch)
  hipLaunchKernelGGL(export_part_kernel<false>, dim3(all), dim3(kPartThreads), 0, s, counters, bins, L.parts, starts,
                     xkey, xpay, share, d_keys, d_vals, d_stamps);
  if ((st = launch_status("export_part_kernel")) != GLEAM_OK) return st;
  hipLaunchKernelGGL(export_part_kernel<true>, dim3(all), dim3(kPartThreads), 0, s, counters, bins, L.parts, starts,
                     xkey, xpay, share, d_keys, d_vals, d_stamps);
  if ((st = launch_status("export_part_kernel")) != GLEAM_OK) return st;
  if (c->capacity <= kPartMax) return GLEAM_OK;  // no part can hold more
  const SortBuf sa{nullptr, xkey, ws_at<uint32_t>(d_ws, L.xidx)};
  const SortBuf sb = sort_other(ws_at<uint8_t>(d_ws, L.sort1), L.m, 1);
  const uint32_t grid = grid_for(L.m) < 1024 ? grid_for(L.m) : 1024;
  hipLaunchKernelGGL(export_unpack_kernel, dim3(grid < kUnpackGrid ? grid : kUnpackGrid), dim3(kThreads), 0, s,
                     counters, sa);
  if ((st = launch_status("export_unpack_kernel")) != GLEAM_OK) return st;
  st = radix_sort_pairs(sa, counters + kWCollected, counters + kWBits, L.m, 1, ws_at<uint8_t>(d_ws, L.sort1), s);
  if (st != GLEAM_OK) return st;
  hipLaunchKernelGGL(export_sorted_kernel, dim3(grid), dim3(kThreads), 0, s, counters, xpay, sa, sb, d_keys, d_vals,
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
