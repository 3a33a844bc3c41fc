// Address-remap interval map (Gleam Sec. 4.1.3, Weight Chunk Sharing: chunks written into
// one client allocation may find their shareable copies in different server allocations,
// so a virtual memory layer maps client device addresses onto those positions; Appendix,
// Implementation Details, Virtual Memory Map: one 1 TB virtual space per task, the
// mappings kept in a red-black tree).
//
// The map is an array of disjoint intervals sorted by start, in caller-owned device
// storage: [256-byte header: u64 count, fence stride, fence length][start x cap]
// [{end, bias} x cap][fence: kFence x u64], end exclusive, bias = target - start (mod
// 2^64, so a translation is one add: p + bias). A sorted array answers the
// same ordered queries as the tree; on the GPU a batch of pointers is translated by
// one search per lane, and a batch of changes is merged in a few passes instead of
// rebalancing node by node.
//
// Translation is bound by lane-divergent loads (each level of a binary search is a
// different cache line for nearly every lane), not by bytes. So every update also
// writes a fence, every S-th start with S = ceil(count / 8192); a translating workgroup
// keeps the fence in LDS and searches it first, leaving log2(S) levels for global
// memory (5 instead of 18 at 208k intervals), and end and bias sit side by side so the
// final step is one 16-byte load and needs no start.
//
// An update never re-sorts the intervals it keeps (they are already in order). It is bound
// by its launches and their chains of dependent reads, so it takes four:
//   1. the removals and the additions are sorted by start in chunks of 2,048, a workgroup
//      per chunk in LDS, each with the running maximum of its ends (more than 16 chunks:
//      one chunk of everything, by the library's radix sort, radix_sort.h; invalid
//      additions take the key kNone and sort last);
//   2. an interval meets a removal of a chunk iff the furthest end among those that start
//      at or before its last address reaches its start: a wave narrows each chunk to its
//      64 intervals first and nearly always finds none. Every interval gets a keep bit and
//      is copied to the workspace; tiles of 1,024 count their survivors;
//   3. an addition meets another one by the same rule over the chunks of additions, and a
//      survivor iff there are survivors (a difference of ranks) among the intervals from
//      the first that ends after its start to the last that starts before its end.
//      Additions that meet nothing are kept and numbered within their chunk;
//   4. the sorted runs are merged by rank: a survivor lands at its own rank plus the kept
//      additions that start before it, a kept addition at its number among all kept ones
//      plus the survivors before it. Nothing is written unless everything fits the
//      capacity, so a refused call changes nothing.
// 209 k intervals, one task's tensors (161 to 2,000) out and another's in: 28 us of kernels,
// against 93 us for eleven launches with bitonic sorts (up to 41 us of them for 2,000
// additions) and a scan and a compaction of their own; 8,000 out and in 64 us a call in
// address order and 120 in any order, against 258 through the radix sorts.

#include <new>

#include "device_scan.h"
#include "gleam_device.h"
#include "gleam_internal.h"
#include "radix_sort.h"

namespace gleam {
namespace {

constexpr int kThreads = 256;
constexpr int kTranslateThreads = 1024;
constexpr uint32_t kMaxGrid = 8192;
constexpr uint64_t kNone = ~0ull;  // sort key of an addition that takes no part; no valid start equals it
constexpr uint64_t kMaxCount = 1ull << 31;

constexpr uint32_t kFence = 8192;  // fence entries (64 KiB of LDS: two translating workgroups per CU)

struct MapRef {
  uint64_t* hdr;   // [0] number of intervals, [1] fence stride S, [2] fence length
  uint64_t* start;
  ulonglong2* et;  // {end, target - start} per interval
  uint64_t* fence; // start[k * S] for k < fence length
  uint64_t cap;
};

MapRef map_ref(const gleam_remap* m) {
  uint64_t* hdr = reinterpret_cast<uint64_t*>(m->storage);
  uint64_t* start = reinterpret_cast<uint64_t*>(m->storage + kHeaderBytes);
  ulonglong2* et = reinterpret_cast<ulonglong2*>(start + m->capacity);
  return MapRef{hdr, start, et, reinterpret_cast<uint64_t*>(et + m->capacity), m->capacity};
}

// Chunks of the sorted removals and additions, and tiles of the intervals.
constexpr int kSmallThreads = 1024;
constexpr uint32_t kSmall = 2 * kSmallThreads;
// Up to 16 chunks: 32,768 of each. A batch in no order makes every wave search every chunk:
// 32,000 out and in take 252 us so (80 in address order), through the radix sorts 305 before
// the update took four launches and about 200 with them.
constexpr uint64_t kMaxChunked = 16ull * kSmall;
constexpr int kTileThreads = 1024;
constexpr uint64_t kTile = kTileThreads;
constexpr uint64_t kTileWords = kTile / 64;
// Tile counts that a workgroup scans in LDS on its way (4 M intervals); more take a launch.
constexpr uint32_t kLdsTiles = 4096;

uint64_t chunk_of(uint64_t n) { return n <= kMaxChunked ? kSmall : n; }

// Workspace of one update (cap = capacity, A = additions, R = removal ranges).
struct UpdLayout {
  uint64_t tiles;
  size_t hdr;                            // [0] R, [1] A (the sorts' counts); [4..7] R's key bits, [8..11] A's; [12] intervals before
  size_t keep, wpre, tcount, tbase;      // cap: keep bits, survivors of the tile before each word; tile counts, their scan
  size_t s_start, s_et;                  // cap: the intervals as they were
  size_t kb, vb, aend, amax, acc, apos, srank;  // A: sorted keys/indices, ends, running max, kept flag, number, survivors before
  size_t below;                          // A: places among the other chunks
  size_t rkb, rmax;                      // R: sorted starts, running max of last addresses
  size_t partial;                        // the scans' tile totals
  size_t ka, aidx, rka, ridx, last, sort;  // past kMaxChunked: the radix sorts' buffers
  size_t total;
};

UpdLayout upd_layout(uint64_t cap, uint64_t n_add, uint64_t n_del) {
  UpdLayout L;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off = (off + bytes + 255) & ~(size_t)255;
    return o;
  };
  L.tiles = (cap + kTile - 1) / kTile;
  L.hdr = take(256);
  L.keep = take(8 * L.tiles * kTileWords);
  L.wpre = take(4 * L.tiles * kTileWords);
  L.tcount = take(8 * (L.tiles + 1));
  L.tbase = take(8 * (L.tiles + 1));
  L.s_start = take(8 * cap);
  L.s_et = take(16 * cap);
  L.kb = take(8 * n_add);
  L.vb = take(8 * n_add);
  L.aend = take(8 * n_add);
  L.amax = take(8 * n_add);
  L.acc = take(8 * n_add);
  L.apos = take(8 * n_add);
  L.srank = take(8 * n_add);
  L.below = off;
  if (n_add > kSmall) take(2 * (kMaxChunked / kSmall) * (n_add < kMaxChunked ? n_add : kMaxChunked));
  L.rkb = take(8 * n_del);
  L.rmax = take(8 * n_del);
  const uint64_t ra = n_add > kMaxChunked ? n_add : 0, rd = n_del > kMaxChunked ? n_del : 0;
  const uint64_t most = ra > rd ? ra : rd;
  L.partial = take(8 * scan_tiles(most > L.tiles + 1 ? most : L.tiles + 1));
  L.ka = L.aidx = L.rka = L.ridx = L.last = L.sort = off;
  if (most) {
    L.ka = take(8 * sort_capacity(ra));
    L.aidx = take(4 * sort_capacity(ra));
    L.rka = take(8 * sort_capacity(rd));
    L.ridx = take(4 * sort_capacity(rd));
    L.last = take(8 * rd);
    L.sort = take(sort_layout(most, 1).total);
  }
  L.total = off;
  return L;
}

uint32_t grid_for(uint64_t n) {
  const uint64_t g = (n + kThreads - 1) / kThreads;
  return (uint32_t)(g == 0 ? 1 : (g < kMaxGrid ? g : kMaxGrid));
}

// Grid of a kernel that folds key bits with one pair of atomics per workgroup: few
// enough workgroups that those atomics on two words do not queue behind each other.
uint32_t fold_grid(uint64_t n) {
  const uint32_t g = grid_for(n);
  return g < 256 ? g : 256;
}

// Entries of the ascending keys[lo, hi) that are <= x (kLe) or < x, plus lo.
template <bool kLe>
__device__ __forceinline__ uint64_t count_below(const uint64_t* keys, uint64_t lo, uint64_t hi, uint64_t x) {
  while (lo < hi) {
    const uint64_t mid = lo + ((hi - lo) >> 1);
    const uint64_t k = keys[mid];
    if (kLe ? k <= x : k < x) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// The same over keys[0, n) for an x that is the same in every lane, by the whole wave: 64
// pivots a round, so 2,048 entries take two dependent reads. Every lane calls it.
template <bool kLe>
__device__ __forceinline__ uint64_t wave_count_below(const uint64_t* keys, uint64_t n, uint64_t x, int lane) {
  uint64_t lo = 0, hi = n;
  while (hi - lo > 64) {
    const uint64_t step = (hi - lo + 63) / 64, idx = lo + (uint64_t)lane * step;
    const uint64_t k = keys[idx < hi ? idx : hi - 1];
    const uint64_t c = (uint64_t)__popcll(__ballot(idx < hi && (kLe ? k <= x : k < x)));
    if (c == 0) return lo;
    hi = min(lo + c * step, hi);
    lo += (c - 1) * step + 1;
  }
  if (lo == hi) return lo;
  const uint64_t idx = lo + (uint64_t)lane;
  const uint64_t k = keys[idx < hi ? idx : hi - 1];
  return lo + (uint64_t)__popcll(__ballot(idx < hi && (kLe ? k <= x : k < x)));
}

__device__ __forceinline__ uint64_t uniform64(uint64_t x, int lane) {
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)x, lane);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(x >> 32), lane);
  return ((uint64_t)hi << 32) | lo;
}

// Batches past kMaxChunked. Counts of the two sorts and the AND/OR words of their keys (see radix_sort.h).
__global__ void update_init_kernel(uint64_t* hdr, uint64_t r, uint64_t n_add) {
  const int t = threadIdx.x;
  if (t < 12) hdr[t] = t == 0 ? r : t == 1 ? n_add : (t == 4 || t == 8) ? ~0ull : 0ull;
}

// Fold a thread's AND/OR of keys into bits[0] (AND) and bits[1] (OR): one pair of
// atomics per workgroup. Every thread of the workgroup calls it.
__device__ void fold_key_bits(uint64_t and_k, uint64_t or_k, uint64_t* bits) {
  __shared__ uint64_t fold[kThreads / 64][2];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
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
  if (threadIdx.x == 0) {
    for (int w = 1; w < kThreads / 64; ++w) {
      and_k &= fold[w][0];
      or_k |= fold[w][1];
    }
    atomicAnd(reinterpret_cast<unsigned long long*>(&bits[0]), (unsigned long long)and_k);
    atomicOr(reinterpret_cast<unsigned long long*>(&bits[1]), (unsigned long long)or_k);
  }
}

// Sort key of removal k: its start, or kNone for an empty range (it sorts last).
__global__ __launch_bounds__(kThreads) void removal_prep_kernel(const uint64_t* d_start, const uint64_t* d_len,
                                                                uint64_t r, uint64_t* key, uint32_t* idx,
                                                                uint64_t* bits) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  uint64_t and_k = ~0ull, or_k = 0;
  for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < r; k += stride) {
    const uint64_t s = d_len[k] ? d_start[k] : kNone;
    key[k] = s;
    idx[k] = (uint32_t)k;
    and_k &= s;
    or_k |= s;
  }
  fold_key_bits(and_k, or_k, bits);
}

// Sorted removals: start, and last address (the running maximum of these tells whether
// any removal starting at or before an address reaches it).
__global__ void removal_unpack_kernel(SortBuf a, SortBuf b, const uint64_t* bits, const uint64_t* d_start,
                                      const uint64_t* d_len, uint64_t r, uint64_t* key, uint64_t* last) {
  const SortBuf sorted = sort_result(a, b, bits, 1);
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < r; k += stride) {
    const uint32_t j = sorted.idx[k];
    const uint64_t s = d_start[j], n = d_len[j];
    key[k] = sorted.lo[k];
    last[k] = n ? (n - 1 > kNone - s ? kNone : s + n - 1) : 0;
  }
}

// Sort key of addition j: its start if valid, else kNone (status INVALID).
__global__ __launch_bounds__(kThreads) void addition_prep_kernel(const uint64_t* a_start, const uint64_t* a_len,
                                                                 const uint64_t* a_target, uint64_t n_add,
                                                                 uint8_t* status, uint64_t* key, uint32_t* idx,
                                                                 uint64_t* bits) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  uint64_t and_k = ~0ull, or_k = 0;
  for (uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n_add; j += stride) {
    const uint64_t s = a_start[j], n = a_len[j], t = a_target[j];
    const bool valid = n != 0 && n <= kNone - s && n <= kNone - t;
    if (!valid && status) status[j] = GLEAM_REMAP_INVALID;
    const uint64_t k = valid ? s : kNone;
    key[j] = k;
    idx[j] = (uint32_t)j;
    and_k &= k;
    or_k |= k;
  }
  fold_key_bits(and_k, or_k, bits);
}

// Sorted additions: start, original index, and end; an invalid one ends at 0 (it sorts
// last, after every valid one, so the running maximum of ends only ever sees real ends
// before it).
__global__ void addition_unpack_kernel(SortBuf a, SortBuf b, const uint64_t* bits, const uint64_t* a_len,
                                       uint64_t n_add, uint64_t* key, uint64_t* val, uint64_t* aend) {
  const SortBuf sorted = sort_result(a, b, bits, 1);
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n_add; k += stride) {
    const uint64_t s = sorted.lo[k];
    const uint32_t j = sorted.idx[k];
    key[k] = s;
    val[k] = j;
    aend[k] = s == kNone ? 0 : s + a_len[j];
  }
}

// ---- chunks sorted in LDS ---------------------------------------------------------------
struct ChunkLds {
  uint64_t key[2][kSmall];
  uint64_t val[kSmall];  // by original place: a removal's last address, an addition's length
  uint32_t idx[2][kSmall];
  uint64_t wave[kSmallThreads / 64];
};

// Sorts (key[0][i], idx[0][i] = i), i < n <= kSmall, by key, stably; returns the buffer that
// holds the result. Batches usually come in address order (a task's tensors as they were
// packed), which one pass sees. Else each wave sorts two runs of 64 in registers, and pairs
// of sorted runs are merged by rank: each entry finds its place in the other run by a
// binary search, one barrier per doubling. Every thread of the workgroup calls it.
__device__ int sort_chunk(ChunkLds& L, uint32_t n) {
  const uint32_t t = threadIdx.x;
  const int lane = t & 63;
  bool bad = false;
  for (uint32_t i = t; i + 1 < n; i += kSmallThreads) bad |= L.key[0][i] > L.key[0][i + 1];
  if (!__syncthreads_or(bad)) return 0;
  const uint32_t i0 = (t / 64) * 128 + lane;
  uint64_t k[2];
  uint32_t id[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {  // places past n sort after every entry: kNone, and the higher index
    id[h] = i0 + 64 * h;
    k[h] = id[h] < n ? L.key[0][id[h]] : kNone;
  }
#pragma unroll
  for (int size = 2; size <= 64; size <<= 1) {
#pragma unroll
    for (int d = size >> 1; d > 0; d >>= 1) {
      const bool low = (lane & d) == 0, up = (lane & size) == 0;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint64_t ok = shfl_xor64(k[h], d);
        const uint32_t oi = (uint32_t)__shfl_xor((int)id[h], d, 64);
        const bool less = ok < k[h] || (ok == k[h] && oi < id[h]);  // the other one comes first
        if (less == (low == up)) {
          k[h] = ok;
          id[h] = oi;
        }
      }
    }
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (i0 + 64 * h < n) {
      L.key[0][i0 + 64 * h] = k[h];
      L.idx[0][i0 + 64 * h] = id[h];
    }
  }
  __syncthreads();
  int b = 0;
  for (uint32_t run = 64; run < n; run *= 2, b ^= 1) {
    for (uint32_t i = t; i < n; i += kSmallThreads) {
      const uint32_t r = i / run, left = (r & ~1u) * run, other = (r ^ 1) * run;
      const uint64_t x = L.key[b][i];
      const uint32_t end = min(other + run, n);
      uint32_t c = 0;
      if (other < end)
        c = (uint32_t)((r & 1) ? count_below<true>(L.key[b], other, end, x) : count_below<false>(L.key[b], other, end, x)) - other;
      const uint32_t to = left + (i - r * run) + c;
      L.key[b ^ 1][to] = x;
      L.idx[b ^ 1][to] = L.idx[b][i];
    }
    __syncthreads();
  }
  return b;
}

// Inclusive scan over the workgroup of two consecutive values per thread. Every thread
// calls it; `wave` is kSmallThreads / 64 words of LDS.
template <class Op>
__device__ __forceinline__ void scan_pairs(uint64_t* v, Op op, uint64_t* wave) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint64_t incl = op(v[0], v[1]);
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint64_t y = shfl_up64(incl, d);
    if (lane >= d) incl = op(y, incl);
  }
  __syncthreads();  // `wave` of an earlier scan read by every thread
  if (lane == 63) wave[w] = incl;
  __syncthreads();
  uint64_t before = 0;
  for (int x = 0; x < w; ++x) before = op(before, wave[x]);
  const uint64_t prev = shfl_up64(incl, 1);
  if (lane) before = op(before, prev);
  v[0] = op(before, v[0]);
  v[1] = op(v[0], v[1]);
}

struct Batches {  // the arguments of one update
  const uint64_t *r_start, *r_len, *a_start, *a_len, *a_target;
  uint64_t n_del, n_add;
  uint8_t* status;
};
struct Removals {  // sorted, in chunks of `chunk`
  uint64_t *key, *max;
  uint64_t n, chunk;
};
struct Additions {  // sorted, in chunks of `chunk`
  uint64_t *key, *idx, *end, *max;
  uint64_t* acc;    // kept: a bit per entry; in one chunk of more than kMaxChunked a word per entry
  uint64_t* pos;    // of such a chunk: the kept ones before each entry
  uint64_t* srank;  // survivors before each
  uint16_t* below;  // [chunk][entry]: entries of that chunk that start before this one (kept entries)
  uint64_t n, chunk;
};

// One workgroup per chunk: `r_chunks` of the removals, then those of the additions.
__global__ __launch_bounds__(kSmallThreads) void sort_chunks_kernel(Batches in, Removals R, Additions A,
                                                                    uint32_t r_chunks) {
  __shared__ ChunkLds L;
  const bool removals = blockIdx.x < r_chunks;
  const uint64_t first = (uint64_t)(removals ? blockIdx.x : blockIdx.x - r_chunks) * kSmall;
  const uint32_t n = (uint32_t)min((removals ? in.n_del : in.n_add) - first, (uint64_t)kSmall);
  for (uint32_t i = threadIdx.x; i < n; i += kSmallThreads) {
    uint64_t k, v;
    if (removals) {
      const uint64_t s = in.r_start[first + i], len = in.r_len[first + i];
      k = len ? s : kNone;
      v = len ? (len - 1 > kNone - s ? kNone : s + len - 1) : 0;
    } else {
      const uint64_t s = in.a_start[first + i], len = in.a_len[first + i], to = in.a_target[first + i];
      const bool valid = len != 0 && len <= kNone - s && len <= kNone - to;
      if (!valid && in.status) in.status[first + i] = GLEAM_REMAP_INVALID;
      k = valid ? s : kNone;
      v = valid ? len : 0;
    }
    L.key[0][i] = k;
    L.idx[0][i] = i;
    L.val[i] = v;
  }
  __syncthreads();
  const int b = sort_chunk(L, n);
  uint64_t e[2], m[2], k[2];
  uint32_t id[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t i = 2 * threadIdx.x + h;
    k[h] = i < n ? L.key[b][i] : kNone;
    id[h] = i < n ? L.idx[b][i] : 0;
    e[h] = i < n ? L.val[id[h]] : 0;
    if (!removals && k[h] != kNone) e[h] += k[h];  // an invalid addition ends at 0
    m[h] = e[h];
  }
  scan_pairs(m, ScanMax(), L.wave);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t i = 2 * threadIdx.x + h;
    if (i >= n) continue;
    if (removals) {
      R.key[first + i] = k[h];
      R.max[first + i] = m[h];
    } else {
      A.key[first + i] = k[h];
      A.idx[first + i] = first + id[h];
      A.end[first + i] = e[h];
      A.max[first + i] = m[h];
    }
  }
}

// ---- survivors --------------------------------------------------------------------------
struct Kept {            // the intervals as they were, and which of them stay
  uint64_t* count;       // [0]
  uint64_t* word;        // keep bits
  uint32_t* wpre;        // survivors of the word's tile before the word
  uint64_t* tcount;      // survivors of each tile
  uint64_t* tbase;       // and their exclusive scan, with the total after the last
  uint64_t* start;
  ulonglong2* et;
};

// The tile's intervals span part of each chunk only (of unsorted batches a few entries of
// every chunk): the tile's waves narrow a chunk each for all of them, so that 16 chunks are
// not searched throughout by each of 16 waves (bound by scattered requests: 32,000 in no order
// and 2 M intervals, removals 147 to 72 us, the merge of the kept additions below 325 to 86).
// Up to six chunks of removals the barrier costs sorted ones what it gives the others (12,000
// and 2 M intervals, the whole call: sorted 71 without and 76 us with it, unsorted 120 and 103).
constexpr uint64_t kNarrowFrom = 6;
constexpr int kMostChunks = (int)(kMaxChunked / kSmall);
static_assert(kMostChunks <= kTileThreads / 64, "one chunk per wave");
struct Narrowed {
  uint64_t lo[kMostChunks], hi[kMostChunks];
};

__global__ __launch_bounds__(kTileThreads) void survive_kernel(MapRef map, Removals R, Kept K) {
  __shared__ uint32_t wcount[kTileWords];
  __shared__ Narrowed near;  // hi 0: the chunk meets nothing here
  const uint64_t count = map.hdr[0];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t tile0 = (uint64_t)blockIdx.x * kTile, p0 = tile0 + 64 * wave, p = p0 + lane;
  if (blockIdx.x == 0 && threadIdx.x == 0) K.count[0] = count;
  bool stay = p < count;
  const uint64_t at = stay ? p : count - 1;
  uint64_t s = 0;
  ulonglong2 et = make_ulonglong2(0, 0);
  if (p0 < count) {
    s = map.start[at];
    et = map.et[at];
  }
  const bool narrow = R.n > kNarrowFrom * R.chunk;
  if (narrow && tile0 < count && (uint64_t)wave * R.chunk < R.n) {
    const uint64_t c = (uint64_t)wave * R.chunk, n = min(R.chunk, R.n - c);
    const uint64_t *key = R.key + c, *max = R.max + c;
    const uint64_t first = map.start[tile0], last = map.et[min(tile0 + kTile, count) - 1].x - 1;
    uint64_t lo = 0, hi = 0;
    if (key[0] <= last && max[n - 1] >= first) {
      hi = wave_count_below<true>(key, n, last, lane);
      if (max[hi - 1] >= first) lo = wave_count_below<true>(key, hi, first, lane);  // (hi >= 1: key[0] <= last)
      else hi = 0;
    }
    if (lane == 0) {
      near.lo[wave] = lo;
      near.hi[wave] = hi;
    }
  }
  if (narrow) __syncthreads();
  if (p0 < count) {  // the wave's intervals lie between `first` and `last`
    const uint64_t first = uniform64(s, 0), last = uniform64(et.x, 63) - 1;
    uint32_t x = 0;
    for (uint64_t c = 0; c < R.n; c += R.chunk, ++x) {
      const uint64_t *key = R.key + c, *max = R.max + c;
      uint64_t lo = 0, hi = min(R.chunk, R.n - c);
      if (narrow) {
        lo = near.lo[x];
        hi = near.hi[x];
        if (hi == 0) continue;
      } else if (key[0] > last || max[hi - 1] < first) {
        continue;
      }
      if (hi - lo > 64) {
        hi = lo + wave_count_below<true>(key + lo, hi - lo, last, lane);
        if (hi == 0 || max[hi - 1] < first) continue;
        lo += wave_count_below<true>(key + lo, hi - lo, first, lane);
      }
      const uint64_t q = count_below<true>(key, lo, hi, et.x - 1);
      if (q && max[q - 1] >= s) stay = false;
    }
    if (p < count) {
      K.start[p] = s;
      K.et[p] = et;
    }
  }
  const uint64_t word = __ballot(stay);
  if (lane == 0) wcount[wave] = (uint32_t)__popcll(word);
  __syncthreads();
  uint32_t before = 0, total = 0;
  for (int w = 0; w < (int)kTileWords; ++w) {
    before += w < wave ? wcount[w] : 0;
    total += wcount[w];
  }
  if (lane == 0) {
    K.word[p0 / 64] = word;
    K.wpre[p0 / 64] = before;
  }
  if (threadIdx.x == 0) {
    K.tcount[blockIdx.x] = total;
    if (blockIdx.x == gridDim.x - 1) K.tcount[gridDim.x] = 0;
  }
}

// Survivors among the first i intervals; `base` the exclusive scan of the tile counts.
template <class T>
__device__ __forceinline__ uint64_t survivors_before(const Kept& K, const T* base, uint64_t i) {
  const uint64_t b = base[i / kTile];
  if (i % kTile == 0) return b;  // (i may be the end of the last tile)
  const uint64_t w = K.word[i / 64];
  return b + K.wpre[i / 64] + (uint64_t)__popcll(w & ((1ull << (i & 63)) - 1));
}

// ---- additions --------------------------------------------------------------------------
__device__ __forceinline__ uint32_t top_bit(uint32_t x) {  // largest power of two <= x (x >= 1)
  return 1u << (31 - __builtin_clz(x));
}

// Does a valid addition [s, e), entry k of the chunk at c, meet another one of its chunk
// (of one that starts before it, the furthest end; the next one's start)?
__device__ __forceinline__ bool meets_own_chunk(const Additions& A, uint64_t c, uint64_t n, uint64_t k, uint64_t s,
                                                uint64_t e) {
  return (k > 0 && A.max[c + k - 1] > s) || (k + 1 < n && A.key[c + k + 1] < e);
}

// Which additions are kept, their places among the other chunks and the survivors before each:
// 256 to a workgroup, as the searches are bound by each CU's rate of scattered requests (16,000 in
// no order and 200,000 intervals: 88 us with a chunk of 2,048 to a workgroup, 33 so; in address
// order 21 and 12). Without additions one workgroup of 1,024. Without `scanned` the tile counts
// are scanned here, by every workgroup for itself; the first one stores the scan.
constexpr int kClassThreads = 256;
static_assert(kSmall % kClassThreads == 0, "a workgroup's additions are of one chunk");
template <int kThreads>
__global__ __launch_bounds__(kThreads) void classify_chunks_kernel(Kept K, Additions A, Batches in, uint32_t tiles,
                                                                   uint32_t scanned) {
  __shared__ uint32_t base[kLdsTiles + 1];
  __shared__ uint32_t wave_sum[kThreads / 64];
  const uint32_t t = threadIdx.x;
  const int lane = t & 63, wave = t >> 6;
  const uint64_t c = (uint64_t)blockIdx.x * kThreads / kSmall * kSmall;
  const uint32_t n = A.n ? (uint32_t)min(A.n - c, (uint64_t)kSmall) : 0;
  const uint32_t k = (uint32_t)((uint64_t)blockIdx.x * kThreads - c) + t;
  const uint64_t at = c + (k < n ? k : 0);
  const uint64_t s = n ? A.key[at] : kNone, e = n ? A.end[at] : 0, id = n ? A.idx[at] : 0;
  const bool valid = k < n && s != kNone;
  bool clash = valid && meets_own_chunk(A, c, n, k, s, e);
  if (!scanned) {
    constexpr uint32_t kMost = kLdsTiles / kThreads;
    const uint32_t each = (tiles + kThreads - 1) / kThreads;  // at most kMost
    uint32_t v[kMost], sum = 0;
#pragma unroll
    for (uint32_t j = 0; j < kMost; ++j) {
      v[j] = j < each && t * each + j < tiles ? (uint32_t)K.tcount[t * each + j] : 0;
      sum += v[j];
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
    for (uint32_t j = 0; j < kMost; ++j) {
      if (j < each && t * each + j < tiles) {
        base[t * each + j] = run;
        if (blockIdx.x == 0) K.tbase[t * each + j] = run;
      }
      run += v[j];
    }
    if (t == kThreads - 1) {
      base[tiles] = run;
      if (blockIdx.x == 0) K.tbase[tiles] = run;
    }
  }
  if (n == 0) return;
  // the wave's additions lie between its first start and the furthest end up to its last
  const uint32_t w0 = k - (uint32_t)lane;
  const uint64_t first = w0 < n ? A.key[c + w0] : kNone, furthest = w0 < n ? A.max[c + min(w0 + 63, n - 1)] : 0;
  const bool some = first != kNone;  // the wave
  // other chunks, four at a time so that their searches wait together
  for (uint64_t c0 = 0; some && c0 < A.n; c0 += 4 * kSmall) {
    const uint64_t* key[4];
    uint32_t len[4], q[4];
    bool any = false;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint64_t cj = c0 + j * kSmall;
      len[j] = cj < A.n && cj != c ? (uint32_t)min(A.n - cj, (uint64_t)kSmall) : 0;
      key[j] = A.key + (len[j] ? cj : 0);
      q[j] = 0;
      if (len[j] && key[j][0] >= furthest) {
        len[j] = 0;
      } else if (len[j] && A.max[cj + len[j] - 1] <= first) {  // they all start (and end) before
        q[j] = len[j];
        len[j] = 0;
      }
      any |= len[j] != 0;
    }
    if (any) {
      for (uint32_t step = kSmall; step; step >>= 1) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (q[j] + step <= len[j] && key[j][q[j] + step - 1] < e) q[j] += step;
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (valid && len[j] && q[j] && A.max[c0 + j * kSmall + q[j] - 1] > s) clash = true;
    }
    if (valid) {  // (of an addition that is kept, those that start before its end start before it)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint64_t cj = c0 + j * kSmall;
        if (cj < A.n && cj != c) A.below[cj / kSmall * A.n + at] = (uint16_t)q[j];
      }
    }
  }
  // The intervals that start before the end (i1) and those that start at or before the
  // start (i0). Usually few lie between the wave's first start and its furthest end: the wave
  // finds those, each lane its own among them.
  uint64_t i0 = 0, i1 = 0;
  if (some) {
    const uint64_t count = K.count[0];
    const uint64_t lo = wave_count_below<true>(K.start, count, first, lane);
    const uint64_t len = wave_count_below<true>(K.start, count, furthest - 1, lane) - lo;
    for (uint64_t step = len ? top_bit((uint32_t)len) : 0; step; step >>= 1) {  // len <= 2^31
      if (i1 + step <= len && K.start[lo + i1 + step - 1] < e) i1 += step;
      if (i0 + step <= len && K.start[lo + i0 + step - 1] <= s) i0 += step;
    }
    i1 += lo;
    i0 += lo;
    if (valid && i0 && K.et[i0 - 1].x > s) --i0;  // those that end at or before the start
  }
  __syncthreads();  // the tile bases
  bool keep = false;
  if (valid) {
    const uint64_t before = scanned ? survivors_before(K, K.tbase, i0) : survivors_before(K, base, i0);
    const uint64_t up_to = scanned ? survivors_before(K, K.tbase, i1) : survivors_before(K, base, i1);
    keep = !clash && up_to == before;
    A.srank[at] = before;
    if (in.status) in.status[id] = keep ? GLEAM_REMAP_ADDED : GLEAM_REMAP_OVERLAP;
  }
  const uint64_t word = __ballot(keep);
  if (lane == 0 && w0 < n) A.acc[(c + w0) / 64] = word;
}

// The same over the whole device, for one chunk of every addition; the numbers come from a
// scan of `acc`.
__global__ __launch_bounds__(kThreads) void classify_all_kernel(Kept K, Additions A, Batches in) {
  const uint64_t count = K.count[0];
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < A.n; k += stride) {
    const uint64_t s = A.key[k];
    uint64_t a = 0;
    if (s != kNone) {
      const uint64_t e = A.end[k];
      const uint64_t i1 = count_below<true>(K.start, 0, count, e - 1);
      uint64_t i0 = count_below<true>(K.start, 0, i1, s);
      if (i0 && K.et[i0 - 1].x > s) --i0;
      const uint64_t before = survivors_before(K, K.tbase, i0);
      const bool clash = meets_own_chunk(A, 0, A.n, k, s, e) || survivors_before(K, K.tbase, i1) > before;
      a = clash ? 0 : 1;
      A.srank[k] = before;
      if (in.status) in.status[A.idx[k]] = clash ? GLEAM_REMAP_OVERLAP : GLEAM_REMAP_ADDED;
    }
    A.acc[k] = a;
  }
}

// ---- merge ------------------------------------------------------------------------------
// The kept additions: how many, and how many among the first k of the chunk at c (of n). In
// chunks they are counted from their bits, which every workgroup scans for itself.
template <bool kChunked>
struct KeptAdditions;

template <>
struct KeptAdditions<true> {
  static constexpr uint32_t kWords = (uint32_t)(kMaxChunked / 64), kOwn = (uint32_t)(kSmall / 64) + 1;
  static_assert(kWords <= (uint32_t)kTileThreads && kOwn <= 64, "one word per thread");
  static constexpr uint32_t kLds = kWords + 1 > kOwn * kTileWords ? kWords + 1 : (uint32_t)(kOwn * kTileWords);
  struct Lds {
    uint64_t word[kLds];
    uint32_t before[kLds], wave[kWords / 64];
  };
  const Lds& lds;
  uint32_t own;  // where the counts of this wave begin
  uint64_t total;
  // Every thread of the workgroup calls it. The words of one chunk are scanned by each wave for
  // itself: the barriers cost 3 of 16 us in a map of 2 M intervals.
  __device__ KeptAdditions(const Additions& A, Lds& l) : lds(l), own(0), total(0) {
    if (A.n == 0) return;
    const uint32_t t = threadIdx.x, wave = t >> 6, lane = t & 63;
    const bool one = A.n <= kSmall;
    const uint32_t at = one ? lane : t;
    const uint64_t word = at < kWords && 64 * (uint64_t)at < A.n ? A.acc[at] : 0;
    const uint32_t c = (uint32_t)__popcll(word);
    uint32_t incl = c;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(incl, d, 64);
      if (lane >= (uint32_t)d) incl += y;
    }
    if (one) {
      own = kOwn * wave;
      total = __shfl(incl, 63, 64);
      if (lane < kOwn) {
        l.word[own + lane] = word;
        l.before[own + lane] = incl - c;
      }
      wave_lds_sync();
      return;
    }
    if (t < kWords) {
      l.word[t] = word;
      if (lane == 63) l.wave[wave] = incl;
    }
    __syncthreads();
    if (t < kWords) {
      for (uint32_t w = 0; w < wave; ++w) incl += l.wave[w];
      l.before[t] = incl - c;
      if (t == kWords - 1) l.before[kWords] = incl;
    }
    __syncthreads();
    total = l.before[kWords];
  }
  __device__ __forceinline__ uint32_t up_to(uint64_t i) const {
    const uint32_t at = own + (uint32_t)(i / 64);
    return lds.before[at] + (i % 64 ? (uint32_t)__popcll(lds.word[at] & ((1ull << (i % 64)) - 1)) : 0);
  }
  __device__ __forceinline__ uint64_t before(const Additions&, uint64_t c, uint64_t, uint64_t k) const {
    return up_to(c + k) - up_to(c);
  }
  __device__ __forceinline__ bool kept(const Additions&, uint64_t k) const {
    return (lds.word[own + k / 64] >> (k % 64)) & 1;
  }
};

template <>
struct KeptAdditions<false> {  // one chunk
  struct Lds {};
  uint64_t total;
  __device__ KeptAdditions(const Additions& A, Lds&) { total = before(A, 0, A.n, A.n); }
  __device__ __forceinline__ uint64_t before(const Additions& A, uint64_t, uint64_t n, uint64_t k) const {
    return k < n ? A.pos[k] : A.pos[n - 1] + A.acc[n - 1];
  }
  __device__ __forceinline__ bool kept(const Additions& A, uint64_t k) const { return A.acc[k] != 0; }
};

// Workgroups [0, tiles): the survivors of a tile each; the others the additions. When
// the result would not fit, the kept additions are FULL instead. The first one also writes
// the header and the counts.
template <bool kChunked>
__global__ __launch_bounds__(kTileThreads) void place_kernel(MapRef map, Kept K, Additions A, Batches in,
                                                             uint32_t tiles, uint64_t* counts) {
  __shared__ typename KeptAdditions<kChunked>::Lds lds;
  __shared__ Narrowed near;  // entries of each chunk that start before the tile's first survivor, and its last
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t before = K.count[0], n_surv = K.tbase[tiles];
  const KeptAdditions<kChunked> kept(A, lds);
  const uint64_t n_acc = kept.total;
  const uint64_t total = n_surv + n_acc;
  const bool fits = total <= map.cap;
  const uint64_t S = total > kFence ? (total + kFence - 1) / kFence : 1;
  auto place = [&](uint64_t q, uint64_t s, ulonglong2 et) {
    map.start[q] = s;
    map.et[q] = et;
    if (q % S == 0) map.fence[q / S] = s;
  };
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    counts[0] = fits ? total : before;
    counts[1] = fits ? n_acc : 0;
    counts[2] = fits ? before - n_surv : 0;
    counts[3] = A.n - (fits ? n_acc : 0);
    if (fits) {
      map.hdr[0] = total;
      map.hdr[1] = S;
      map.hdr[2] = (total + S - 1) / S;
    }
  }
  if (blockIdx.x < tiles) {
    const uint64_t tile0 = (uint64_t)blockIdx.x * kTile, p0 = tile0 + 64 * wave, p = p0 + lane;
    if (!fits || tile0 >= before) return;  // the workgroup
    const bool narrow = A.n > A.chunk;
    if (narrow && (uint64_t)wave * A.chunk < A.n) {
      const uint64_t c = (uint64_t)wave * A.chunk, n = min(A.chunk, A.n - c);
      const uint64_t* key = A.key + c;
      const uint64_t first = K.start[tile0], last = K.start[min(tile0 + kTile, before) - 1];
      uint64_t lo = 0, hi = 0;
      if (key[0] < last) {
        lo = hi = n;
        if (key[n - 1] >= first) {
          lo = wave_count_below<false>(key, n, first, lane);
          hi = lo + wave_count_below<false>(key + lo, n - lo, last, lane);
        }
      }
      if (lane == 0) {
        near.lo[wave] = lo;
        near.hi[wave] = hi;
      }
    }
    if (narrow) __syncthreads();
    if (p0 >= before) return;  // the wave
    const uint64_t at = p < before ? p : before - 1;
    const uint64_t s = K.start[at], word = K.word[p0 / 64];
    const uint64_t first = uniform64(s, 0), last = uniform64(s, 63);
    uint64_t q = K.tbase[blockIdx.x] + K.wpre[p0 / 64] + (uint64_t)__popcll(word & ((1ull << lane) - 1));
    uint32_t x = 0;
    for (uint64_t c = 0; c < A.n; c += A.chunk, ++x) {
      const uint64_t n = min(A.chunk, A.n - c);
      const uint64_t* key = A.key + c;
      uint64_t lo = 0, hi = n;
      if (narrow) {
        lo = near.lo[x];
        hi = near.hi[x];
      } else if (key[0] >= last) {
        continue;
      } else if (key[n - 1] < first) {
        lo = n;
      }
      if (hi - lo > 64) {
        const uint64_t from = lo;
        lo += wave_count_below<false>(key + from, hi - from, first, lane);
        hi = from + wave_count_below<false>(key + from, hi - from, last, lane);
      }
      q += kept.before(A, c, n, lo == hi ? lo : count_below<false>(key, lo, hi, s));
    }
    if ((word >> lane) & 1) place(q, s, K.et[p]);
    return;
  }
  for (uint64_t k = (uint64_t)(blockIdx.x - tiles) * kTile + threadIdx.x; k < A.n;
       k += (uint64_t)(gridDim.x - tiles) * kTile) {
    if (!kept.kept(A, k)) continue;
    if (!fits) {
      if (in.status) in.status[A.idx[k]] = GLEAM_REMAP_FULL;
      continue;
    }
    const uint64_t s = A.key[k], own = k / A.chunk * A.chunk;
    uint64_t q = A.srank[k] + kept.before(A, own, min(A.chunk, A.n - own), k - own);
    uint32_t x = 0;
    for (uint64_t c = 0; c < A.n; c += A.chunk, ++x)
      if (c != own) q += kept.before(A, c, min(A.chunk, A.n - c), A.below[x * A.n + k]);
    place(q, s, make_ulonglong2(A.end[k], in.a_target[A.idx[k]] - s));
  }
}

// Translation. The interval that can hold address a is the last one starting at or
// before a. The fence (in LDS) narrows it to one run of S starts: if f fence entries
// are <= a, the answer lies in [(f - 1) S, f S), whose first start is known <= a. Both
// searches count the entries <= a by binary lifting, a fixed number of halving steps
// that the lanes of a wave take together. Each global step is a different cache line
// for nearly every lane, so the kernel is bound by the L2's request rate, not by bytes
// or by latency (carrying several addresses per lane measured no faster, and reading a run
// once, as whole lines by 16 lanes for each address, 43.7 against 41.3 us for 2^20 pointers
// over 209 k intervals, though 82 against 117 over 2 M). The fence is read with all its loads
// in flight together: 41.3 to 39.3 us.
__global__ void __launch_bounds__(kTranslateThreads)
translate_kernel(MapRef map, const uint64_t* addr, uint64_t n, uint64_t* out) {
  __shared__ uint64_t fence[kFence];
  // count <= 2^31 intervals, so every index and run length fits in 32 bits
  const uint32_t count = (uint32_t)map.hdr[0], S = (uint32_t)map.hdr[1], F = (uint32_t)map.hdr[2];
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  // the first address and the fence, read together; later addresses one round ahead
  uint64_t next = addr[i < n ? i : n - 1];
  constexpr uint32_t kEach = kFence / kTranslateThreads;
  uint64_t v[kEach];
#pragma unroll
  for (uint32_t j = 0; j < kEach; ++j) {
    const uint32_t k = j * kTranslateThreads + threadIdx.x;
    if (j * kTranslateThreads < F) v[j] = map.fence[k < F ? k : 0];  // (uniform)
  }
#pragma unroll
  for (uint32_t j = 0; j < kEach; ++j)
    if (j * kTranslateThreads < F) fence[j * kTranslateThreads + threadIdx.x] = v[j];
  __syncthreads();
  const uint32_t f_top = F ? top_bit(F) : 0, s_top = S > 1 ? top_bit(S - 1) : 0;
  for (; i < n; i += stride) {
    const uint64_t a = next;
    next = addr[i + stride < n ? i + stride : n - 1];
    uint32_t f = 0;
    for (uint32_t step = f_top; step; step >>= 1)
      if (f + step <= F && fence[f + step - 1] <= a) f += step;
    uint64_t r = GLEAM_UNMAPPED;
    if (f) {
      // the starts in (lo, hi) that are <= a
      const uint32_t lo = (f - 1) * S;
      const uint32_t len = (count - lo > S ? S : count - lo) - 1;
      uint32_t c = 0;
      for (uint32_t step = s_top; step; step >>= 1)
        if (c + step <= len && map.start[lo + c + step] <= a) c += step;
      const ulonglong2 et = map.et[lo + c];  // start[lo + c] <= a: inside iff a < end
      if (a < et.x) r = a + et.y;
    }
    out[i] = r;
  }
}

__global__ void export_kernel(MapRef map, uint64_t* d_start, uint64_t* d_len, uint64_t* d_target,
                              uint64_t* d_count) {
  const uint64_t count = map.hdr[0];
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  const uint64_t first = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (first == 0) d_count[0] = count;
  for (uint64_t p = first; p < count; p += stride) {
    const uint64_t s = map.start[p];
    const ulonglong2 et = map.et[p];
    d_start[p] = s;
    d_len[p] = et.x - s;
    d_target[p] = et.y + s;
  }
}

gleam_status hip_call(hipError_t e, const char* what) {
  if (e != hipSuccess) {
    set_error("%s: %s", what, hipGetErrorString(e));
    return GLEAM_E_HIP;
  }
  return launch_status(what);
}

}  // namespace
// Loads this file's GPU code object on the current device (gleam_preload).
hipError_t preload_remap() {
  hipFuncAttributes attr;
  return hipFuncGetAttributes(&attr, reinterpret_cast<const void*>(&export_kernel));
}

}  // namespace gleam

extern "C" size_t gleam_remap_bytes(uint64_t capacity) {
  if (capacity == 0 || capacity > gleam::kMaxCount) return 0;
  return gleam::kHeaderBytes + 24 * (size_t)capacity + 8 * (size_t)gleam::kFence;
}

extern "C" gleam_status gleam_remap_create(void* d_storage, size_t bytes, uint64_t capacity, gleam_remap** out,
                                           void* stream) {
  using namespace gleam;
  clear_error();
  if (!out) {
    set_error("gleam_remap_create: null output handle");
    return GLEAM_E_INVALID;
  }
  *out = nullptr;
  const size_t need = gleam_remap_bytes(capacity);
  if (need == 0) {
    set_error("gleam_remap_create: capacity must be in [1, 2^31]");
    return GLEAM_E_INVALID;
  }
  if (!d_storage || !aligned256(d_storage)) {
    set_error("gleam_remap_create: storage must be non-null and 256-byte aligned");
    return GLEAM_E_INVALID;
  }
  if (bytes < need) {
    set_error("gleam_remap_create: storage of %zu bytes, %zu needed", bytes, need);
    return GLEAM_E_INVALID;
  }
  gleam_remap* m = new (std::nothrow) gleam_remap;
  if (!m) {
    set_error("gleam_remap_create: out of host memory");
    return GLEAM_E_INVALID;
  }
  m->storage = static_cast<uint8_t*>(d_storage);
  m->capacity = capacity;
  const gleam_status st = fill_u64(reinterpret_cast<uint64_t*>(m->storage), kHeaderBytes / 8, 0,
                                   (hipStream_t)stream);
  if (st != GLEAM_OK) {
    delete m;
    return st;
  }
  *out = m;
  return GLEAM_OK;
}

extern "C" gleam_status gleam_remap_destroy(gleam_remap* m) {
  delete m;
  return GLEAM_OK;
}

extern "C" size_t gleam_remap_update_bytes(const gleam_remap* m, uint64_t n_add, uint64_t n_del) {
  if (!m || n_add > gleam::kMaxCount || n_del > gleam::kMaxCount) return 0;
  return gleam::upd_layout(m->capacity, n_add, n_del).total;
}

extern "C" gleam_status gleam_remap_update(gleam_remap* m, const uint64_t* d_del_start, const uint64_t* d_del_len,
                                           uint64_t n_del, const uint64_t* d_add_start, const uint64_t* d_add_len,
                                           const uint64_t* d_add_target, uint64_t n_add, uint8_t* d_add_status,
                                           uint64_t* d_counts, void* d_ws, size_t ws_bytes, void* stream) {
  using namespace gleam;
  clear_error();
  if (!m || !d_counts) {
    set_error("gleam_remap_update: null map or counts");
    return GLEAM_E_INVALID;
  }
  if ((n_del > 0 && (!d_del_start || !d_del_len)) || (n_add > 0 && (!d_add_start || !d_add_len || !d_add_target))) {
    set_error("gleam_remap_update: null removal or addition array");
    return GLEAM_E_INVALID;
  }
  if (n_add > kMaxCount || n_del > kMaxCount) {
    set_error("gleam_remap_update: more than 2^31 additions or removals");
    return GLEAM_E_UNSUPPORTED;
  }
  const UpdLayout L = upd_layout(m->capacity, n_add, n_del);
  if (!d_ws || !aligned256(d_ws)) {
    set_error("gleam_remap_update: workspace must be non-null and 256-byte aligned");
    return GLEAM_E_INVALID;
  }
  if (ws_bytes < L.total) {
    set_error("gleam_remap_update: workspace of %zu bytes, %zu needed", ws_bytes, L.total);
    return GLEAM_E_WORKSPACE;
  }
  hipStream_t s = (hipStream_t)stream;
  uint8_t* b = static_cast<uint8_t*>(d_ws);
  auto at = [&](size_t off) { return reinterpret_cast<uint64_t*>(b + off); };
  uint64_t* hdr = at(L.hdr);
  uint64_t* partial = at(L.partial);
  void* sort_ws = b + L.sort;
  const MapRef map = map_ref(m);
  const uint64_t cap = m->capacity;
  gleam_status st;
  const Batches in{d_del_start, d_del_len, d_add_start, d_add_len, d_add_target, n_del, n_add, d_add_status};
  const Removals R{at(L.rkb), at(L.rmax), n_del, chunk_of(n_del)};
  const Additions A{at(L.kb), at(L.vb), at(L.aend), at(L.amax), at(L.acc), at(L.apos), at(L.srank),
                    reinterpret_cast<uint16_t*>(b + L.below), n_add, chunk_of(n_add)};
  const Kept K{hdr + 12, at(L.keep), reinterpret_cast<uint32_t*>(b + L.wpre), at(L.tcount), at(L.tbase),
               at(L.s_start), reinterpret_cast<ulonglong2*>(b + L.s_et)};
  const bool many_del = n_del > kMaxChunked, many_add = n_add > kMaxChunked;
  const uint32_t tiles = (uint32_t)L.tiles;

  // 1. both batches sorted
  const uint32_t r_chunks = many_del ? 0 : (uint32_t)((n_del + kSmall - 1) / kSmall);
  const uint32_t a_chunks = many_add ? 0 : (uint32_t)((n_add + kSmall - 1) / kSmall);
  if (r_chunks + a_chunks > 0) {
    hipLaunchKernelGGL(sort_chunks_kernel, dim3(r_chunks + a_chunks), dim3(kSmallThreads), 0, s, in, R, A, r_chunks);
    if ((st = launch_status("sort_chunks_kernel")) != GLEAM_OK) return st;
  }
  if (many_del || many_add) {
    hipLaunchKernelGGL(update_init_kernel, dim3(1), dim3(64), 0, s, hdr, n_del, n_add);
    if ((st = launch_status("update_init_kernel")) != GLEAM_OK) return st;
  }
  if (many_del) {
    const SortBuf ra{nullptr, at(L.rka), reinterpret_cast<uint32_t*>(b + L.ridx)};
    const SortBuf rb = sort_other(sort_ws, n_del, 1);
    hipLaunchKernelGGL(removal_prep_kernel, dim3(fold_grid(n_del)), dim3(kThreads), 0, s, d_del_start, d_del_len,
                       n_del, ra.lo, ra.idx, hdr + 4);
    if ((st = launch_status("removal_prep_kernel")) != GLEAM_OK) return st;
    if ((st = radix_sort_pairs(ra, hdr, hdr + 4, n_del, 1, sort_ws, s)) != GLEAM_OK) return st;
    hipLaunchKernelGGL(removal_unpack_kernel, dim3(grid_for(n_del)), dim3(kThreads), 0, s, ra, rb, hdr + 4,
                       d_del_start, d_del_len, n_del, R.key, at(L.last));
    if ((st = launch_status("removal_unpack_kernel")) != GLEAM_OK) return st;
    if ((st = device_scan<ScanMax, false>(at(L.last), R.max, n_del, partial, s)) != GLEAM_OK) return st;
  }
  if (many_add) {
    const SortBuf aa{nullptr, at(L.ka), reinterpret_cast<uint32_t*>(b + L.aidx)};
    const SortBuf ab = sort_other(sort_ws, n_add, 1);
    hipLaunchKernelGGL(addition_prep_kernel, dim3(fold_grid(n_add)), dim3(kThreads), 0, s, d_add_start, d_add_len,
                       d_add_target, n_add, d_add_status, aa.lo, aa.idx, hdr + 8);
    if ((st = launch_status("addition_prep_kernel")) != GLEAM_OK) return st;
    if ((st = radix_sort_pairs(aa, hdr + 1, hdr + 8, n_add, 1, sort_ws, s)) != GLEAM_OK) return st;
    hipLaunchKernelGGL(addition_unpack_kernel, dim3(grid_for(n_add)), dim3(kThreads), 0, s, aa, ab, hdr + 8,
                       d_add_len, n_add, A.key, A.idx, A.end);
    if ((st = launch_status("addition_unpack_kernel")) != GLEAM_OK) return st;
    if ((st = device_scan<ScanMax, false>(A.end, A.max, n_add, partial, s)) != GLEAM_OK) return st;
  }

  // 2. survivors
  hipLaunchKernelGGL(survive_kernel, dim3(tiles), dim3(kTileThreads), 0, s, map, R, K);
  if ((st = launch_status("survive_kernel")) != GLEAM_OK) return st;
  const bool scanned = many_add || L.tiles > kLdsTiles;
  if (scanned && (st = device_scan<ScanSum, true>(K.tcount, K.tbase, L.tiles + 1, partial, s)) != GLEAM_OK) return st;

  // 3. additions checked against each other and the survivors, and numbered
  if (many_add) {
    hipLaunchKernelGGL(classify_all_kernel, dim3(grid_for(n_add)), dim3(kThreads), 0, s, K, A, in);
    if ((st = launch_status("classify_all_kernel")) != GLEAM_OK) return st;
    if ((st = device_scan<ScanSum, true>(A.acc, A.pos, n_add, partial, s)) != GLEAM_OK) return st;
  } else {
    if (n_add)
      hipLaunchKernelGGL(classify_chunks_kernel<kClassThreads>, dim3((uint32_t)((n_add + kClassThreads - 1) / kClassThreads)),
                         dim3(kClassThreads), 0, s, K, A, in, tiles, scanned ? 1u : 0u);
    else
      hipLaunchKernelGGL(classify_chunks_kernel<kTileThreads>, dim3(1), dim3(kTileThreads), 0, s, K, A, in, tiles,
                         scanned ? 1u : 0u);
    if ((st = launch_status("classify_chunks_kernel")) != GLEAM_OK) return st;
  }

  // 4. merge by rank into the storage (only if everything fits), the header and the counts
  const uint64_t groups = (n_add + kTile - 1) / kTile;
  const uint32_t a_groups = (uint32_t)(groups < kMaxGrid ? groups : kMaxGrid);
  hipLaunchKernelGGL(many_add ? place_kernel<false> : place_kernel<true>, dim3(tiles + a_groups), dim3(kTileThreads), 0, s,
                     map, K, A, in, tiles, d_counts);
  return launch_status("place_kernel");
}

extern "C" gleam_status gleam_remap_translate(const gleam_remap* m, const uint64_t* d_addr, uint64_t n,
                                              uint64_t* d_out, void* stream) {
  using namespace gleam;
  clear_error();
  if (!m || (n > 0 && (!d_addr || !d_out))) {
    set_error("gleam_remap_translate: null map, addresses or output");
    return GLEAM_E_INVALID;
  }
  if (n == 0) return GLEAM_OK;
  int cus = 0;
  const gleam_status st = device_cu_count(&cus);
  if (st != GLEAM_OK) return st;
  // as many 1024-lane workgroups per CU as the LDS holds fences (at most two, 32 waves);
  // each loads the fence once
  const uint64_t per_cu = kFence * 8 <= 80 * 1024 ? 2 : 1;
  const uint64_t want = (n + kTranslateThreads - 1) / kTranslateThreads;
  const uint64_t grid = want < per_cu * cus ? want : per_cu * cus;
  hipLaunchKernelGGL(translate_kernel, dim3((uint32_t)grid), dim3(kTranslateThreads), 0, (hipStream_t)stream,
                     map_ref(m), d_addr, n, d_out);
  return launch_status("translate_kernel");
}

extern "C" gleam_status gleam_remap_export(const gleam_remap* m, uint64_t* d_start, uint64_t* d_len,
                                           uint64_t* d_target, uint64_t* d_count, void* stream) {
  using namespace gleam;
  clear_error();
  if (!m || !d_start || !d_len || !d_target || !d_count) {
    set_error("gleam_remap_export: null map or output");
    return GLEAM_E_INVALID;
  }
  hipLaunchKernelGGL(export_kernel, dim3(grid_for(m->capacity)), dim3(kThreads), 0, (hipStream_t)stream, map_ref(m),
                     d_start, d_len, d_target, d_count);
  return launch_status("export_kernel");
}
