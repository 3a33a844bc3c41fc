// Device-wide LSD radix sort of (key, index) pairs for the table's maintenance calls
// (eviction order and export order) and the address map's update (removals and
// additions by start), written for gfx950 so those calls enqueue kernels only (no
// library sort, no memsets): a caller may capture them in a HIP graph. Published methods: one
// histogram of every pass ahead of the passes is Onesweep's (Adinets and Merrill, "Onesweep:
// A Faster Least Significant Digit Radix Sort for GPUs", 2022), the running sums passed from
// workgroup to workgroup are decoupled look-back (Merrill and Garland, "Single-pass Parallel
// Prefix Scan with Decoupled Look-back", 2016).
//
// Keys are 64 or 128 bits (hi:lo), indices u32. Each pass sorts by one 8-bit digit,
// stably, over 4096-element tiles. Launches: one clear, one histogram of every digit of
// every pass (a digit's counts do not depend on the order), then one kernel per pass:
//   - a workgroup takes the next chunk of tiles by a ticket (one tile, or as many as keep
//     the chunks to kSortChunks); each wave of a tile owns consecutive elements and
//     ranks them stably (the lanes holding one digit find each other with eight ballots, a
//     running per-digit count in LDS carries the rank across the wave's rounds);
//   - it publishes the chunk's count of each digit (of a chunk of several tiles counted
//     beforehand), and thread d sums digit d's counts of the chunks before it, back to the
//     nearest one that has already published its running sum. A chunk's counts are
//     published before its workgroup waits for any other, and the chunks before it have
//     smaller tickets, so they are running or done: every wait ends, however few workgroups
//     the GPU holds at once;
//   - the tile is reordered in LDS by digit and written out word by word, so consecutive
//     lanes store consecutive addresses of one digit's run.
// What it is bound by: launches below about a million elements (three launches per pass,
// with separate histograms and scans, took 24 and 48 launches of at least 4 us), and the
// scattered writes of the passes above. (Chunks of one tile throughout: 20 M elements,
// 4,883 tiles, 0.7 ms per two-word pass, the running sums crossing the XCDs tile by tile.)
// A pass whose digit is the same for every key moves nothing and is skipped on the
// device: the caller supplies the AND and the OR of all key words, the pass kernels
// return at once for such a pass, and the buffers' roles (which holds the input) follow
// from how many passes before it were not skipped. Nothing is decided on the host, so
// the launches are fixed and a graph of them replays correctly for any keys.
// The sort is stable: equal keys keep their input order (the address map's callers
// number their entries in input order, so ties go to the lower index).
#pragma once

#include "gleam_device.h"
#include "gleam_internal.h"

namespace gleam {
namespace {

constexpr int kSortThreads = 256;
constexpr int kSortWaves = kSortThreads / 64;
constexpr int kSortItems = 16;                               // per lane
constexpr uint32_t kSortTile = kSortThreads * kSortItems;    // 4096 elements
constexpr uint32_t kSortWaveSpan = 64 * kSortItems;          // 1024 elements per wave
constexpr int kDigits = 256;

struct SortBuf {
  uint64_t* hi;  // null for 64-bit keys
  uint64_t* lo;
  uint32_t* idx;
};

// bits = {AND of lo words, OR of lo words, AND of hi words, OR of hi words} over the
// keys being sorted. Pass p's digit is bits 8p..8p+7 of the 128-bit key.
__device__ __forceinline__ bool pass_trivial(const uint64_t* bits, uint32_t p) {
  const uint32_t w = p >= 8 ? 2u : 0u;
  const uint64_t differ = bits[w] ^ bits[w + 1];
  return ((differ >> ((8 * p) & 63)) & 0xFFu) == 0;
}

// Whether pass p reads the workspace buffer (b) rather than the caller's (a).
__device__ __forceinline__ bool reads_b(const uint64_t* bits, uint32_t p) {
  uint32_t moved = 0;
  for (uint32_t q = 0; q < p; ++q) moved += pass_trivial(bits, q) ? 0u : 1u;
  return (moved & 1u) != 0;
}

// Where the sorted pairs are after all 8 * words passes.
__device__ __forceinline__ SortBuf sort_result(const SortBuf& a, const SortBuf& b, const uint64_t* bits, int words) {
  return reads_b(bits, 8u * (uint32_t)words) ? b : a;
}

// Zeroes the digit totals, the passes' tickets and the chunks' states.
__global__ __launch_bounds__(kSortThreads) void sort_clear_kernel(uint64_t* words, uint64_t n) {
  const uint64_t stride = (uint64_t)gridDim.x * kSortThreads;
  for (uint64_t i = (uint64_t)blockIdx.x * kSortThreads + threadIdx.x; i < n; i += stride) words[i] = 0;
}

// totals[pass][digit] of every pass that moves anything. A grid of at most
// kSortHistGrid workgroups walks the tiles, so that their final atomics stay few.
constexpr uint32_t kSortHistGrid = 256;
template <int kWords>
__global__ __launch_bounds__(kSortThreads) void sort_hist_kernel(SortBuf a, const uint64_t* n_dev, const uint64_t* bits,
                                                                 uint32_t* totals) {
  constexpr uint32_t kPasses = 8u * kWords;
  __shared__ uint32_t h[kPasses][kDigits];
  const uint64_t n = *n_dev;
  if ((uint64_t)blockIdx.x * kSortTile >= n) return;
  for (uint32_t p = 0; p < kPasses; ++p) h[p][threadIdx.x] = 0;
  __syncthreads();
  uint32_t moves = 0;  // bit p: pass p moves something
  for (uint32_t p = 0; p < kPasses; ++p) moves |= pass_trivial(bits, p) ? 0u : 1u << p;
  for (uint64_t base = (uint64_t)blockIdx.x * kSortTile; base < n; base += (uint64_t)gridDim.x * kSortTile) {
    uint64_t lo[kSortItems], hi[kSortItems];
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {  // unconditional (clamped) loads, issued together
      const uint64_t i = base + (uint64_t)r * kSortThreads + threadIdx.x;
      const uint64_t at = i < n ? i : n - 1;
      lo[r] = a.lo[at];
      hi[r] = kWords == 2 ? a.hi[at] : 0;
    }
    for (uint32_t p = 0; p < kPasses; ++p) {
      if (!((moves >> p) & 1u)) continue;
      const uint32_t sh = (8 * p) & 63;
#pragma unroll
      for (int r = 0; r < kSortItems; ++r) {
        const uint64_t i = base + (uint64_t)r * kSortThreads + threadIdx.x;
        const uint64_t w = kWords == 2 && p >= 8 ? hi[r] : lo[r];
        if (i < n) atomicAdd(&h[p][(uint32_t)(w >> sh) & 0xFFu], 1u);
      }
    }
  }
  __syncthreads();
  for (uint32_t p = 0; p < kPasses; ++p) {
    const uint32_t c = h[p][threadIdx.x];
    if (c) atomicAdd(&totals[p * kDigits + threadIdx.x], c);
  }
}

// The pass kernel: 512 threads of 8 elements (with 256 of 16, a two-word pass takes 172
// registers, 256 where the compiler keeps addresses across tiles, and half the waves).
constexpr int kPassThreads = 512;
constexpr int kPassWaves = kPassThreads / 64;
constexpr int kPassItems = (int)kSortTile / kPassThreads;

// Exclusive prefix over the workgroup's threads of two values at once.
__device__ __forceinline__ void block_excl_scan2(uint32_t& x, uint32_t& y, uint32_t (*tmp)[2]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t ix = x, iy = y;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t px = __shfl_up(ix, d, 64), py = __shfl_up(iy, d, 64);
    if (lane >= d) {
      ix += px;
      iy += py;
    }
  }
  if (lane == 63) {
    tmp[wave][0] = ix;
    tmp[wave][1] = iy;
  }
  __syncthreads();
  uint32_t bx = 0, by = 0;
#pragma unroll
  for (int w = 0; w < kPassWaves; ++w) {
    if (w < wave) {
      bx += tmp[w][0];
      by += tmp[w][1];
    }
  }
  x = bx + ix - x;
  y = by + iy - y;
}

// A chunk's published words, one per digit: {tag, count}. The tags of pass p are 2p + 1
// (the chunk's own count) and 2p + 2 (the count of this chunk and all before it), so the
// words of an earlier pass read as not yet published.
__device__ __forceinline__ uint64_t sort_state(uint32_t tag, uint32_t count) { return ((uint64_t)tag << 32) | count; }

// The elements with digit threadIdx.x in the chunks before `tile`. Reads kSortAhead chunks'
// words at once, from the nearest back.
template <uint32_t kSortAhead>
__device__ __forceinline__ uint32_t sort_before(uint64_t* state, uint64_t tile, uint32_t pass) {
  const uint32_t own = 2 * pass + 1, sum = 2 * pass + 2;
  uint32_t before = 0;
  uint64_t t = tile;
  while (t > 0) {
    uint64_t w[kSortAhead];
#pragma unroll
    for (uint32_t k = 0; k < kSortAhead; ++k) {
      const uint64_t at = t > k + 1 ? t - 1 - k : 0;
      w[k] = __hip_atomic_load(&state[at * kDigits + threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    bool stop = false;
#pragma unroll
    for (uint32_t k = 0; k < kSortAhead; ++k) {
      if (stop || t == 0) continue;
      const uint32_t tag = (uint32_t)(w[k] >> 32);
      if (tag != own && tag != sum) {  // not published yet: read again from here
        stop = true;
        continue;
      }
      before += (uint32_t)w[k];
      t = tag == sum ? 0 : t - 1;
    }
    if (stop) __builtin_amdgcn_s_sleep(1);
  }
  return before;
}

struct SortLds {
  uint32_t run[kPassWaves][kDigits];  // per wave: running digit counts, then first local positions
  uint32_t gdelta[kDigits];           // global position = gdelta[d] + local sorted position
  uint32_t scan_tmp[kPassWaves][2];
  uint64_t xch[kSortTile];            // the tile in local sorted order, one word at a time
  uint8_t xdig[kSortTile];            // digit of each local sorted position
  uint32_t my_tile;
};

// Up to kSortFineMax elements the tiles are a quarter (kSortItems 2 instead of 8): a pass of a
// few tiles takes as long as one workgroup does, which is mostly the chain of its ranking
// rounds. Two-word keys take half tiles up to kSortMidMax, as whole ones would leave half of
// the CUs idle (341,000 of 681,000 entries evicted: 322 to 275 us a call, all of 996,000 387 to
// 373; sorting the million keys of an export, one word each, 308 to 342, so those do not).
constexpr uint64_t kSortFineMax = 1u << 18;
constexpr uint32_t kSortFineTile = kSortTile / 4;
constexpr uint64_t kSortMidMax = 1u << 20;
constexpr uint32_t kSortMidTile = kSortTile / 2;
constexpr uint64_t kSortChunks = 512;  // two workgroups on each CU

template <int kWords, int kSortItems>
__device__ __forceinline__ void sort_pass(SortLds& lds, SortBuf a, SortBuf b, uint64_t n, const uint64_t* bits,
                                          uint32_t pass, const uint32_t* totals, uint64_t* state, uint32_t* ticket) {
  constexpr uint32_t kSortTile = kPassThreads * kSortItems, kSortWaveSpan = 64 * kSortItems;
  auto& run = lds.run;
  auto& gdelta = lds.gdelta;
  auto& scan_tmp = lds.scan_tmp;
  auto& xch = lds.xch;
  auto& xdig = lds.xdig;
  auto& my_tile = lds.my_tile;
  const uint64_t tiles = (n + kSortTile - 1) / kSortTile;
  const uint64_t chunk = (tiles + kSortChunks - 1) / kSortChunks;  // tiles per chunk
  // uniform over the workgroup; the workgroups below the chunk count take every ticket
  if ((uint64_t)blockIdx.x * chunk >= tiles || pass_trivial(bits, pass)) return;
  const bool from_b = reads_b(bits, pass);
  const SortBuf in = from_b ? b : a, out = from_b ? a : b;
  const uint32_t sh = (8 * pass) & 63;
  const bool digit_in_hi = kWords == 2 && pass >= 8;
  const uint32_t digit_total = threadIdx.x < kDigits ? totals[threadIdx.x] : 0;

  for (;;) {
    if (threadIdx.x == 0) my_tile = atomicAdd(ticket, 1u);
    if (threadIdx.x < kDigits) gdelta[threadIdx.x] = 0;
    __syncthreads();  // my_tile known, gdelta cleared
    const uint64_t mine_at = my_tile, first_tile = mine_at * chunk;
    if (first_tile >= tiles) return;
    const uint64_t end_tile = first_tile + chunk < tiles ? first_tile + chunk : tiles;
    const bool digit = threadIdx.x < kDigits;  // threads that look after digit threadIdx.x
    uint64_t* mine = &state[mine_at * kDigits + (digit ? threadIdx.x : 0)];
    uint32_t before = 0;  // elements with that digit before the next tile
    if (chunk > 1) {
      const uint64_t* word = digit_in_hi ? in.hi : in.lo;
      const uint64_t end = end_tile * kSortTile < n ? end_tile * kSortTile : n;
      for (uint64_t at0 = first_tile * kSortTile; at0 < end; at0 += kSortTile) {
        uint64_t w[kSortItems];
#pragma unroll
        for (int r = 0; r < kSortItems; ++r) {  // unconditional (clamped) loads, issued together
          const uint64_t i = at0 + (uint64_t)r * kPassThreads + threadIdx.x;
          w[r] = word[i < end ? i : end - 1];
        }
#pragma unroll
        for (int r = 0; r < kSortItems; ++r)
          if (at0 + (uint64_t)r * kPassThreads + threadIdx.x < end) atomicAdd(&gdelta[(uint32_t)(w[r] >> sh) & 0xFFu], 1u);
      }
      __syncthreads();
      if (digit) {
        const uint32_t count = gdelta[threadIdx.x];
        __hip_atomic_store(mine, sort_state(2 * pass + (mine_at ? 1 : 2), count), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        before = sort_before<8>(state, mine_at, pass);
        if (mine_at)
          __hip_atomic_store(mine, sort_state(2 * pass + 2, before + count), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    for (uint64_t tile = first_tile; tile < end_tile; ++tile) {
      // the thread number, opaque to the compiler: otherwise it keeps every round's element
      // numbers and LDS addresses in registers across the loop (256, one workgroup per CU)
      uint32_t tid = threadIdx.x;
      asm volatile("" : "+v"(tid));
      const int lane = tid & 63, wave = tid >> 6;
      const uint64_t lt_mask = lane ? (~0ull >> (64 - lane)) : 0ull;
      const uint64_t tile0 = tile * kSortTile;
      for (int k = tid; k < kPassWaves * kDigits; k += kPassThreads) (&run[0][0])[k] = 0;
      __syncthreads();  // run[] cleared
      const uint32_t in_tile = (uint32_t)(n - tile0 < kSortTile ? n - tile0 : kSortTile);

      uint64_t lo[kSortItems], hi[kSortItems];
      uint32_t ix[kSortItems], dg[kSortItems], pos[kSortItems];
#pragma unroll
      for (int r = 0; r < kSortItems; ++r) {  // unconditional (clamped) loads, issued together
        const uint32_t li = wave * kSortWaveSpan + r * 64 + lane;
        const uint64_t at = tile0 + (li < in_tile ? li : in_tile - 1);
        lo[r] = in.lo[at];
        hi[r] = kWords == 2 ? in.hi[at] : 0;
        ix[r] = in.idx[at];
      }

      // rank inside the wave, in element order: earlier rounds through run[wave][d], this
      // round through the peers below this lane
#pragma unroll
      for (int r = 0; r < kSortItems; ++r) {
        const uint32_t li = wave * kSortWaveSpan + r * 64 + lane;
        const bool valid = li < in_tile;
        const uint32_t d = (uint32_t)((digit_in_hi ? hi[r] : lo[r]) >> sh) & 0xFFu;
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int bit = 0; bit < 8; ++bit) {
          const uint64_t ones = __ballot(valid && ((d >> bit) & 1u));
          peers &= ((d >> bit) & 1u) ? ones : ~ones;
        }
        const uint32_t below = (uint32_t)__popcll(peers & lt_mask);
        const uint32_t prior = run[wave][d];
        dg[r] = d;
        pos[r] = prior + below;
        if (valid && below == 0) run[wave][d] = prior + (uint32_t)__popcll(peers);
        wave_lds_sync();  // this round's counts before the next round's reads
      }
      __syncthreads();  // every wave's digit counts complete

      {
        const uint32_t d = digit ? tid : 0;
        uint32_t c[kPassWaves], count = 0;
#pragma unroll
        for (int w = 0; w < kPassWaves; ++w) {
          c[w] = digit ? run[w][d] : 0;
          count += c[w];
        }
        if (chunk == 1 && digit)
          __hip_atomic_store(mine, sort_state(2 * pass + (mine_at ? 1 : 2), count), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
        uint32_t local = count;         // becomes the digit's first local position
        uint32_t global = digit_total;  // becomes the digit's first global position
        block_excl_scan2(local, global, scan_tmp);
        if (digit) {
          if (chunk == 1) {
            before = sort_before<4>(state, mine_at, pass);  // (few: the tile's elements hold the registers)
            if (mine_at)
              __hip_atomic_store(mine, sort_state(2 * pass + 2, before + count), __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
          }
          gdelta[d] = global + before - local;
          before += count;
          // (only this thread touches column d)
#pragma unroll
          for (int w = 0; w < kPassWaves; ++w) {
            run[w][d] = local;
            local += c[w];
          }
        }
      }
      __syncthreads();

#pragma unroll
      for (int r = 0; r < kSortItems; ++r) {
        const uint32_t li = wave * kSortWaveSpan + r * 64 + lane;
        if (li < in_tile) {
          pos[r] += run[wave][dg[r]];
          xdig[pos[r]] = (uint8_t)dg[r];
          xch[pos[r]] = lo[r];
        }
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < kSortItems; ++k) {
        const uint32_t j = k * kPassThreads + tid;
        if (j < in_tile) out.lo[gdelta[xdig[j]] + j] = xch[j];
      }
      if (kWords == 2) {
        __syncthreads();  // xch read out before it is refilled
#pragma unroll
        for (int r = 0; r < kSortItems; ++r) {
          const uint32_t li = wave * kSortWaveSpan + r * 64 + lane;
          if (li < in_tile) xch[pos[r]] = hi[r];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kSortItems; ++k) {
          const uint32_t j = k * kPassThreads + tid;
          if (j < in_tile) out.hi[gdelta[xdig[j]] + j] = xch[j];
        }
      }
      __syncthreads();
      uint32_t* xidx = reinterpret_cast<uint32_t*>(xch);
#pragma unroll
      for (int r = 0; r < kSortItems; ++r) {
        const uint32_t li = wave * kSortWaveSpan + r * 64 + lane;
        if (li < in_tile) xidx[pos[r]] = ix[r];
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < kSortItems; ++k) {
        const uint32_t j = k * kPassThreads + tid;
        if (j < in_tile) out.idx[gdelta[xdig[j]] + j] = xidx[j];
      }
      __syncthreads();  // run, xch and xdig read out before the next tile
    }
  }
}

// (three workgroups of eight waves per CU: as many as their LDS allows)
template <int kWords>
__global__ __launch_bounds__(kPassThreads, 4) void sort_pass_kernel(SortBuf a, SortBuf b, const uint64_t* n_dev,
                                                                 const uint64_t* bits, uint32_t pass,
                                                                 const uint32_t* totals, uint64_t* state,
                                                                 uint32_t* ticket) {
  __shared__ SortLds lds;
  const uint64_t n = *n_dev;
  if (n <= kSortFineMax)
    sort_pass<kWords, kPassItems / 4>(lds, a, b, n, bits, pass, totals, state, ticket);
  else if (kWords == 2 && n <= kSortMidMax)
    sort_pass<kWords, kPassItems / 2>(lds, a, b, n, bits, pass, totals, state, ticket);
  else
    sort_pass<kWords, kPassItems>(lds, a, b, n, bits, pass, totals, state, ticket);
}

// Sorts of at most kSortSmallMax elements run whole in one 1024-lane workgroup: every
// pass in one launch instead of a launch per pass. Wave w owns 64 * kSortItems consecutive
// elements, kSortItems per lane (element w * 64 * kSortItems + 64 r + lane in round r).
// A pass loads the digit word of the wave's share, ranks it stably with the same
// ballots and a running per-digit count in the wave's own LDS row (so no barrier
// between rounds), and turns the row totals into each wave's offset within each digit
// and a scan over digits into each digit's first position. It then moves the elements
// one word at a time through LDS: each lane reads its elements' word again (coalesced;
// the share does not fit in registers beside the ranks) and places it at its sorted
// position in LDS, and the workgroup writes LDS out in order, so the global stores
// are coalesced (a single CU scattering 8-byte stores is slow). Passes alternate
// between the two buffers through global memory, a workgroup barrier apart, and skip
// exactly the passes the large sort skips, so the result is where sort_result() says.
constexpr int kSortSmallThreads = 1024;
constexpr int kSortSmallWaves = kSortSmallThreads / 64;
constexpr uint32_t kSortSmallMax = (uint32_t)kSortSmallThreads * kSortItems;  // 16384

// A lane's 16 elements first + 64 r of src, loaded without a guard (the buffers hold
// sort_capacity(n_max) elements, a whole number of wave spans, so a wave that holds any
// element may read its whole span), so that the loads issue together rather than as one
// guarded round trip each. Elements past n are read but never used.
template <typename T, int kItems>
__device__ __forceinline__ void small_share(const T* src, uint32_t first, T (&x)[kItems]) {
#pragma unroll
  for (int r = 0; r < kItems; ++r) x[r] = src[first + r * 64];
}

struct SortSmallLds {
  uint32_t run[kSortSmallWaves][kDigits];  // per wave: digit counts, then offsets within each digit
  uint32_t dstart[kDigits];                // each digit's first position
  uint32_t wsum[kDigits / 64];
  uint64_t xch[kSortSmallMax];             // one word of every element, in sorted order
};

template <int kWords, int kSortItems>
__device__ __forceinline__ void sort_small(SortSmallLds& lds, SortBuf a, SortBuf b, uint32_t n, const uint64_t* bits) {
  constexpr uint32_t kSortWaveSpan = 64 * kSortItems;
  auto& run = lds.run;
  auto& dstart = lds.dstart;
  auto& wsum = lds.wsum;
  auto& xch = lds.xch;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t lt_mask = lane ? (~0ull >> (64 - lane)) : 0ull;
  const uint32_t span0 = (uint32_t)wave * kSortWaveSpan;
  const bool has = span0 < n;  // this wave's span holds elements (uniform over the wave)
  SortBuf in = a, out = b;
  for (uint32_t pass = 0; pass < 8u * kWords; ++pass) {
    if (pass_trivial(bits, pass)) continue;  // uniform: every lane reads the same words

    const uint32_t sh = (8 * pass) & 63;
    const uint64_t* word = (kWords == 2 && pass >= 8) ? in.hi : in.lo;
    for (int k = threadIdx.x; k < kSortSmallWaves * kDigits; k += kSortSmallThreads) (&run[0][0])[k] = 0;
    uint32_t rank[kSortItems];  // (position within the wave's share of the digit) << 8 | digit
    {
      uint64_t w[kSortItems] = {};
      if (has) small_share(word, span0 + lane, w);
#pragma unroll
      for (int r = 0; r < kSortItems; ++r) rank[r] = (uint32_t)(w[r] >> sh) & 0xFFu;
    }
    __syncthreads();  // run[] cleared
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
      const bool valid = span0 + r * 64 + lane < n;
      const uint32_t d = rank[r];
      uint64_t peers = __ballot(valid);
#pragma unroll
      for (int bit = 0; bit < 8; ++bit) {
        const uint64_t ones = __ballot(valid && ((d >> bit) & 1u));
        peers &= ((d >> bit) & 1u) ? ones : ~ones;
      }
      const uint32_t below = (uint32_t)__popcll(peers & lt_mask);
      const uint32_t prior = run[wave][d];
      rank[r] = (prior + below) << 8 | d;
      if (valid && below == 0) run[wave][d] = prior + (uint32_t)__popcll(peers);
      wave_lds_sync();  // this round's counts before the next round's reads
    }
    __syncthreads();  // every wave's digit counts complete
    uint32_t tot = 0, incl = 0;
    if (threadIdx.x < kDigits) {  // digit d = threadIdx.x: each wave's offset within d
      const int d = threadIdx.x;
      for (int w = 0; w < kSortSmallWaves; ++w) {
        const uint32_t c = run[w][d];
        run[w][d] = tot;
        tot += c;
      }
      incl = tot;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
      }
      if (lane == 63) wsum[wave] = incl;
    }
    __syncthreads();
    if (threadIdx.x < kDigits) {
      uint32_t before = 0;
      for (int w = 0; w < wave; ++w) before += wsum[w];
      dstart[threadIdx.x] = before + incl - tot;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {  // rank becomes the sorted position
      const uint32_t d = rank[r] & 0xFFu;
      rank[r] = dstart[d] + run[wave][d] + (rank[r] >> 8);
    }
    // move every element's words and index to its position through LDS, one array at a
    // time, so that the global stores are in order
    uint64_t x[kSortItems] = {};
    uint32_t xi[kSortItems] = {};
    if (has) {
      small_share(in.lo, span0 + lane, x);
      small_share(in.idx, span0 + lane, xi);
    }
#pragma unroll
    for (int r = 0; r < kSortItems; ++r)
      if (span0 + r * 64 + lane < n) xch[rank[r]] = x[r];
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < n; j += kSortSmallThreads) out.lo[j] = xch[j];
    if (kWords == 2) {
      if (has) small_share(in.hi, span0 + lane, x);
      __syncthreads();  // xch read out before it is refilled
#pragma unroll
      for (int r = 0; r < kSortItems; ++r)
        if (span0 + r * 64 + lane < n) xch[rank[r]] = x[r];
      __syncthreads();
      for (uint32_t j = threadIdx.x; j < n; j += kSortSmallThreads) out.hi[j] = xch[j];
    }
    __syncthreads();
    uint32_t* xidx = reinterpret_cast<uint32_t*>(xch);
#pragma unroll
    for (int r = 0; r < kSortItems; ++r)
      if (span0 + r * 64 + lane < n) xidx[rank[r]] = xi[r];
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < n; j += kSortSmallThreads) out.idx[j] = xidx[j];
    __syncthreads();  // this pass's stores visible to the workgroup before the next pass loads
    const SortBuf t = in;
    in = out;
    out = t;
  }
}

// The elements per lane follow the number sorted (1, 4 or 16), so that all sixteen waves
// take part in ranking a few thousand.
template <int kWords>
__global__ __launch_bounds__(kSortSmallThreads) void sort_small_kernel(SortBuf a, SortBuf b, const uint64_t* n_dev,
                                                                       const uint64_t* bits, uint64_t n_max) {
  __shared__ SortSmallLds lds;
  const uint64_t n_all = *n_dev;
  const uint32_t n = (uint32_t)(n_all < n_max ? n_all : n_max);
  if (n == 0) return;
  if (n <= kSortSmallThreads)
    sort_small<kWords, 1>(lds, a, b, n, bits);
  else if (n <= 4 * kSortSmallThreads)
    sort_small<kWords, 4>(lds, a, b, n, bits);
  else
    sort_small<kWords, kSortItems>(lds, a, b, n, bits);
}

// Workspace of a sort of n elements with `words` 64-bit key words: the second key/index
// buffer (b), the digit totals and tickets of the passes, and the chunks' states.
struct SortLayout {
  uint64_t tiles, chunks;
  size_t hi, lo, idx, totals, state, total;
};
constexpr uint64_t kSortTotalWords = 16 * kDigits / 2 + 8;  // u64 words: u32 totals[16][256], u32 tickets[16]

// Elements to allocate in each key/index buffer of a sort of at most n elements (the
// caller's buffer a too): a one-workgroup sort reads whole wave spans.
inline uint64_t sort_capacity(uint64_t n) {
  return n <= kSortSmallMax ? (n + kSortWaveSpan - 1) / kSortWaveSpan * kSortWaveSpan : n;
}

inline SortLayout sort_layout(uint64_t n_max, int words) {
  SortLayout L;
  const uint64_t n = sort_capacity(n_max);
  L.tiles = (n_max + kSortTile - 1) / kSortTile;
  const uint64_t fine = ((n_max < kSortFineMax ? n_max : kSortFineMax) + kSortFineTile - 1) / kSortFineTile;
  const uint64_t mid = ((n_max < kSortMidMax ? n_max : kSortMidMax) + kSortMidTile - 1) / kSortMidTile;
  uint64_t most = fine > L.tiles ? fine : L.tiles;  // (a sort for n_max may sort fewer)
  if (words == 2 && n_max > kSortFineMax && mid > most) most = mid;
  L.chunks = most < kSortChunks ? most : kSortChunks;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off = (off + bytes + 255) & ~(size_t)255;
    return o;
  };
  L.hi = take(words == 2 ? 8 * n : 0);
  L.lo = take(8 * n);
  L.idx = take(4 * n);
  L.totals = off;  // the states follow the totals: one clear
  L.state = off + 8 * kSortTotalWords;
  if (n_max > kSortSmallMax) take(8 * (kSortTotalWords + (size_t)kDigits * L.chunks));
  L.total = off;
  return L;
}

inline SortBuf sort_other(void* ws, uint64_t n_max, int words) {
  const SortLayout L = sort_layout(n_max, words);
  uint8_t* p = static_cast<uint8_t*>(ws);
  return SortBuf{words == 2 ? reinterpret_cast<uint64_t*>(p + L.hi) : nullptr, reinterpret_cast<uint64_t*>(p + L.lo),
                 reinterpret_cast<uint32_t*>(p + L.idx)};
}

// Sorts the first *n_dev (at most n_max, a device count the host does not read) pairs of
// `a` (keys of `words` 64-bit words, 1 or 2; n_max below 2^32) by key, ascending. Each
// of a's arrays holds sort_capacity(n_max) elements.
// `bits` (device u64[4], see pass_trivial) must describe those keys. The result is in `a`
// or in the workspace's buffer (sort_other), as sort_result() tells on the device. Grids
// are sized for n_max, up to kSortMaxGrid workgroups; those past *n_dev do nothing.
constexpr uint64_t kSortMaxGrid = kSortChunks;
template <int kWords>
gleam_status radix_sort_passes(SortBuf a, const uint64_t* n_dev, const uint64_t* bits, uint64_t n_max, void* ws,
                               hipStream_t s) {
  const SortBuf b = sort_other(ws, n_max, kWords);
  if (n_max <= kSortSmallMax) {
    hipLaunchKernelGGL(sort_small_kernel<kWords>, dim3(1), dim3(kSortSmallThreads), 0, s, a, b, n_dev, bits, n_max);
    return launch_status("sort_small_kernel");
  }
  const SortLayout L = sort_layout(n_max, kWords);
  uint8_t* p = static_cast<uint8_t*>(ws);
  uint32_t* totals = reinterpret_cast<uint32_t*>(p + L.totals);
  uint64_t* state = reinterpret_cast<uint64_t*>(p + L.state);
  uint32_t* tickets = totals + 16 * kDigits;
  const uint64_t clear = kSortTotalWords + kDigits * L.chunks;  // the states follow the totals
  const uint64_t clear_grid = (clear + 4 * kSortThreads - 1) / (4 * kSortThreads);
  hipLaunchKernelGGL(sort_clear_kernel, dim3((uint32_t)(clear_grid < kSortMaxGrid ? clear_grid : kSortMaxGrid)),
                     dim3(kSortThreads), 0, s, reinterpret_cast<uint64_t*>(totals), clear);
  gleam_status st = launch_status("sort_clear_kernel");
  if (st != GLEAM_OK) return st;
  const uint32_t hist_grid = (uint32_t)(L.tiles < kSortHistGrid ? L.tiles : kSortHistGrid);
  hipLaunchKernelGGL(sort_hist_kernel<kWords>, dim3(hist_grid), dim3(kSortThreads), 0, s, a, n_dev, bits, totals);
  if ((st = launch_status("sort_hist_kernel")) != GLEAM_OK) return st;
  const uint32_t grid = (uint32_t)L.chunks;
  for (uint32_t q = 0; q < 8u * kWords; ++q) {
    hipLaunchKernelGGL(sort_pass_kernel<kWords>, dim3(grid), dim3(kPassThreads), 0, s, a, b, n_dev, bits, q,
                       totals + q * kDigits, state, tickets + q);
    if ((st = launch_status("sort_pass_kernel")) != GLEAM_OK) return st;
  }
  return GLEAM_OK;
}

inline gleam_status radix_sort_pairs(SortBuf a, const uint64_t* n_dev, const uint64_t* bits, uint64_t n_max,
                                     int words, void* ws, hipStream_t s) {
  if (n_max == 0) return GLEAM_OK;
  return words == 2 ? radix_sort_passes<2>(a, n_dev, bits, n_max, ws, s)
                    : radix_sort_passes<1>(a, n_dev, bits, n_max, ws, s);
}

}  // namespace
}  // namespace gleam
