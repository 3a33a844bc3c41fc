// The data path around the decision (Gleam Sec. 4.1.2): the sender turns each block's
// status into a record, packs the bytes that must travel into one buffer, and the
// receiver rebuilds every payload from the records, that buffer and the bytes it
// already holds.
//
//   gleam_send_plan       one record per block; MISS blocks get 16-byte-aligned offsets
//                         in the packed buffer (an order-preserving scan of lengths)
//   gleam_pack_misses     copy every MISS block's bytes to its offset
//   gleam_restore_blocks  write every block of the destination payloads: MISS from the
//                         packed buffer, HIT_CACHE from the holder's copy, HIT_BATCH from
//                         the packed bytes of the earlier block it repeats
//
// The copies are HBM-bound: one read and one write per byte moved.

#include "gleam_device.h"
#include "gleam_internal.h"
#include "launch_shape.h"

namespace gleam {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
static_assert(kThreads == (int)kCopyThreads, "copy_shape's workgroups");
constexpr int kScanThreads = 1024;
// The plan's tiles: kThreads consecutive blocks times `rounds` (1, 2, 4 or 8), the
// fewest rounds that keep the tiles within kPlanTiles, so that a small batch spreads over
// many CUs and the write pass can sum the tiles before its own by itself: two launches.
// 69,882 blocks of 20,000 payloads: 11 us, against 36 us in three launches with a one-
// workgroup scan over tiles of 2,048 blocks and a thread walking 8 blocks at a time.
constexpr uint64_t kPlanTiles = 2048;
constexpr uint32_t kPlanRounds = (uint32_t)(kTileItems / kThreads);  // at most 8
__device__ __forceinline__ uint64_t round16(uint64_t n) { return (n + 15) & ~15ull; }

__device__ __forceinline__ uint64_t wave_inclusive_scan64(uint64_t x, int lane) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t lo = __shfl_up((uint32_t)x, d, 64);
    const uint32_t hi = __shfl_up((uint32_t)(x >> 32), d, 64);
    if (lane >= d) x += ((uint64_t)hi << 32) | lo;
  }
  return x;
}

// Exclusive scan of one u64 per thread over a workgroup of kWaves waves.
template <int kWaves>
__device__ __forceinline__ uint64_t block_exclusive_scan64(uint64_t x, uint64_t* wave_sums, uint64_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t incl = wave_inclusive_scan64(x, lane);
  if (lane == 63) wave_sums[wave] = incl;
  __syncthreads();
  uint64_t before = 0, sum = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const uint64_t s = wave_sums[w];
    before += w < wave ? s : 0;
    sum += s;
  }
  __syncthreads();
  *total = sum;
  return before + incl - x;
}

struct Geo {
  const uint64_t* seg_len;
  const uint64_t* blk_first;
  uint64_t n_seg;
  uint64_t n_blocks;
  uint64_t block_bytes;
};

// One block of the batch: its payload, and its place in it.
struct Block {
  uint64_t payload, offset, length;
};

// Blocks g_first + lane, one per lane (g_first the same in every lane and below n_blocks):
// the wave finds the first one's payload with 64 pivots a round, then each lane its own
// among the next 64 payload starts. One thread walking 8 blocks from a binary search of
// its own spent about 15 dependent reads (69,882 blocks of 20,000 payloads: 10 us of a
// pass). Every lane must call this; lanes past the batch get length 0.
__device__ __forceinline__ Block wave_block(const Geo& geo, uint64_t g_first, int lane) {
  const uint64_t g = g_first + (uint64_t)lane;
  const uint64_t s0 = wave_find_segment(geo.blk_first, geo.n_seg, g_first, lane);
  const bool valid = g < geo.n_blocks;
  const uint64_t s = lane_segment(geo.blk_first, geo.n_seg, s0, valid ? g : geo.n_blocks - 1, lane);
  const uint64_t start = (valid ? g - geo.blk_first[s] : 0) * geo.block_bytes;
  const uint64_t len_s = geo.seg_len[s];
  return Block{s, start, valid && start < len_s ? min(len_s - start, geo.block_bytes) : 0};
}

__device__ __forceinline__ uint64_t block_sum64(uint64_t x, uint64_t* wave_sums) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) x += shfl_xor64(x, o);
  if ((threadIdx.x & 63) == 0) wave_sums[threadIdx.x >> 6] = x;
  __syncthreads();
  uint64_t sum = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) sum += wave_sums[w];
  __syncthreads();
  return sum;
}

// Per tile: {packed bytes of its MISS blocks, MISS | HIT_CACHE | HIT_BATCH counts in 21
// bits each (a tile has at most 2,048 blocks)}.
__global__ __launch_bounds__(kThreads) void plan_tile_kernel(Geo geo, const uint8_t* status, uint32_t rounds,
                                                             uint64_t* tiles) {
  __shared__ uint64_t sums[kWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint64_t counts = 0, bytes = 0;
  for (uint32_t r = 0; r < rounds; ++r) {
    const uint64_t g0 = ((uint64_t)blockIdx.x * rounds + r) * kThreads + (uint64_t)wave * 64;
    if (g0 >= geo.n_blocks) break;  // uniform over the wave
    const uint64_t g = g0 + (uint64_t)lane;
    const uint8_t st = status[min(g, geo.n_blocks - 1)];
    const Block b = wave_block(geo, g0, lane);
    if (g >= geo.n_blocks) continue;
    if (st == GLEAM_MISS) bytes += round16(b.length);
    counts += 1ull << (st == GLEAM_MISS ? 0 : st == GLEAM_HIT_CACHE ? 21 : 42);
  }
  bytes = block_sum64(bytes, sums);
  counts = block_sum64(counts, sums);
  if (threadIdx.x == 0) {
    tiles[2 * blockIdx.x] = bytes;
    tiles[2 * blockIdx.x + 1] = counts;
  }
}

constexpr uint64_t kCountMask = (1ull << 21) - 1;

// More than kPlanTiles tiles (and the empty batch): one workgroup turns the tiles' bytes
// into their offsets and writes the totals.
__global__ __launch_bounds__(kScanThreads) void plan_scan_kernel(uint64_t* tiles, uint64_t n_tiles, uint64_t* offs,
                                                                 uint64_t* totals) {
  __shared__ uint64_t sums[kScanThreads / 64];
  uint64_t carry = 0, miss = 0, hit = 0, dup = 0;
  for (uint64_t base = 0; base < n_tiles; base += kScanThreads) {
    const uint64_t t = base + threadIdx.x;
    const uint64_t b = t < n_tiles ? tiles[2 * t] : 0;
    const uint64_t c = t < n_tiles ? tiles[2 * t + 1] : 0;
    uint64_t total;
    const uint64_t excl = block_exclusive_scan64<kScanThreads / 64>(b, sums, &total);
    if (t < n_tiles) offs[t] = carry + excl;
    carry += total;
    uint64_t m = c & kCountMask, h = (c >> 21) & kCountMask, d = c >> 42, sum;
    block_exclusive_scan64<kScanThreads / 64>(m, sums, &sum);
    miss += sum;
    block_exclusive_scan64<kScanThreads / 64>(h, sums, &sum);
    hit += sum;
    block_exclusive_scan64<kScanThreads / 64>(d, sums, &sum);
    dup += sum;
  }
  if (threadIdx.x == 0) {
    totals[0] = miss;
    totals[1] = hit;
    totals[2] = dup;
    totals[3] = carry;
  }
}

// The records. A tile's first packed offset comes from `offs`, or (offs null: at most
// kPlanTiles tiles) from summing the bytes of the tiles before it, in which case the last
// tile also writes the totals.
__global__ __launch_bounds__(kThreads) void plan_write_kernel(Geo geo, const uint64_t* digest, const uint8_t* status,
                                                              const uint64_t* ref, uint32_t rounds,
                                                              const uint64_t* tiles, const uint64_t* offs,
                                                              gleam_send_record* rec, uint64_t* totals) {
  __shared__ uint64_t sums[kWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint64_t pos = 0;
  if (offs) {
    pos = offs[blockIdx.x];
  } else {
    const bool last = blockIdx.x + 1 == gridDim.x;
    uint64_t bytes = 0, miss = 0, hit = 0, dup = 0;
    const uint64_t end = last ? (uint64_t)gridDim.x : (uint64_t)blockIdx.x;
    for (uint64_t t = threadIdx.x; t < end; t += kThreads) {
      const uint64_t b = tiles[2 * t];
      if (t < blockIdx.x) bytes += b;
      if (last) {
        const uint64_t c = tiles[2 * t + 1];
        miss += c & kCountMask;
        hit += (c >> 21) & kCountMask;
        dup += c >> 42;
      }
    }
    pos = block_sum64(bytes, sums);
    if (last) {  // uniform over the workgroup
      miss = block_sum64(miss, sums);
      hit = block_sum64(hit, sums);
      dup = block_sum64(dup, sums);
      if (threadIdx.x == 0) {
        totals[0] = miss;
        totals[1] = hit;
        totals[2] = dup;
        totals[3] = pos + tiles[2 * (uint64_t)blockIdx.x];
      }
    }
  }
  for (uint32_t r = 0; r < rounds; ++r) {
    const uint64_t round0 = ((uint64_t)blockIdx.x * rounds + r) * kThreads;
    if (round0 >= geo.n_blocks) break;  // uniform over the workgroup
    const uint64_t g0 = round0 + (uint64_t)wave * 64, g = g0 + (uint64_t)lane;
    const uint64_t at = min(g, geo.n_blocks - 1);
    const uint8_t st = status[at];
    const uint64_t dg = digest[at], rf = ref[at];
    Block b{0, 0, 0};
    if (g0 < geo.n_blocks) b = wave_block(geo, g0, lane);  // uniform over the wave
    const uint64_t mine = g < geo.n_blocks && st == GLEAM_MISS ? round16(b.length) : 0;
    uint64_t total;
    const uint64_t excl = block_exclusive_scan64<kWaves>(mine, sums, &total);
    if (g < geo.n_blocks) {
      gleam_send_record out;
      out.block = g;
      out.payload = b.payload;
      out.offset = b.offset;
      out.ident = st == GLEAM_MISS ? pos + excl : st == GLEAM_HIT_CACHE ? dg : rf;
      out.length = (uint32_t)b.length;
      out.kind = st;
      rec[g] = out;
    }
    pos += total;
  }
}

__device__ __forceinline__ uint64_t uniform64(uint64_t x) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(x >> 32));
  return ((uint64_t)hi << 32) | lo;
}

// Copy len <= kPiece bytes with one wave: 16-byte non-temporal words from either end's
// start at any alignment (gfx950 under HSA runs with unaligned access enabled; each word
// covers 16 bytes of the range, so every byte is touched once and none outside it), then
// the last len mod 16 bytes one by one. The addresses name the global address space (they
// come from integers, from which the compiler would make flat accesses).
typedef u32x4 u32x4_any __attribute__((aligned(1)));
typedef __attribute__((address_space(1))) u32x4_any global_u32x4;
typedef const __attribute__((address_space(1))) u32x4_any const_global_u32x4;
typedef __attribute__((address_space(1))) uint8_t global_u8;
typedef const __attribute__((address_space(1))) uint8_t const_global_u8;
template <uint32_t kPiece>
__device__ __forceinline__ void wave_copy(uint64_t dst, uint64_t src, uint32_t len, int lane) {
  const_global_u32x4* s = (const_global_u32x4*)src + lane;
  global_u32x4* d = (global_u32x4*)dst + lane;
  if (len == kPiece) {
    constexpr int kWords = kPiece / 1024;  // per lane
    u32x4 v[kWords];
#pragma unroll
    for (int j = 0; j < kWords; ++j) v[j] = __builtin_nontemporal_load(s + 64 * j);
#pragma unroll
    for (int j = 0; j < kWords; ++j) __builtin_nontemporal_store(v[j], d + 64 * j);
    return;
  }
  const uint32_t words = len >> 4, tail = (words << 4) + (uint32_t)lane;
  uint8_t byte = 0;
  if (tail < len) byte = ((const_global_u8*)src)[tail];
  for (uint32_t w0 = 0; w0 < words; w0 += 256) {
    u32x4 v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (w0 + lane + 64 * j < words) v[j] = __builtin_nontemporal_load(s + w0 + 64 * j);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (w0 + lane + 64 * j < words) __builtin_nontemporal_store(v[j], d + w0 + 64 * j);
  }
  if (tail < len) ((global_u8*)dst)[tail] = byte;
}

// [at, at + len) lies inside [0, size), without overflow.
__device__ __forceinline__ bool inside(uint64_t at, uint64_t len, uint64_t size) {
  return at <= size && len <= size - at;
}

// The record's block lies inside its payload of the batch.
__device__ __forceinline__ bool block_in_batch(const gleam_send_record& r, const uint64_t* seg_len, uint64_t n_seg) {
  return r.payload < n_seg && inside(r.offset, r.length, seg_len[r.payload]);
}

// Work items: (block, piece of it), 1 << per_log2 pieces per block, one wave each.
// Records whose block is not inside its payload, or whose bytes are not inside the packed
// buffer, are skipped.
template <uint32_t kPiece>
__global__ __launch_bounds__(kThreads) void pack_kernel(const uint64_t* __restrict__ seg_addr,
                                                        const uint64_t* __restrict__ seg_len, uint64_t n_seg,
                                                        const gleam_send_record* __restrict__ rec, uint64_t n,
                                                        uint32_t per_log2, uint8_t* out, uint64_t out_bytes) {
  const int lane = threadIdx.x & 63;
  const uint64_t stride = (uint64_t)gridDim.x * kWaves;
  for (uint64_t item = uniform64((uint64_t)blockIdx.x * kWaves + (threadIdx.x >> 6)); item < n << per_log2;
       item += stride) {
    const uint64_t g = item >> per_log2, c0 = (item - (g << per_log2)) * kPiece;
    const gleam_send_record r = rec[g];
    if (r.kind != GLEAM_MISS || c0 >= r.length || !inside(r.ident, r.length, out_bytes) ||
        !block_in_batch(r, seg_len, n_seg))
      continue;
    wave_copy<kPiece>((uint64_t)out + r.ident + c0, seg_addr[r.payload] + r.offset + c0,
              (uint32_t)min((uint64_t)r.length - c0, (uint64_t)kPiece), lane);
  }
}

template <uint32_t kPiece>
__global__ __launch_bounds__(kThreads) void restore_kernel(const uint64_t* __restrict__ dst_addr,
                                                           const uint64_t* __restrict__ dst_len, uint64_t n_seg,
                                                           const gleam_send_record* __restrict__ rec, uint64_t n,
                                                           uint32_t per_log2, const uint8_t* packed,
                                                           uint64_t packed_bytes, const uint64_t* __restrict__ held) {
  const int lane = threadIdx.x & 63;
  const uint64_t stride = (uint64_t)gridDim.x * kWaves;
  for (uint64_t item = uniform64((uint64_t)blockIdx.x * kWaves + (threadIdx.x >> 6)); item < n << per_log2;
       item += stride) {
    const uint64_t g = item >> per_log2, c0 = (item - (g << per_log2)) * kPiece;
    // the held address does not depend on the record: read both at once, so the range
    // check of the record is the only dependent read before the copy
    const uint64_t held_addr = held ? held[g] : 0;
    const gleam_send_record r = rec[g];
    if (c0 >= r.length || !block_in_batch(r, dst_len, n_seg)) continue;
    uint64_t src = 0;
    if (r.kind == GLEAM_MISS) {
      if (inside(r.ident, r.length, packed_bytes)) src = (uint64_t)packed + r.ident;
    } else if (r.kind == GLEAM_HIT_CACHE) {
      src = held_addr;
    } else if (r.kind == GLEAM_HIT_BATCH && r.ident < n) {
      const gleam_send_record first = rec[r.ident];
      if (first.kind == GLEAM_MISS && first.length == r.length && inside(first.ident, r.length, packed_bytes))
        src = (uint64_t)packed + first.ident;
    }
    if (!src) continue;
    wave_copy<kPiece>(dst_addr[r.payload] + r.offset + c0, src + c0, (uint32_t)min((uint64_t)r.length - c0, (uint64_t)kPiece),
              lane);
  }
}

}  // namespace
// Loads this file's GPU code object on the current device (gleam_preload).
hipError_t preload_transfer() {
  hipFuncAttributes attr;
  return hipFuncGetAttributes(&attr, reinterpret_cast<const void*>(&plan_scan_kernel));
}

}  // namespace gleam

extern "C" gleam_status gleam_send_plan(const gleam_batch* b, const uint64_t* d_digest, const uint8_t* d_status,
                                        const uint64_t* d_ref, gleam_send_record* d_records, uint64_t* d_totals,
                                        void* d_ws, size_t ws_bytes, void* stream) {
  using namespace gleam;
  clear_error();
  gleam_status st = validate_batch(b, "gleam_send_plan");
  if (st != GLEAM_OK) return st;
  if (!d_totals || (b->n_blocks > 0 && (!d_digest || !d_status || !d_ref || !d_records))) {
    set_error("gleam_send_plan: null input or output");
    return GLEAM_E_INVALID;
  }
  const WsLayout L = ws_layout(b->n_blocks);
  st = check_workspace(L, d_ws, ws_bytes, "gleam_send_plan");
  if (st != GLEAM_OK) return st;
  if (L.tiles > max_workgroups(kThreads)) {
    set_error("gleam_send_plan: more tiles than one launch has workgroups (2^24)");
    return GLEAM_E_UNSUPPORTED;
  }
  hipStream_t s = (hipStream_t)stream;
  // the scratch holds at least 4 n_blocks words; the tiles take three words for every
  // kThreads blocks or more
  uint64_t* tiles = reinterpret_cast<uint64_t*>(static_cast<uint8_t*>(d_ws) + L.scratch_off);
  const Geo geo{b->seg_len, b->blk_first, b->n_seg, b->n_blocks, b->block_bytes};
  uint32_t rounds = 1;
  while (rounds < kPlanRounds && b->n_blocks > kPlanTiles * kThreads * rounds) rounds *= 2;
  const uint64_t n_tiles = (b->n_blocks + (uint64_t)kThreads * rounds - 1) / ((uint64_t)kThreads * rounds);
  uint64_t* offs = nullptr;
  if (b->n_blocks > 0) {
    hipLaunchKernelGGL(plan_tile_kernel, dim3((uint32_t)n_tiles), dim3(kThreads), 0, s, geo, d_status, rounds, tiles);
    if ((st = launch_status("plan_tile_kernel")) != GLEAM_OK) return st;
  }
  if (n_tiles == 0 || n_tiles > kPlanTiles) {
    offs = tiles + 2 * n_tiles;
    hipLaunchKernelGGL(plan_scan_kernel, dim3(1), dim3(kScanThreads), 0, s, tiles, n_tiles, offs, d_totals);
    if ((st = launch_status("plan_scan_kernel")) != GLEAM_OK) return st;
  }
  if (b->n_blocks == 0) return GLEAM_OK;
  hipLaunchKernelGGL(plan_write_kernel, dim3((uint32_t)n_tiles), dim3(kThreads), 0, s, geo, d_digest, d_status, d_ref,
                     rounds, tiles, offs, d_records, d_totals);
  return launch_status("plan_write_kernel");
}

extern "C" gleam_status gleam_pack_misses(const gleam_batch* b, const gleam_send_record* d_records, uint8_t* d_out,
                                          uint64_t out_bytes, void* stream) {
  using namespace gleam;
  clear_error();
  gleam_status st = validate_batch(b, "gleam_pack_misses");
  if (st != GLEAM_OK) return st;
  if (b->n_blocks == 0) return GLEAM_OK;
  if (!d_records || (!d_out && out_bytes > 0)) {
    set_error("gleam_pack_misses: null records or output");
    return GLEAM_E_INVALID;
  }
  const CopyShape c = copy_shape(b->n_blocks, b->block_bytes, true);
  hipLaunchKernelGGL(c.large ? pack_kernel<kLargePiece> : pack_kernel<kSmallPiece>, dim3(c.groups), dim3(kThreads), 0,
                     (hipStream_t)stream, b->seg_addr, b->seg_len, b->n_seg, d_records, b->n_blocks, c.per_log2, d_out,
                     out_bytes);
  return launch_status("pack_kernel");
}

extern "C" gleam_status gleam_restore_blocks(const gleam_batch* dst, const gleam_send_record* d_records,
                                             const uint8_t* d_packed, uint64_t packed_bytes, const uint64_t* d_held,
                                             void* stream) {
  using namespace gleam;
  clear_error();
  gleam_status st = validate_batch(dst, "gleam_restore_blocks");
  if (st != GLEAM_OK) return st;
  if (dst->n_blocks == 0) return GLEAM_OK;
  if (!d_records || (!d_packed && packed_bytes > 0)) {
    set_error("gleam_restore_blocks: null records or packed buffer");
    return GLEAM_E_INVALID;
  }
  // at most one block of each payload is short: with four blocks per payload or more, at
  // least three in four are full
  const CopyShape c = copy_shape(dst->n_blocks, dst->block_bytes, dst->n_blocks / 4 < dst->n_seg);
  hipLaunchKernelGGL(c.large ? restore_kernel<kLargePiece> : restore_kernel<kSmallPiece>, dim3(c.groups),
                     dim3(kThreads), 0, (hipStream_t)stream, dst->seg_addr, dst->seg_len, dst->n_seg, d_records,
                     dst->n_blocks, c.per_log2, d_packed, packed_bytes, d_held);
  return launch_status("restore_kernel");
}
