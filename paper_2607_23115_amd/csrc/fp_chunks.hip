// gleam_fp_chunks: block digests of a batch of payloads on gfx950.
//
// Identifier of a block (Gleam Sec. 4.1.2, hash of the source bytes): XXH64 with
// seed 0 of each 4 KiB leaf over its actual bytes, folded by a bottom-up pairwise
// tree (node = XXH64 of LE64(left) || LE64(right); an odd last element moves up).
//
// Work decomposition. Leaf slot = g * LPB + k (block g, leaf k, LPB = leaves per
// block). Two lanes own one slot: the even lane keeps XXH64 accumulators 1 and 2, the
// odd lane 3 and 4, so each lane runs two independent chains of 128 rounds and a
// wave covers 32 leaves. A workgroup of 4 waves owns GROUP = 128 consecutive slots
// (LPB <= GROUP), or one whole block walked GROUP slots at a time (LPB > GROUP). In a
// large batch of blocks of up to 64 KiB, the last kQuadTailSlots slots go to workgroups
// of four lanes per leaf (64 slots each, half the stages): the batch's last round of
// workgroups, during which part of the GPU already idles, then ends sooner.
//
// Occupancy. HBM read rate on MI355X rises as fewer waves stream at once: one 4-wave
// workgroup per CU reads faster than two or more (measured with plain read kernels and
// with this one). For blocks of 1 MiB and up the workgroup's LDS is padded past half
// of the CU's 160 KiB, so each CU holds exactly one, and a grid of 4 per CU walks the
// blocks. Smaller blocks keep one workgroup per item at normal occupancy: their
// gathered waves need the extra waves to hide latency.
//
// Memory path (the kernel is HBM-bound; XXH64 itself runs far above HBM rate).
// A wave whose 32 leaves are full and contiguous streams them with non-temporal
// 16-byte loads in which 32 consecutive lanes read one 512-byte run of one leaf (2
// leaves per load instruction, 16 loads = 32 leaves x 512 B per stage). Each stage goes
// through a per-wave LDS tile, 512 B per leaf, whose 32-byte stripes are XOR-swizzled by
// the leaf index, so both the stores and each lane's 16-byte reads of its own
// half-stripes are free of bank conflicts; the next stage's loads are in flight while
// the current one is hashed. Waves that are not one contiguous full run (payload ends,
// small payloads) use the same tile with per-instruction leaf addresses read from the
// registers of the lanes that hash each leaf. Every load covers 16 bytes of its own leaf
// from the leaf's start, at any
// alignment (see load_stream16_any), so a leaf's bytes reach the tile in order and no
// path shifts them.
//
// Tree: levels inside a wave's 32 leaves use cross-lane shuffles; the roots of
// 32-leaf groups meet in LDS. Pairing by aligned position level by level is the same
// computation as the plain bottom-up definition.

#include "fp_core.h"
#include "launch_shape.h"

namespace gleam {
namespace {

constexpr int kThreads = 256;
constexpr int kSoloPad = 24 << 10;  // takes the workgroup's LDS past 80 KiB: one per CU
constexpr uint64_t kQuadTailSlots = 16384;
constexpr uint64_t kSparseUnits = 2048;

template <bool kSolo, typename Out>
__global__ __launch_bounds__(kThreads) void fp_kernel(FpArgs a, Out out) {
  constexpr int W = kThreads / 64;
  constexpr uint32_t GROUP = W * kLeavesPerWave;
  __shared__ __attribute__((aligned(16))) uint8_t lds[W * kWaveLds + (kSolo ? kSoloPad : 0)];
  __shared__ uint64_t roots[2][kMaxRoots];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  uint8_t* tile = lds + wave * kWaveLds;
  const uint32_t L2 = a.lpb_log2;
  const uint32_t lpb = 1u << L2;
  const bool even = (lane & 1) == 0;

  // The last slots of a batch of small blocks, past a.items groups: four lanes per leaf,
  // W * kQuadLeaves slots per workgroup (see launch_fp).
  if (!kSolo && blockIdx.x >= a.items) {
    constexpr uint64_t kPerGroup = GROUP / (W * kQuadLeaves);
    quad_pass<W, false>(a, a.items * kPerGroup + (blockIdx.x - a.items), lds, nullptr, out);
    return;
  }

  // Persistent workgroups: a grid of a few workgroups per CU walks the work items.
  for (uint64_t item = blockIdx.x; item < a.items; item += gridDim.x) {
    __syncthreads();  // the previous item's roots have been consumed
    if (lpb <= GROUP) {
      // GROUP consecutive slots: GROUP / LPB whole blocks.
      const uint64_t wave_slot0 = uniform64(item * GROUP + (uint64_t)wave * kLeavesPerWave);
      const uint64_t slot = wave_slot0 + (lane >> 1);
      const uint64_t g = slot >> L2;
      const uint32_t k = (uint32_t)(slot & (lpb - 1));
      const Leaf lf = locate_wave(a, wave_slot0 >> L2, g, k, lane);
      typename Out::Before before_hash{};
      if constexpr (Out::kReadsBefore)
        before_hash = out.before(lpb <= kLeavesPerWave && even && k == 0 && g < a.n_blocks, g);
      const uint64_t d = hash_slot(lf, tile, lane);
      if (a.leaf_out && even && g < a.n_blocks) a.leaf_out[slot] = lf.len ? d : 0;
      const uint32_t G = lpb <= kLeavesPerWave ? lpb : (uint32_t)kLeavesPerWave;
      const uint32_t p = k & (G - 1);
      uint32_t n = lf.blk_leaves;
      if (lpb > kLeavesPerWave) {
        const uint32_t before = k & ~(uint32_t)(kLeavesPerWave - 1);
        n = n > before ? min(n - before, (uint32_t)kLeavesPerWave) : 0u;
      }
      const uint64_t v = tree_reduce_lanes(d, p, n, G, 2);
      if (lpb <= kLeavesPerWave) {
        out(a, even && p == 0 && g < a.n_blocks, g, v, lf.seg, before_hash);
      } else {
        if (lane == 0) roots[0][wave] = v;
        __syncthreads();
        if (wave == 0) {
          // W wave roots = GROUP / LPB blocks of G2 = LPB / 32 roots each
          const uint32_t G2 = lpb / kLeavesPerWave;
          const uint64_t g2 = ((item * GROUP) >> L2) + (uint64_t)(lane / G2);
          uint32_t n2 = 0;
          uint64_t v2 = 0;
          const Leaf head = locate_wave(a, (item * GROUP) >> L2, g2, 0, lane);
          typename Out::Before before2{};
          if constexpr (Out::kReadsBefore)
            before2 = out.before(lane < W && (lane & (G2 - 1)) == 0 && g2 < a.n_blocks, g2);
          if (lane < W && g2 < a.n_blocks) {
            n2 = (head.blk_leaves + kLeavesPerWave - 1) / kLeavesPerWave;
            v2 = roots[0][lane];
          }
          v2 = tree_reduce_lanes(v2, lane & (G2 - 1), n2, G2);
          out(a, lane < W && (lane & (G2 - 1)) == 0 && g2 < a.n_blocks, g2, v2, head.seg, before2);
        }
      }
    } else {
      // One block of LPB > GROUP leaves, GROUP slots at a time.
      const uint64_t g = item;
      const uint64_t s0 = uniform64(find_segment(a.blk_first, a.n_seg, g));
      const Leaf head = locate(a, g, 0, s0);
      const uint32_t nleaf = head.blk_leaves;
      typename Out::Before before_hash{};
      if constexpr (Out::kReadsBefore) before_hash = out.before(threadIdx.x == 0, g);
      const uint32_t groups = a.leaf_out ? lpb / GROUP : (nleaf + GROUP - 1) / GROUP;
      for (uint32_t grp = 0; grp < groups; ++grp) {
        const uint32_t k = grp * GROUP + (uint32_t)wave * kLeavesPerWave + (lane >> 1);
        const Leaf lf = locate(a, g, k, s0);
        const uint64_t d = hash_slot(lf, tile, lane);
        if (a.leaf_out && even) a.leaf_out[((uint64_t)g << L2) + k] = lf.len ? d : 0;
        const uint32_t before = k & ~(uint32_t)(kLeavesPerWave - 1);
        const uint32_t n = nleaf > before ? min(nleaf - before, (uint32_t)kLeavesPerWave) : 0u;
        const uint64_t v = tree_reduce_lanes(d, (uint32_t)(lane >> 1), n, kLeavesPerWave, 2);
        if (lane == 0) roots[0][grp * W + wave] = v;
      }
      __syncthreads();
      if (wave == 0) {
        const uint32_t n2 = (nleaf + kLeavesPerWave - 1) / kLeavesPerWave;  // <= kMaxRoots
        const uint64_t r = tree_reduce_lds(roots[0], roots[1], n2, lane);
        out(a, lane == 0, g, r, head.seg, before_hash, true);
      }
    }
  }
}


// One workgroup of W waves per W * kQuadLeaves slots; LPB <= kQuadLeaves, so every wave
// holds whole blocks. W = 1 for the smallest batches (more CUs then share the loads; each
// wave loads all its stages into LDS at once), 4 otherwise.
template <int W, typename Out>
__global__ __launch_bounds__(64 * W) void fp_quad_kernel(FpArgs a, Out out) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[W == 1 ? kQuadDirectLds : W * kQuadWaveLds];
  quad_pass<W, false, W == 1>(a, blockIdx.x, lds, nullptr, out);
}

// ---- Comparison with recorded digests -------------------------------------------------
// The kernels above with the comparison in the place of the store: the digests never reach
// memory, and no second pass reads them (30,000 small copies: 80.6 to 76.4 us a call; 2.9 GB
// of a decoder in 1 MiB blocks, located to the leaf: 474 to 428 us, most of it from
// leaf_pass). A lane keeps the payload it found when it located its leaf: searching for it
// again where digests differ cost the small copies 6 us. The recorded digest is read before
// the leaves are hashed: a wave that reads it at its end keeps its LDS, and with it the next
// workgroup, waiting for a round trip of memory.
struct FirstDiff {
  uint64_t s, at;
};

// first_diff[s] = min(first_diff[s], x) for the lanes with `differs`. When every such lane of
// the wave lies in one payload (all but the waves at payload boundaries), the wave takes the
// minimum itself and one lane issues the atomic, unless the word is already as low: a payload
// whose blocks all changed (a layer updated in place) would otherwise queue one atomic per
// block on its word (262,144 leaves of one payload: 3.2 ms). That word is read at the end
// (read before hashing, the waves that start together all find it high and queue: 425 us for
// 1 GB changed throughout in 4 KiB blocks), and those reads queue too: 203 us with one for
// each wave, 175 where the four waves of a workgroup leave their differences in `late` for one
// (Compare::finish), 182 with the comparison in a pass of its own. Where the calls are `rare`,
// one for a whole block of 1 MiB or more, the word is not read. Every lane of the wave calls it.
__device__ __forceinline__ void lower_first_diff(uint64_t* first_diff, uint64_t s, bool differs, uint64_t x,
                                                 bool rare, FirstDiff* late) {
  const int lane = threadIdx.x & 63;
  const uint64_t active = __ballot(differs);
  if (late && lane == 0) late->at = ~0ull;
  if (active == 0) return;  // the wave
  const int leader = __ffsll((unsigned long long)active) - 1;
  const uint64_t s0 = shfl64(s, leader);
  bool issue = differs;
  uint64_t m = differs ? x : ~0ull;
  if (__ballot(differs && s != s0) == 0) {  // one payload for every differing lane
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      const uint64_t y = shfl_xor64(m, o);
      m = y < m ? y : m;
    }
    issue = lane == leader;
    if (late) {
      if (issue) *late = FirstDiff{s, m};
      return;
    }
  } else {
    rare = true;
  }
  if (issue && (rare || m < __hip_atomic_load(&first_diff[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)))
    atomicMin(reinterpret_cast<unsigned long long*>(&first_diff[s]), (unsigned long long)m);
}

struct Compare {
  const uint64_t* recorded;
  uint8_t* match;  // nullable
  uint64_t* first_diff;
  typedef uint64_t Before;  // the recorded digest
  // The waves' differences, for one read of the payload's word instead of one per wave.
  static constexpr bool kReadsBefore = true, kFinishes = true;
  template <int W>
  struct Late {
    FirstDiff wave[W];
  };
  // Every thread of the workgroup calls it. Later waves hold later slots.
  template <int W>
  __device__ __forceinline__ void finish(const Late<W>& late) const {
    __syncthreads();
    if (threadIdx.x >= W) return;
    const FirstDiff mine = late.wave[threadIdx.x];
    bool issue = mine.at != ~0ull;
    for (uint32_t w = 0; w < threadIdx.x; ++w) issue = issue && !(late.wave[w].s == mine.s && late.wave[w].at != ~0ull);
    if (issue && mine.at < __hip_atomic_load(&first_diff[mine.s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      atomicMin(reinterpret_cast<unsigned long long*>(&first_diff[mine.s]), (unsigned long long)mine.at);
  }
  __device__ __forceinline__ uint64_t before(bool valid, uint64_t at) const { return valid ? recorded[at] : 0; }
};

// Block g: equal digests? The first differing block of each payload.
struct CompareBlocks : Compare {
  __device__ __forceinline__ void operator()(const FpArgs& a, bool valid, uint64_t g, uint64_t v, uint64_t s,
                                             uint64_t was, bool rare = false, FirstDiff* late = nullptr) const {
    const bool same = !valid || was == v;
    if (valid && match) match[g] = same ? 1 : 0;
    lower_first_diff(first_diff, s, !same, same ? 0 : g - a.blk_first[s], rare, late);
  }
};

// Leaf slot (slot = g * LPB + k): equal digests? Slots past a short block's last leaf hold 0
// on both sides, so they always agree. The first differing leaf of each payload by its index
// within the payload, (g - blk_first[s]) * LPB + k.
struct CompareLeaves : Compare {
  __device__ __forceinline__ void operator()(const FpArgs& a, bool valid, uint64_t slot, uint64_t v, uint64_t s,
                                             uint64_t was, bool rare = false, FirstDiff* late = nullptr) const {
    const bool same = !valid || was == v;
    if (valid && match) match[slot] = same ? 1 : 0;
    lower_first_diff(first_diff, s, !same, same ? 0 : slot - (a.blk_first[s] << a.lpb_log2), rare, late);
  }
  // Slots [slot0, end) of payload s, which hold no leaf: 0 on this side. Every thread of the
  // workgroup calls it; end - slot0 is a multiple of 128.
  __device__ __forceinline__ void absent(const FpArgs& a, uint64_t slot0, uint64_t end, uint64_t s) const {
    constexpr int kEach = 4;
    for (uint64_t at = slot0; at < end; at += kEach * kThreads) {
      uint64_t r[kEach], any = 0;
#pragma unroll
      for (int j = 0; j < kEach; ++j) {  // unconditional (clamped) loads, issued together
        const uint64_t slot = at + (uint64_t)j * kThreads + threadIdx.x;
        r[j] = recorded[slot < end ? slot : end - 1];
      }
#pragma unroll
      for (int j = 0; j < kEach; ++j) {
        const uint64_t slot = at + (uint64_t)j * kThreads + threadIdx.x;
        if (slot >= end) r[j] = 0;
        else if (match) match[slot] = r[j] == 0 ? 1 : 0;
        any |= r[j];
      }
      if (!__any(any != 0)) continue;  // as it is unless the recorded digests are of other payloads
#pragma unroll
      for (int j = 0; j < kEach; ++j) {
        const uint64_t slot = at + (uint64_t)j * kThreads + threadIdx.x;
        lower_first_diff(first_diff, s, r[j] != 0, slot - (a.blk_first[s] << a.lpb_log2), false, nullptr);
      }
    }
  }
};

// The leaf digests of one wave's consecutive slots alone: no tree, so a workgroup takes the
// same few slots in blocks of any size (1 MiB blocks by whole blocks end unevenly: 2,829 of
// them are 11.05 rounds of the 256 CUs). `slot0` in slots.
template <typename Out>
__device__ __forceinline__ void leaf_pass(const FpArgs& a, uint64_t slot0, uint8_t* tile, int lane, const Out& out,
                                          FirstDiff* late) {
  const uint64_t slot = slot0 + (lane >> 1), g = slot >> a.lpb_log2;
  const uint32_t k = (uint32_t)(slot & ((1u << a.lpb_log2) - 1));
  const Leaf lf = locate_wave(a, slot0 >> a.lpb_log2, g, k, lane);
  const bool valid = (lane & 1) == 0 && g < a.n_blocks;
  const typename Out::Before before = out.before(valid, slot);
  const uint64_t d = hash_slot(lf, tile, lane);
  out(a, valid, slot, lf.len ? d : 0, lf.seg, before, false, late);
}

template <bool kDirect, typename Out>
__device__ __forceinline__ void leaf_pass_quad(const FpArgs& a, uint64_t slot0, uint8_t* tile, int lane,
                                               const Out& out, FirstDiff* late = nullptr) {
  const uint64_t slot = slot0 + (lane >> 2), g = slot >> a.lpb_log2;
  const uint32_t k = (uint32_t)(slot & ((1u << a.lpb_log2) - 1));
  const Leaf lf = locate_wave(a, slot0 >> a.lpb_log2, g, k, lane);
  const bool valid = (lane & 3) == 0 && g < a.n_blocks;
  const typename Out::Before before = out.before(valid, slot);
  const uint64_t d = kDirect ? hash_slot_quad_direct(lf, tile, lane) : hash_slot_quad(lf, tile, lane);
  out(a, valid, slot, lf.len ? d : 0, lf.seg, before, false, late);
}

// Two lanes per leaf in the first a.items workgroups, four in those after them (as fp_kernel).
// `first`: the workgroups launched before these.
template <typename Out>
__global__ __launch_bounds__(kThreads) void fp_leaf_kernel(FpArgs a, uint64_t first, Out out) {
  constexpr int W = kThreads / 64;
  __shared__ __attribute__((aligned(16))) uint8_t lds[W * kWaveLds];
  static_assert(kQuadWaveLds <= kWaveLds, "one tile per wave");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint8_t* tile = lds + wave * kWaveLds;
  __shared__ typename Out::template Late<W> late;
  const uint64_t group = first + blockIdx.x;
  if (group < a.items) {
    leaf_pass(a, uniform64((group * W + wave) * kLeavesPerWave), tile, lane, out, &late.wave[wave]);
  } else {
    const uint64_t slot0 = a.items * W * kLeavesPerWave + ((group - a.items) * W + wave) * kQuadLeaves;
    leaf_pass_quad<false>(a, uniform64(slot0), tile, lane, out, &late.wave[wave]);
  }
  out.finish(late);
}

// Blocks of which most are short: a workgroup takes 1 << unit_log2 consecutive slots of one
// block (128 to lpb), finds the block's payload once, hashes its leaves 128 slots at a time and
// reads past the slots that hold none. The blocks' first units come first, then their second
// ones: those with leaves are then spread over the XCDs, to which workgroups go in turn (of
// four units a block, the first with all its leaves, they would go to two of the eight).
// 20,000 payloads of 12 KB in 1 MiB blocks 0.86 ms, in 16 MiB blocks 1.17 (with a workgroup, and
// a search for the payload in each of its waves, for every 64 slots 2.3 and 21; with the slots
// written by the fingerprint kernel and compared in a pass of their own 1.75 and 4.2).
template <typename Out>
__global__ __launch_bounds__(kThreads) void fp_leaf_sparse_kernel(FpArgs a, uint64_t first, uint32_t unit_log2,
                                                                  Out out) {
  constexpr int W = kThreads / 64;
  constexpr uint32_t GROUP = W * kLeavesPerWave;
  __shared__ __attribute__((aligned(16))) uint8_t lds[W * kWaveLds];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint8_t* tile = lds + wave * kWaveLds;
  const uint64_t unit = first + blockIdx.x, part = unit / a.n_blocks, g = unit - part * a.n_blocks;
  const uint64_t base = g << a.lpb_log2;
  const uint64_t s = uniform64(wave_find_segment(a.blk_first, a.n_seg, g, lane));
  const uint32_t leaves = locate_at(a, g, 0, s).blk_leaves;
  uint32_t k = (uint32_t)part << unit_log2;
  const uint32_t end = k + (1u << unit_log2);
  for (; k < end && k < leaves; k += GROUP) {
    const uint32_t mine = k + (uint32_t)wave * kLeavesPerWave + (lane >> 1);
    const Leaf lf = locate_at(a, g, mine, s);
    const bool valid = (lane & 1) == 0;
    const typename Out::Before before = out.before(valid, base + mine);
    const uint64_t d = hash_slot(lf, tile, lane);
    out(a, valid, base + mine, lf.len ? d : 0, s, before);
  }
  out.absent(a, base + k, base + end, s);
}

// One-wave workgroups, every stage at once into LDS.
template <typename Out>
__global__ __launch_bounds__(64) void fp_leaf_small_kernel(FpArgs a, Out out) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[kQuadDirectLds];
  leaf_pass_quad<true>(a, (uint64_t)blockIdx.x * kQuadLeaves, lds, threadIdx.x, out);
}

}  // namespace

gleam_status validate_batch(const gleam_batch* b, const char* who) {
  if (!b) {
    set_error("%s: null batch", who);
    return GLEAM_E_INVALID;
  }
  if (b->leaf_bytes != GLEAM_LEAF_BYTES || !valid_block_bytes(b->block_bytes)) {
    set_error("%s: leaf_bytes must be 4096 and block_bytes 4096 << k (k <= 12)", who);
    return GLEAM_E_INVALID;
  }
  if (b->n_blocks > 0 && (b->n_seg == 0 || !b->seg_addr || !b->seg_len || !b->blk_first)) {
    set_error("%s: null descriptor for a non-empty batch", who);
    return GLEAM_E_INVALID;
  }
  if (b->n_blocks > (UINT64_MAX >> 13)) {
    set_error("%s: batch too large", who);
    return GLEAM_E_UNSUPPORTED;
  }
  return GLEAM_OK;
}

namespace {

template <typename Out>
gleam_status launch_fp_out(const gleam_batch* b, uint64_t* d_block_digest, uint64_t* d_leaf_digest, const Out& out,
                           hipStream_t stream) {
  if (b->n_blocks == 0) return GLEAM_OK;
  const int lpb_log2 = log2_exact(b->block_bytes) - 12;
  const uint64_t lpb = 1ull << lpb_log2;
  const uint64_t slots = b->n_blocks * lpb;  // n_blocks < 2^51: no overflow
  // (a large batch takes the four-lanes kernel only while one launch holds its grid of one
  // 4-wave workgroup per 64 slots)
  if (lpb <= (uint64_t)kQuadLeaves &&
      (slots <= kQuadMaxSlots ||
       (slots / kQuadLargePayloadSlots >= b->n_seg && slots / (4 * kQuadLeaves) < max_workgroups(kThreads)))) {
    int cus = 0;
    gleam_status st = device_cu_count(&cus);
    if (st != GLEAM_OK) return st;
    const uint64_t waves = (b->n_blocks * lpb + kQuadLeaves - 1) / kQuadLeaves;
    FpArgs a{b->seg_addr, b->seg_len, b->blk_first, b->n_seg, b->n_blocks, d_block_digest, d_leaf_digest,
             (uint32_t)lpb_log2, waves};
    // one-wave workgroups while they spread the batch over more CUs (16 MiB, 256 waves:
    // 10.1 vs 11.2 us), 4-wave ones above two waves per CU (ResNet-50, 895 waves: 16.6 vs
    // 17.9 us with one-wave workgroups)
    if (waves <= 2ull * (uint64_t)cus) {
      hipLaunchKernelGGL((fp_quad_kernel<1, Out>), dim3((uint32_t)waves), dim3(64), 0, stream, a, out);
    } else {
      hipLaunchKernelGGL((fp_quad_kernel<4, Out>), dim3((uint32_t)((waves + 3) / 4)), dim3(256), 0, stream, a, out);
    }
    return launch_status("fp_quad_kernel");
  }
  constexpr uint64_t group = (kThreads / 64) * kLeavesPerWave;
  uint64_t items = lpb <= group ? (b->n_blocks * lpb + group - 1) / group : b->n_blocks;
  // 1 MiB blocks and up: one workgroup resident per CU, a grid of 4 per CU walking the
  // blocks. Smaller blocks: one workgroup per item (both measured best on MI355X).
  const bool solo = lpb >= 256;
  uint64_t grid = items;
  // Blocks of up to 64 KiB in a batch of several rounds of workgroups: the last
  // kQuadTailSlots slots (rounded to whole groups) run as workgroups of four lanes per
  // leaf, which finish in half the time, so the GPU drains faster at the end.
  if (lpb <= (uint64_t)kQuadLeaves && slots > 4 * kQuadTailSlots) {
    items = (slots - kQuadTailSlots) / group;
    const uint64_t quad_group = (kThreads / 64) * kQuadLeaves;
    grid = items + (slots - items * group + quad_group - 1) / quad_group;
  }
  if (solo) {
    int cus = 0;
    gleam_status st = device_cu_count(&cus);
    if (st != GLEAM_OK) return st;
    grid = items < 4ull * (uint64_t)cus ? items : 4ull * (uint64_t)cus;
  }
  if (grid > max_workgroups(kThreads)) {
    set_error("fingerprint: batch needs more workgroups than one launch has (2^24)");
    return GLEAM_E_UNSUPPORTED;
  }
  FpArgs a{b->seg_addr, b->seg_len, b->blk_first, b->n_seg, b->n_blocks, d_block_digest, d_leaf_digest,
           (uint32_t)lpb_log2, items};
  if (solo)
    hipLaunchKernelGGL((fp_kernel<true, Out>), dim3((uint32_t)grid), dim3(kThreads), 0, stream, a, out);
  else
    hipLaunchKernelGGL((fp_kernel<false, Out>), dim3((uint32_t)grid), dim3(kThreads), 0, stream, a, out);
  return launch_status("fp_kernel");
}

}  // namespace

gleam_status launch_fp(const gleam_batch* b, uint64_t* d_block_digest, uint64_t* d_leaf_digest, hipStream_t stream) {
  return launch_fp_out(b, d_block_digest, d_leaf_digest, StoreBlocks{}, stream);
}

gleam_status launch_fp_compare(const gleam_batch* b, const uint64_t* recorded, uint8_t* match, uint64_t* first_diff,
                               hipStream_t stream) {
  return launch_fp_out(b, nullptr, nullptr, CompareBlocks{{recorded, match, first_diff}}, stream);
}

// The launch rules of launch_fp for blocks of up to 64 KiB, here for blocks of any size.
gleam_status launch_leaf_compare(const gleam_batch* b, const uint64_t* recorded, uint8_t* match, uint64_t* first_diff,
                                 hipStream_t stream) {
  if (b->n_blocks == 0) return GLEAM_OK;
  const int lpb_log2 = log2_exact(b->block_bytes) - 12;
  const uint64_t slots = b->n_blocks << lpb_log2;
  const CompareLeaves out{{recorded, match, first_diff}};
  FpArgs a{b->seg_addr, b->seg_len, b->blk_first, b->n_seg, b->n_blocks, nullptr, nullptr, (uint32_t)lpb_log2, 0};
  if (slots <= kQuadMaxSlots) {
    int cus = 0;
    gleam_status st = device_cu_count(&cus);
    if (st != GLEAM_OK) return st;
    const uint64_t waves = (slots + kQuadLeaves - 1) / kQuadLeaves;
    if (waves <= 2ull * (uint64_t)cus) {
      hipLaunchKernelGGL(fp_leaf_small_kernel<CompareLeaves>, dim3((uint32_t)waves), dim3(64), 0, stream, a, out);
      return launch_status("fp_leaf_small_kernel");
    }
  }
  constexpr uint64_t group = (kThreads / 64) * kLeavesPerWave, quad_group = (kThreads / 64) * kQuadLeaves;
  // Fewer than four blocks per payload: a quarter of the blocks or more may be short. The units
  // are 128 to 1,024 slots, as large as leaves kSparseUnits of them, four for every workgroup
  // that the GPU holds (2,000 payloads of 300 KB in 4 MiB blocks: 117 us, 850 with 64 slots);
  // smaller batches have idle CUs to spare.
  if (slots > kQuadMaxSlots && b->n_blocks / 4 < b->n_seg && slots / group >= kSparseUnits && lpb_log2 >= 7) {
    uint32_t unit_log2 = 7;
    while (unit_log2 < 10 && unit_log2 < (uint32_t)lpb_log2 && slots >> (unit_log2 + 1) >= kSparseUnits) ++unit_log2;
    return launch_in_parts(slots >> unit_log2, max_workgroups(kThreads), [&](uint64_t first, uint32_t groups) {
      hipLaunchKernelGGL(fp_leaf_sparse_kernel<CompareLeaves>, dim3(groups), dim3(kThreads), 0, stream, a, first,
                         unit_log2, out);
      return launch_status("fp_leaf_sparse_kernel");
    });
  }
  // Two lanes per leaf where payloads average fewer than kQuadLargePayloadSlots slots, or 1.5
  // blocks, which may be nearly empty (100,000 payloads of 300 bytes in 256 KiB blocks: 537 us,
  // 1,111 with four lanes).
  if (slots > kQuadMaxSlots && (slots / kQuadLargePayloadSlots < b->n_seg ||
                                b->n_blocks - b->n_blocks / 3 < b->n_seg || slots / quad_group >= 0x7fffffffull))
    a.items = (slots - kQuadTailSlots) / group;
  const uint64_t grid = a.items + (slots - a.items * group + quad_group - 1) / quad_group;
  if (grid > 0x7fffffffull) {
    set_error("fingerprint: batch needs more than 2^31 workgroups");
    return GLEAM_E_UNSUPPORTED;
  }
  return launch_in_parts(grid, max_workgroups(kThreads), [&](uint64_t first, uint32_t groups) {
    hipLaunchKernelGGL(fp_leaf_kernel<CompareLeaves>, dim3(groups), dim3(kThreads), 0, stream, a, first, out);
    return launch_status("fp_leaf_kernel");
  });
}

// Loads this file's GPU code object on the current device (gleam_preload).
hipError_t preload_fp_chunks() {
  hipFuncAttributes attr;
  return hipFuncGetAttributes(&attr, reinterpret_cast<const void*>(&fp_kernel<true, StoreBlocks>));
}

}  // namespace gleam

extern "C" gleam_status gleam_fp_chunks(const gleam_batch* b, uint64_t* d_block_digest, uint64_t* d_leaf_digest,
                                        void* stream) {
  using namespace gleam;
  clear_error();
  gleam_status st = validate_batch(b, "gleam_fp_chunks");
  if (st != GLEAM_OK) return st;
  if (b->n_blocks == 0) return GLEAM_OK;
  if (!d_block_digest) {
    set_error("gleam_fp_chunks: null output for a non-empty batch");
    return GLEAM_E_INVALID;
  }
  return launch_fp(b, d_block_digest, d_leaf_digest, (hipStream_t)stream);
}
