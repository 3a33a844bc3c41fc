// How launches of many workgroups are cut, as plain arithmetic (a CPU test compiles this
// file by itself).
#pragma once

#include <stdint.h>

namespace gleam {

// One launch has fewer than 2^32 threads: 2^24 - 1 workgroups of 256. HIP starts a larger one
// with its count of threads modulo 2^32, so workgroups are missing, and reports an error only
// where nothing is left of it.
constexpr uint64_t max_workgroups(uint32_t threads) { return UINT32_MAX / threads; }

// Calls launch(first, count) for workgroups [first, first + count) of `groups`, at most `most`
// at once, in order; stops at the first status that is not 0 and returns it.
template <class Launch>
int32_t launch_in_parts(uint64_t groups, uint64_t most, const Launch& launch) {
  for (uint64_t first = 0; first < groups; first += most) {
    const uint64_t left = groups - first;
    const int32_t status = launch(first, (uint32_t)(left < most ? left : most));
    if (status != 0) return status;
  }
  return 0;
}

// Copy pieces: one wave copies one piece of a block, a whole piece loaded before its first
// word is stored. Copying is bound by HBM (one read and one write per byte). Measured on
// 4 GiB (read + write traffic), four waves per workgroup: 4 KiB per wave (four 16-byte
// words per lane) 6.0-6.1 TB/s, 16 KiB 5.9-6.0; 8 KiB 5.1, 16 KiB in four rounds 5.5; a
// 256-thread workgroup striding over 64 KiB with four words per thread 5.4; persistent
// grids 5.2-5.8. A block of 4 KiB, the small copies' block size, is one piece, so its wave
// waits for the record once and keeps no other wave waiting.
// The larger piece is for grids in which most waves find nothing to copy, in blocks of
// kLargePieceBlock and up: the GPU starts about 1.2 workgroups per ns, so such a grid costs
// by its size. Packing takes it (held blocks have nothing to pack: a 3.8 GB decoder shard
// with about a tenth missing 98-148 us against 133-185), and restoring batches of mostly
// short payloads (20,000 of 12 KB in 64 KiB blocks 92 us against 133); restoring mostly
// full blocks does not (the shard 1,327 us against 1,262).
constexpr uint32_t kCopyThreads = 256, kCopyWaves = kCopyThreads / 64;
constexpr uint32_t kSmallPiece = 4096, kLargePiece = 16384;
constexpr uint32_t kLargePieceBlock = 65536;

struct CopyShape {
  bool large;         // kLargePiece
  uint32_t per_log2;  // log2 of the pieces per block
  uint32_t groups;    // workgroups of kCopyWaves pieces; they stride where there are more pieces
};

// `sparse`: many of the blocks may have nothing to copy. n_blocks below 2^51, block_bytes a
// power of two of kSmallPiece or more (validate_batch).
inline CopyShape copy_shape(uint64_t n_blocks, uint32_t block_bytes, bool sparse) {
  CopyShape c;
  c.large = sparse && block_bytes >= kLargePieceBlock;
  c.per_log2 = 0;
  for (uint32_t piece = c.large ? kLargePiece : kSmallPiece; piece < block_bytes; piece *= 2) ++c.per_log2;
  const uint64_t want = ((n_blocks << c.per_log2) + kCopyWaves - 1) / kCopyWaves;
  c.groups = (uint32_t)(want < max_workgroups(kCopyThreads) ? want : max_workgroups(kCopyThreads));
  return c;
}

}  // namespace gleam
