// gleam_identify_weights: weight identification at free time (Gleam Sec. 4.1.1,
// "Weight Block Identification"). An allocation holds weights only if every payload
// recorded at its first host-to-device write still has the same bytes when the
// allocation is freed; in-place activations or inputs make it non-weights (Appendix,
// discussion of corner cases). Instead of the recorded bytes, the digests recorded
// at write time are compared with digests of the current device bytes, by the fingerprint
// kernels with the comparison in the place of their stores (fp_chunks.hip), between two
// small launches that set up and fold the results per payload and per allocation.

#include "gleam_device.h"
#include "gleam_internal.h"
#include "launch_shape.h"

namespace gleam {
namespace {

constexpr int kThreads = 256;

__global__ void identify_init_kernel(uint64_t* first_diff, uint64_t n_seg, const uint64_t* region_first,
                                     uint64_t n_regions, uint8_t* region_weight) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (uint64_t s = t; s < n_seg; s += stride) first_diff[s] = ~0ull;
  for (uint64_t r = t; r < n_regions; r += stride) region_weight[r] = region_first[r + 1] > region_first[r] ? 1 : 0;
}

// Per payload: a difference clears its allocation's weight flag.
__global__ void identify_region_kernel(const uint64_t* first_diff, uint64_t n_seg, const uint64_t* region_first,
                                       uint64_t n_regions, uint8_t* region_weight) {
  const uint64_t s = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n_seg || first_diff[s] == ~0ull) return;
  if (s < region_first[0] || s >= region_first[n_regions]) return;
  const uint64_t r = find_segment(region_first, n_regions, s);
  region_weight[r] = 0;
}

constexpr uint64_t kMaxIdentify = 1ull << 39;

uint32_t grid_for(uint64_t n, uint64_t cap = max_workgroups(kThreads)) {
  const uint64_t g = (n + kThreads - 1) / kThreads;
  return (uint32_t)(g < cap ? (g ? g : 1) : cap);
}

}  // namespace
// Loads this file's GPU code object on the current device (gleam_preload).
hipError_t preload_identify() {
  hipFuncAttributes attr;
  return hipFuncGetAttributes(&attr, reinterpret_cast<const void*>(&identify_init_kernel));
}

}  // namespace gleam

extern "C" gleam_status gleam_identify_weights(const gleam_batch* b, const uint64_t* d_recorded,
                                               const uint64_t* d_region_first, uint64_t n_regions,
                                               uint8_t* d_block_match, uint64_t* d_seg_first_diff,
                                               uint8_t* d_region_weight, void* d_ws, size_t ws_bytes, void* stream) {
  using namespace gleam;
  clear_error();
  gleam_status st = validate_batch(b, "gleam_identify_weights");
  if (st != GLEAM_OK) return st;
  if ((b->n_blocks > 0 && !d_recorded) || (n_regions > 0 && (!d_region_first || !d_region_weight))) {
    set_error("gleam_identify_weights: null recorded digests, region list or output");
    return GLEAM_E_INVALID;
  }
  if (b->n_seg > max_workgroups(kThreads) * kThreads || n_regions > kMaxIdentify || b->n_blocks > kMaxIdentify) {
    set_error("gleam_identify_weights: more than 2^32 payloads, or 2^39 regions or blocks");
    return GLEAM_E_UNSUPPORTED;
  }
  const WsLayout L = ws_layout(b->n_blocks + b->n_seg);
  st = check_workspace(L, d_ws, ws_bytes, "gleam_identify_weights");
  if (st != GLEAM_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  uint64_t* first_diff = d_seg_first_diff
                             ? d_seg_first_diff
                             : reinterpret_cast<uint64_t*>(static_cast<uint8_t*>(d_ws) + L.scratch_off);
  const uint64_t init_n = b->n_seg > n_regions ? b->n_seg : n_regions;
  hipLaunchKernelGGL(identify_init_kernel, dim3(grid_for(init_n, 4096)), dim3(kThreads), 0, s, first_diff, b->n_seg,
                     d_region_first, n_regions, d_region_weight);
  if ((st = launch_status("identify_init_kernel")) != GLEAM_OK) return st;
  if (b->n_blocks == 0) return GLEAM_OK;
  if ((st = launch_fp_compare(b, d_recorded, d_block_match, first_diff, s)) != GLEAM_OK) return st;
  if (n_regions == 0) return GLEAM_OK;
  hipLaunchKernelGGL(identify_region_kernel, dim3(grid_for(b->n_seg)), dim3(kThreads), 0, s, first_diff, b->n_seg,
                     d_region_first, n_regions, d_region_weight);
  return launch_status("identify_region_kernel");
}

extern "C" gleam_status gleam_identify_leaves(const gleam_batch* b, const uint64_t* d_recorded_leaf,
                                              const uint64_t* d_region_first, uint64_t n_regions,
                                              uint8_t* d_leaf_match, uint64_t* d_seg_first_diff,
                                              uint8_t* d_region_weight, void* d_ws, size_t ws_bytes, void* stream) {
  using namespace gleam;
  clear_error();
  gleam_status st = validate_batch(b, "gleam_identify_leaves");
  if (st != GLEAM_OK) return st;
  if ((b->n_blocks > 0 && !d_recorded_leaf) || (n_regions > 0 && (!d_region_first || !d_region_weight))) {
    set_error("gleam_identify_leaves: null recorded leaf digests, region list or output");
    return GLEAM_E_INVALID;
  }
  const uint32_t lpb_log2 = (uint32_t)(log2_exact(b->block_bytes) - 12);
  const uint64_t n_slots = b->n_blocks << lpb_log2;  // n_blocks < 2^51 (validate_batch)
  if (b->n_seg > max_workgroups(kThreads) * kThreads || n_regions > kMaxIdentify || n_slots > kMaxIdentify) {
    set_error("gleam_identify_leaves: more than 2^32 payloads, or 2^39 regions or leaf slots");
    return GLEAM_E_UNSUPPORTED;
  }
  const WsLayout L = ws_layout(n_slots + b->n_seg);
  st = check_workspace(L, d_ws, ws_bytes, "gleam_identify_leaves");
  if (st != GLEAM_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  uint64_t* first_diff = d_seg_first_diff
                             ? d_seg_first_diff
                             : reinterpret_cast<uint64_t*>(static_cast<uint8_t*>(d_ws) + L.scratch_off);
  const uint64_t init_n = b->n_seg > n_regions ? b->n_seg : n_regions;
  hipLaunchKernelGGL(identify_init_kernel, dim3(grid_for(init_n, 4096)), dim3(kThreads), 0, s, first_diff, b->n_seg,
                     d_region_first, n_regions, d_region_weight);
  if ((st = launch_status("identify_init_kernel")) != GLEAM_OK) return st;
  if (b->n_blocks == 0) return GLEAM_OK;
  if ((st = launch_leaf_compare(b, d_recorded_leaf, d_leaf_match, first_diff, s)) != GLEAM_OK) return st;
  if (n_regions == 0) return GLEAM_OK;
  hipLaunchKernelGGL(identify_region_kernel, dim3(grid_for(b->n_seg)), dim3(kThreads), 0, s, first_diff, b->n_seg,
                     d_region_first, n_regions, d_region_weight);
  return launch_status("identify_region_kernel");
}
