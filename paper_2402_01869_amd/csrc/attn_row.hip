// Row kernel (decode rows, and spans row by row when asked) and the split-KV merge.
#include <algorithm>

#include "row_body.h"

namespace ic {

namespace {

using namespace rowp;

template <int D, int PF, bool NT>
__global__ __launch_bounds__(kRowWaves * 64) void row_attn_kernel(AttnParams p) {
  __shared__ __attribute__((aligned(16))) float lds[row_lds_bytes<D>() / sizeof(float)];
  __shared__ int s_last;
  const int H = p.num_heads;
  const uint32_t wg = blockIdx.x;
  const int item_idx = wg / H;
  const int head = wg - item_idx * H;
  const RowItem it = p.row_items[item_idx];
  row_body<D, PF, NT, false, true>(p, it, head, lds, &s_last);
}

// Persistent launch of the same body: `slots` workgroups (one per CU) pull (item, head) pairs from a
// queue with an atomic counter (zeroed by the descriptor upload).  Measured on MI355X:
// 256 resident workgroups read 6.65 TB/s, 4 % more than one workgroup per work item, because no
// workgroup launch or drain sits between two items.
template <int D, int PF>
__global__ __launch_bounds__(kRowWaves * 64) void row_persist_kernel(AttnParams p) {
  __shared__ __attribute__((aligned(16))) float lds[row_lds_bytes<D>() / sizeof(float)];
  __shared__ int s_next;
  const int H = p.num_heads;
  const uint32_t n_r = (uint32_t)p.n_vec_items * (uint32_t)H;
  const bool queued = n_r > gridDim.x;
  for (uint32_t idx = blockIdx.x; idx < n_r;) {
    const uint32_t item = idx / (uint32_t)H;  // head fastest: neighbours read adjacent tiles of a block
    const RowItem it = p.row_items[item];
    row_body<D, PF, true>(p, it, (int)(idx - item * (uint32_t)H), lds);
    if (!queued) return;
    idx = queue_pull(&p.counters[kCtrRowQueue], gridDim.x, &s_next);
  }
  if (!queued) return;
  queue_leave(p.counters, kCtrRowQueue, 1, -1, kCtrRowLeft);
}

// Merge pass for the rows of split tiles, and for split decode rows that their last partition has not merged (merge_body.h).
// The partial results of a row are [H][D] fp32 per partition, contiguous: a workgroup of 256 threads takes 1024
// consecutive values of one row, 16 bytes per thread and load.  Bound by memory.  Measured against one workgroup of D
// threads per (row, head), which read 4 bytes per thread and needed the maximum before the first value: 8 rows of 64
// heads in 2 to 11 partitions 7.3 -> 5.7 us.
constexpr int kMergeThreads = 256, kMergeElems = 4 * kMergeThreads;

template <int D>
__global__ __launch_bounds__(kMergeThreads) void merge_kernel(AttnParams p, uint32_t chunks) {
  const uint32_t mi = blockIdx.x / chunks;
  const uint32_t e = (blockIdx.x - mi * chunks) * kMergeElems + threadIdx.x * 4u;
  if (e >= (uint32_t)p.num_heads * D) return;
  const MergeItem it = p.merge_items[p.merge_first + mi];
  mergep::merge_four<D, 4, false>(p, it.qrow, it.slot0, it.nparts, e);
}

}  // namespace

hipError_t launch_row_kernel(const AttnParams& p, int head_dim, hipStream_t st) {
  if (p.n_vec_items <= 0) return hipSuccess;
  const uint64_t grid = (uint64_t)p.n_vec_items * p.num_heads;
  if (grid > 0x7fffffffull) return hipErrorInvalidValue;
  const dim3 g((uint32_t)grid), b(kRowWaves * 64);
#define IC_ROW_CASE(DD)                                                                       \
  case DD:                                                                                    \
    switch (p.row_variant & 3) {                                                              \
      case 0: hipLaunchKernelGGL((row_attn_kernel<DD, 1, true>), g, b, 0, st, p); break;       \
      case 1: hipLaunchKernelGGL((row_attn_kernel<DD, 2, true>), g, b, 0, st, p); break;       \
      case 2: hipLaunchKernelGGL((row_attn_kernel<DD, 1, false>), g, b, 0, st, p); break;      \
      default: hipLaunchKernelGGL((row_attn_kernel<DD, 2, false>), g, b, 0, st, p); break;     \
    }                                                                                         \
    break;
  switch (head_dim) {
    IC_ROW_CASE(64)
    IC_ROW_CASE(128)
    IC_ROW_CASE(256)
    default: return hipErrorInvalidValue;
  }
#undef IC_ROW_CASE
  return hipGetLastError();
}

// Slim build of the persistent row kernel for running BESIDE the tile kernel: no register prefetch
// (measured not to matter there: the CU's memory pipe, not the wave, holds the loads in flight)
// and at most 80 VGPRs (head_dim 256: 96, with blocks taken in two halves), so that one of these workgroups fits
// on a CU next to a tile workgroup.
template <int D>
__global__ __launch_bounds__(kRowWaves * 64, (D <= 128 ? 6 : 5)) void row_persist_slim_kernel(AttnParams p) {
  __shared__ __attribute__((aligned(16))) float lds[row_lds_bytes<D>() / sizeof(float)];
  __shared__ int s_next;
  const int H = p.num_heads;
  const uint32_t n_r = (uint32_t)p.n_vec_items * (uint32_t)H;
  const bool queued = n_r > gridDim.x;
  for (uint32_t idx = blockIdx.x; idx < n_r;) {
    const uint32_t item = idx / (uint32_t)H;
    const RowItem it = p.row_items[item];
    row_body<D, 0, true, (D > 128)>(p, it, (int)(idx - item * (uint32_t)H), lds);
    if (!queued) return;
    idx = queue_pull(&p.counters[kCtrRowQueue], gridDim.x, &s_next);
  }
  if (!queued) return;
  queue_leave(p.counters, kCtrRowQueue, 1, -1, kCtrRowLeft);
}

hipError_t launch_row_persist(const AttnParams& p, int head_dim, int slots, hipStream_t st) {
  if (p.n_vec_items <= 0) return hipSuccess;
  if (!p.counters || slots < 1) return hipErrorInvalidValue;
  const dim3 g((uint32_t)std::min<uint64_t>((uint64_t)slots, (uint64_t)p.n_vec_items * p.num_heads)), b(kRowWaves * 64);
  switch (head_dim) {
    case 64: hipLaunchKernelGGL((row_persist_kernel<64, 1>), g, b, 0, st, p); break;
    case 128: hipLaunchKernelGGL((row_persist_kernel<128, 1>), g, b, 0, st, p); break;
    case 256: hipLaunchKernelGGL((row_persist_kernel<256, 1>), g, b, 0, st, p); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_row_persist_slim(const AttnParams& p, int head_dim, int slots, hipStream_t st) {
  if (p.n_vec_items <= 0) return hipSuccess;
  if (!p.counters || slots < 1) return hipErrorInvalidValue;
  const dim3 g((uint32_t)std::min<uint64_t>((uint64_t)slots, (uint64_t)p.n_vec_items * p.num_heads)), b(kRowWaves * 64);
  switch (head_dim) {
    case 64: hipLaunchKernelGGL(row_persist_slim_kernel<64>, g, b, 0, st, p); break;
    case 128: hipLaunchKernelGGL(row_persist_slim_kernel<128>, g, b, 0, st, p); break;
    case 256: hipLaunchKernelGGL(row_persist_slim_kernel<256>, g, b, 0, st, p); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_merge_kernel(const AttnParams& p, int head_dim, hipStream_t st) {
  if (p.n_merge_items <= 0) return hipSuccess;
  const uint32_t chunks = ((uint32_t)(p.num_heads * head_dim) + kMergeElems - 1) / kMergeElems;
  const uint64_t grid = (uint64_t)p.n_merge_items * chunks;
  if (grid > 0x7fffffffull) return hipErrorInvalidValue;
  const dim3 g((uint32_t)grid), b(kMergeThreads);
  switch (head_dim) {
    case 64: hipLaunchKernelGGL(merge_kernel<64>, g, b, 0, st, p, chunks); break;
    case 128: hipLaunchKernelGGL(merge_kernel<128>, g, b, 0, st, p, chunks); break;
    case 256: hipLaunchKernelGGL(merge_kernel<256>, g, b, 0, st, p, chunks); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace ic
