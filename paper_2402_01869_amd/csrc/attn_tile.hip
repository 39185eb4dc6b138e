// Tile kernels: recomputation spans on the matrix cores.  head_dim <= 128: 32 query rows per wave (tile32_body.h);
// head_dim 256: 16 rows per wave (tile16_body.h).  Either way a workgroup is 8 waves, two per SIMD.  The rows of a span
// that see fewer than 64 keys are units of their own (few_body.h), handed out after the tile items.
#include <algorithm>

#include "few_body.h"
#include "tile32_body.h"

namespace ic {

namespace {

using namespace tilep;

// What a workgroup of the tile kernels is for head_dim D.
template <int D>
struct Impl {
  static constexpr int kThreads = tile32::G32<D>::kThreads;
  static constexpr int kLdsBytes = std::max(tile32::tile32_lds_bytes<D>(), fewp::few_lds_bytes<D>());
  static __device__ __forceinline__ void body(const AttnParams& p, const TileItem& it, int th, uint16_t* lds) {
    tile32::tile32_body<D>(p, it, th, lds);
  }
};
template <>
struct Impl<tile16::kDim> {
  static constexpr int kThreads = tile16::kThreads;
  static constexpr int kLdsBytes = std::max(tile16::kLdsBytes, fewp::few_lds_bytes<tile16::kDim>());
  static __device__ __forceinline__ void body(const AttnParams& p, const TileItem& it, int th, uint16_t* lds) {
    tile16::tile16_body(p, it, th, lds);
  }
};

// Few-key units of a launch: pairs of query heads per few item.
__host__ __device__ inline uint32_t few_units(const AttnParams& p) { return (uint32_t)p.n_few_items * (uint32_t)((p.num_heads + 1) / 2); }

// Workgroups (of one XCD where each has its queue) that hand out everything in one round; XCD 0 has the most to do.
__host__ __device__ inline uint32_t tile_round(const AttnParams& p) {
  const uint32_t n_th = (uint32_t)p.num_heads >> p.tile_g_shift;
  if (n_th < 8u) return (uint32_t)p.n_tile_items * n_th + few_units(p);
  return (uint32_t)p.n_tile_items * ((n_th + 7u) / 8u) + (few_units(p) + 7u) / 8u;
}

template <int D>
__device__ __forceinline__ void run_few(const AttnParams& p, uint32_t unit, uint16_t* lds) {
  static_assert(fewp::few_lds_bytes<D>() <= Impl<D>::kLdsBytes && Impl<D>::kThreads == 512, "few-key units run in the tile kernels");
  const uint32_t pairs = (uint32_t)(p.num_heads + 1) / 2u;
  const uint32_t f = unit / pairs;
  fewp::few_body<D>(p, p.few_items[f], (int)(unit - f * pairs), lds);
}

// One workgroup per work item: head_dim 256 where the tiles run alone.  (At head_dim 64 and 128 the persistent launch is as fast there
// or faster: 16 chunks of 2048 rows on 16384 keys, 32 heads of 128, 8.49 against 9.06 ms, 8 chunks of 512 the same.)
template <int D>
__global__ __launch_bounds__(Impl<D>::kThreads, 2) void tile_attn_kernel(AttnParams p) {
  __shared__ __attribute__((aligned(1024))) uint16_t lds[Impl<D>::kLdsBytes / 2];
  const int n_th = p.num_heads >> p.tile_g_shift;  // head groups, each served by one workgroup per item
  const uint32_t wg = blockIdx.x;
  const uint32_t n_tile = (uint32_t)p.n_tile_items * (uint32_t)n_th;
  if (wg >= n_tile) {
    run_few<D>(p, wg - n_tile, lds);
    return;
  }
  const int item_idx = wg / n_th;
  const int th = wg - item_idx * n_th;
  const TileItem it = p.tile_items[item_idx];
  Impl<D>::body(p, it, th, lds);
}

// Persistent launch of the same body, for running beside the row kernel: `slots` workgroups (one
// per CU; two do not fit) pull tile items from one queue per XCD with atomic counters
// (counters[0..7], zeroed by the descriptor upload).  Workgroups are dealt round-robin to the 8 XCDs
// (L2 domains) by block index, so XCD x = index % 8 owns the tile items of the heads h = x (mod 8),
// in head-major order: the query tiles of one (sequence, head), which read the same keys, run on
// one L2 at the same time, and each span's keys are fetched from HBM about once.
// Register budget: at most 208 per lane, vector and accumulation registers together (checked by the test-suite
// from the compiler's resource report and listing).  Two waves of this kernel and one of the slim row kernel (80, head_dim
// 256: 96) or of the slim group kernel (96) fill the 512 of a SIMD, which is what lets one workgroup of each
// share a CU.
// kBeside only names the build (side by side with a row or group kernel, or on its own), so that a kernel trace
// tells the two uses apart; the code is the same.
// amdgpu_num_vgpr: on this target vector and accumulation registers share one file and the compiler doubles the
// figure it is given, so 104 caps the kernel at 208 registers (launch bounds alone would allow 256).
template <int D, bool kBeside>
__global__ __launch_bounds__(Impl<D>::kThreads, 2) __attribute__((amdgpu_num_vgpr(104))) void tile_persist_kernel(AttnParams p) {
  __shared__ __attribute__((aligned(1024))) uint16_t lds[Impl<D>::kLdsBytes / 2];
  __shared__ int s_next;
  if (p.tile_first) __builtin_amdgcn_s_setprio(3);
  const int H = p.num_heads >> p.tile_g_shift;               // head groups
  const bool per_xcd = H >= 8;   // with fewer head groups than XCDs, one shared queue instead
  const uint32_t x = blockIdx.x & 7u;
  const uint32_t heads_x = (uint32_t)(H - (int)x + 7) / 8u;  // head groups congruent to x mod 8
  const uint32_t n_t = (uint32_t)p.n_tile_items * (per_xcd ? heads_x : (uint32_t)H);
  const uint32_t units = few_units(p);  // dealt to the XCDs by unit index, after the tile items
  const uint32_t n_all = n_t + (per_xcd ? (units - x + 7u) / 8u : units);
  // the first round is handed out by index: workgroup blockIdx of XCD x takes the XCD's item blockIdx / 8
  const uint32_t round = per_xcd ? gridDim.x / 8u : gridDim.x;
  const bool queued = tile_round(p) > round;  // the same for every XCD
  int32_t* const queue = &p.counters[per_xcd ? x : (uint32_t)kCtrTileShared];
  const auto next = [&]() -> uint32_t { return queued ? queue_pull(queue, round, &s_next) : n_all; };
  uint32_t idx = per_xcd ? blockIdx.x / 8u : blockIdx.x;
  while (idx < n_t) {
    uint32_t item, th;
    if (per_xcd) {
      const uint32_t hsel = idx / (uint32_t)p.n_tile_items;
      item = idx - hsel * (uint32_t)p.n_tile_items;
      th = x + 8u * hsel;
    } else {
      item = idx / (uint32_t)H;
      th = idx - item * (uint32_t)H;
    }
    const TileItem it = p.tile_items[item];
    Impl<D>::body(p, it, (int)th, lds);
    idx = next();
  }
  // (a loop of its own: values of one body kept in registers across the other would not fit)
  while (idx < n_all) {
    run_few<D>(p, per_xcd ? x + 8u * (idx - n_t) : idx - n_t, lds);
    idx = next();
  }
  if (queued) queue_leave(p.counters, 0, 8, kCtrTileShared, kCtrTileLeft);
}

}  // namespace

hipError_t launch_tile_kernel(const AttnParams& p, int head_dim, hipStream_t st) {
  if (head_dim != tile16::kDim) return hipErrorInvalidValue;
  const uint64_t grid = (uint64_t)p.n_tile_items * (uint64_t)(p.num_heads >> p.tile_g_shift) + few_units(p);
  if (grid == 0) return hipSuccess;
  if (grid > 0x7fffffffull) return hipErrorInvalidValue;
  hipLaunchKernelGGL(tile_attn_kernel<tile16::kDim>, dim3((uint32_t)grid), dim3(Impl<tile16::kDim>::kThreads), 0, st, p);
  return hipGetLastError();
}

// slots is rounded down to a multiple of 8 so that every XCD gets the same number of workgroups.
hipError_t launch_tile_persist(const AttnParams& p, int head_dim, int slots, bool beside, hipStream_t st) {
  if (p.n_tile_items <= 0 && p.n_few_items <= 0) return hipSuccess;
  if (!p.counters || slots < 8) return hipErrorInvalidValue;
  // no more workgroups than one round needs, and as many per XCD as its queue's share where each has its own
  const bool per_xcd = (p.num_heads >> p.tile_g_shift) >= 8;
  const dim3 g(per_xcd ? 8u * std::min((uint32_t)slots / 8u, tile_round(p)) : std::min((uint32_t)(slots - slots % 8), tile_round(p)));
#define IC_TILE_CASE(DD)                                                                                          \
  case DD:                                                                                                        \
    if (beside) hipLaunchKernelGGL((tile_persist_kernel<DD, true>), g, dim3(Impl<DD>::kThreads), 0, st, p);        \
    else hipLaunchKernelGGL((tile_persist_kernel<DD, false>), g, dim3(Impl<DD>::kThreads), 0, st, p);              \
    break;
  switch (head_dim) {
    IC_TILE_CASE(64)
    IC_TILE_CASE(128)
    IC_TILE_CASE(256)
    default: return hipErrorInvalidValue;
  }
#undef IC_TILE_CASE
  return hipGetLastError();
}

}  // namespace ic
