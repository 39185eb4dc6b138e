// Split-KV merge: out = sum_p o_p 2^(m_p - m) / sum_p l_p 2^(m_p - m), m = max_p m_p, over the partial results that
// the partitions of a row left in part_o / part_ml.  Used by the merge kernel and, where the launches of one
// workgroup per item run rows that the planner split, by whichever partition's workgroup finishes last.
#pragma once

#include "ic_internal.h"

namespace ic {
namespace mergep {

typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;

// Partial results that another workgroup of the same launch will read or has written: single accesses at agent scope, which
// go through the XCD's L2 (the L2s of the XCDs are not coherent with each other) to the memory they share.  Also where the
// merge kernel reads them: plain stores stay in the L2s and are written back when the kernel ends (196 rows of 15000 keys in
// 4096-key items, 64 heads over 8: 1897 us a layer, 1866 this way).
__device__ __forceinline__ void store_shared(float* a, float v) {
  __hip_atomic_store(a, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ f32x2 load_shared(const float* a) {
  return __builtin_bit_cast(f32x2, __hip_atomic_load((const uint64_t*)a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// Four consecutive values of one row, e = head * D + dim of the first.  The partitions are read kBatch at a time, values and
// (m, l) together, and combined in ascending order with a running maximum: nothing waits for the maximum first.
// kShared: the partial results come from this launch.
template <int D, int kBatch, bool kShared>
__device__ __forceinline__ void merge_four(const AttnParams& p, int qrow, int slot0, int nparts, uint32_t e) {
  const uint32_t row_elems = (uint32_t)p.num_heads * D;
  const float* po = p.part_o + (int64_t)slot0 * row_elems + e;
  const float* pm = p.part_ml + ((int64_t)slot0 * p.num_heads + e / D) * 2;
  float M = -1.0e30f, L = 0.f;
  f32x4 O = {0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < nparts; k0 += kBatch) {
    f32x4 o[kBatch];
    f32x2 ml[kBatch];
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      const int64_t part = min(k0 + k, nparts - 1);
      if constexpr (kShared) {
        ml[k] = load_shared(pm + part * p.num_heads * 2);
        const f32x2 a = load_shared(po + part * row_elems), b = load_shared(po + part * row_elems + 2);
        o[k] = (f32x4){a[0], a[1], b[0], b[1]};
      } else {
        ml[k] = *(const f32x2*)(pm + part * p.num_heads * 2);
        o[k] = *(const f32x4*)(po + part * row_elems);
      }
    }
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      if (k0 + k >= nparts) break;
      const float m_new = __builtin_fmaxf(M, ml[k][0]);
      const float was = __builtin_amdgcn_exp2f(M - m_new), wgt = __builtin_amdgcn_exp2f(ml[k][0] - m_new);
      M = m_new;
      L = __builtin_fmaf(ml[k][1], wgt, L * was);
#pragma unroll
      for (int i = 0; i < 4; ++i) O[i] = __builtin_fmaf(o[k][i], wgt, O[i] * was);
    }
  }
  bf16x4 out;
#pragma unroll
  for (int i = 0; i < 4; ++i) out[i] = (__bf16)(O[i] / L);  // round to nearest even
  *(bf16x4*)(p.out + (int64_t)qrow * row_elems + e) = out;
}

// End of a partition of a split decode row: the workgroup that finds the others' partial results already there merges
// them (all of them, in partition order, so the result does not depend on who is last) and puts the counter back to zero.
// A merge pass of its own costs 4-6 us of launch and latency behind a kernel of 10 to 30 us.  Measured: four layers of one row of
// 3000 keys (40 heads) 78 -> 72.5 us, of 8 rows of 1000..8000 keys (64 heads over 8 K/V heads) 168 -> 158 us.
// The partitions' workgroups run on any XCDs: partial results are stored and loaded at agent scope (store_shared,
// load_shared), every wave waits until its stores have got there before the count, and the count is one atomic.  (Plain
// stores with an agent-scope release fence write back the whole L2 in every wave: the same kernels took 1.4 to 2.4
// times as long.)
// unit: which of the row's units (heads, or K/V heads with n_heads query heads each) this workgroup has, head0 the first head.
template <int D, int kBatch>
__device__ __forceinline__ void finish_split(const AttnParams& p, int slot, int unit, int head0, int n_heads, int* s_last) {
  const int mi = p.slot_merge[slot];
  const int nparts = p.merge_items[mi].nparts;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t* const arrived = p.arrived + (int64_t)mi * p.split_units + unit;
    const int before = __hip_atomic_fetch_add(arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (before == nparts - 1) __hip_atomic_store(arrived, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *s_last = before;
  }
  __syncthreads();
  if (*s_last != nparts - 1) return;  // the same for the whole workgroup
  const MergeItem mg = p.merge_items[mi];
  for (uint32_t e = 4u * threadIdx.x; e < (uint32_t)(n_heads * D); e += 4u * blockDim.x)
    merge_four<D, kBatch, true>(p, mg.qrow, mg.slot0, mg.nparts, (uint32_t)head0 * D + e);
}

}  // namespace mergep
}  // namespace ic
