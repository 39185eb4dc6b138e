// What the matrix-core kernels share: vector types, the constants of the online softmax, LDS rows of staged keys and values in the
// 32x32x16 shape's kernels that copy them through registers (the group kernel), and their V operand.
#pragma once

#include "ic_internal.h"

namespace ic {
namespace tilep {

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

constexpr float kNegBig = -1.0e30f;
constexpr float kLazyLog2 = 8.0f;  // slack of the online softmax's reference maximum, in log2 units
constexpr int kTileK = 64;    // keys per staged tile

template <int D>
struct TG {
  static constexpr int kKStride = D + 8;        // bf16 per LDS row of K (16-byte pad)
  static constexpr int kVStride = D + 32;       // bf16 per LDS row of V: rows shift by 16 banks
  static constexpr int kQSteps = D / 16;        // MFMA k-steps of Q K^T
  static constexpr int kDTiles = D / 32;        // 32-row tiles of O^T
};

// A operand of O^T += V^T P^T for MFMA rows d = d0 .. d0+31 (this lane: d0 + lane % 32) and the 8 keys
// of k-step ksp that belong to this lane half, read with the LDS transpose load.  In each group of
// 16 lanes, lane i supplies the address of an 8-byte row and receives column i % 4 of the rows
// supplied by lanes i/4, i/4 + 4, i/4 + 8, i/4 + 12 (layout measured on gfx950).  So lane j points at
// V[key j/4][dims 4 (j % 4) ..+3] of its group's 16 dims, and lane i gets V[4 keys][dim i]: two loads
// give the 8 keys in accumulator order (slots 0-3: keys 4 hl ..+3, slots 4-7: keys 8 + 4 hl ..+3).
template <int D>
__device__ __forceinline__ bf16x8 read_vt_operand(const uint16_t* vs, int d0, int ksp, int lane) {
  using G = TG<D>;
  typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
  const int hl = lane >> 5;
  const int j = lane & 15;
  const uint16_t* a = vs + (16 * ksp + 4 * hl + (j >> 2)) * G::kVStride + d0 + 16 * ((lane & 31) >> 4) + 4 * (j & 3);
  const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)a);
  const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(a + 8 * G::kVStride));
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

}  // namespace tilep
}  // namespace ic
