// The leading rows of a recomputation chunk that see fewer than 64 keys (a discarded request's context is recomputed
// from position 0, Section 4.2): at most 63 rows of one sequence against at most 63 keys, for one query head per half
// of a workgroup.  As row items these rows cost a workgroup per (row, head), each a chain of dependent loads (item,
// block table, keys) around a few hundred multiply-adds: 4 fresh chunks of a 40-head pool are 10080 of them, 240 us.
// Here a (sequence, head) is ONE unit: its keys are staged in LDS once, 16 rows per wave on the matrix cores.
//   - The weights keep their 24 bits of significand on the way into the PV product: p = hi + mid + lo, all bf16, one MFMA
//     each (against the one rounding, 2^-9, that the tile bodies make; with a handful of keys a single weight's
//     rounding shows in the result).  With two parts (16 bits) 0.17 % of the results were not the bf16 value nearest to the
//     exact one, with three 0.01 %, as on the vector kernel, for 0.3 us a launch.  The normaliser is the fp32 sum of the weights, the
//     maximum the row's own.
//   - A product of a zero weight and an infinite value is NaN on the matrix core, also for keys the row does not
//     see.  If a wave's result is not finite it is computed again key by key on the vector ALU, over the row's own
//     keys only.
// Bound by latency (two dependent loads and one barrier per unit); units are the tail of the tile kernels' queues.
// Measured, two layer steps of 16 decode rows + 4 chunks of 300..1500 rows from position 0 (40 heads, head_dim 128): 676 ->
// 454 us; one chunk of some 100 rows from position 17, 32 heads over one K/V head: 44 -> 19 us a layer.
#pragma once

#include "tile16_body.h"

namespace ic {
namespace fewp {

using namespace tilep;

// LDS: one 64-key tile of K and of V per half of the workgroup, in the 16-row tile's row strides.
template <int D>
constexpr int few_lds_bytes() {
  return 2 * tile16::tile16_buf_elems<D>() * 2;
}

// Unit (f, pair): rows f.first .. f.first + f.n_rows - 1 of the row items (one sequence, ascending positions) for
// query heads 2 pair (threads 0..255) and 2 pair + 1 (threads 256..511).  lds: few_lds_bytes<D>() bytes.
template <int D>
__device__ __forceinline__ void few_body(const AttnParams& p, const FewItem& f, int pair, uint16_t* lds) {
  using G = tile16::G16<D>;
  const int32_t offs = first_offsets(p);
  const int H = p.num_heads, Hk = p.num_kv_heads;
  int tid0 = threadIdx.x;
  asm volatile("" : "+v"(tid0));  // values derived from it are not kept in registers across the tile items before
  const int half = __builtin_amdgcn_readfirstlane(tid0 >> 8);
  const int tid = tid0 & 255;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, g = lane >> 4;
  const bool live = 2 * pair + half < H;  // an odd last head leaves the second half without one
  const int head = min(2 * pair + half, H - 1);
  const int kvh = head / p.group;

  const RowItem* rows = p.row_items + f.first;
  const int n = f.n_rows;
  const int r = 16 * w + col;
  const RowItem* mine = rows + min(r, n - 1);  // dead rows mirror the last live one
  const int qrow = mine->qrow, pos = mine->k_end - 1;
  const int n_keys = rows[n - 1].k_end;  // <= 63

  uint16_t* ks = lds + half * tile16::tile16_buf_elems<D>();
  uint16_t* vs = ks + kTileK * G::kKStride;
  {
    typedef __attribute__((address_space(4))) const int32_t const_i32;
    const_i32* bt = (const_i32*)(p.bt_flat + table_start(p, offs, rows[0].seq));
    constexpr int kTileBytes = kBlockSize * D * 2;
    constexpr int kLoads = kTileK * G::kChunks / 256;
    const char* base = (const char*)p.pool + (int64_t)kvh * kTileBytes;
    const int last_blk = (n_keys - 1) / kBlockSize;
    u32x4 k[kLoads], v[kLoads];
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      const int u = tid + 256 * j, tok = u / G::kChunks, c = u % G::kChunks;
      const int blk = __builtin_amdgcn_readfirstlane(tok / kBlockSize);  // a wave's chunks never straddle a block
      const char* a = base + (int64_t)bt[min(blk, last_blk)] * ((int64_t)2 * Hk * kTileBytes) + (tok % kBlockSize) * (D * 2) + c * 16;
      k[j] = v[j] = (u32x4){0u, 0u, 0u, 0u};
      if (tok < n_keys) {  // slots past the last key may hold anything
        k[j] = *(const u32x4*)a;
        v[j] = *(const u32x4*)(a + (int64_t)Hk * kTileBytes);
      }
    }
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      const int u = tid + 256 * j, tok = u / G::kChunks, c = u % G::kChunks;
      *(u32x4*)(ks + tok * G::kKStride + c * 8) = k[j];
      *(u32x4*)(vs + tok * G::kVStride + c * 8) = v[j];
    }
  }
  bf16x8 qreg[G::kQSteps];
  {
    const uint16_t* qp = p.q + ((int64_t)qrow * H + head) * D + 8 * g;
#pragma unroll
    for (int t = 0; t < G::kQSteps; ++t) qreg[t] = *(const bf16x8*)(qp + 32 * t);
  }
  __syncthreads();
  if (16 * w >= n || !live) return;  // wave-uniform; no barrier follows

  // S^T = K Q^T: this lane holds query column col, keys 16 u + 4 g + i
  f32x4 s[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    s[u] = (f32x4){0.f, 0.f, 0.f, 0.f};
    const uint16_t* kp = ks + (16 * u + col) * G::kKStride + 8 * g;
#pragma unroll
    for (int t = 0; t < G::kQSteps; ++t)
      s[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(const bf16x8*)(kp + 32 * t), qreg[t], s[u], 0, 0, 0);
  }
  const float sc = p.scale_log2e;
  float m = kNegBig;
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s[u][i] = 16 * u + 4 * g + i > pos ? -__builtin_inff() : s[u][i] * sc;
      m = __builtin_fmaxf(m, s[u][i]);
    }
  m = __builtin_fmaxf(m, __shfl_xor(m, 16));
  m = __builtin_fmaxf(m, __shfl_xor(m, 32));
  float l = 0.f;
  bf16x8 hi[2], mid[2], lo[2];
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s[u][i] = __builtin_amdgcn_exp2f(s[u][i] - m);
      l += s[u][i];
      const __bf16 h = (__bf16)s[u][i];
      const float r1 = s[u][i] - (float)h;  // exact, and so is what is left after mid
      const __bf16 d = (__bf16)r1;
      hi[u >> 1][4 * (u & 1) + i] = h;
      mid[u >> 1][4 * (u & 1) + i] = d;
      lo[u >> 1][4 * (u & 1) + i] = (__bf16)(r1 - (float)d);
    }
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);

  // O^T += V^T P^T: this lane holds dims 16 dt + 4 g + i of its column
  f32x4 acc[G::kDTiles];
  float worst = 0.f;
#pragma unroll
  for (int dt = 0; dt < G::kDTiles; ++dt) {
    acc[dt] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const bf16x8 a = tile16::read_vt16<D>(vs, 16 * dt, h, lane);
      acc[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, hi[h], acc[dt], 0, 0, 0);
      acc[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, mid[h], acc[dt], 0, 0, 0);
      acc[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, lo[h], acc[dt], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) worst += acc[dt][i] * 0.f;  // 0, or NaN for an infinity or a NaN
  }
  if (__builtin_amdgcn_ballot_w64(!(worst == 0.f)) != 0) {
#pragma unroll
    for (int dt = 0; dt < G::kDTiles; ++dt) acc[dt] = (f32x4){0.f, 0.f, 0.f, 0.f};
    for (int gs = 0; gs < 4; ++gs)
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int key = 16 * u + 4 * gs + i;
          const float pk = __shfl(s[u][i], 16 * gs + col);
          if (key > pos) continue;
#pragma unroll
          for (int dt = 0; dt < G::kDTiles; ++dt) {
            const bf16x4 vv = *(const bf16x4*)(vs + key * G::kVStride + 16 * dt + 4 * g);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[dt][e] = __builtin_fmaf(pk, (float)vv[e], acc[dt][e]);
          }
        }
  }
  if (r < n) {
    uint16_t* op = p.out + ((int64_t)qrow * H + head) * D + 4 * g;
#pragma unroll
    for (int dt = 0; dt < G::kDTiles; ++dt) {
      bf16x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (__bf16)(acc[dt][e] / l);  // round to nearest even
      *(bf16x4*)(op + 16 * dt) = o;
    }
  }
}

}  // namespace fewp
}  // namespace ic
