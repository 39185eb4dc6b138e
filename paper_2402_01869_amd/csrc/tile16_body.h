// Tile path for head_dim 256: the work item, steps and schedule of tile32_body.h (recomputation chunks, Section 4.2, on the
// matrix cores), with 16 query rows per wave instead of 32.
//
// Why 16: 32 rows x 256 dims of fp32 accumulators (128 registers) plus the wave's Q^T (64) leave no room for a second
// wave on a SIMD, and a lone wave has nothing to hide its LDS and memory waits behind.  With 16 rows per wave
// (v_mfma_f32_16x16x32_bf16, 16 cycles) a wave holds 64 accumulator and 32 Q^T registers, a workgroup is 8 waves of 16 rows
// (128 rows), and two waves share every SIMD.  The price is LDS traffic: every K and V operand read now
// feeds half as many multiply-adds, 1 KiB per MFMA, which is what LDS delivers (256 bytes a cycle and CU) when all four SIMDs multiply.
//   - S^T = K Q^T per 16-key subtile: A = K[16 keys][32 dims] from LDS (lane: key = lane % 16, dims 8 (lane / 16) ..+7),
//     B = Q^T from registers; result: lane holds query column lane % 16, keys 4 (lane / 16) ..+3 of the subtile.
//   - O^T += V^T P^T per 32 keys (two subtiles, one half of a tile) and 16 dims: the two subtiles' weights of a lane, rounded to
//     bf16, ARE the B operand (slot j < 4 of lane group g <-> key 4 g + j of the first subtile, slot 4 + j <-> the same key of the
//     second); the A operand comes from two LDS transpose loads in that key order.
// What bounds it: at two waves a SIMD and an LDS operand per 16-cycle MFMA, LDS reads and issue; on N(0,1) data the power cap.
// Before, a wave did the scores, the weights and the products of a 64-key tile one after the other, K and V went through 32
// registers, the weights were summed by v_dot2 (which waits for the MFMAs in flight), and the matrix pipe was idle for 70 % of the
// time.  Measured, before and now: 8 chunks of 2048 rows on 8192 keys, 16 heads, 3.15 -> 2.53 ms (786 -> 979 TFLOP/s;
// all-zero data 2.84 -> 1.98 ms); 8 chunks of 512 on 512..2048, 146.6 -> 121.7 us, beside 64 decode rows the call 300 -> 293 us.
// 512 threads, 208 registers: as many as the 32-row shape's kernel, so the same neighbours fit beside it.
#pragma once

#include "tile32_body.h"

namespace ic {
namespace tile16 {

using namespace tilep;
using tile32::barrier;
using tile32::copy_region;
using tile32::here;
using tile32::pin;
using tile32::unroll;

// The 16-row shape with tiles staged as padded rows (the few-key units).
template <int D>
struct G16 {
  // bf16 per LDS row of K and of V: rows shift by 8 of the 64 banks (32 bytes).  An operand read of K takes 16 bytes of
  // 16 keys per quarter wave, a transpose read of V 32 bytes of 8 keys per half wave: both then cover all banks once.
  static constexpr int kKStride = D + 16;
  static constexpr int kVStride = D + 16;
  static constexpr int kChunks = D / 8;                   // 16-byte chunks per token row
  static constexpr int kQSteps = D / 32;                  // MFMA k-steps of Q K^T
  static constexpr int kDTiles = D / 16;                  // 16-row tiles of O^T
};

// A operand of O^T += V^T P^T for dims d0 .. d0 + 15 and the 32 keys of half h of the tile, in the key order of the
// weights (see the head of this file).  The LDS transpose load (layout measured on gfx950): in a group of 16 lanes,
// lane j points at 8 bytes and lane i receives element i % 4 of the pieces of lanes i / 4, i / 4 + 4, i / 4 + 8,
// i / 4 + 12.  Lane j of group g points at V[key 4 g + j / 4][dims d0 + 4 (j % 4) ..+3]; lane i then holds dim d0 + i
// of keys 4 g ..+3.
template <int D>
__device__ __forceinline__ bf16x8 read_vt16(const uint16_t* vs, int d0, int h, int lane) {
  using G = G16<D>;
  typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
  const int g = lane >> 4, j = lane & 15;
  const uint16_t* a = vs + (32 * h + 4 * g + (j >> 2)) * G::kVStride + d0 + 4 * (j & 3);
  const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)a);
  const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(a + 16 * G::kVStride));
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

template <int D>
constexpr int tile16_buf_elems() {
  return kTileK * G16<D>::kKStride + kTileK * G16<D>::kVStride;
}
// Staged tiles: as tile32_body.h's, 1 KiB regions of 8 keys x 64 dims, region (key / 8) * 4 + dim / 64, copied by one load of a wave
// each.  Chunk c of key k sits at chunk c ^ spread(k) of the key's 128 bytes.  A transpose read of V takes two neighbouring chunks of 8
// keys.  A K operand read, in one pass, takes chunk c of 8 keys and chunk c ^ 1 of the other 8 (lanes 0-3, 12-15 and 20-27, as measured:
// with bit 0 of the spread depending on the key half of these passes conflict).  Either then covers all banks once.
__device__ __forceinline__ int spread(int key) { return ((key >> 1) & 1) << 2 | ((key >> 2) & 1) << 1; }

constexpr int kDim = 256, kRows = 16, kWaves = 8, kThreads = 64 * kWaves;  // query rows (x heads of a group) per wave
constexpr int kTileBytes = kTileK * kDim * 2;               // one staged tile of K or of V
constexpr int kRegions = kTileBytes / 1024 / kWaves;        // regions of a tile that one wave copies: keys 8 w .. 8 w + 7
constexpr int kKeyGroup = 16 * kDim * 2;                    // bytes from 16 keys to the next 16
constexpr int kQ = 2 * (kDim / 32), kP = kDim / 16;         // MFMAs of a half's scores (two subtiles) and of its products
constexpr int kLdsBytes = 4 * kTileBytes;                   // two tiles of K, two of V
static_assert(tile_rows(kDim) == kRows * kWaves && kRegions == kDim / 64, "a workgroup's rows, and a wave's keys");

// Accumulation registers by number, all 104 of them, as in tile32_body.h: O^T of 16-dim tile dt, Q^T of k-step t, the normaliser, ones.
constexpr int acc_o(int dt) { return 4 * dt; }
constexpr int acc_q(int t) { return kDim / 4 + 4 * t; }
constexpr int kAccL = kDim / 4 + kDim / 8, kAccOnes = kAccL + 4;

// s (vector registers) = a * Q^T(0), or += a * Q^T(T)
template <int T>
__device__ __forceinline__ void mfma_qk(f32x4& s, const u32x4 a) {
  constexpr int R = acc_q(T);
  if constexpr (T == 0) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, a[%2:%3], 0" : "=&v"(s) : "v"(a), "n"(R), "n"(R + 3) : IC_ACC_104);
  else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, a[%2:%3], %0" : "+v"(s) : "v"(a), "n"(R), "n"(R + 3) : IC_ACC_104);
}
// O^T(DT) += v * p
template <int DT>
__device__ __forceinline__ void mfma_pv(const bf16x8 v, const bf16x8 p) {
  constexpr int R = acc_o(DT);
  asm volatile("v_mfma_f32_16x16x32_bf16 a[%2:%3], %0, %1, a[%2:%3]" ::"v"(v), "v"(p), "n"(R), "n"(R + 3) : IC_ACC_104);
}
// Normaliser += the weights of p, as rounded (a product with ones: every row of the result is the sum of a column's 32
// weights).  kFirst: of a step, whose weights are summed by themselves before they join the running total.
template <bool kFirst>
__device__ __forceinline__ void normaliser(const bf16x8 p) {
  if constexpr (kFirst) asm volatile("v_mfma_f32_16x16x32_bf16 a[%1:%2], a[%3:%4], %0, 0" ::"v"(p), "n"(kAccL), "n"(kAccL + 3), "n"(kAccOnes), "n"(kAccOnes + 3) : IC_ACC_104);
  else asm volatile("v_mfma_f32_16x16x32_bf16 a[%1:%2], a[%3:%4], %0, a[%1:%2]" ::"v"(p), "n"(kAccL), "n"(kAccL + 3), "n"(kAccOnes), "n"(kAccOnes + 3) : IC_ACC_104);
}

// The 8 scores of a lane become weights in 12 operations of two instructions (the last kind one): kind 0 the exponents of pair j,
// 1 their exponentials, 2 rounding to bf16.  K counts them in an order that keeps each a pair behind the one it needs.
template <int K>
__device__ __forceinline__ void weight_op(f32x4 (&s)[2], bf16x8& pw, float negm, float sc) {
  constexpr int kind = K < 2 ? 0 : K == 2 ? 1 : K < 9 ? (K - 3) % 3 : K == 9 ? 1 : 2;
  constexpr int j = K < 2 ? K : K == 2 ? 0 : K < 9 ? (K - 3) / 3 + 2 - kind : K == 9 ? 3 : K - 8;
  constexpr int u = j / 2, i = 2 * (j % 2);
  if constexpr (kind == 0) {
    s[u][i] = __builtin_fmaf(s[u][i], sc, negm);
    s[u][i + 1] = __builtin_fmaf(s[u][i + 1], sc, negm);
  } else if constexpr (kind == 1) {
    s[u][i] = __builtin_amdgcn_exp2f(s[u][i]);
    s[u][i + 1] = __builtin_amdgcn_exp2f(s[u][i + 1]);
  } else {
    pw[2 * j] = (__bf16)s[u][i];
    pw[2 * j + 1] = (__bf16)s[u][i + 1];
  }
}

// One TileItem x one group of (1 << p.tile_g_shift) query heads that share a K/V head, executed by a workgroup of kWaves
// waves (see tile32_body() for the row mapping and for the steps, which are the same).  lds: kLdsBytes, 1 KiB aligned.
__device__ __forceinline__ void tile16_body(const AttnParams& p, const TileItem& it, int th, uint16_t* lds) {
  const int32_t offs = first_offsets(p);
  constexpr int D = kDim, kS = kQ + kP, kR = kRegions;
  typedef __attribute__((address_space(3))) const char lds_char;
  typedef __attribute__((address_space(3))) const u32x4 lds_u32x4;
  typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
  const int H = p.num_heads, Hk = p.num_kv_heads, gs = p.tile_g_shift;
  const int head0 = th << gs;
  const int kvh = head0 / p.group;
  const int n_rows_t = it.n_rows << gs;  // rows of the tile: query rows x heads of the group
  const int lane = here();
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int col = lane & 15, g = lane >> 4;

  // row of the tile (dead rows mirror the last live one), and the last key it sees
  auto row_of = [&](int ln) { return min(kRows * w + (ln & 15), n_rows_t - 1); };
  auto pos_of = [&](int ln) { return it.pos0 + (row_of(ln) >> gs); };
  const int wave_pos_lo = it.pos0 + min((kRows * w) >> gs, it.n_rows - 1);
  const int wave_pos_hi = it.pos0 + min((kRows * w + kRows - 1) >> gs, it.n_rows - 1);
  const float sc = p.scale_log2e;

  // ---- this wave's Q^T, beside the block ids and before the first copy (see tile32_body.h)
  const int r = row_of(lane);
  const int head = head0 + (r & ((1 << gs) - 1));
  const uint16_t* qp = p.q + ((int64_t)(it.qrow0 + (r >> gs)) * H + head) * D + 8 * g;
  u32x4 q[D / 32];
#pragma unroll
  for (int t = 0; t < D / 32; ++t) q[t] = *(const u32x4*)(qp + 32 * t);

  // ---- keys and values: this wave copies keys 8 w .. 8 w + 7 of every tile, half of block w / 2 of the tile's four
  typedef __attribute__((address_space(4))) const int32_t const_i32;
  const_i32* bt = (const_i32*)(p.bt_flat + table_start(p, offs, it.seq));
  const int last_blk = (it.k_end - 1) / kBlockSize;   // last table entry this item may touch
  const int n_tiles = (it.k_end - it.k_begin + kTileK - 1) / kTileK;
  constexpr int kBlockBytes = kBlockSize * D * 2;     // one (K or V, head) tile of a block
  const uint32_t blk_stride = 2u * (uint32_t)Hk * kBlockBytes;
  const char* const kbase = (const char*)p.pool + (int64_t)kvh * kBlockBytes;
  const int64_t vplane = (int64_t)Hk * kBlockBytes;
  const int my_key = 8 * (w & 1) + (lane >> 3);       // inside the block
  const uint32_t lane_off = (uint32_t)(my_key * (D * 2) + ((lane & 7) ^ spread(my_key)) * 16);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)lds;
  const uint32_t my_lds = lds0 + (uint32_t)(kR * w) * 1024u;
  constexpr int kVBuf = 2 * kTileBytes;               // the two buffers of V follow those of K
  // Tiles past the item's end re-read its last block and are never used.
  auto block_id = [&](int t) { return bt[min((it.k_begin + t * kTileK) / kBlockSize + w / 2, last_blk)]; };
  auto copy_tile = [&](int id, int64_t plane, int buf) __attribute__((always_inline)) {
    const char* b = kbase + plane + (uint64_t)(uint32_t)id * blk_stride;
#pragma unroll
    for (int j = 0; j < kR; ++j) copy_region(b + 128 * j, lane_off, my_lds + (uint32_t)(buf + 1024 * j));
  };
  int id_u = block_id(0), id_1 = block_id(1), id_2 = block_id(2);  // blocks of tiles u, u + 1, u + 2
#pragma unroll
  for (int s = 0; s < D / 32; ++s) asm volatile("" ::"v"(q[s]));  // waits
  copy_tile(id_u, 0, 0);
  if (n_tiles > 1) copy_tile(id_1, 0, kTileBytes);
  copy_tile(id_u, vplane, kVBuf);

  // ---- Q^T, O^T = 0, normaliser = 0
  {
    tile32::acc_mine<128>();
    unroll<D / 4>([&](auto i) __attribute__((always_inline)) { tile32::acc_write<decltype(i)::value>(0u); });
    unroll<D / 8>([&](auto i) __attribute__((always_inline)) {
      constexpr int e = decltype(i)::value;
      tile32::acc_write<acc_q(0) + e>(q[e / 4][e % 4]);
    });
    unroll<4>([&](auto i) __attribute__((always_inline)) {
      tile32::acc_write<kAccL + decltype(i)::value>(0u);
      tile32::acc_write<kAccOnes + decltype(i)::value>(0x3f803f80u);
    });
    tile32::acc_mine<128>();
  }
  float m = kNegBig;                    // reference of the weights, in log2 units
  float l = 0.f;                        // normaliser of this lane's column, without the last step's sums
  float top = -__builtin_inff();        // this lane's largest raw score in the half that is weighed next
  f32x4 sa[2], sb[2];                   // scores of even and odd halves, two subtiles each
  bf16x8 pa = {}, pb = {};              // weights of even and odd halves
#pragma unroll
  for (int u = 0; u < 2; ++u) sa[u] = sb[u] = (f32x4){0.f, 0.f, 0.f, 0.f};

  // Operand reads.  K (MFMA i of a half: subtile i % 2, k-step i / 2): keys 16 (i % 2) + col, dims 32 (i / 2) + 8 g ..+7.
  // V (transpose load, see read_vt16): dims 16 dt ..+15 of the 32 keys of half h.
  lds_char* const lb = (lds_char*)lds;
  lds_char* const k_row = lb + (col >> 3) * (kR * 1024) + (col & 7) * 128;
  lds_char* k_at[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) k_at[c] = k_row + ((4 * c + g) ^ spread(col)) * 16;
  auto read_k = [&](int i, int at) __attribute__((always_inline)) {
    return *(lds_u32x4*)(k_at[(i >> 1) & 1] + at + (i & 1) * kKeyGroup + (i >> 2) * 1024);
  };
  const int vj = lane & 15, vk = 4 * g + (vj >> 2);
  lds_char* v_at[4];  // [dt & 3]
#pragma unroll
  for (int o = 0; o < 4; ++o)
    v_at[o] = lb + kVBuf + (vk >> 3) * (kR * 1024) + (vk & 7) * 128 + ((2 * o + ((vj >> 1) & 1)) ^ spread(vk)) * 16 + (vj & 1) * 8;
  auto read_v = [&](int dt, int h, int at) __attribute__((always_inline)) {
    lds_char* const a = v_at[dt & 3] + at + 2 * h * kKeyGroup + (dt >> 2) * 1024;
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)a);
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(a + kKeyGroup));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  };

  const int n_half = wave_pos_hi < it.k_begin ? 0 : min(2 * n_tiles, (wave_pos_hi - it.k_begin) / 32 + 1);  // halves this wave sees
  u32x4 kop[kQ];    // K operands; the first four are read at the end of the stage before
  bf16x8 vop[kP];   // V operands
  auto must_move = [&]() { return __builtin_amdgcn_ballot_w64(top * sc > m + kLazyLog2) != 0; };
  auto move = [&]() __attribute__((always_inline)) {  // the factor of what has the reference before
    float t = __builtin_fmaxf(top, tile32::from_lane(top, here() ^ 16));
    t = __builtin_fmaxf(t, tile32::from_lane(t, here() ^ 32));
    const float cand = __builtin_fmaxf(m, t * sc);
    const bool grew = cand > m + kLazyLog2;  // the same in the four lanes of a column
    const float alpha = grew ? __builtin_amdgcn_exp2f(m - cand) : 1.0f;
    m = grew ? cand : m;
    return alpha;
  };
  auto rescale = [&](float alpha) __attribute__((always_inline)) {
    tile32::acc_settle<128>();
    unroll<D / 16>([&](auto ci) __attribute__((always_inline)) {
      constexpr int c = 4 * decltype(ci)::value;
      float x[4];
      unroll<4>([&](auto e) __attribute__((always_inline)) { x[decltype(e)::value] = tile32::acc_read<c + decltype(e)::value>(); });
      unroll<4>([&](auto e) __attribute__((always_inline)) { tile32::acc_write<c + decltype(e)::value>(__builtin_bit_cast(uint32_t, x[decltype(e)::value] * alpha)); });
    });
    l *= alpha;
    tile32::acc_write<kAccL>(__builtin_bit_cast(uint32_t, tile32::acc_read<kAccL>() * alpha));
    tile32::acc_settle<128>();
  };
  auto sum_up = [&]() __attribute__((always_inline)) {  // a step's sums join the normaliser
    tile32::acc_settle<128>();
    l += tile32::acc_read<kAccL>();
    tile32::acc_write<kAccL>(0u);  // the next normaliser() is a barrier away
  };
  auto next_ids = [&](int u) __attribute__((always_inline)) {
    id_u = id_1;
    id_1 = id_2;
    id_2 = block_id(u + 3);
  };
  auto hide = [&](f32x4 (&s)[2], int k0) __attribute__((always_inline)) {  // scores of keys past the lane's row; returns the largest left
    const int ln = here();
    const int room = pos_of(ln) - k0 - 4 * (ln >> 4);
    asm volatile("" ::: "memory");  // keeps the caller's condition a branch instead of always-on selects
    float t = -__builtin_inff();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      s[i / 4][i % 4] = 16 * (i / 4) + (i % 4) > room ? -__builtin_inff() : s[i / 4][i % 4];
      t = __builtin_fmaxf(t, s[i / 4][i % 4]);
    }
    return t;
  };
  auto largest = [&](const f32x4 (&s)[2]) __attribute__((always_inline)) {
    float t = -__builtin_inff();
#pragma unroll
    for (int i = 0; i < 8; ++i) t = __builtin_fmaxf(t, s[i / 4][i % 4]);
    return t;
  };
  auto products = [&](auto half_tag, const bf16x8& pw, int at) __attribute__((always_inline)) {  // operands four MFMAs ahead
    constexpr int kHalf = decltype(half_tag)::value;
    bf16x8 v[kP];
    auto operand = [&](auto vi) __attribute__((always_inline)) { v[decltype(vi)::value] = read_v(decltype(vi)::value, kHalf, at); };
    unroll<4>(operand);
    pin();
    unroll<kP>([&](auto ii) __attribute__((always_inline)) {
      constexpr int i = decltype(ii)::value;
      mfma_pv<i>(v[i], pw);
      if constexpr (i + 4 < kP) operand(std::integral_constant<int, i + 4>{});
      pin();
    });
  };
  auto serial_step = [&](int u) __attribute__((always_inline)) {
    const int par = (u & 1) * kTileBytes, other = par ^ kTileBytes;
    const int kt = it.k_begin + u * kTileK;
    const int n_valid = it.k_end - (kt - kTileK);
    if (u >= n_tiles - 1 && u > 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no copy follows V of tile u - 1
    if (n_valid < kTileK) {  // dead slots of that tile: zero (0 * NaN would poison the product)
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      const int at = here();
      if (8 * w + (at >> 3) >= n_valid) {
#pragma unroll
        for (int j = 0; j < kR; ++j)
          *(__attribute__((address_space(3))) u32x4*)(uintptr_t)(my_lds + (uint32_t)(kVBuf + other + 1024 * j) + 16 * at) = (u32x4){0u, 0u, 0u, 0u};
      }
    }
    if (u == 0 && n_tiles > 1) barrier<2 * kR>();  // K of the second tile and V of the first may be on their way
    else barrier<kR>();
    const int vt = n_tiles == 2 ? u + 1 : u;  // (no third tile needs the wait for V of the second to be by count)
    if (vt > 0 && vt < n_tiles) copy_tile(vt == u ? id_u : id_1, vplane, __builtin_amdgcn_readfirstlane(kVBuf + (vt & 1) * kTileBytes));
    if (u > 0 && 2 * u - 2 < n_half) {
      products(std::integral_constant<int, 0>{}, pa, other);
      normaliser<false>(pa);
      if (kt - 1 > wave_pos_lo) top = hide(sb, kt - 32);
      if (must_move()) rescale(move());
      unroll<12>([&](auto k) __attribute__((always_inline)) { weight_op<decltype(k)::value>(sb, pb, -m, sc); });
      asm volatile("s_nop 3" : "+v"(pb));
      products(std::integral_constant<int, 1>{}, pb, other);
      normaliser<false>(pb);
      sum_up();
    }
    if (u == n_tiles) return;
    if (2 * u < n_half) {
      u32x4 ka[kQ], kb[kQ];
      unroll<3>([&](auto ii) __attribute__((always_inline)) {
        ka[decltype(ii)::value] = read_k(decltype(ii)::value, par);
        kb[decltype(ii)::value] = read_k(decltype(ii)::value, par + 2 * kKeyGroup);
      });
      pin();
      unroll<kQ>([&](auto ii) __attribute__((always_inline)) {
        constexpr int i = decltype(ii)::value;
        mfma_qk<i / 2>(sa[i % 2], ka[i]);
        mfma_qk<i / 2>(sb[i % 2], kb[i]);
        if constexpr (i + 3 < kQ) {
          ka[i + 3] = read_k(i + 3, par);
          kb[i + 3] = read_k(i + 3, par + 2 * kKeyGroup);
        }
        pin();
      });
      asm volatile("s_nop 15" : "+v"(sa[0]), "+v"(sa[1]), "+v"(sb[0]), "+v"(sb[1]));
      float first;
      if (kt + kTileK - 1 > wave_pos_lo) {
        first = hide(sa, kt);
        top = hide(sb, kt + 32);
      } else {
        first = largest(sa);
        top = largest(sb);
      }
      // Lazy reference, as in tile32_body.h; here from the largest of 64 scores.
      const float second = top;
      top = __builtin_fmaxf(top, first);
      if (must_move()) {
        const float alpha = move();
        if (u > 0) rescale(alpha);  // (before, there is nothing to rescale)
      }
      top = second;
      unroll<12>([&](auto k) __attribute__((always_inline)) { weight_op<decltype(k)::value>(sa, pa, -m, sc); });
      asm volatile("s_nop 3" : "+v"(pa));
    }
    // No tile to publish, and no copy into the buffer that this one leaves.  (From three tiles on the last step is some waves' fast one,
    // which has the barrier; the waves of a workgroup must meet at the same ones.)
    if (n_tiles <= 2 && u + 1 == n_tiles) return;
    barrier<kR>();
    if (u + 2 < n_tiles) copy_tile(id_2, 0, par);
    next_ids(u);
  };

  // Operands are read four MFMAs ahead (an MFMA is half as long as the 32-row shape's).
  auto fast_stage = [&](auto half_tag, auto par_tag, int u, f32x4 (&scur)[2], f32x4 (&snext)[2], bf16x8& pcur, bf16x8& pprev) __attribute__((always_inline)) {
    constexpr int kHalf = decltype(half_tag)::value, kPar = decltype(par_tag)::value;
    constexpr int kAt = kPar * kTileBytes + kHalf * 2 * kKeyGroup;
    constexpr int kNextAt = kHalf == 0 ? kAt + 2 * kKeyGroup : (kPar ^ 1) * kTileBytes;
    constexpr int kVAt = (kPar ^ 1) * kTileBytes;
    const bool moved = must_move();
    float alpha = 1.f;
    if (__builtin_expect(moved, 0)) alpha = move();
    const float negm = -m;
    auto weights = [&](auto slot) __attribute__((always_inline)) {  // this slot's share of the 12 operations
      constexpr int a = decltype(slot)::value * 12 / kS, b = (decltype(slot)::value + 1) * 12 / kS;
      unroll<b - a>([&](auto k) __attribute__((always_inline)) { weight_op<a + decltype(k)::value>(scur, pcur, negm, sc); });
    };
    auto operand_v = [&](auto vi) __attribute__((always_inline)) { vop[decltype(vi)::value] = read_v(decltype(vi)::value, kHalf, kVAt); };
    pin();
    unroll<kQ>([&](auto ii) __attribute__((always_inline)) {
      constexpr int i = decltype(ii)::value;
      if constexpr (i == kQ - 4) {
        barrier<kR>();
        pin();
      }
      if constexpr (i % 2 == 0) asm volatile("" ::"v"(kop[i]), "v"(kop[i + 1]));  // one wait for the two
      mfma_qk<i / 2>(snext[i % 2], kop[i]);
      if constexpr (i % 2 == 0 && i + 4 < kQ) {
        kop[i + 4] = read_k(i + 4, kAt);
        kop[i + 5] = read_k(i + 5, kAt);
      }
      if constexpr (i >= kQ - 4) operand_v(std::integral_constant<int, i - (kQ - 4)>{});
      if constexpr (kHalf == 0 && i == kQ - 2) l += tile32::acc_read<kAccL>();  // the step before
      weights(ii);
      pin();
    });
    unroll<kP>([&](auto ii) __attribute__((always_inline)) {
      constexpr int i = decltype(ii)::value;
      if constexpr (i % 2 == 0) asm volatile("" ::"v"(vop[i]), "v"(vop[i + 1]));
      mfma_pv<i>(vop[i], pprev);
      if constexpr (i == kP - 1) normaliser<kHalf == 0>(pprev);
      if constexpr (i % 2 == 0 && i + 4 < kP) {
        operand_v(std::integral_constant<int, i + 4>{});
        operand_v(std::integral_constant<int, i + 5>{});
      }
      if constexpr (i == 0 && kHalf == 0) copy_tile(id_u, vplane, kVBuf + kPar * kTileBytes);
      if constexpr (i == 0 && kHalf == 1) {
        copy_tile(id_2, 0, kPar * kTileBytes);
        next_ids(u);
      }
      if constexpr (i >= kP - 4) kop[i - (kP - 4)] = read_k(i - (kP - 4), kNextAt);
      weights(std::integral_constant<int, kQ + i>{});
      constexpr int m0 = kP / 2;  // the largest score of half h + 1, four pairs over the last slots
      if constexpr (i >= m0) {
        if constexpr (i == m0) top = -__builtin_inff();
#pragma unroll
        for (int k = (i - m0) * 4 / (kP - m0); k < (i - m0 + 1) * 4 / (kP - m0); ++k) top = __builtin_fmaxf(__builtin_fmaxf(top, snext[k / 2][2 * (k % 2)]), snext[k / 2][2 * (k % 2) + 1]);
      }
      pin();
    });
    asm volatile("" : "+v"(pcur), "+v"(top));  // are worked out here, not in the next stage, where they are used
    if (__builtin_expect(moved, 0)) rescale(alpha);  // the products so far have the old reference, those of half h the new one
  };

  // Steps 1 .. fast_end of this wave have three full parts in both stages, nothing to hide and a whole tile of V to publish.
  const int fast_end = min(min((n_half - 2) >> 1, (wave_pos_lo - it.k_begin - 31) >> 6), (it.k_end - it.k_begin) >> 6);
  constexpr std::integral_constant<int, 0> A{}, even{};
  constexpr std::integral_constant<int, 1> B{}, odd{};
  for (int u = 0; u <= n_tiles;) {
    serial_step(u);
    ++u;
    if (u + 1 <= fast_end) {
#pragma unroll
      for (int i = 0; i < 4; ++i) kop[i] = read_k(i, kTileBytes);
      do {
        fast_stage(A, odd, u, sb, sa, pb, pa);
        fast_stage(B, odd, u, sa, sb, pa, pb);
        fast_stage(A, even, u + 1, sb, sa, pb, pa);
        fast_stage(B, even, u + 1, sa, sb, pa, pb);
        u += 2;
      } while (u + 1 <= fast_end);
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // copies still in flight write LDS that the next item uses

  // ---- epilogue: lane holds O^T[d][col] for d = 16 dt + 4 g + i
  tile32::acc_settle<128>();
  const float lsum = l + tile32::acc_read<kAccL>();
  const int lane_e = here();
  const int r_e = kRows * w + (lane_e & 15), d0 = 4 * (lane_e >> 4);
  if (r_e < n_rows_t) {
    const int qr = r_e >> gs;
    const int head = head0 + (r_e & ((1 << gs) - 1));
    if (it.slot0 < 0) {
      const float inv = 1.0f / lsum;
      uint16_t* op = p.out + ((int64_t)(it.qrow0 + qr) * H + head) * D;
      unroll<kP>([&](auto ci) __attribute__((always_inline)) {
        constexpr int c = decltype(ci)::value;
        bf16x4 o;
        unroll<4>([&](auto e) __attribute__((always_inline)) { o[decltype(e)::value] = (__bf16)(tile32::acc_read<4 * c + decltype(e)::value>() * inv); });  // round to nearest even
        *(bf16x4*)(op + 16 * c + d0) = o;
      });
    } else {
      const int64_t ps = (int64_t)(it.slot0 + qr * it.nparts) * H + head;
      float* op = p.part_o + ps * D;
      unroll<kP>([&](auto ci) __attribute__((always_inline)) {
        constexpr int c = decltype(ci)::value;
        f32x4 o;
        unroll<4>([&](auto e) __attribute__((always_inline)) { o[decltype(e)::value] = tile32::acc_read<4 * c + decltype(e)::value>(); });
        *(f32x4*)(op + 16 * c + d0) = o;
      });
      if (d0 == 0) {
        p.part_ml[ps * 2] = m;
        p.part_ml[ps * 2 + 1] = lsum;
      }
    }
  }
}

}  // namespace tile16
}  // namespace ic
