// Tile path of the attention kernels: the query rows of a recomputation chunk (Section 4.2) against a range of their
// sequence's paged keys.  Here QK^T and PV are dense contractions (hundreds of rows share every
// key), so they run on the matrix cores: v_mfma_f32_32x32x16_bf16, fp32 accumulation.  (The kernels use this body for
// head_dim 64 and 128; head_dim 256 runs tile16_body.h, where a wave takes 16 rows.)
//
// One workgroup = one TileItem x one head group (one head with multi-head attention; with grouped
// queries the G heads that share a K/V head): up to tile_rows(D) rows = query rows x heads of the
// group, one wave per 32 rows, two waves per SIMD.
//   - S^T = K Q^T: A operand = 32 keys x 16 dims from LDS, B operand = this wave's Q^T kept in accumulation
//     registers for the whole item.  In the 32x32 accumulator layout every lane then owns ONE
//     query column (lane % 32) and 16 of the 32 keys.
//   - O^T += V^T P^T: the accumulator registers of S^T, rounded to bf16, already ARE the B
//     operand (8 keys per lane per MFMA, slot j of lane half hl <-> key 8*(j/4) + 4*hl + j%4).
//     V stays [key][dim] in LDS; the A operand (one dim, 8 keys per lane, in that key order) comes
//     from two ds_read_b64_tr_b16 transpose loads, so no register transposition is needed.
//   - The normaliser is one more product of the same P^T, with ones (normaliser(), below).
//   - Causality: query row r of the item sits at position pos0 + r and sees keys <= that position.
//     Only halves of a tile that straddle a wave's diagonal are masked; what lies beyond it is skipped.
// Dead slots (keys >= k_end, possibly NaN) get score -inf by select and V = 0 in LDS.
//
// What bounds it: the rate at which a wave issues (one instruction per 6 to 8 cycles from one wave, one vector instruction per 4 from
// two) beside 32 cycles a MFMA, and on N(0,1) data the power cap.  So:
//   - The work of three consecutive halves of a tile (32 keys) runs in one instruction stream: the scores of half h + 1, the
//     weights of half h and the products of half h - 1, dealt out slot by slot (one MFMA, its share of the weights, its LDS
//     reads) and pinned there.  With the three one after the other, two waves of a SIMD that reach them together leave the
//     matrix pipe idle while both are in the weights.
//   - No dot-product instructions: v_dot2_f32_bf16 waits for the MFMAs in flight to leave the matrix pipe and holds the next
//     one back (a probe of two waves: MFMA + 4 fma 33 cycles, MFMA + 2 dot2 53).
//   - K and V go from the pool straight into LDS (copy_region()): no registers, no LDS writes and no wait in the stream.
// O^T and Q^T live in accumulation registers that are named by number (acc_o, acc_q): as values of the program the compiler
// moved them to vector registers and back around every branch of the key loop, 64 moves a half.
// Tried: 64 query rows per wave, one wave per SIMD (half the LDS reads per MFMA; 9.03 ms on all-zero data where two waves of 32 rows take
// 7.43 in the old schedule: one wave cannot issue enough).
// Measured, before (registers to LDS, weights between the products) and now: 16 chunks of 2048 rows on 16384 keys, 32 heads of 128,
// 9.92 -> 8.2 ms (942 -> 1140 TFLOP/s; all-zero data 7.43 -> 5.79 ms), 8 chunks of 512 on 1024..4096, 64 heads over 8, 395 -> 350 us;
// beside decode rows the long-context call 10.78 -> 9.6-9.75 ms, the grouped one 498 -> 452 us.
#pragma once

#include <type_traits>
#include <utility>

#include "tile_body.h"

namespace ic {
namespace tile32 {

using namespace tilep;

// Staged tiles: 64 keys of K, or of V, as 1 KiB regions of 8 keys x 64 dims, region (key / 8) * (D / 64) + dim / 64.  A region is what
// one wave copies with one load (lane i: key i / 8 and one 16-byte chunk of its eight: whole 128-byte lines), so its bytes are 64
// consecutive lanes' and cannot be padded; chunk c of key k sits at chunk c ^ spread(k) of the key's 128 bytes instead, which puts the 16
// keys of a K operand, and the 4 keys x 64 bytes of a V operand, that are read together on all 64 banks.  Operand reads are a
// lane's base address plus a constant.
__device__ __forceinline__ int spread(int key) { return ((key >> 1) & 1) << 2 | ((key >> 2) & 3); }

template <int D>
struct G32 {
  static constexpr int kWaves = tile_rows(D) / 32;
  static constexpr int kThreads = 64 * kWaves;
  static constexpr int kTileBytes = kTileK * D * 2;                    // one staged tile of K or of V
  static constexpr int kRegions = kTileBytes / 1024 / kWaves;          // regions of a tile that one wave copies
  static constexpr int kKeyGroup = (D / 32) * 1024;                    // bytes from 16 keys to the next 16
  static constexpr int kQSteps = D / 16;                               // MFMA k-steps of Q K^T
  static constexpr int kDTiles = D / 32;                               // 32-row tiles of O^T
  static_assert(kWaves == 8 && kRegions == D / 64, "wave w copies keys 8 w .. 8 w + 7");
};

template <int D>
constexpr int tile32_lds_bytes() {
  return 4 * G32<D>::kTileBytes;  // two tiles of K, two of V
}

__device__ __forceinline__ void pin() { __builtin_amdgcn_sched_barrier(0); }
template <class F, int... I>
__device__ __forceinline__ void each(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void unroll(F&& f) {
  each(f, std::make_integer_sequence<int, N>{});
}

// Accumulation registers, by number: O^T of 32-dim tile dt, Q^T of k-step s, the normaliser and its ones.  Every MFMA names all of
// them as clobbered, so the compiler keeps nothing of its own in them while a tile item runs (the test-suite reads the
// listing).  It does not know either that an MFMA writes them, nor what the scores' MFMAs write in vector registers: what reads those is
// at least an acc_settle() or four MFMAs behind.
template <int D> constexpr int acc_o(int dt) { return 16 * dt; }
template <int D> constexpr int acc_q(int s) { return D / 2 + 4 * s; }
template <int D> constexpr int acc_l() { return D / 2 + D / 4; }
template <int D> constexpr int acc_ones() { return D / 2 + D / 4 + 4; }

#define IC_A10(n) "a" #n "0", "a" #n "1", "a" #n "2", "a" #n "3", "a" #n "4", "a" #n "5", "a" #n "6", "a" #n "7", "a" #n "8", "a" #n "9"
#define IC_ACC_56 "a0", "a1", "a2", "a3", "a4", "a5", "a6", "a7", "a8", "a9", IC_A10(1), IC_A10(2), IC_A10(3), IC_A10(4), \
                  "a50", "a51", "a52", "a53", "a54", "a55"
#define IC_ACC_104 IC_ACC_56, "a56", "a57", "a58", "a59", IC_A10(6), IC_A10(7), IC_A10(8), IC_A10(9), "a100", "a101", "a102", "a103"

// s (vector registers) = a * Q^T(0), or += a * Q^T(S)
template <int D, int S>
__device__ __forceinline__ void mfma_qk(f32x16& s, const u32x4 a) {
  constexpr int R = acc_q<D>(S);
  if constexpr (D == 128) {
    if constexpr (S == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, a[%2:%3], 0" : "=&v"(s) : "v"(a), "n"(R), "n"(R + 3) : IC_ACC_104);
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, a[%2:%3], %0" : "+v"(s) : "v"(a), "n"(R), "n"(R + 3) : IC_ACC_104);
  } else {
    if constexpr (S == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, a[%2:%3], 0" : "=&v"(s) : "v"(a), "n"(R), "n"(R + 3) : IC_ACC_56);
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, a[%2:%3], %0" : "+v"(s) : "v"(a), "n"(R), "n"(R + 3) : IC_ACC_56);
  }
}
// O^T(DT) += v * p
template <int D, int DT>
__device__ __forceinline__ void mfma_pv(const bf16x8 v, const bf16x8 p) {
  constexpr int R = acc_o<D>(DT);
  if constexpr (D == 128) asm volatile("v_mfma_f32_32x32x16_bf16 a[%2:%3], %0, %1, a[%2:%3]" ::"v"(v), "v"(p), "n"(R), "n"(R + 15) : IC_ACC_104);
  else asm volatile("v_mfma_f32_32x32x16_bf16 a[%2:%3], %0, %1, a[%2:%3]" ::"v"(v), "v"(p), "n"(R), "n"(R + 15) : IC_ACC_56);
}
// Normaliser += the weights of p, as rounded: it counts exactly what the matrix core multiplies, so the output stays an exact convex
// combination of the values.  p is the B operand of the 32x32x16 shape (lane: column lane % 32, keys by lane / 32); read as the B operand of
// 16x16x32 its four groups of 16 lanes are four groups of 8 keys, of which the even ones hold columns 0..15 and the odd ones
// columns 16..31.  A row of the A operand that is 1 for the even (odd) groups and 0 for the others gives the sums of one half of
// the columns: even result rows columns 0..15, odd rows columns 16..31, so every lane gets both in its first two results.
// 0 times a weight of the other half is 0 because every weight is finite (see move()).
// 16 cycles of the matrix pipe for 16 keys, and no vector instruction.  (Without zeros: the two operands of a half regrouped by columns with
// v_permlane16_swap_b32, or the 4x4x4 shape, in which a lane gets the sum of its own weights, cost the grouped and the
// long-context call 1 to 3 %.)  kFirst: of a step (64 keys), whose weights are summed by themselves before they join the running
// total: that is then rounded once a step.
template <int D, bool kFirst>
__device__ __forceinline__ void normaliser(const bf16x8 p) {
  constexpr int L = acc_l<D>(), A = acc_ones<D>();
  if constexpr (D == 128) {
    if constexpr (kFirst) asm volatile("v_mfma_f32_16x16x32_bf16 a[%1:%2], a[%3:%4], %0, 0" ::"v"(p), "n"(L), "n"(L + 3), "n"(A), "n"(A + 3) : IC_ACC_104);
    else asm volatile("v_mfma_f32_16x16x32_bf16 a[%1:%2], a[%3:%4], %0, a[%1:%2]" ::"v"(p), "n"(L), "n"(L + 3), "n"(A), "n"(A + 3) : IC_ACC_104);
  } else {
    if constexpr (kFirst) asm volatile("v_mfma_f32_16x16x32_bf16 a[%1:%2], a[%3:%4], %0, 0" ::"v"(p), "n"(L), "n"(L + 3), "n"(A), "n"(A + 3) : IC_ACC_56);
    else asm volatile("v_mfma_f32_16x16x32_bf16 a[%1:%2], a[%3:%4], %0, a[%1:%2]" ::"v"(p), "n"(L), "n"(L + 3), "n"(A), "n"(A + 3) : IC_ACC_56);
  }
}
template <int R>
__device__ __forceinline__ void acc_write(uint32_t v) {
  asm volatile("v_accvgpr_write_b32 a[%1], %0" ::"v"(v), "n"(R));
}
template <int R>
__device__ __forceinline__ float acc_read() {
  float v;
  asm volatile("v_accvgpr_read_b32 %0, a[%1]" : "=v"(v) : "n"(R));
  return v;
}
// Wait states between an MFMA and other accesses to its registers, and the other way round (the longest is 16 + 3).
template <int D>
__device__ __forceinline__ void acc_settle() {
  if constexpr (D == 128) asm volatile("s_nop 15\n\ts_nop 3" ::: "memory", IC_ACC_104);
  else asm volatile("s_nop 15\n\ts_nop 3" ::: "memory", IC_ACC_56);
}

// Lane numbers worked out where they are needed: kept across the key loop they would take registers.
__device__ __forceinline__ int here() {
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  return lane;
}
__device__ __forceinline__ float from_lane(float v, int lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(lane << 2, __builtin_bit_cast(int, v)));
}
__device__ __forceinline__ float other_half(float v) { return from_lane(v, here() ^ 32); }
__device__ __forceinline__ float largest_of(float a, float b) { return __builtin_elementwise_maximum(a, b); }  // NaN if one of them is

// Nothing of the compiler's own is in the accumulation registers from here on.
template <int D>
__device__ __forceinline__ void acc_mine() {
  if constexpr (D == 128) asm volatile("" ::: "memory", IC_ACC_104);
  else asm volatile("" ::: "memory", IC_ACC_56);
}

// One 16-byte piece per lane, 1 KiB per wave, from base + offset of the lane to LDS byte address lds_at + 16 * lane.  As assembly,
// because the compiler would make every LDS read wait for all such copies in flight; barrier() waits for them by count.  (clang warns
// that m0 is a reserved register, once a use; what it would put there of its own it has to know to be overwritten.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void copy_region(const char* base, uint32_t lane_off, uint32_t lds_at) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_at), "v"(lane_off), "s"(base) : "memory", "m0");
}
#pragma clang diagnostic pop
// Every wave's LDS reads before are done, and so are its copies but the last kPending.
template <int kPending>
__device__ __forceinline__ void barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(kPending) : "memory");
}

// The 16 scores of a lane become weights in 24 operations of two instructions (the last kind one): kind 0 the exponents of pair j,
// 1 their exponentials, 2 rounding to bf16 (one v_cvt_pk_bf16_f32).  K counts them in an order that keeps each a pair behind the one it needs.
template <int K>
__device__ __forceinline__ void weight_op(f32x16& s, bf16x8 (&pw)[2], float negm, float sc) {
  constexpr int kind = K < 2 ? 0 : K == 2 ? 1 : K < 21 ? (K - 3) % 3 : K == 21 ? 1 : 2;
  constexpr int j = K < 2 ? K : K == 2 ? 0 : K < 21 ? (K - 3) / 3 + 2 - kind : K == 21 ? 7 : K - 16;
  constexpr int i = 2 * j;
  if constexpr (kind == 0) {
    s[i] = __builtin_fmaf(s[i], sc, negm);
    s[i + 1] = __builtin_fmaf(s[i + 1], sc, negm);
  } else if constexpr (kind == 1) {
    s[i] = __builtin_amdgcn_exp2f(s[i]);
    s[i + 1] = __builtin_amdgcn_exp2f(s[i + 1]);
  } else {
    pw[i / 8][i % 8] = (__bf16)s[i];
    pw[i / 8][i % 8 + 1] = (__bf16)s[i + 1];
  }
}

// One TileItem x one group of (1 << p.tile_g_shift) query heads that share a K/V head, executed by a
// workgroup of tile_rows(D) / 32 waves.  th = index of the head group: its heads are
// th << shift .. ((th + 1) << shift) - 1.  Row r of the tile is query row r >> shift of the item for
// head (th << shift) + (r & mask): with multi-head attention (shift 0) a tile is 256 rows of one head,
// with grouped-query attention the heads of a group ride on one staging of their common keys.
// lds: at least tile32_lds_bytes<D>() bytes of workgroup LDS, 1 KiB aligned.
template <int D>
__device__ __forceinline__ void tile32_body(const AttnParams& p, const TileItem& it, int th, uint16_t* lds) {
  using G = G32<D>;
  constexpr int kQ = G::kQSteps, kP = 2 * G::kDTiles, kS = kQ + kP, kR = G::kRegions;
  const int32_t offs = first_offsets(p);
  typedef __attribute__((address_space(3))) const char lds_char;
  typedef __attribute__((address_space(3))) const u32x4 lds_u32x4;
  typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;

  const int H = p.num_heads;
  const int Hk = p.num_kv_heads;
  const int gs = p.tile_g_shift;
  const int head0 = th << gs;
  const int kvh = head0 / p.group;
  const int n_rows_t = it.n_rows << gs;               // rows of the tile: query rows x heads of the group
  const int lane = here();
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int col = lane & 31;  // query column of this lane inside the wave's 32 rows
  const int hl = lane >> 5;

  // row of the tile (dead rows mirror the last live one), and the last key it sees
  auto row_of = [&](int ln) { return min(32 * w + (ln & 31), n_rows_t - 1); };
  auto pos_of = [&](int ln) { return it.pos0 + (row_of(ln) >> gs); };
  const int wave_pos_lo = it.pos0 + min((32 * w) >> gs, it.n_rows - 1);        // smallest limit in the wave
  const int wave_pos_hi = it.pos0 + min((32 * w + 31) >> gs, it.n_rows - 1);   // largest limit in the wave
  const float sc = p.scale_log2e;

  // ---- this wave's Q^T, asked for beside the block ids and there before the first copy: loads return in order, and the compiler, which
  // does not know of the copies, waits for every load in flight.  Behind the copies the first scores waited for K of a second
  // tile and V of the first (2 rows and 2 chunks of 32, 4 heads of 64: 12.75 us a call, now 12.5; one 512-row chunk on 2500 keys, 64
  // heads over 8, two layers: 126.2, 124.5).  A call on a single tile copies no second one.
  const int r = row_of(lane);
  const int head = head0 + (r & ((1 << gs) - 1));
  const uint16_t* qp = p.q + ((int64_t)(it.qrow0 + (r >> gs)) * H + head) * D + 8 * hl;
  u32x4 q[kQ];
#pragma unroll
  for (int s = 0; s < kQ; ++s) q[s] = *(const u32x4*)(qp + 16 * s);

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
  constexpr int kVBuf = 2 * G::kTileBytes;            // the two buffers of V follow those of K
  // Tiles past the item's end re-read its last block and are never used.
  auto block_id = [&](int t) { return bt[min((it.k_begin + t * kTileK) / kBlockSize + w / 2, last_blk)]; };
  auto copy_tile = [&](int id, int64_t plane, int buf) __attribute__((always_inline)) {
    const char* b = kbase + plane + (uint64_t)(uint32_t)id * blk_stride;
#pragma unroll
    for (int j = 0; j < kR; ++j) copy_region(b + 128 * j, lane_off, my_lds + (uint32_t)(buf + 1024 * j));
  };
  int id_u = block_id(0), id_1 = block_id(1), id_2 = block_id(2);  // blocks of tiles u, u + 1, u + 2
#pragma unroll
  for (int s = 0; s < kQ; ++s) asm volatile("" ::"v"(q[s]));  // waits
  copy_tile(id_u, 0, 0);
  if (n_tiles > 1) copy_tile(id_1, 0, G::kTileBytes);
  copy_tile(id_u, vplane, kVBuf);

  // ---- Q^T, O^T = 0, normaliser = 0
  {
    acc_mine<D>();
    unroll<D / 2>([&](auto i) __attribute__((always_inline)) { acc_write<decltype(i)::value>(0u); });
    unroll<4 * kQ>([&](auto i) __attribute__((always_inline)) {
      constexpr int e = decltype(i)::value;
      acc_write<acc_q<D>(0) + e>(q[e / 4][e % 4]);
    });
    const uint32_t one = ((lane >> 4) & 1) == (lane & 1) ? 0x3f803f80u : 0u;
    unroll<4>([&](auto i) __attribute__((always_inline)) {
      acc_write<acc_l<D>() + decltype(i)::value>(0u);
      acc_write<acc_ones<D>() + decltype(i)::value>(one);
    });
    acc_mine<D>();
  }
  float m = kNegBig;                    // reference of the weights, in log2 units
  float l[2] = {0.f, 0.f};              // normalisers of columns lane % 16 and 16 + lane % 16, without the last step's sums
  float top = -__builtin_inff();        // this lane's largest raw score in the half that is weighed next
  f32x16 sa, sb;                        // scores of even and odd halves
  bf16x8 pa[2] = {}, pb[2] = {};        // weights of even and odd halves: P^T operands of their two k-steps
#pragma unroll
  for (int i = 0; i < 16; ++i) sa[i] = sb[i] = 0.f;

  // Operand reads.  K: keys 32 * half + col, dims 16 s + 8 hl ..+7.  V (transpose load: in each group of 16 lanes, lane i supplies the
  // address of an 8-byte row and receives column i % 4 of the rows supplied by lanes i / 4, i / 4 + 4, i / 4 + 8, i / 4 + 12; layout
  // measured on gfx950): lane j points at V[key j / 4][dims 4 (j % 4) ..+3] of its group's 16 dims, and two loads give the 8 keys in
  // accumulator order (slots 0-3: keys 4 hl ..+3, slots 4-7: keys 8 + 4 hl ..+3).
  lds_char* const lb = (lds_char*)lds;
  const int key = col & 15;
  lds_char* const k_row = lb + (col >> 4) * G::kKeyGroup + (key >> 3) * (kR * 1024) + (key & 7) * 128;
  lds_char* k_at[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) k_at[c] = k_row + ((2 * c + hl) ^ spread(key)) * 16;
  auto read_k = [&](int s, int at) __attribute__((always_inline)) { return *(lds_u32x4*)(k_at[s & 3] + at + (s >> 2) * 1024); };
  const int vj = lane & 15, vc = 2 * ((lane >> 4) & 1) + ((vj >> 1) & 1), vk = 4 * hl + (vj >> 2);
  lds_char* v_at[2][2];  // [dt & 1][keys vk, vk + 8]
#pragma unroll
  for (int o = 0; o < 2; ++o)
#pragma unroll
    for (int e = 0; e < 2; ++e) v_at[o][e] = lb + kVBuf + e * (kR * 1024) + vk * 128 + ((4 * o + vc) ^ spread(vk + 8 * e)) * 16 + (vj & 1) * 8;
  auto read_v = [&](int dt, int ksp, int at) __attribute__((always_inline)) {
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(v_at[dt & 1][0] + at + ksp * G::kKeyGroup + (dt >> 1) * 1024));
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(v_at[dt & 1][1] + at + ksp * G::kKeyGroup + (dt >> 1) * 1024));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  };

  // ---- Steps.  Step u has two barriers.  Barrier A publishes V of tile u - 1 (the first one K of tile 0) and frees the buffer of tile
  // u - 2, into which V of tile u is copied then; barrier B publishes K of tile u + 1 and frees the buffer of tile u for K of tile
  // u + 2.  So every copy has a whole step to arrive, and a wave waits for all but the last tile's worth (kR) it has issued.
  // Between them a wave does one of two things, whatever the others do:
  //   serial  A(u); products of tile u - 1, second half of its weights first; scores of tile u, weights of its first half; B(u)
  //   fast    scores of half 2 u | A(u) | weights of half 2 u - 1 | O += P(2 u - 2);  scores of half 2 u + 1 | B(u) | weights of half 2 u | O += P(2 u - 1),
  //           each of the two stages as one interleaved stream
  // Both start from the scores of half 2 u - 1 (sb) and the weights of half 2 u - 2 (pa) and leave those of the next tile.  The serial step
  // does the first and the last tiles, hidden keys and all; there is one copy of it, for a call on a few tiles is over before
  // more code has been fetched.
  const int n_half = wave_pos_hi < it.k_begin ? 0 : min(2 * n_tiles, (wave_pos_hi - it.k_begin) / 32 + 1);  // halves this wave sees
  u32x4 kop[kQ];    // K operands; the first two are read at the end of the stage before
  bf16x8 vop[kP];   // V operands
  auto must_move = [&]() { return __builtin_amdgcn_ballot_w64(!(top * sc <= m + kLazyLog2)) != 0; };
  // The factor of what has the reference before; s: the scores that are weighed next.  A column whose largest score is NaN or
  // overflows (a NaN or an infinity in its query row, or in a key that it sees) has no result: its factor is NaN, once, which its sums
  // and its normaliser keep, and these scores become -inf.  So no weight is ever NaN or infinite, and none gets into
  // another column's normaliser.
  auto move = [&](f32x16& s) __attribute__((always_inline)) {
    const float cand = largest_of(m, largest_of(top, other_half(top)) * sc);
    const bool bad = !(cand < __builtin_inff());  // the same in both lanes of a column
    const bool grew = cand > m + kLazyLog2 && !bad;
    float alpha = grew ? __builtin_amdgcn_exp2f(m - cand) : 1.0f;
    m = grew ? cand : m;
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(bad) != 0, 0)) {
      const float l0 = l[0], l1 = l[1], own = here() & 16 ? l1 : l0;
      if (bad && own == own) alpha = __builtin_nanf("");
#pragma unroll
      for (int i = 0; i < 16; ++i) s[i] = bad ? -__builtin_inff() : s[i];
    }
    return alpha;
  };
  auto rescale = [&](float alpha) __attribute__((always_inline)) {
    acc_settle<D>();
    unroll<D / 8>([&](auto ci) __attribute__((always_inline)) {
      constexpr int c = 4 * decltype(ci)::value;
      float x[4];
      unroll<4>([&](auto e) __attribute__((always_inline)) { x[decltype(e)::value] = acc_read<c + decltype(e)::value>(); });
      unroll<4>([&](auto e) __attribute__((always_inline)) { acc_write<c + decltype(e)::value>(__builtin_bit_cast(uint32_t, x[decltype(e)::value] * alpha)); });
    });
    const float a0 = from_lane(alpha, here() & 15), a1 = from_lane(alpha, (here() & 15) + 16);  // of the columns this lane has the sums of
    l[0] *= a0;
    l[1] *= a1;
    acc_write<acc_l<D>()>(__builtin_bit_cast(uint32_t, acc_read<acc_l<D>()>() * a0));
    acc_write<acc_l<D>() + 1>(__builtin_bit_cast(uint32_t, acc_read<acc_l<D>() + 1>() * a1));
    acc_settle<D>();
  };
  auto sum_up = [&]() __attribute__((always_inline)) {  // a step's sums join the normaliser
    acc_settle<D>();
    unroll<2>([&](auto i) __attribute__((always_inline)) {
      l[decltype(i)::value] += acc_read<acc_l<D>() + decltype(i)::value>();
      acc_write<acc_l<D>() + decltype(i)::value>(0u);  // the next normaliser() is a barrier away
    });
  };
  auto next_ids = [&](int u) __attribute__((always_inline)) {
    id_u = id_1;
    id_1 = id_2;
    id_2 = block_id(u + 3);
  };

  auto hide = [&](f32x16& s, int k0) __attribute__((always_inline)) {  // scores of keys past the lane's row; returns the largest left
    const int ln = here();
    const int room = pos_of(ln) - k0 - 4 * (ln >> 5);
    asm volatile("" ::: "memory");  // keeps the caller's condition a branch instead of always-on selects
    float t = -__builtin_inff();
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      s[i] = 8 * (i / 4) + (i % 4) > room ? -__builtin_inff() : s[i];
      t = largest_of(t, s[i]);
    }
    return t;
  };
  auto largest = [&](const f32x16& s) __attribute__((always_inline)) {
    float t = -__builtin_inff();
#pragma unroll
    for (int i = 0; i < 16; ++i) t = largest_of(t, s[i]);
    return t;
  };
  auto products = [&](auto half_tag, const bf16x8 (&pw)[2], int at) __attribute__((always_inline)) {  // operands four MFMAs ahead
    constexpr int kStep = 2 * decltype(half_tag)::value;
    bf16x8 v[kP];
    auto operand = [&](auto vi) __attribute__((always_inline)) { v[decltype(vi)::value] = read_v(decltype(vi)::value % G::kDTiles, kStep + decltype(vi)::value / G::kDTiles, at); };
    unroll<4>(operand);
    pin();
    unroll<kP>([&](auto ii) __attribute__((always_inline)) {
      constexpr int i = decltype(ii)::value;
      mfma_pv<D, i % G::kDTiles>(v[i], pw[i / G::kDTiles]);
      if constexpr (i + 4 < kP) operand(std::integral_constant<int, i + 4>{});
      pin();
    });
  };
  auto serial_step = [&](int u) __attribute__((always_inline)) {
    const int par = (u & 1) * G::kTileBytes, other = par ^ G::kTileBytes;
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
    if (vt > 0 && vt < n_tiles) copy_tile(vt == u ? id_u : id_1, vplane, __builtin_amdgcn_readfirstlane(kVBuf + (vt & 1) * G::kTileBytes));
    if (u > 0 && 2 * u - 2 < n_half) {
      products(std::integral_constant<int, 0>{}, pa, other);
      normaliser<D, false>(pa[0]);
      normaliser<D, false>(pa[1]);
      if (kt - 1 > wave_pos_lo) top = hide(sb, kt - 32);
      if (must_move()) rescale(move(sb));
      unroll<24>([&](auto k) __attribute__((always_inline)) { weight_op<decltype(k)::value>(sb, pb, -m, sc); });
      asm volatile("s_nop 3" : "+v"(pb[0]), "+v"(pb[1]));
      products(std::integral_constant<int, 1>{}, pb, other);
      normaliser<D, false>(pb[0]);
      normaliser<D, false>(pb[1]);
      sum_up();
    }
    if (u == n_tiles) return;
    if (2 * u < n_half) {
      u32x4 ka[kQ], kb[kQ];  // operands three k-steps ahead: left to itself the compiler reads each right before its use
      unroll<3>([&](auto si) __attribute__((always_inline)) {
        ka[decltype(si)::value] = read_k(decltype(si)::value, par);
        kb[decltype(si)::value] = read_k(decltype(si)::value, par + 2 * G::kKeyGroup);
      });
      pin();
      unroll<kQ>([&](auto si) __attribute__((always_inline)) {
        constexpr int s = decltype(si)::value;
        mfma_qk<D, s>(sa, ka[s]);
        mfma_qk<D, s>(sb, kb[s]);
        if constexpr (s + 3 < kQ) {
          ka[s + 3] = read_k(s + 3, par);
          kb[s + 3] = read_k(s + 3, par + 2 * G::kKeyGroup);
        }
        pin();
      });
      asm volatile("s_nop 15\n\ts_nop 3" : "+v"(sa), "+v"(sb));
      float first;
      if (kt + kTileK - 1 > wave_pos_lo) {
        first = hide(sa, kt);
        top = hide(sb, kt + 32);
      } else {
        first = largest(sa);
        top = largest(sb);
      }
      // Lazy reference: m only has to bound the scores loosely.  It is moved (and the accumulators rescaled) only when a score exceeds
      // it by more than kLazyLog2; until then weights may reach 2^kLazyLog2, which fp32 sums and bf16 weights hold easily.  A lane
      // looks at its own scores; the two lanes of a column meet only when some lane of the wave has to move.
      // Here it is the largest of 64 scores: the weight of a row's largest score is then more often exactly 1, the one weight that
      // rounding does not touch (chunks of 300..1500 rows from position 0: relative error 1.908e-3, with 32 scores 1.923e-3).
      const float second = top;
      top = largest_of(top, first);
      if (must_move()) {
        const float alpha = move(sa);
        if (u > 0 || __builtin_amdgcn_ballot_w64(alpha != alpha) != 0) rescale(alpha);  // (at first there is nothing to rescale)
      }
      top = second;
      unroll<24>([&](auto k) __attribute__((always_inline)) { weight_op<decltype(k)::value>(sa, pa, -m, sc); });
      asm volatile("s_nop 3" : "+v"(pa[0]), "+v"(pa[1]));
    }
    // No tile to publish, and no copy into the buffer that this one leaves.  (From three tiles on the last step is some waves' fast one,
    // which has the barrier; the waves of a workgroup must meet at the same ones.)
    if (n_tiles <= 2 && u + 1 == n_tiles) return;
    barrier<kR>();
    if (u + 2 < n_tiles) copy_tile(id_2, 0, par);
    next_ids(u);
  };

  auto fast_stage = [&](auto half_tag, auto par_tag, int u, f32x16& scur, f32x16& snext, bf16x8 (&pcur)[2], bf16x8 (&pprev)[2]) __attribute__((always_inline)) {
    constexpr int kHalf = decltype(half_tag)::value, kPar = decltype(par_tag)::value;
    constexpr int kAt = kPar * G::kTileBytes + kHalf * 2 * G::kKeyGroup;
    constexpr int kNextAt = kHalf == 0 ? kAt + 2 * G::kKeyGroup : (kPar ^ 1) * G::kTileBytes;
    constexpr int kVAt = (kPar ^ 1) * G::kTileBytes, kVStep = 2 * kHalf;
    bool moved = must_move();
    float alpha = 1.f;
    if (__builtin_expect(moved, 0)) {
      alpha = move(scur);
      moved = __builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0;
    }
    const float negm = -m;
    auto weights = [&](auto slot) __attribute__((always_inline)) {  // this slot's share of the 24 operations
      constexpr int a = decltype(slot)::value * 24 / kS, b = (decltype(slot)::value + 1) * 24 / kS;
      unroll<b - a>([&](auto k) __attribute__((always_inline)) { weight_op<a + decltype(k)::value>(scur, pcur, negm, sc); });
    };
    auto operand_v = [&](auto vi) __attribute__((always_inline)) {
      constexpr int v = decltype(vi)::value;
      vop[v] = read_v(v % G::kDTiles, kVStep + v / G::kDTiles, kVAt);
    };
    pin();
    unroll<kQ>([&](auto ii) __attribute__((always_inline)) {
      constexpr int i = decltype(ii)::value;
      if constexpr (i == kQ - 2) {
        barrier<kR>();
        pin();
      }
      if constexpr (i % 2 == 0) asm volatile("" ::"v"(kop[i]), "v"(kop[i + 1]));  // one wait for the two
      mfma_qk<D, i>(snext, kop[i]);
      if constexpr (i % 2 == 0 && i + 2 < kQ) {
        kop[i + 2] = read_k(i + 2, kAt);
        kop[i + 3] = read_k(i + 3, kAt);
      }
      if constexpr (i >= kQ - 2) operand_v(std::integral_constant<int, i - (kQ - 2)>{});
      if constexpr (kHalf == 0 && (i == kQ - 2 || i == kQ - 1)) l[i - (kQ - 2)] += acc_read<acc_l<D>() + i - (kQ - 2)>();  // the step before
      weights(ii);
      pin();
    });
    unroll<kP>([&](auto ii) __attribute__((always_inline)) {
      constexpr int i = decltype(ii)::value, dt = i % G::kDTiles, ks = i / G::kDTiles;
      if constexpr (i % 2 == 0) asm volatile("" ::"v"(vop[i]), "v"(vop[i + 1]));
      mfma_pv<D, dt>(vop[i], pprev[ks]);
      if constexpr (dt == G::kDTiles - 1) normaliser<D, kHalf == 0 && ks == 0>(pprev[ks]);
      if constexpr (i % 2 == 0 && i + 2 < kP) {
        operand_v(std::integral_constant<int, i + 2>{});
        operand_v(std::integral_constant<int, i + 3>{});
      }
      if constexpr (i == 0 && kHalf == 0) copy_tile(id_u, vplane, kVBuf + kPar * G::kTileBytes);
      if constexpr (i == 0 && kHalf == 1) {
        copy_tile(id_2, 0, kPar * G::kTileBytes);
        next_ids(u);
      }
      if constexpr (i >= kP - 2) kop[i - (kP - 2)] = read_k(i - (kP - 2), kNextAt);
      weights(std::integral_constant<int, kQ + i>{});
      constexpr int m0 = kP / 2;  // the largest score of half h + 1, eight pairs over the last slots
      if constexpr (i >= m0) {
        if constexpr (i == m0) top = -__builtin_inff();
#pragma unroll
        for (int k = (i - m0) * 8 / (kP - m0); k < (i - m0 + 1) * 8 / (kP - m0); ++k) top = largest_of(largest_of(top, snext[2 * k]), snext[2 * k + 1]);
      }
      pin();
    });
    asm volatile("" : "+v"(pcur[0]), "+v"(pcur[1]), "+v"(top));  // are worked out here, not in the next stage, where they are used
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
      for (int s = 0; s < 2; ++s) kop[s] = read_k(s, G::kTileBytes);
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

  // ---- epilogue: lane holds O^T[d][col] for d = 32 dt + 8 (i/4) + 4 hl + i%4
  acc_settle<D>();
  const float l0 = l[0] + acc_read<acc_l<D>()>(), l1 = l[1] + acc_read<acc_l<D>() + 1>();
  const int lane_e = here();
  const float lsum = lane_e & 16 ? l1 : l0;
  const int r_e = 32 * w + (lane_e & 31), d0 = 4 * (lane_e >> 5);
  if (r_e < n_rows_t) {
    const int qr = r_e >> gs;
    const int head = head0 + (r_e & ((1 << gs) - 1));
    if (it.slot0 < 0) {
      const float inv = 1.0f / lsum;
      uint16_t* op = p.out + ((int64_t)(it.qrow0 + qr) * H + head) * D;
      unroll<D / 8>([&](auto ci) __attribute__((always_inline)) {
        constexpr int c = decltype(ci)::value;
        bf16x4 o;
        unroll<4>([&](auto e) __attribute__((always_inline)) { o[decltype(e)::value] = (__bf16)(acc_read<4 * c + decltype(e)::value>() * inv); });  // round to nearest even
        *(bf16x4*)(op + 8 * c + d0) = o;
      });
    } else {
      const int64_t ps = (int64_t)(it.slot0 + qr * it.nparts) * H + head;
      float* op = p.part_o + ps * D;
      unroll<D / 8>([&](auto ci) __attribute__((always_inline)) {
        constexpr int c = decltype(ci)::value;
        f32x4 o;
        unroll<4>([&](auto e) __attribute__((always_inline)) { o[decltype(e)::value] = acc_read<4 * c + decltype(e)::value>(); });
        *(f32x4*)(op + 8 * c + d0) = o;
      });
      if (d0 == 0) {
        p.part_ml[ps * 2] = m;
        p.part_ml[ps * 2 + 1] = lsum;
      }
    }
  }
}

}  // namespace tile32
}  // namespace ic
