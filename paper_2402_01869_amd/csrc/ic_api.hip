// C ABI, host-side validation and launch planning for the intercept hot path.
// See include/infercept_hot.h for the contract of every entry point.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <vector>

#include "ic_internal.h"

using namespace ic;

namespace {

constexpr int kStagingSlots = 4;       // pinned host buffers, each filled by successive calls, then the next
// Keys per decode work item: 4096 (the most a row item can hold).  Measured on the 13B-shaped batches: contexts up to
// 4096 keys as ONE item each (no partial results, no merge pass) are 1 % faster than 2048-key items, alone and beside
// the tile kernel; 512- and 1024-key items are 1-5 % slower (head_dim 256, GPT-J-shaped decode: 6 % slower at 512).
constexpr int kDefaultRowPart = 4096;
constexpr int kWholeSpan = 1 << 30;    // span partition: none
constexpr int kUnsplitWorkgroups = 1024;  // tile workgroups (4 per CU) from which spans are not split at all
// The weights of rows that see fewer keys than this are not rounded to bf16.  The matrix-core kernels round them
// before the PV product; with a handful of keys a single weight's rounding (2^-9 relative) shows in the
// output, with dozens the roundings average out.  The vector path keeps the weights in fp32, the
// few-key units split them into three bf16 parts.
constexpr int kShareKeys = 8192;  // sequences at least this long keep their tile items side by side
constexpr int kMfmaMinKeys = 64;
constexpr int kExpectedCus = 256;        // the planner runs without a device; the launches use the device's own count
// Mean K/V bytes of a row item below which one workgroup per item beats the persistent launch: its queue hands out one
// item per 12.5 ns (atomics on one address), whatever the number of workgroups.  Measured, us per call, persistent /
// one per item: head_dim 128, 8000 items of 16 keys 101 / 23, of 100 keys 119 / 71; 10240 of 200 keys (100 KB) 210 / 172,
// 7800 of 300 keys 212 / 195, 2920 of 800 keys (400 KB) 187.5 / 188.2, 1440 of 1600 keys 179 / 184; head_dim 256, 3200
// items of 48 keys 52 / 33, 3904 of 300 keys (300 KB) 189.3 / 189.5, 1456 of 800 keys 182 / 184.
constexpr double kShortItemBytes = 300e3;

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

struct StagingSlot {
  char* host = nullptr;
  size_t cap = 0;
  size_t used = 0;       // bytes handed out since the slot was entered
  hipEvent_t ev = nullptr;
  bool pending = false;  // ev marks the last upload out of this slot
};

struct ProfState {
  bool on = false;
  std::vector<hipEvent_t> ev;       // pairs
  std::vector<int> kind;            // per pair
  int used = 0;                     // pairs recorded
};

}  // namespace

struct ic_pool {
  ic_pool_cfg cfg;
  char* base;
  size_t bytes;
  size_t block_bytes;
  ic_tuning tune;
  // library-owned runtime state (created lazily by the first GPU call)
  StagingSlot slots[kStagingSlots];
  int next_slot;
  // Device-side int32 lists, one per use (block ids of a pack, of an unpack, row destinations of an append), each
  // with the host copy of what it holds: a call whose list equals the previous one's (the same blocks moved for
  // every layer of a model, say) skips the upload and the checks that list already passed.
  struct DevList {
    int32_t* dev = nullptr;
    size_t cap = 0;
    std::vector<int32_t> held;  // contents of dev (from the last upload queued), empty = nothing usable
    bool checked = false;       // ... which have passed the host checks (false: uploaded under IC_FLAG_TRUSTED)
  };
  DevList lists[3];
  std::vector<void*> retired_dev;   // id lists that were outgrown: earlier launches may still read them, freed at destroy
  std::vector<void*> retired_host;  // the same for pinned descriptor buffers
  int num_cus;           // compute units of the pool's device (0 until the first attention call)
  hipStream_t side;      // second stream: the tile kernel runs beside the row kernel
  hipEvent_t ev_fork, ev_join;
  ProfState prof;
};

namespace ic {
PoolView pool_view(const ic_pool* pool) { return PoolView{pool->cfg, pool->base, pool->bytes, pool->block_bytes}; }
}  // namespace ic

namespace {

int check_cfg(const ic_pool_cfg* c) {
  if (!c) return IC_ENULL;
  if (c->num_blocks < 1 || c->num_heads < 1 || c->num_kv_heads < 1 || c->head_dim < 1 ||
      c->block_size < 1)
    return IC_EINVAL;
  if (c->dtype != 0 || c->layout != 0) return IC_EUNSUPPORTED;
  if (c->block_size != kBlockSize) return IC_EUNSUPPORTED;
  if (c->num_kv_heads > c->num_heads || c->num_heads % c->num_kv_heads != 0) return IC_EINVAL;
  if (c->head_dim != 64 && c->head_dim != 128 && c->head_dim != 256) return IC_EUNSUPPORTED;
  if (c->num_heads > 4096) return IC_EINVAL;
  return IC_OK;
}

size_t cfg_block_bytes(const ic_pool_cfg& c) {
  return (size_t)c.block_size * 2 * c.num_kv_heads * c.head_dim * 2;
}

// Structural checks (always done) and content checks (skipped when trusted).
int check_batch(const ic_pool_cfg& cfg, const ic_batch_desc* d, bool trusted) {
  if (!d) return IC_ENULL;
  if (!d->ctx_len || !d->q_len || !d->q_start || !d->block_tables) return IC_ENULL;
  if (d->num_seqs < 1 || d->max_blocks_per_seq < 1 || d->total_q_rows < 1) return IC_EINVAL;
  if (!(d->scale > 0.f) || d->scale > 3.0e38f) return IC_EINVAL;  // NaN fails the first comparison
  int64_t rows = 0;
  for (int s = 0; s < d->num_seqs; ++s) {
    const int32_t c = d->ctx_len[s], n = d->q_len[s];
    if (c < 1 || n < 1 || n > c) return IC_EINVAL;
    if ((c + kBlockSize - 1) / kBlockSize > d->max_blocks_per_seq) return IC_ESIZE;
    const int64_t r0 = d->q_start[s];
    if (r0 < 0 || r0 + n > d->total_q_rows) return IC_EOVERLAP;
    rows += n;
  }
  if (rows > d->total_q_rows) return IC_EOVERLAP;
  if (trusted) return IC_OK;
  std::vector<uint8_t> taken((size_t)d->total_q_rows, 0);
  for (int s = 0; s < d->num_seqs; ++s) {
    for (int32_t r = d->q_start[s]; r < d->q_start[s] + d->q_len[s]; ++r) {
      if (taken[r]) return IC_EOVERLAP;
      taken[r] = 1;
    }
    const int nb = (d->ctx_len[s] + kBlockSize - 1) / kBlockSize;
    const int32_t* row = d->block_tables + (int64_t)s * d->max_blocks_per_seq;
    for (int j = 0; j < nb; ++j)
      if (row[j] < 0 || row[j] >= cfg.num_blocks) return IC_ERANGE;
  }
  return IC_OK;
}

int check_ids(const ic_pool_cfg& cfg, const int32_t* ids, int32_t n, bool distinct) {
  if (n < 0) return IC_EINVAL;
  if (n == 0) return IC_OK;
  if (!ids) return IC_ENULL;
  for (int32_t i = 0; i < n; ++i)
    if (ids[i] < 0 || ids[i] >= cfg.num_blocks) return IC_ERANGE;
  if (distinct) {
    std::vector<uint8_t> seen((size_t)cfg.num_blocks, 0);
    for (int32_t i = 0; i < n; ++i) {
      if (seen[ids[i]]) return IC_EDUP;
      seen[ids[i]] = 1;
    }
  }
  return IC_OK;
}

// Destination of every query row's new K/V: block * block_size + slot (rows no sequence owns keep -1).
void append_destinations(const ic_batch_desc* desc, int32_t* dst) {
  for (int s = 0; s < desc->num_seqs; ++s) {
    const int32_t* table = desc->block_tables + (int64_t)s * desc->max_blocks_per_seq;
    const int t0 = desc->ctx_len[s] - desc->q_len[s];
    for (int i = 0; i < desc->q_len[s]; ++i) {
      const int t = t0 + i;
      dst[desc->q_start[s] + i] = table[t / kBlockSize] * kBlockSize + t % kBlockSize;
    }
  }
}

// Two rows on one slot would make the result depend on the order of the writes.
bool destinations_distinct(const ic_pool_cfg& cfg, const int32_t* dst, size_t rows) {
  std::vector<uint8_t> seen((size_t)cfg.num_blocks * kBlockSize, 0);
  for (size_t r = 0; r < rows; ++r) {
    if (dst[r] < 0) continue;
    if (seen[dst[r]]) return false;
    seen[dst[r]] = 1;
  }
  return true;
}

// ---------------------------------------------------------------------------------------
// Launch plan.  Sizes only (plan_sizes) or the filled descriptor image (plan_fill).
// Device image layout (all sections 256-byte aligned, in this order):
//   counters[16] | bt_off[num_seqs] | bt_flat[table_entries] | row_items | tile_items | few_items | merge_items | row_dst | slot_merge | arrived
// followed in the workspace by part_o[slots][H][D] and part_ml[slots][H][2].
// ---------------------------------------------------------------------------------------
struct PlanSizes {
  ic_plan_info info;
  int row_part, span_part, tile_rows;  // tile_rows: QUERY rows per tile item
  int min_keys;                        // rows that see fewer keys are vector row items whatever their kind
  int vec_items;                       // row items [0, vec_items) do not round their weights to bf16, the rest run on the group kernel
  int few_runs, few_rows;              // ... of which the last few_rows are the rows of few_runs few-key units (tile kernels)
                                       // and the others the vector kernel's
  int tile_g_shift;                    // log2 of the query heads one tile workgroup serves
  bool spans_as_rows;
  bool few_as_units;                   // few-key rows of spans go to the tile kernels' few-key body
  bool decode_as_tiles;                // grouped pools, span_kernel = 2: decode rows as one-row tile items
  bool decode_as_group;                // grouped pools: decode rows stay row items, run by the group kernel
  bool slim_group;                     // the group kernel has a slim build for the shape
  bool side_by_side;                   // the tile kernel beside the slim row or group kernel, on two streams
  bool row_per_item;                   // the vector kernel's items are short, or split by choose_row_part: one workgroup each, no queue
  bool tile_leads;                     // side by side: the tile kernel is the one on the caller's stream
  size_t off_ctr, off_bt_off, off_bt_flat, off_row, off_tile, off_few, off_merge, off_row_dst, off_slot_merge, off_arrived, image_bytes;
  int row_slots, row_merges;           // partial slots and merge items of split decode rows: the first of each
  size_t off_part_o, off_part_ml, total_bytes;
};

int round64(int x) { return (x + 63) / 64 * 64; }

}  // namespace

struct ic_plan {
  PlanSizes ps;
  ic_pool_cfg cfg;   // shape the plan was made for
  ic_tuning tune;    // launch knobs it was made with
  float scale;
  char* ws;          // the caller's workspace: descriptor image + partial results
  int32_t total_q_rows;
  bool append_checked;  // the rows' cache slots were found distinct (or the descriptor was trusted)
};

namespace {

// Where the rows of one sequence go.  Rows [0, n_few) see fewer than min_keys keys and are row items whatever their
// kind, run by the vector kernel or, several to a unit, by the tile kernels' few-key body; the rest are row items
// (vector or group kernel) or tile items.
struct SeqRoute {
  int n_few;        // leading rows of the sequence whose weights must not be rounded to bf16
  bool few_unit;    // ... run as one few-key unit (else: one by one on the vector kernel)
  bool rest_rows;   // the other rows are row items (else: tile items)
  bool rest_group;  // ... run by the group kernel
};

SeqRoute route(const PlanSizes& ps, int c, int n) {
  SeqRoute r;
  r.n_few = std::min(n, std::max(0, ps.min_keys - 1 - (c - n)));
  r.rest_rows = n == 1 ? !ps.decode_as_tiles : ps.spans_as_rows;
  r.rest_group = r.rest_rows && n == 1 && ps.decode_as_group;
  // A decode row stays with the vector kernel: alone in its sequence it would fill one of a unit's 64 rows.
  r.few_unit = r.n_few > 0 && n > 1 && ps.few_as_units;
  return r;
}

// Expected times of a batch with both kinds of work, in us, for the choice between the two launches of it and of the decode
// rows' partition.  Fitted to 4184 calls of 892 batches (4 to 40 K/V heads of 64, 128, 256 dims, 1 to 2000 decode rows of 40 to
// 9600 keys, 1 to 22 chunks, the rows whole and in partitions of 384 to 2048 keys; rms 7 %).  What these times choose took 1.6 %
// longer in the mean than the best of what was measured for the batch (at most 17 %); whole rows always side by side 16 % (up
// to 3.5 times: thousands of rows of 40 keys), and one after the other below a threshold on the shorter kernel's time 6 %.
// Measured again with the tile kernels that run their products and weights as one stream: with tile_flops of head_dim 128 and 256
// as now (before: 1.29 and 1.15) these times are 10 % off (rms, before 12) and choose 1.8 % more than the best (before 1.9; head_dim
// 256 2.3, before 2.8).  At head_dim 64 and for grouped pools the rates that fit best, 1.27 and 1.55, chose no better.  With
// these rates and those of tile_step_us() as now, 81 batches of 969 got another plan, which takes 4 % less time in the
// mean (16 % less to 9 % more).
struct RowLoad {
  int64_t items = 0;                  // work items x (query heads on the vector kernel, K/V heads on the group kernel)
  double bytes = 0.0, longest = 0.0;  // K/V bytes they read, of the longest item
  int64_t long_items = 0;             // items of at least 3/4 of the longest
  bool group = false;                 // some are the group kernel's
  bool split = false;                 // some are parts of a row
};

// What differs between head_dim 64, 128, 256 and the group kernel's pools.
struct LaunchRates {
  double tile_flops;  // per us, all CUs: 64-key steps of tile workgroups
  double row_many;    // K/V bytes per us of a persistent row workgroup among many,
  double row_one;     // ... of the longest item's, beside a tile workgroup,
  double row_rate;    // ... of all of them: one slim workgroup per CU (alone at head_dim 64 there are two: 32 heads, 224 rows of
                      // 3000 keys 1051 us beside one short chunk, 789 after it)
  double row_alone;   // ... of a workgroup of the stand-alone launches on a CU of its own
  double pair_us;     // fork, join and upload
  double lead;        // the tile kernel leads while the rows' time (queued_rows_us) is below so much of its own (see tile_leads)
};
const LaunchRates& launch_rates(int head_dim, bool group) {
  static const LaunchRates rates[4] = {{1.11e9, 40e3, 39e3, 5.2e6, 22e3, 29.0, 0.65}, {1.42e9, 92e3, 41e3, 6.2e6, 38e3, 26.0, 1.0},
                                       {1.45e9, 100e3, 38e3, 6.1e6, 50e3, 35.5, 0.95}, {1.44e9, 28e3, 64e3, 6.05e6, 38e3, 32.0, 1.5}};
  return rates[group ? 3 : head_dim == 64 ? 0 : head_dim == 128 ? 1 : 2];
}

// Tile items, two steps more per item, and half an item where more than one round leaves the last ones running alone.
double tiles_us(const LaunchRates& rate, int head_dim, int64_t items, int64_t steps, int64_t most) {
  if (items == 0) return 0.0;
  const double step = 4.0 * tile_rows(head_dim) * 64 * head_dim / (rate.tile_flops / kExpectedCus);
  const double one = most + 2.0, all = (steps + 2.0 * items) / kExpectedCus + (items > kExpectedCus ? 0.54 * one : 0.0);
  return step * std::max(one, all);
}

// Side by side the rows come from the queue of one workgroup per CU, 2.7 us an item; up to two rounds of long ones run one
// after the other.  The shorter of the two kernels costs the longer one 0.4 of its own time.
double queued_rows_us(const LaunchRates& rate, const RowLoad& r) {
  const int64_t rounds = (r.long_items + kExpectedCus - 1) / kExpectedCus;
  return std::max({r.bytes / rate.row_rate, (r.items * 2.7 + r.bytes / rate.row_many) / kExpectedCus,
                   (rounds <= 2 ? rounds : 1) * (r.longest / rate.row_one + 2.7)});
}
double side_by_side_us(const LaunchRates& rate, double tiles, const RowLoad& r) {
  const double rows = queued_rows_us(rate, r);
  return rate.pair_us + std::max(tiles, rows) + 0.4 * std::min(tiles, rows);
}

// One after the other the rows run at the memory's rate, or as long as the longest item takes.  Few-key units cost less than
// behind tile items that share the CUs.
double serial_us(const LaunchRates& rate, double tiles, const RowLoad& r, bool few_units) {
  return (few_units ? 17.5 : 24.5) + tiles + std::max(r.bytes / 6.2e6, r.longest / rate.row_alone);
}

// Keys per decode work item when the caller leaves the choice to the library.  Whole rows (up to kDefaultRowPart keys)
// as long as they give every workgroup two items; fewer, and part of the chip may idle while the longest rows run: then
// the partition that is expected to end soonest.  The model, in us:
//   - the keys' bytes at 6.6 TB/s, or at what the launch's workgroups reach where they are few; a workgroup alone on its
//     CU reads 22 / 38 / 50 GB/s at head_dim 64 / 128 / 256 (one tile of K and V in flight per wave), and that is the
//     least the longest item takes; the group kernel's, two to a CU, reach 6.6 TB/s times the root of their share of the
//     places (measured 3.2 TB/s at 112 of 512, 4.4 expected and 5.2 measured at 224); a quarter of the longest item's
//     time comes on top, for the end where only the longest are left, half from a second round on;
//   - 3.5 us between two items of a persistent workgroup (whole rows), 1 us per round of the others, which overlap;
//   - a split: 1.5 us, and 0.8 us for every four partitions the last one has to read back.
// Measured per layer, with the append (us), chosen partition / whole rows: 13B shape, one row of 3000 keys 18 (512) / 45,
// 4 of 1000..2000 33 (1536) / 36, 10 of 1000..3000 76 (1024) / 75.5; GPT-J shape, 2 of 2000 22 (384) / 44, 16 of 512..2048
// 66 (640) / 64; 70B shape, one of 6000 16.5 (384) / 61, 8 of 1000..8000 40 (768) / 66, 32 of 1000..5000 75 (768) / 80;
// 32 heads of 64 dims, 8 of 1000..3000 31 (768) / 40.  From two rounds on whole rows win: 13B shape, 20 rows of 500..3000
// 115, in partitions of 1024 keys 123.
int choose_row_part(const ic_pool* pool, const ic_batch_desc* d, const PlanSizes& ps) {
  const bool group = ps.decode_as_group;
  const int D = pool->cfg.head_dim;
  const int64_t units = group ? pool->cfg.num_kv_heads : pool->cfg.num_heads;
  bool spans = false;
  for (int s = 0; s < d->num_seqs && !spans; ++s) spans = d->q_len[s] > 1;
  // Decode rows as one-row tiles are not what this model is about; and where spans run row by row, their rows take the
  // partition too, in numbers that fill the chip whole.
  if (ps.decode_as_tiles || (spans && ps.spans_as_rows)) return kDefaultRowPart;
  const int64_t slots = group && !spans ? 2 * kExpectedCus : kExpectedCus;  // two group workgroups per CU; behind tile workgroups fewer at first
  const int64_t enough = 2 * slots;
  int64_t items = 0, keys = 0;
  int longest = 0;
  for (int s = 0; s < d->num_seqs && items * units < enough; ++s) {
    if (d->q_len[s] != 1) continue;
    items += (d->ctx_len[s] + kDefaultRowPart - 1) / kDefaultRowPart;
    keys += d->ctx_len[s];
    longest = std::max(longest, d->ctx_len[s]);
  }
  if (items == 0 || items * units >= enough) return kDefaultRowPart;
  const double key_bytes = 4.0 * D, alone = D == 64 ? 22e3 : D == 128 ? 38e3 : 50e3;  // bytes per us
  static const int parts[] = {kDefaultRowPart, 3072, 2048, 1536, 1280, 1024, 768, 640, 512, 448, 384, 320, 256, 192, 128};
  int best = kDefaultRowPart;
  double best_us = 0.0;
  for (const int part : parts) {
    if (part >= longest && part != kDefaultRowPart) continue;  // no other plan than whole rows
    int64_t n = 0;
    for (int s = 0; s < d->num_seqs; ++s)
      if (d->q_len[s] == 1) n += (d->ctx_len[s] + part - 1) / part;
    n *= units;
    const double last = std::min(longest, part) * key_bytes / alone;
    const double rate = group ? 6.6e6 * std::min(1.0, std::sqrt((double)n / slots)) : std::min(6.6e6, 0.8 * alone * n);
    double us = std::max(last, keys * units * key_bytes / rate) + (n > slots ? 0.5 : 0.25) * last;
    us += (part == kDefaultRowPart && !group ? 3.5 : 1.0) * n / slots;
    if (longest > part) us += 1.5 + 0.8 * ((longest + 4 * part - 1) / (4 * part));
    if (best_us == 0.0 || us < std::min(0.985 * best_us, best_us - 0.5)) {
      best = part;
      best_us = us;
    }
  }
  return best;
}

// The row items of a batch whose decode rows are cut into items of `part` keys.
RowLoad row_load(const ic_pool* pool, const ic_batch_desc* d, const PlanSizes& ps, int part) {
  const double key_bytes = 4.0 * pool->cfg.head_dim;
  RowLoad load;
  int longest = 0;
  const auto is_row = [&](int s) {  // decode rows that are row items (span_kernel = 2: only those of few keys)
    const SeqRoute rt = route(ps, d->ctx_len[s], d->q_len[s]);
    return d->q_len[s] == 1 && (rt.rest_rows || rt.n_few > 0);
  };
  for (int s = 0; s < d->num_seqs; ++s)
    if (is_row(s)) longest = std::max(longest, std::min(d->ctx_len[s], part));
  for (int s = 0; s < d->num_seqs; ++s) {
    const int c = d->ctx_len[s], n = d->q_len[s];
    const SeqRoute rt = route(ps, c, n);
    if (is_row(s)) {
      const bool group = rt.rest_group && rt.n_few == 0;
      const int64_t units = group ? pool->cfg.num_kv_heads : pool->cfg.num_heads;
      load.group = load.group || group;
      load.split = load.split || c > part;
      load.items += (c + part - 1) / part * units;
      load.bytes += key_bytes * c * units;
      load.long_items += (c / part + (4 * (int64_t)(c % part) >= 3 * (int64_t)longest)) * units;
    } else if (n > 1 && rt.n_few > 0 && !rt.few_unit) {
      const int last = c - n + rt.n_few;  // keys of the last of these rows
      load.items += (int64_t)rt.n_few * pool->cfg.num_heads;
      load.bytes += key_bytes * pool->cfg.num_heads * rt.n_few * (last - 0.5 * (rt.n_few - 1));
    }
  }
  load.longest = key_bytes * longest;
  return load;
}

// Its tile items; *alone: without rows beside them.  From six rounds on the persistent tile kernel, whose queues keep the tiles
// of a sequence on one L2, is the faster one at head_dim 256 too, where it only runs side by side (one row of 100 keys, 16 heads, 8
// chunks of 2048 on 2048 keys: 899 us side by side, 996 one after the other; 16 of 1024 on 3000: 1147, 1423; 8 of 2048 on 8192: 2553,
// 2615; with four rounds 8 of 1024 on 512: 193, 190).
double tile_load_us(const ic_pool* pool, const ic_batch_desc* d, const PlanSizes& ps, double* alone) {
  int64_t items = 0, steps = 0, most = 0;
  for (int s = 0; s < d->num_seqs; ++s) {
    const int c = d->ctx_len[s], n = d->q_len[s], part = n == 1 ? ps.row_part : ps.span_part;
    const SeqRoute rt = route(ps, c, n);
    if (rt.rest_rows) continue;
    for (int r0 = rt.n_few; r0 < n; r0 += ps.tile_rows) {
      const int klen = c - n + std::min(n, r0 + ps.tile_rows);
      items += (klen - 1) / part + 1;
      steps += (klen + 63) / 64;
      most = std::max<int64_t>(most, (std::min(klen, part) + 63) / 64);
    }
  }
  const int64_t n_th = pool->cfg.num_heads >> ps.tile_g_shift;
  const double t = tiles_us(launch_rates(pool->cfg.head_dim, ps.decode_as_group), pool->cfg.head_dim, items * n_th, steps * n_th, most);
  *alone = pool->cfg.head_dim > 128 && items * n_th >= 6 * kExpectedCus ? 1.07 * t : t;
  return t;
}

// The merge launch of rows that are split, where the spans need none anyway.
double merge_launch_us(const PlanSizes& ps, const RowLoad& rows) { return rows.split && ps.span_part == kWholeSpan ? 5.0 : 0.0; }

// Keys per decode work item beside tile items that are expected to take tiles_time.  While whole rows give fewer items than
// CUs the finer partition wins ties, because one long item slows the tile workgroup on its CU and the next CU has none; from
// then on it has to be expected to save 1.5 %.  Measured, whole rows / 1024 keys an item: 40 heads, 3 rows of 4000 keys and
// 2 chunks of 512 on 2000 116 / 94, 7 such rows and 3 chunks on 1500 159 / 132, 16 heads of 256 dims, 6 and 2 161 / 113; where
// the tiles lead, 40 heads, 5 and 4 chunks on 2500 200 / 204.
// rows: the load of whole rows, replaced by that of the choice.
int choose_row_part_beside(const ic_pool* pool, const ic_batch_desc* d, const PlanSizes& ps, double tiles_time, RowLoad& rows) {
  static const int parts[] = {2048, 1024, 768, 512, 384};
  const LaunchRates& rate = launch_rates(pool->cfg.head_dim, ps.decode_as_group);
  int best = ps.row_part, longest = 0;
  for (int s = 0; s < d->num_seqs; ++s)
    if (d->q_len[s] == 1) longest = std::max(longest, d->ctx_len[s]);
  double least = side_by_side_us(rate, tiles_time, rows) + merge_launch_us(ps, rows);
  int64_t tried = rows.items;
  for (const int part : parts) {
    if (ps.decode_as_tiles || tried >= 4 * kExpectedCus) break;  // rounds enough: a finer partition only adds items
    if (part >= longest) continue;                               // no other plan than whole rows
    const RowLoad finer = row_load(pool, d, ps, part);
    const double t = side_by_side_us(rate, tiles_time, finer) + merge_launch_us(ps, finer);
    if (t < (rows.items < kExpectedCus ? 1.02 : 0.985) * least) {
      best = part;
      rows = finer;
      least = std::min(least, t);
    }
    tried = finer.items;
  }
  return best;
}

// Time of one 64-key step of a tile workgroup among 256 (1.0 PFLOP/s, head_dim 256: 0.85); it takes the same time however many of
// the tile's rows are live.  Of 77 batches of chunks, each measured in up to 12 partitions, the ones chosen with it take 0.9 % longer
// than the best in the mean and 14 % at most (with the 0.9 and 0.5 of the tile kernels before: 1.15 %, 18 %).
double tile_step_us(int head_dim) {
  return 4.0 * tile_rows(head_dim) * 64 * head_dim / ((head_dim > 128 ? 0.85e9 : 1.0e9) / kExpectedCus);
}

// Keys per span work item when the caller leaves the choice to the library: the partition expected to end soonest.
// Splitting buys parallelism at the price of fp32 partial results for every row and a merge pass (4.5 us, and its bytes
// written and read at some 4 TB/s; on the long-context shape, which has four rounds of whole tiles, 7 % of the call), so
// it is looked at only when whole tiles give fewer than four rounds, and pays where one round is not full or the longest
// tiles run alone at the end.  An item costs two steps besides its keys.  row_us: time of the row items, beside which
// shorter spans gain nothing.  Measured: one 512-row chunk on 2500 keys, 64 heads over 8 K/V heads (128 whole tiles):
// 98 -> 62 us + 9 us of merge; 3 chunks of 67 rows on 8900 keys, 16 heads over 2 K/V heads: call 176 -> 34 us.
int choose_span_part(const ic_pool* pool, const ic_batch_desc* d, const PlanSizes& ps, double row_us) {
  const int H = pool->cfg.num_heads, D = pool->cfg.head_dim;
  const int64_t n_th = H >> ps.tile_g_shift;
  const double step_us = tile_step_us(D);
  constexpr double kItemSteps = 2.0;
  static const int parts[] = {kWholeSpan, 8192, 6144, 4096, 3072, 2560, 2048, 1536, 1280, 1024, 768, 640, 512, 384, 256};
  int best = kWholeSpan, longest = 0;
  for (int s = 0; s < d->num_seqs; ++s)
    if (d->q_len[s] > 1) longest = std::max(longest, d->ctx_len[s]);
  double best_us = 0.0;
  for (const int part : parts) {
    if (part >= longest && part != kWholeSpan) continue;  // no other plan than whole tiles
    int64_t items = 0, steps = 0, full = 0, most = 0, split_rows = 0;
    for (int s = 0; s < d->num_seqs; ++s) {
      const int c = d->ctx_len[s], n = d->q_len[s];
      if (n == 1) continue;
      for (int r0 = route(ps, c, n).n_few; r0 < n; r0 += ps.tile_rows) {
        const int nr = std::min(ps.tile_rows, n - r0), klen = c - n + r0 + nr;
        const int64_t np = (klen - 1) / part + 1;
        items += np;
        steps += (klen + 63) / 64;
        full += klen / part;
        most = std::max<int64_t>(most, (std::min(klen, part) + 63) / 64);
        if (np > 1) split_rows += np * nr;
      }
    }
    items *= n_th;
    steps *= n_th;
    full *= n_th;
    double cost = std::max((double)most, (double)((full + kExpectedCus - 1) / kExpectedCus) * (std::min<double>(part, 64.0 * most) / 64)) + kItemSteps;
    if (items > kExpectedCus) cost = std::max(cost, (steps + items * kItemSteps) / kExpectedCus + 0.5 * (most + kItemSteps));
    double us = cost * step_us;
    if (split_rows > 0) us += 4.5 + split_rows * H * (D + 2.0) * 4 * 2 / 4e6;
    if (best_us == 0.0 || us < best_us) {
      best = part;
      best_us = us;
    }
    if (best_us <= row_us) break;
  }
  return best;
}

// Units of a split decode row that are merged by their last partition: K/V heads on the group kernel, query heads on the
// vector kernel (in a pool whose decode rows are the group kernel's, the vector kernel only has rows too short to
// split).  0: the merge kernel merges them.  A partition's end takes 2-3 us longer that way (its stores have to reach
// memory, then a counter), which overlaps only where several workgroups share a CU: on the launches of one workgroup
// per item, which rows that choose_row_part splits run on.  Rows split beside tile items come from a queue.  From the queue of a persistent kernel it adds up: 44 rows
// of 600..10200 keys, 40 heads, in 4096-key items 729 us a layer against 710 with the merge kernel.
int split_units(const ic_pool* pool, const PlanSizes& ps) {
  const ic_tuning& t = pool->tune;
  if (t.decode_part_tokens > 0 || t.row_launch > 1 || t.row_slots > 0 || ps.row_part >= kDefaultRowPart || ps.side_by_side) return 0;
  return ps.decode_as_group ? pool->cfg.num_kv_heads : pool->cfg.num_heads;
}

// How much workspace a plan may take.  kFull is what paged_attn_mixed_workspace_bytes sizes; the others are for a caller whose
// workspace is smaller (one allocated for another batch, say): no split that only buys time, and, the least a batch
// can run in, no few-key units either.
enum Room { kFull = 0, kUnsplit = 1, kLeast = 2 };

void plan_sizes(const ic_pool* pool, const ic_batch_desc* d, PlanSizes& ps, Room room = kFull) {
  std::memset(&ps, 0, sizeof ps);
  // Grouped-query attention: the G = H / Hkv query heads of a group read the same keys.  When G is a
  // power of two up to 32, a tile workgroup takes all of them (G rows per query row), so keys are
  // staged once per group, and decode rows (G rows of one query token) go to the matrix cores too:
  // as row items run by the group kernel, or (span_kernel = 2) as one-row tile items.
  const int G = pool->cfg.num_heads / pool->cfg.num_kv_heads;
  ps.tile_g_shift = 0;
  if (G >= 2 && G <= 32 && (G & (G - 1)) == 0)
    while ((1 << ps.tile_g_shift) < G) ++ps.tile_g_shift;
  const int kTileRows = tile_rows(pool->cfg.head_dim) >> ps.tile_g_shift;
  ps.tile_rows = kTileRows;
  const ic_tuning& t = pool->tune;
  ps.span_part = t.span_part_tokens > 0 ? round64(t.span_part_tokens) : kWholeSpan;
  ps.min_keys = t.mfma_min_keys > 0 ? std::min(t.mfma_min_keys, 64) : kMfmaMinKeys;  // <= the smallest partition
  ps.spans_as_rows = (t.span_kernel == 1);  // default: MFMA tiles
  ps.decode_as_tiles = ps.tile_g_shift > 0 && t.span_kernel == 2;
  ps.decode_as_group = ps.tile_g_shift > 0 && t.span_kernel == 0;
  ps.row_part = std::min(t.decode_part_tokens > 0 ? round64(t.decode_part_tokens) : kDefaultRowPart, kMaxRowPart);
  int64_t tiles = 0, few = 0;  // unsplit query tiles; rows of spans with few keys
  for (int s = 0; s < d->num_seqs; ++s)
    if (d->q_len[s] > 1) {
      const int n_few = route(ps, d->ctx_len[s], d->q_len[s]).n_few;
      tiles += (d->q_len[s] - n_few + kTileRows - 1) / kTileRows;
      few += n_few;
    }
  // Without tile items the few-key units would be a launch of their own (4-5 us); up to two rounds of one-row items on
  // the vector kernel take no longer.  Measured: 4 chunks of 2 rows from position 0 + 1 decode row, 16 heads, two
  // layers: 30 us as row items, 36 as units.
  ps.few_as_units = room != kLeast && !ps.spans_as_rows && (tiles > 0 || few * pool->cfg.num_heads > 2 * kExpectedCus);
  if (t.span_part_tokens == 0) {
    const int64_t head_groups = pool->cfg.num_heads >> ps.tile_g_shift;
    double row_us = 0.0;
    for (int s = 0; s < d->num_seqs; ++s)
      if (d->q_len[s] == 1) row_us += d->ctx_len[s] * (4.0 * pool->cfg.head_dim * pool->cfg.num_kv_heads / 5.5e6);
    ps.span_part = room != kFull || ps.spans_as_rows || tiles * head_groups >= kUnsplitWorkgroups ? kWholeSpan : choose_span_part(pool, d, ps, row_us);
  }
  // Side by side: tile items or few-key units beside rows of a kernel that has a slim build, unless one after the other is
  // expected to take less by 4 % or a fifth of the shorter kernel (where the rows are split: not 2 % more, their last
  // partitions merge them there), or because the caller asks for persistent row workgroups.  The decode rows' partition
  // goes with the launch.
  ps.slim_group = pool->cfg.head_dim == 128 && G <= 16;
  {
    const bool choose = t.decode_part_tokens == 0 && room == kFull, few_units = ps.few_as_units && few > 0;
    const int part_alone = choose ? choose_row_part(pool, d, ps) : ps.row_part;
    double tiles_alone = 0.0;
    const double tiles_time = t.serial_spans ? 0.0 : tile_load_us(pool, d, ps, &tiles_alone);
    if (tiles_time > 0.0 || (few_units && !t.serial_spans)) {
      RowLoad rows = row_load(pool, d, ps, ps.row_part);
      ps.side_by_side = rows.items > 0 && (ps.decode_as_group ? rows.group && ps.slim_group : true);
      const RowLoad alone = !ps.side_by_side || part_alone == ps.row_part ? rows : row_load(pool, d, ps, part_alone);
      const int part_beside = ps.side_by_side && choose ? choose_row_part_beside(pool, d, ps, tiles_time, rows) : ps.row_part;
      if (ps.side_by_side && t.row_launch < 2 && t.row_slots == 0) {
        const LaunchRates& rate = launch_rates(pool->cfg.head_dim, ps.decode_as_group);
        const double serial = serial_us(rate, tiles_alone, alone, few_units);
        const double hidden = std::min(tiles_time, queued_rows_us(rate, rows));  // all that can be: the shorter kernel
        const double slack = part_beside < ps.row_part ? -0.02 * serial : std::min(0.04 * serial, 0.2 * hidden);
        ps.side_by_side = side_by_side_us(rate, tiles_time, rows) + merge_launch_us(ps, rows) < serial + slack;
      }
      ps.row_part = ps.side_by_side ? part_beside : part_alone;
      // Which of the two kernels goes on the caller's stream, with issue priority if it is the tile kernel; the other one goes
      // through the fork and join of the second stream.  The line is where the calls take the same time either way, between
      // these ratios of the rows' time to the tiles' (tile kernel first / rows first, us, well off the line): 40 heads of
      // 128, 0.95 and 1.1 (8 chunks of 512 on 2000 and 15 rows of 2500 keys 278 / 303, 29 rows 377 / 362); 32 heads of 64,
      // 0.6 and 0.7 (11 rows 128 / 135, 25 rows 182 / 154); 16 heads of 256, 0.8 and 1.2 (15 rows 234 / 247, 25 rows 288 /
      // 280); 64 heads over 8 and 16 over 4 and 2, 1.2 to 2 (199 rows of 2500 504 / 551, 85 of 9000 697 / 694, 110 855 / 829).
      ps.tile_leads = queued_rows_us(launch_rates(pool->cfg.head_dim, ps.decode_as_group), rows) <
                      launch_rates(pool->cfg.head_dim, ps.decode_as_group).lead * tiles_time;
    } else {
      ps.row_part = part_alone;
    }
  }
  ic_plan_info& in = ps.info;
  double vec_keys = 0;  // of the row items on the vector kernel
  for (int s = 0; s < d->num_seqs; ++s) {
    const int c = d->ctx_len[s], n = d->q_len[s];
    in.table_entries += (c + kBlockSize - 1) / kBlockSize;
    if (n == 1) in.decode_rows += 1; else in.span_rows += n;
    const SeqRoute rt = route(ps, c, n);
    const int n_as_rows = rt.rest_rows ? n : rt.n_few;
    if (rt.few_unit) {
      ps.few_runs += 1;
      ps.few_rows += rt.n_few;
    }
    for (int i = 0; i < n_as_rows; ++i) {
      const int klen = c - n + i + 1;
      const int parts = (klen + ps.row_part - 1) / ps.row_part;
      in.row_items += parts;
      if (!rt.few_unit && (i < rt.n_few || !rt.rest_group)) vec_keys += klen;
      if (i < rt.n_few || !rt.rest_group) ps.vec_items += parts;
      if (parts > 1) { in.partial_slots += parts; in.merge_rows += 1; ps.row_slots += parts; ps.row_merges += 1; }
    }
    if (!rt.rest_rows) {
      const int part = n == 1 ? ps.row_part : ps.span_part;
      for (int r0 = rt.n_few; r0 < n; r0 += kTileRows) {
        const int nr = std::min(kTileRows, n - r0);
        const int klen = c - n + r0 + nr;  // keys visible to the tile's last row
        const int parts = (klen + part - 1) / part;
        in.tile_items += parts;
        if (parts > 1) { in.partial_slots += parts * nr; in.merge_rows += nr; }
      }
    }
  }
  const int H = pool->cfg.num_heads, D = pool->cfg.head_dim;
  const int n_vec = ps.vec_items - ps.few_rows;
  const bool short_rows = n_vec > 0 && vec_keys * (4.0 * D) < n_vec * kShortItemBytes;
  ps.row_per_item = short_rows || (t.decode_part_tokens == 0 && ps.row_part < kDefaultRowPart);
  size_t o = 0;
  ps.off_ctr = o;     o = align_up(o + sizeof(int32_t) * 16, 256);
  ps.off_bt_off = o;  o = align_up(o + sizeof(int32_t) * (size_t)d->num_seqs, 256);
  ps.off_bt_flat = o; o = align_up(o + sizeof(int32_t) * (size_t)in.table_entries, 256);
  ps.off_row = o;     o = align_up(o + sizeof(RowItem) * (size_t)in.row_items, 256);
  ps.off_tile = o;    o = align_up(o + sizeof(TileItem) * (size_t)in.tile_items, 256);
  ps.off_few = o;     o = align_up(o + sizeof(FewItem) * (size_t)ps.few_runs, 256);
  ps.off_merge = o;   o = align_up(o + sizeof(MergeItem) * (size_t)in.merge_rows, 256);
  ps.off_row_dst = o; o = align_up(o + sizeof(int32_t) * (size_t)d->total_q_rows, 256);  // for kv_write_span_planned
  const int units = split_units(pool, ps);
  ps.off_slot_merge = o; if (units > 0) o = align_up(o + sizeof(int32_t) * (size_t)ps.row_slots, 256);
  ps.off_arrived = o;    o = align_up(o + sizeof(int32_t) * (size_t)ps.row_merges * units, 256);
  ps.image_bytes = o;
  ps.off_part_o = o;  o = align_up(o + sizeof(float) * (size_t)in.partial_slots * H * D, 256);
  ps.off_part_ml = o; o = align_up(o + sizeof(float) * (size_t)in.partial_slots * H * 2, 256);
  ps.total_bytes = o;
}

// The plan for a workspace of so many bytes.
int plan_within(const ic_pool* pool, const ic_batch_desc* d, size_t bytes, PlanSizes& ps) {
  for (const Room room : {kFull, kUnsplit, kLeast}) {
    plan_sizes(pool, d, ps, room);
    if (bytes >= ps.total_bytes) return IC_OK;
  }
  return IC_ESIZE;
}

// The kernels that run a plan, and how.
struct PlanLaunches {
  bool side_by_side;     // the tile kernel beside the slim builds, on two streams; else one kernel after the other
  int tile, row, group;  // IC_LAUNCH_*
};

// Decode rows are memory-bound and span tiles are MFMA-bound (the complementarity Section 4.2
// builds on): a batch that has both runs them as two persistent kernels side by side, one
// workgroup of each per CU, the tile kernel on the pool's second stream (forked from and joined
// back into the caller's stream by events).  The kernel beside the tile kernel is the slim row
// kernel (multi-head pools) or the slim group kernel (grouped pools: head_dim 128, groups of up
// to 16 heads).  serial_spans = 1, the other grouped shapes and, unless the caller asks for persistent row workgroups
// (row_launch 2 or 3, row_slots), batches too small to pay for the second stream run one kernel after the other instead.
PlanLaunches plan_launches(const ic_pool* pool, const PlanSizes& ps) {
  const ic_tuning& t = pool->tune;
  const int D = pool->cfg.head_dim;
  const bool tiles = ps.info.tile_items > 0 || ps.few_runs > 0;
  const bool rows = ps.vec_items > ps.few_rows, groups = ps.info.row_items > ps.vec_items;
  PlanLaunches how;
  how.side_by_side = ps.side_by_side;
  // head_dim <= 128: the persistent tile launch also when no other kernel runs beside it.  Its per-XCD queues keep the
  // query tiles of one (sequence, head) on one L2: 16 chunks of 2048 rows on 16384 keys, 32 heads of 128, then fetch 2.2 x instead
  // of 6.5 x their keys from HBM and take 8.49 instead of 9.06 ms; 8 chunks of 512, 40 heads or 64 over 8, the same either way.
  // head_dim 256: one workgroup per work item.  Neither is the better one throughout: 8 chunks of 512 rows on 512..2048 keys, 16
  // heads, 124 us either way, 4 chunks of 200..400 on 1000..6000, 16 heads over 4, 118 us against 124 (persistent), 8 of 2048 on
  // 8192 2.58 ms against 2.53 and, with one short row beside the chunks, 16 of 1024 on 3000 1.42 ms against 1.15.
  how.tile = !tiles ? IC_LAUNCH_NONE : how.side_by_side || D <= 128 ? IC_LAUNCH_PERSISTENT : IC_LAUNCH_PER_ITEM;
  // row_launch = 3: the side-by-side builds, alone
  how.group = !groups ? IC_LAUNCH_NONE : how.side_by_side || (t.row_launch == 3 && ps.slim_group) ? IC_LAUNCH_SLIM : IC_LAUNCH_PER_ITEM;
  how.row = !rows ? IC_LAUNCH_NONE
            : how.side_by_side || t.row_launch == 3 ? IC_LAUNCH_SLIM
            : t.row_launch == 1 || (t.row_launch == 0 && t.row_slots == 0 && ps.row_per_item) ? IC_LAUNCH_PER_ITEM
                                                                                              : IC_LAUNCH_PERSISTENT;
  return how;
}

// May throw std::bad_alloc (per-sequence scratch vectors); callers at the ABI catch it.
void plan_fill(const ic_batch_desc* d, const PlanSizes& ps, char* img) {
  const int kTileRows = ps.tile_rows;
  std::memset(img + ps.off_ctr, 0, sizeof(int32_t) * 16);  // work-queue counters start at zero
  std::memset(img + ps.off_arrived, 0, ps.image_bytes - ps.off_arrived);
  int32_t* slot_merge = (int32_t*)(img + ps.off_slot_merge);
  int32_t* bt_off = (int32_t*)(img + ps.off_bt_off);
  int32_t* bt_flat = (int32_t*)(img + ps.off_bt_flat);
  RowItem* rows = (RowItem*)(img + ps.off_row);
  TileItem* tiles = (TileItem*)(img + ps.off_tile);
  FewItem* fews = (FewItem*)(img + ps.off_few);
  MergeItem* merges = (MergeItem*)(img + ps.off_merge);
  {
    int32_t* row_dst = (int32_t*)(img + ps.off_row_dst);
    std::fill(row_dst, row_dst + (ps.off_slot_merge - ps.off_row_dst) / sizeof(int32_t), -1);
    append_destinations(d, row_dst);
  }
  int64_t nbt = 0;
  // vector items first, then the rows of the few-key units, then the group kernel's items
  const int few_first = ps.vec_items - ps.few_rows;
  int nvec = 0, nfew = few_first, ngrp = ps.vec_items, nruns = 0;
  // the split decode rows' slots and merge items come before those of split tiles
  int ntiles = 0, nmerge = ps.row_merges, slot = ps.row_slots, nrmerge = 0, rslot = 0;
  std::vector<int> tile_slot0, tile_parts;
  for (int s = 0; s < d->num_seqs; ++s) {
    const int c = d->ctx_len[s], n = d->q_len[s];
    const int nb = (c + kBlockSize - 1) / kBlockSize;
    bt_off[s] = (int32_t)nbt;
    std::memcpy(bt_flat + nbt, d->block_tables + (int64_t)s * d->max_blocks_per_seq,
                sizeof(int32_t) * (size_t)nb);
    nbt += nb;
    const SeqRoute rt = route(ps, c, n);
    const int n_as_rows = rt.rest_rows ? n : rt.n_few;
    if (rt.few_unit) fews[nruns++] = FewItem{nfew, rt.n_few};
    for (int i = 0; i < n_as_rows; ++i) {
      const int klen = c - n + i + 1;
      const int parts = (klen + ps.row_part - 1) / ps.row_part;
      const int qrow = d->q_start[s] + i;
      const bool vec = i < rt.n_few || !rt.rest_group;
      if (parts > 1) {
        if (ps.off_arrived > ps.off_slot_merge)
          for (int k = 0; k < parts; ++k) slot_merge[rslot + k] = nrmerge;
        merges[nrmerge++] = MergeItem{qrow, rslot, parts, 0};
      }
      for (int k = 0; k < parts; ++k) {
        RowItem& it = rows[rt.few_unit ? nfew++ : vec ? nvec++ : ngrp++];
        it.seq = s;
        it.qrow = qrow;
        it.k_begin = k * ps.row_part;
        it.k_end = std::min(klen, (k + 1) * ps.row_part);
        it.slot = parts > 1 ? rslot++ : -1;
        it.pad[0] = it.pad[1] = it.pad[2] = 0;
      }
    }
    if (!rt.rest_rows && rt.n_few < n) {
      // slots first (per tile: rows x partitions), then items ordered partition-major so that the
      // query tiles which read the same keys are dispatched next to each other
      const int first = rt.n_few;
      const int ntile = (n - first + kTileRows - 1) / kTileRows;
      const int part = n == 1 ? ps.row_part : ps.span_part;
      int max_parts = 0;
      tile_slot0.assign((size_t)ntile, -1);
      tile_parts.assign((size_t)ntile, 0);
      for (int ti = 0; ti < ntile; ++ti) {
        const int r0 = first + ti * kTileRows;
        const int nr = std::min(kTileRows, n - r0);
        const int klen = c - n + r0 + nr;
        const int parts = (klen + part - 1) / part;
        tile_parts[ti] = parts;
        max_parts = std::max(max_parts, parts);
        if (parts > 1) {
          tile_slot0[ti] = slot;
          for (int r = 0; r < nr; ++r)
            merges[nmerge++] = MergeItem{d->q_start[s] + r0 + r, slot + r * parts, parts, 0};
          slot += parts * nr;
        }
      }
      for (int k = 0; k < max_parts; ++k)
        for (int ti = 0; ti < ntile; ++ti) {
          if (k >= tile_parts[ti]) continue;
          const int r0 = first + ti * kTileRows;
          const int nr = std::min(kTileRows, n - r0);
          const int pos0 = c - n + r0;
          const int klen = pos0 + nr;
          TileItem& it = tiles[ntiles++];
          it.seq = s;
          it.qrow0 = d->q_start[s] + r0;
          it.n_rows = nr;
          it.pos0 = pos0;
          it.k_begin = k * part;
          it.k_end = std::min(klen, (k + 1) * part);
          it.slot0 = tile_parts[ti] > 1 ? tile_slot0[ti] + k : -1;
          it.nparts = tile_parts[ti];
        }
    }
  }
  // Longest tile items first: workgroups are handed out in item order (per head), and a few hundred items of
  // unequal length (contexts differ 3 : 1) over 256 CUs otherwise end with the longest ones running alone.
  // The items of one long sequence count as equally long (the stable sort then leaves them side by side, in
  // the order made above): they read the same keys, which no longer stay in an L2 from one item to the next
  // (8192 keys of one head are 4 MiB), so they have to run at the same time to share them.  Measured on one
  // box: 2048-row chunks on 16384-token prefixes 3 % faster side by side than longest-item-first, 512-row
  // chunks on prefixes of 512..2048 tokens 2 % slower.
  const auto weight = [d](const TileItem& t) {
    return d->ctx_len[t.seq] >= kShareKeys ? (int64_t)d->ctx_len[t.seq] * 256 : (int64_t)(t.k_end - t.k_begin) * t.n_rows;
  };
  std::stable_sort(tiles, tiles + ntiles, [&](const TileItem& a, const TileItem& b) { return weight(a) > weight(b); });
  // The same for row items, within the vector kernel's and the group kernel's share: decode contexts differ 16 : 1.
  const auto longer = [](const RowItem& a, const RowItem& b) { return a.k_end - a.k_begin > b.k_end - b.k_begin; };
  std::stable_sort(rows, rows + few_first, longer);
  std::stable_sort(rows + ps.vec_items, rows + ps.info.row_items, longer);
}

// ---------------------------------------------------------------------------------------
// Runtime helpers
// ---------------------------------------------------------------------------------------
// The second stream of the side-by-side launch.  ONE per device for the whole process, shared by all
// pools (a model has one pool per layer): a process gets few hardware queues (four by default), streams
// are dealt onto them round-robin, and two streams on one queue run in order; a side stream per pool
// would sooner or later share the caller's queue and silently serialise the two kernels.  Lives until
// the process ends.
hipStream_t shared_side_stream() {
  static std::mutex mu;
  static hipStream_t side[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  std::lock_guard<std::mutex> lock(mu);
  if (!side[dev] && hipStreamCreateWithFlags(&side[dev], hipStreamNonBlocking) != hipSuccess) side[dev] = nullptr;
  return side[dev];
}

// Sizes of the pool's own buffers, fixed at the first GPU call from the pool's shape so that later calls
// allocate nothing: a descriptor image is block tables (at most one entry per block while sequences
// share none), work items and one int per query row; an id list is at most one entry per block (a
// swap, one list each for packs and unpacks) or per cache slot (an append).  Only a call beyond these sizes grows a buffer, and then the
// old one is kept until kv_pool_destroy (launches in flight may still read it) instead of being
// freed behind a device-wide wait.
size_t pinned_slot_bytes(const ic_pool* pool) { return align_up(((size_t)256 << 10) + 8 * (size_t)pool->cfg.num_blocks, 4096); }
enum { kListPack = 0, kListUnpack = 1, kListAppend = 2 };
size_t dev_list_bytes(const ic_pool* pool, int which) {
  const size_t entries = (size_t)pool->cfg.num_blocks * (which == kListAppend ? (size_t)kBlockSize : 1);
  return align_up(std::max((size_t)1 << 16, sizeof(int32_t) * entries), 4096);
}

// `bytes` of pinned memory for an upload that will be queued on `st`.  A slot serves calls until it is full; only then is
// an event recorded behind its last upload (on the stream of the call that leaves it: successive calls of a pool are
// ordered), and only a slot that comes round again waits for its event.  An event after every upload kept the kernel
// behind it from starting for 5.5 us: a call of two decode rows and two 32-row chunks 17.2 -> 12.4 us,
// a plan and four layers of one decoding row 81.1 -> 76.7 us.
int acquire_pinned(ic_pool* pool, size_t bytes, hipStream_t st, char** out) {
  const size_t want = align_up(bytes, 256);
  StagingSlot* s = &pool->slots[pool->next_slot];
  if (s->used > 0 && s->used + want > s->cap) {  // leave it
    if (!s->ev && hipEventCreateWithFlags(&s->ev, hipEventDisableTiming) != hipSuccess) return IC_EHIP;
    if (hipEventRecord(s->ev, st) != hipSuccess) return IC_EHIP;
    s->pending = true;
    pool->next_slot = (pool->next_slot + 1) % kStagingSlots;
    s = &pool->slots[pool->next_slot];
    s->used = 0;
  }
  if (s->pending) {
    if (hipEventSynchronize(s->ev) != hipSuccess) return IC_EHIP;
    s->pending = false;
  }
  if (s->cap < want) {
    const size_t cap = std::max(align_up(want, 4096), pinned_slot_bytes(pool));
    void* fresh = nullptr;
    if (hipHostMalloc(&fresh, cap, hipHostMallocDefault) != hipSuccess) return IC_EHIP;
    if (s->host) pool->retired_host.push_back(s->host);
    s->host = (char*)fresh;
    s->cap = cap;
  }
  *out = s->host + s->used;
  s->used += want;
  return IC_OK;
}

struct ProfScope {
  ic_pool* pool;
  hipStream_t st;
  int idx;
  ProfScope(ic_pool* p, int kind, hipStream_t s) : pool(p), st(s), idx(-1) {
    ProfState& pr = p->prof;
    if (pr.on && (size_t)(pr.used + 1) * 2 <= pr.ev.size()) {
      idx = pr.used++;
      pr.kind[idx] = kind;
      (void)hipEventRecord(pr.ev[2 * idx], st);
    }
  }
  ~ProfScope() {
    if (idx >= 0) (void)hipEventRecord(pool->prof.ev[2 * idx + 1], st);
  }
};

bool misaligned(const void* p) { return ((uintptr_t)p & 15u) != 0; }

// Nothing may be thrown through the C ABI: the host-side checks and the planner use std::vector.
template <class F>
int guarded(F&& body) noexcept {
  try {
    return body();
  } catch (const std::bad_alloc&) {
    return IC_ENOMEM;
  } catch (...) {
    return IC_EINVAL;
  }
}

}  // namespace

// =========================================================================================
extern "C" {

const char* ic_strerror(int code) {
  switch (code) {
    case IC_OK: return "ok";
    case IC_ENULL: return "null pointer argument";
    case IC_EINVAL: return "size, length or count out of range";
    case IC_ERANGE: return "block id outside the pool";
    case IC_ESIZE: return "caller buffer too small";
    case IC_EALIGN: return "device pointer not 16-byte aligned";
    case IC_EDUP: return "duplicate destination block id";
    case IC_EUNSUPPORTED: return "configuration not supported by this build";
    case IC_EOVERLAP: return "query-row ranges overlap or leave the packed array";
    case IC_EHIP: return "HIP runtime error";
    case IC_ENOMEM: return "host allocation failed";
    case IC_ELIMIT: return "more than the fixed capacity of this allocation-free entry point";
    default: return "unknown error code";
  }
}

int kv_pool_init(const ic_pool_cfg* cfg, void* dev_pool_base, size_t pool_bytes, ic_pool** out) {
  if (!cfg || !dev_pool_base || !out) return IC_ENULL;
  const int rc = check_cfg(cfg);
  if (rc != IC_OK) return rc;
  if (misaligned(dev_pool_base)) return IC_EALIGN;
  const size_t bb = cfg_block_bytes(*cfg);
  if (pool_bytes / bb < (size_t)cfg->num_blocks) return IC_ESIZE;
  ic_pool* p = new (std::nothrow) ic_pool();
  if (!p) return IC_ENOMEM;
  p->cfg = *cfg;
  p->base = (char*)dev_pool_base;
  p->bytes = pool_bytes;
  p->block_bytes = bb;
  std::memset(&p->tune, 0, sizeof p->tune);
  p->next_slot = 0;
  p->num_cus = 0;
  p->side = nullptr;
  p->ev_fork = p->ev_join = nullptr;
  *out = p;
  return IC_OK;
}

int kv_pool_destroy(ic_pool* pool) {
  if (!pool) return IC_ENULL;
  int rc = IC_OK;
  // uploads out of the slot in use have no event behind them yet
  const StagingSlot& open = pool->slots[pool->next_slot];
  if (open.used > 0 && hipDeviceSynchronize() != hipSuccess) rc = IC_EHIP;
  for (StagingSlot& s : pool->slots) {
    if (s.pending && hipEventSynchronize(s.ev) != hipSuccess) rc = IC_EHIP;
    if (s.ev) (void)hipEventDestroy(s.ev);
    if (s.host) (void)hipHostFree(s.host);
  }
  for (hipEvent_t e : pool->prof.ev) (void)hipEventDestroy(e);
  for (ic_pool::DevList& dl : pool->lists)
    if (dl.dev) (void)hipFree(dl.dev);
  for (void* p : pool->retired_dev) (void)hipFree(p);
  for (void* p : pool->retired_host) (void)hipHostFree(p);
  if (pool->side && hipStreamSynchronize(pool->side) != hipSuccess) rc = IC_EHIP;  // shared: never destroyed
  if (pool->ev_fork) (void)hipEventDestroy(pool->ev_fork);
  if (pool->ev_join) (void)hipEventDestroy(pool->ev_join);
  delete pool;
  return rc;
}

size_t kv_block_bytes(const ic_pool* pool) { return pool ? pool->block_bytes : 0; }

int ic_check_batch(const ic_pool_cfg* cfg, const ic_batch_desc* desc) {
  const int rc = check_cfg(cfg);
  if (rc != IC_OK) return rc;
  return guarded([&] { return check_batch(*cfg, desc, false); });
}

int ic_check_ids(const ic_pool_cfg* cfg, const int32_t* host_ids, int32_t n, int require_distinct) {
  const int rc = check_cfg(cfg);
  if (rc != IC_OK) return rc;
  return guarded([&] { return check_ids(*cfg, host_ids, n, require_distinct != 0); });
}

int ic_pool_set_tuning(ic_pool* pool, const ic_tuning* tuning) {
  if (!pool || !tuning) return IC_ENULL;
  if (tuning->decode_part_tokens < 0 || tuning->span_part_tokens < 0 || tuning->span_kernel < 0 ||
      tuning->span_kernel > 2 || tuning->row_variant < 0 || tuning->row_variant > 3 ||
      tuning->serial_spans < 0 || tuning->serial_spans > 1 || tuning->row_launch < 0 || tuning->row_launch > 3 ||
      tuning->row_slots < 0 || tuning->row_slots > 65536 || tuning->mfma_min_keys < 0 ||
      tuning->mfma_min_keys > 64 || tuning->reserved[0])
    return IC_EINVAL;
  pool->tune = *tuning;
  return IC_OK;
}

int ic_plan_query(const ic_pool* pool, const ic_batch_desc* desc, ic_plan_info* out) {
  if (!pool || !desc || !out) return IC_ENULL;
  const int rc = check_batch(pool->cfg, desc, true);
  if (rc != IC_OK) return rc;
  PlanSizes ps;
  plan_sizes(pool, desc, ps);
  *out = ps.info;
  return IC_OK;
}

int ic_plan_image(const ic_pool* pool, const ic_batch_desc* desc, void* host_image, size_t host_bytes,
                  ic_plan_layout* out) {
  if (!pool || !desc || !out) return IC_ENULL;
  return guarded([&]() -> int {
  const int rc = check_batch(pool->cfg, desc, false);
  if (rc != IC_OK) return rc;
  PlanSizes ps;
  plan_sizes(pool, desc, ps);
  std::memset(out, 0, sizeof *out);
  out->image_bytes = (int64_t)ps.image_bytes;
  out->off_counters = (int64_t)ps.off_ctr;
  out->off_bt_off = (int64_t)ps.off_bt_off;
  out->off_bt_flat = (int64_t)ps.off_bt_flat;
  out->off_row_items = (int64_t)ps.off_row;
  out->off_tile_items = (int64_t)ps.off_tile;
  out->off_merge_items = (int64_t)ps.off_merge;
  out->off_row_dst = (int64_t)ps.off_row_dst;
  out->row_part_tokens = ps.row_part;
  out->span_part_tokens = ps.span_part;
  out->tile_query_rows = ps.tile_rows;
  out->tile_head_shift = ps.tile_g_shift;
  out->n_row_items = ps.info.row_items;
  out->n_tile_items = ps.info.tile_items;
  out->n_merge_items = ps.info.merge_rows;
  out->n_vector_row_items = ps.vec_items;
  if (host_image) {
    if (host_bytes < ps.image_bytes) return IC_ESIZE;
    std::memset(host_image, 0, ps.image_bytes);
    plan_fill(desc, ps, (char*)host_image);
  }
  return IC_OK;
  });
}

int ic_plan_launches(const ic_pool* pool, const ic_batch_desc* desc, ic_plan_launch_info* out) {
  if (!pool || !desc || !out) return IC_ENULL;
  return guarded([&]() -> int {
  const int rc = check_batch(pool->cfg, desc, false);
  if (rc != IC_OK) return rc;
  PlanSizes ps;
  plan_sizes(pool, desc, ps);
  const PlanLaunches how = plan_launches(pool, ps);
  const int units = split_units(pool, ps);
  std::memset(out, 0, sizeof *out);
  out->off_few_items = (int64_t)ps.off_few;
  out->off_slot_merge = (int64_t)ps.off_slot_merge;
  out->off_arrived = (int64_t)ps.off_arrived;
  out->side_by_side = how.side_by_side;
  out->tile_launch = how.tile;
  out->row_launch = how.row;
  out->group_launch = how.group;
  out->n_few_items = ps.few_runs;
  out->n_few_rows = ps.few_rows;
  out->n_merged_inside = units > 0 ? ps.row_merges : 0;
  out->n_split_slots = units > 0 ? ps.row_slots : 0;
  out->n_split_units = units;
  return IC_OK;
  });
}

size_t paged_attn_mixed_workspace_bytes(const ic_pool* pool, const ic_batch_desc* desc) {
  if (!pool || !desc) return 0;
  if (check_batch(pool->cfg, desc, true) != IC_OK) return 0;
  PlanSizes ps;
  plan_sizes(pool, desc, ps);
  return ps.total_bytes;
}

// Upload of the descriptor image of a planned batch into the workspace (through the pinned ring).
static int upload_plan(ic_pool* pool, const ic_batch_desc* desc, const PlanSizes& ps, char* ws, hipStream_t st) {
  char* host = nullptr;
  const int rc = acquire_pinned(pool, ps.image_bytes, st, &host);
  if (rc != IC_OK) return rc;
  plan_fill(desc, ps, host);
  ProfScope ps_(pool, IC_K_UPLOAD, st);
  return launch_upload(ws, host, ps.image_bytes, st) == hipSuccess ? IC_OK : IC_EHIP;
}

// The kernels of one attention call, for a descriptor image that is already in the workspace.
static int launch_attention(ic_pool* pool, const PlanSizes& ps, float scale, const void* dev_q, void* dev_out,
                            char* ws, hipStream_t st) {
  const int D = pool->cfg.head_dim;
  if (pool->num_cus == 0) {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 8)
      return IC_EHIP;
    pool->num_cus = cus;
  }
  AttnParams p;
  p.pool = (const uint16_t*)pool->base;
  p.q = (const uint16_t*)dev_q;
  p.out = (uint16_t*)dev_out;
  p.bt_off = (const int32_t*)(ws + ps.off_bt_off);
  p.bt_flat = (const int32_t*)(ws + ps.off_bt_flat);
  p.row_items = (const RowItem*)(ws + ps.off_row);
  p.tile_items = (const TileItem*)(ws + ps.off_tile);
  p.few_items = (const FewItem*)(ws + ps.off_few);
  p.merge_items = (const MergeItem*)(ws + ps.off_merge);
  p.slot_merge = (const int32_t*)(ws + ps.off_slot_merge);
  p.arrived = (int32_t*)(ws + ps.off_arrived);
  p.part_o = (float*)(ws + ps.off_part_o);
  p.part_ml = (float*)(ws + ps.off_part_ml);
  p.num_heads = pool->cfg.num_heads;
  p.num_kv_heads = pool->cfg.num_kv_heads;
  p.group = pool->cfg.num_heads / pool->cfg.num_kv_heads;
  p.tile_g_shift = ps.tile_g_shift;
  p.n_row_items = ps.info.row_items;
  p.n_vec_items = ps.vec_items - ps.few_rows;
  p.group_first = ps.vec_items;
  p.n_tile_items = ps.info.tile_items;
  p.n_few_items = ps.few_runs;
  p.split_units = split_units(pool, ps);
  p.merge_first = p.split_units > 0 ? ps.row_merges : 0;
  p.n_merge_items = ps.info.merge_rows - p.merge_first;
  p.scale_log2e = scale * 1.4426950408889634f;
  p.row_variant = pool->tune.row_variant;
  p.tile_first = 0;
  p.counters = (int32_t*)(ws + ps.off_ctr);

  const PlanLaunches how = plan_launches(pool, ps);
  // One persistent row workgroup per CU; alone at head_dim 64, where a wave has half as many bytes in flight, two
  // (5856 items of 800 keys: 259 -> 192 us, 2912 of 1600 keys: 239 -> 179 us).
  const int row_slots = pool->tune.row_slots > 0 ? pool->tune.row_slots : pool->num_cus;
  const int alone_slots = pool->tune.row_slots > 0 || D > 64 ? row_slots : 2 * row_slots;
  if (how.side_by_side) {
    if (!pool->side) {  // the stream is assigned last: a half-made set is retried by the next call
      if (!pool->ev_fork && hipEventCreateWithFlags(&pool->ev_fork, hipEventDisableTiming) != hipSuccess) return IC_EHIP;
      if (!pool->ev_join && hipEventCreateWithFlags(&pool->ev_join, hipEventDisableTiming) != hipSuccess) return IC_EHIP;
      if (!(pool->side = shared_side_stream())) return IC_EHIP;
    }
    if (hipEventRecord(pool->ev_fork, st) != hipSuccess) return IC_EHIP;
    if (hipStreamWaitEvent(pool->side, pool->ev_fork, 0) != hipSuccess) return IC_EHIP;
    // From here on the side stream may hold work that writes dev_out and the workspace: whatever fails
    // below, the caller's stream is still made to wait for it (or, failing that, the host does).
    // The kernel that leads runs on the caller's stream, where nothing but the upload is in front of it;
    // the other one pays the two cross-stream waits (some 10 us each).  Measured on 128 decode rows and 8 chunks of 512, 64 heads over
    // 8: tile kernel first 0.437 ms a call, rows first 0.495; 256 rows and 16 chunks of 2048 on 16384, 32 heads: 9.32 against
    // 9.52 ms.  A tile kernel that leads also asks for issue priority: what it loses to its neighbour's waves is lost to the
    // call (the same calls without: 0.441 and 9.35 ms, hardly more than runs differ).
    const bool tile_main = ps.tile_leads;
    hipStream_t s_tile = tile_main ? st : pool->side, s_rows = tile_main ? pool->side : st;
    p.tile_first = tile_main;
    bool ok = true;
    auto run_tile = [&] {
      ProfScope ps_(pool, IC_K_TILE, s_tile);
      ok = launch_tile_persist(p, D, pool->num_cus, true, s_tile) == hipSuccess;
    };
    auto run_rows = [&] {
      if (ok && how.group == IC_LAUNCH_SLIM) {
        ProfScope ps_(pool, IC_K_GROUP, s_rows);
        ok = launch_group_slim(p, D, row_slots, s_rows) == hipSuccess;
      }
      if (ok && how.row == IC_LAUNCH_SLIM) {  // in a grouped pool: the rows with too few keys for the matrix cores
        ProfScope ps_(pool, IC_K_ROW, s_rows);
        ok = launch_row_persist_slim(p, D, row_slots, s_rows) == hipSuccess;
      }
    };
    // the tile workgroups are placed first either way: one per CU, the row workgroups fill in beside them
    bool joined;
    if (tile_main) {
      run_tile();
      run_rows();
      joined = hipEventRecord(pool->ev_join, pool->side) == hipSuccess;
    } else {
      run_tile();
      joined = hipEventRecord(pool->ev_join, pool->side) == hipSuccess;
      run_rows();
    }
    if (!joined || hipStreamWaitEvent(st, pool->ev_join, 0) != hipSuccess) {
      (void)hipStreamSynchronize(pool->side);
      return IC_EHIP;
    }
    if (!ok) return IC_EHIP;
  } else {
    if (how.tile != IC_LAUNCH_NONE) {
      ProfScope ps_(pool, IC_K_TILE, st);
      const hipError_t e = how.tile == IC_LAUNCH_PERSISTENT ? launch_tile_persist(p, D, pool->num_cus, false, st)
                                                            : launch_tile_kernel(p, D, st);
      if (e != hipSuccess) return IC_EHIP;
    }
    if (how.group != IC_LAUNCH_NONE) {
      ProfScope ps_(pool, IC_K_GROUP, st);
      if ((how.group == IC_LAUNCH_SLIM ? launch_group_slim(p, D, row_slots, st) : launch_group_kernel(p, D, st)) != hipSuccess) return IC_EHIP;
    }
    if (how.row != IC_LAUNCH_NONE) {
      ProfScope ps_(pool, IC_K_ROW, st);
      const hipError_t e = how.row == IC_LAUNCH_SLIM       ? launch_row_persist_slim(p, D, row_slots, st)
                           : how.row == IC_LAUNCH_PER_ITEM ? launch_row_kernel(p, D, st)
                                                           : launch_row_persist(p, D, alone_slots, st);
      if (e != hipSuccess) return IC_EHIP;
    }
  }
  if (p.n_merge_items > 0) {
    ProfScope ps_(pool, IC_K_MERGE, st);
    if (launch_merge_kernel(p, D, st) != hipSuccess) return IC_EHIP;
  }
  return IC_OK;
}


int paged_attn_mixed(ic_pool* pool, const ic_batch_desc* desc, const void* dev_q, void* dev_out,
                     void* dev_workspace, size_t workspace_bytes, void* hip_stream) {
  if (!pool || !desc || !dev_q || !dev_out || !dev_workspace) return IC_ENULL;
  return guarded([&]() -> int {
    int rc = check_batch(pool->cfg, desc, (desc->flags & IC_FLAG_TRUSTED) != 0);
    if (rc != IC_OK) return rc;
    if (misaligned(dev_q) || misaligned(dev_out) || ((uintptr_t)dev_workspace & 255u)) return IC_EALIGN;
    PlanSizes ps;
    if ((rc = plan_within(pool, desc, workspace_bytes, ps)) != IC_OK) return rc;
    hipStream_t st = (hipStream_t)hip_stream;
    char* ws = (char*)dev_workspace;
    if ((rc = upload_plan(pool, desc, ps, ws, st)) != IC_OK) return rc;
    return launch_attention(pool, ps, desc->scale, dev_q, dev_out, ws, st);
  });
}

int paged_attn_plan_create(ic_pool* pool, const ic_batch_desc* desc, void* dev_workspace, size_t workspace_bytes,
                           void* hip_stream, ic_plan** out) {
  if (!pool || !desc || !dev_workspace || !out) return IC_ENULL;
  return guarded([&]() -> int {
  int rc = check_batch(pool->cfg, desc, (desc->flags & IC_FLAG_TRUSTED) != 0);
  if (rc != IC_OK) return rc;
  if ((uintptr_t)dev_workspace & 255u) return IC_EALIGN;
  std::unique_ptr<ic_plan> pl(new ic_plan());
  if ((rc = plan_within(pool, desc, workspace_bytes, pl->ps)) != IC_OK) return rc;
  pl->cfg = pool->cfg;
  pl->tune = pool->tune;
  pl->scale = desc->scale;
  pl->ws = (char*)dev_workspace;
  pl->total_q_rows = desc->total_q_rows;
  pl->append_checked = true;
  if (!(desc->flags & IC_FLAG_TRUSTED)) {
    std::vector<int32_t> dst((size_t)desc->total_q_rows, -1);
    append_destinations(desc, dst.data());
    pl->append_checked = destinations_distinct(pool->cfg, dst.data(), dst.size());
  }
  if ((rc = upload_plan(pool, desc, pl->ps, pl->ws, (hipStream_t)hip_stream)) != IC_OK) return rc;
  *out = pl.release();
  return IC_OK;
  });
}

int paged_attn_planned(ic_pool* pool, const ic_plan* plan, const void* dev_q, void* dev_out, void* hip_stream) {
  if (!pool || !plan || !dev_q || !dev_out) return IC_ENULL;
  const ic_pool_cfg &a = pool->cfg, &b = plan->cfg;
  if (a.num_blocks != b.num_blocks || a.block_size != b.block_size || a.num_heads != b.num_heads ||
      a.num_kv_heads != b.num_kv_heads || a.head_dim != b.head_dim || a.dtype != b.dtype || a.layout != b.layout)
    return IC_EINVAL;  // the plan was made for another shape
  if (std::memcmp(&pool->tune, &plan->tune, sizeof(ic_tuning)) != 0) return IC_EINVAL;  // or another launch plan
  if (misaligned(dev_q) || misaligned(dev_out)) return IC_EALIGN;
  return launch_attention(pool, plan->ps, plan->scale, dev_q, dev_out, plan->ws, (hipStream_t)hip_stream);
}

int kv_write_span_planned(ic_pool* pool, const ic_plan* plan, const void* dev_k_new, const void* dev_v_new,
                          void* hip_stream) {
  if (!pool || !plan || !dev_k_new || !dev_v_new) return IC_ENULL;
  const ic_pool_cfg &a = pool->cfg, &b = plan->cfg;
  if (a.num_blocks != b.num_blocks || a.block_size != b.block_size || a.num_heads != b.num_heads ||
      a.num_kv_heads != b.num_kv_heads || a.head_dim != b.head_dim || a.dtype != b.dtype || a.layout != b.layout)
    return IC_EINVAL;
  if (!plan->append_checked) return IC_EDUP;
  if (misaligned(dev_k_new) || misaligned(dev_v_new)) return IC_EALIGN;
  hipStream_t st = (hipStream_t)hip_stream;
  ProfScope ps_(pool, IC_K_APPEND, st);
  const hipError_t e = launch_append(pool->base, dev_k_new, dev_v_new, (const int32_t*)(plan->ws + plan->ps.off_row_dst),
                                     plan->total_q_rows, a.num_kv_heads, a.head_dim, st);
  return e == hipSuccess ? IC_OK : IC_EHIP;
}

int paged_attn_plan_destroy(ic_plan* plan) {
  if (!plan) return IC_ENULL;
  delete plan;
  return IC_OK;
}

// The pool's device-side int32 list (block ids of a swap, row destinations of an append).
static int ensure_dev_list(ic_pool* pool, int which, size_t bytes) {
  ic_pool::DevList& dl = pool->lists[which];
  if (dl.cap >= bytes) return IC_OK;
  const size_t cap = std::max(align_up(bytes, 4096), dev_list_bytes(pool, which));
  int32_t* fresh = nullptr;
  if (hipMalloc((void**)&fresh, cap) != hipSuccess) return IC_EHIP;
  if (dl.dev) pool->retired_dev.push_back(dl.dev);  // earlier launches may still read it
  dl.dev = fresh;
  dl.cap = cap;
  dl.held.clear();
  return IC_OK;
}

// Bring `n` ints into the pool's device list `which` on `st`, unless it holds exactly these already.
static int upload_list(ic_pool* pool, int which, const int32_t* host, size_t n, bool checked, hipStream_t st) {
  ic_pool::DevList& dl = pool->lists[which];
  const size_t bytes = align_up(sizeof(int32_t) * n, 16);
  int rc = ensure_dev_list(pool, which, bytes);
  if (rc != IC_OK) return rc;
  if (dl.held.size() == n && std::memcmp(dl.held.data(), host, sizeof(int32_t) * n) == 0) {
    dl.checked = dl.checked || checked;
    return IC_OK;
  }
  dl.held.clear();  // whatever fails below, the device copy is no longer known
  dl.checked = checked;
  char* pinned = nullptr;
  if ((rc = acquire_pinned(pool, bytes, st, &pinned)) != IC_OK) return rc;
  std::memcpy(pinned, host, sizeof(int32_t) * n);
  std::memset(pinned + sizeof(int32_t) * n, 0xff, bytes - sizeof(int32_t) * n);
  {
    ProfScope ps_(pool, IC_K_UPLOAD, st);
    if (launch_upload(dl.dev, pinned, bytes, st) != hipSuccess) return IC_EHIP;
  }
  dl.held.assign(host, host + n);
  return IC_OK;
}

// The device list holds exactly these ints and they have passed the host checks.
static bool list_is_held(const ic_pool* pool, int which, const int32_t* host, size_t n) {
  const ic_pool::DevList& dl = pool->lists[which];
  return dl.checked && dl.held.size() == n && std::memcmp(dl.held.data(), host, sizeof(int32_t) * n) == 0;
}

static int swap_common(ic_pool* pool, const int32_t* host_ids, int32_t n, const void* dev_staging,
                       size_t staging_bytes, void* hip_stream, bool pack) {
  if (!pool) return IC_ENULL;
  if (n < 0) return IC_EINVAL;
  if (n == 0) return IC_OK;
  if (!host_ids || !dev_staging) return IC_ENULL;
  return guarded([&]() -> int {
  const int which = pack ? kListPack : kListUnpack;
  // a list the device copy already holds has passed these checks
  int rc = list_is_held(pool, which, host_ids, (size_t)n) ? IC_OK : check_ids(pool->cfg, host_ids, n, !pack);
  if (rc != IC_OK) return rc;
  if (misaligned(dev_staging)) return IC_EALIGN;
  if (staging_bytes / pool->block_bytes < (size_t)n) return IC_ESIZE;
  {  // staging must not overlap the pool
    const char* s0 = (const char*)dev_staging;
    const char* s1 = s0 + (size_t)n * pool->block_bytes;
    if (s0 < pool->base + pool->bytes && pool->base < s1) return IC_EINVAL;
  }
  hipStream_t st = (hipStream_t)hip_stream;
  if ((rc = upload_list(pool, which, host_ids, (size_t)n, true, st)) != IC_OK) return rc;
  const int32_t* dev_ids = pool->lists[which].dev;
  hipError_t e;
  {
    ProfScope ps_(pool, pack ? IC_K_PACK : IC_K_UNPACK, st);
    e = pack ? launch_pack(pool->base, (void*)dev_staging, dev_ids, n, pool->block_bytes, st)
             : launch_unpack(pool->base, dev_staging, dev_ids, n, pool->block_bytes, st);
  }
  return e == hipSuccess ? IC_OK : IC_EHIP;
  });
}

int kv_pack_blocks(ic_pool* pool, const int32_t* host_ids, int32_t n, void* dev_staging,
                   size_t staging_bytes, void* hip_stream) {
  return swap_common(pool, host_ids, n, dev_staging, staging_bytes, hip_stream, true);
}

int kv_unpack_blocks(ic_pool* pool, const int32_t* host_ids, int32_t n, const void* dev_staging,
                     size_t staging_bytes, void* hip_stream) {
  return swap_common(pool, host_ids, n, dev_staging, staging_bytes, hip_stream, false);
}

int kv_write_span(ic_pool* pool, const ic_batch_desc* desc, const void* dev_k_new, const void* dev_v_new,
                  void* hip_stream) {
  if (!pool || !desc || !dev_k_new || !dev_v_new) return IC_ENULL;
  return guarded([&]() -> int {
  const bool trusted = (desc->flags & IC_FLAG_TRUSTED) != 0;
  int rc = check_batch(pool->cfg, desc, trusted);
  if (rc != IC_OK) return rc;
  if (misaligned(dev_k_new) || misaligned(dev_v_new)) return IC_EALIGN;
  const size_t rows = (size_t)desc->total_q_rows;
  std::vector<int32_t> dst(rows, -1);
  append_destinations(desc, dst.data());
  if (!trusted && !list_is_held(pool, kListAppend, dst.data(), rows) && !destinations_distinct(pool->cfg, dst.data(), rows))
    return IC_EDUP;
  hipStream_t st = (hipStream_t)hip_stream;
  if ((rc = upload_list(pool, kListAppend, dst.data(), rows, !trusted, st)) != IC_OK) return rc;
  hipError_t e;
  {
    ProfScope ps_(pool, IC_K_APPEND, st);
    e = launch_append(pool->base, dev_k_new, dev_v_new, pool->lists[kListAppend].dev, desc->total_q_rows,
                      pool->cfg.num_kv_heads, pool->cfg.head_dim, st);
  }
  return e == hipSuccess ? IC_OK : IC_EHIP;
  });
}

int ic_prof_begin(ic_pool* pool, int32_t max_launches) {
  if (!pool) return IC_ENULL;
  if (max_launches < 1 || max_launches > (1 << 20)) return IC_EINVAL;
  return guarded([&]() -> int {
    ProfState& pr = pool->prof;
    pr.ev.reserve((size_t)max_launches * 2);
    while (pr.ev.size() < (size_t)max_launches * 2) {
      hipEvent_t e;
      if (hipEventCreate(&e) != hipSuccess) return IC_EHIP;
      pr.ev.push_back(e);
    }
    pr.kind.assign(pr.ev.size() / 2, 0);
    pr.used = 0;
    pr.on = true;
    return IC_OK;
  });
}

int ic_prof_end(ic_pool* pool, ic_prof_stats* out) {
  if (!pool || !out) return IC_ENULL;
  ProfState& pr = pool->prof;
  std::memset(out, 0, sizeof *out);
  pr.on = false;
  for (int i = 0; i < pr.used; ++i) {
    if (hipEventSynchronize(pr.ev[2 * i + 1]) != hipSuccess) return IC_EHIP;
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, pr.ev[2 * i], pr.ev[2 * i + 1]) != hipSuccess) return IC_EHIP;
    const int k = pr.kind[i];
    if (out->launches[k] == 0 || ms < out->min_ms[k]) out->min_ms[k] = ms;
    if (out->launches[k] == 0 || ms > out->max_ms[k]) out->max_ms[k] = ms;
    out->launches[k] += 1;
    out->total_ms[k] += ms;
  }
  pr.used = 0;
  return IC_OK;
}

}  // extern "C"
