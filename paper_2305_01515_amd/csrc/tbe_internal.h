// Internal declarations shared by the HIP translation units of libtbe (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tbe {

constexpr int kWave = 64;                 // CDNA wavefront width
constexpr uint32_t kNoSet = 0xFFFFFFFFu;  // global set id of rows of a table without cache
// Backward work classes by the number of lookups a distinct row has in the batch:
//   1            : updated bag by bag (the gradient is the bag's), flagged in the location word
//   2..kLongRun  : one lane group per row, gradient rows gathered per lookup
//   above        : "heavy" rows.  In all but the largest batches a workgroup for each entry of a row in the heavy list, gradient
//                  rows gathered per lookup (long_rows_in_rest); else the table's gradient slice is streamed through LDS, once per
//                  (chunk of up to heavy_chunk_rows of the table's heavy rows, bag range),
//                  and every lane group adds up, from LDS, the lookups of its rows that fall into the tile;
//                  the partial sums of a row, one per bag range, are added up by the combine kernel.
//                  (Max pooling, whose gradient is masked per lookup, takes these rows one workgroup each.)
constexpr int kLongRun = 64;
constexpr int kHeavyThreads = 1024;       // workgroup of the tile kernel: 1024 / lanes-per-row lane groups
// rows whose sums a lane group keeps in registers (8 fp16 elements per lane need twice the registers of 4 fp32)
__host__ __device__ constexpr int heavy_rows_per_group(int dtype) { return dtype == 0 ? 8 : 6; }
// A heavy row with many lookups is entered into the heavy list in several parts (heavy_split, heavy_parts).  For the tile kernel:
// from kHeavySplit lookups on, kHeavyMaxParts at most, each taking every parts-th window of G lookups, so that no lane group has a
// hot row's lookups all to itself.
constexpr int kHeavySplit = 2048;
constexpr int kHeavyMaxParts = 64;
// Gradient tile in LDS (wide rows padded by 16 bytes against bank conflicts).  A big tile matters: the lane groups
// of a wavefront run in lockstep, each over its own row's lookups inside the tile, and the more lookups a tile
// holds per row the less their counts differ (benchmark workload, tile kernel: 32 KB 0.145 ms, 64 KB 0.125, 96 KB 0.110).
#ifndef TBE_HEAVY_TILE_BYTES
#define TBE_HEAVY_TILE_BYTES 98304
#endif
constexpr int kHeavyTileBytes = TBE_HEAVY_TILE_BYTES;    // gradient tile in LDS (rows padded by 16 bytes against bank conflicts)
// (chunk, bag range) work items the ranges are chosen for: one workgroup of 1024 threads per CU that is free for
// them (Geometry::heavy_target: all CUs less those the transfer kernel keeps to itself).  Measured on the benchmark workload (32 chunks, 256 CUs; tile kernel + combine alone, ms): 256 items
// 0.110 + 0.024, 512 items 0.124 + 0.039, 1024 items 0.148 + 0.079 -- more ranges mean more partial sums to write
// and to add up; beside the transfer kernel, which holds 48 CUs: 256 items 0.20 (two rounds), 192 items 0.15.
constexpr int kLinkCus = 48;              // workgroups of the transfer kernel: 1024 threads each, a CU each
constexpr int kHeavyMaxRanges = 128;
#ifndef TBE_HEAVY_ROUNDS
#define TBE_HEAVY_ROUNDS 4
#endif
constexpr int kHeavyRounds = TBE_HEAVY_ROUNDS;  // rounds of (chunk, bag range) work items when one round would make them too long

constexpr uint32_t kWhereOverflow = 0x80000000u;  // in the overflow copies of the batch before
constexpr uint32_t kWhereParked = 0x40000000u;    // among the victims the batch before parked
constexpr uint32_t kWhereIndex = 0x3FFFFFFFu;
// With a pipeline several batches deep the overflow copies of more than one batch are alive: the code of such a
// copy also names its batch buffer (bits 26..29; the index is then 26 bits wide).  Zero in the one-deep pipeline.
constexpr int kWhereBufShift = 26;
constexpr uint32_t kWhereBufIndex = (1u << kWhereBufShift) - 1u;
constexpr int kMaxBatchBufs = 16;

// Per-lookup location word (BatchBuf::loc): where the lookup's row is while its batch trains.
constexpr uint32_t kLocOverflow = 0x80000000u;  // index = overflow slot of a bypassed row, else global cache slot
constexpr uint32_t kLocSingle = 0x40000000u;    // the row has exactly one lookup in this batch
constexpr uint32_t kLocIndex = 0x3FFFFFFFu;

enum Status : uint8_t { ST_MISS = 0, ST_HIT = 1, ST_INSERT = 2, ST_BYPASS = 3 };

// Per-table constants, resident in device memory (array of T).
//
// Sort key of (table t, row r): key_base + (r mod S) * rows_per_set + r div S when the table
// has S > 0 sets, key_base + r otherwise.  It is a bijection of (t, r), ascending in
// (table, set, row), so one radix sort groups the lookups by table, set and row at once.
struct TableMeta {
  int64_t rows;
  uint32_t key_base;      // first sort key of this table
  uint32_t rows_per_set;  // ceil(rows / sets); 0 when sets == 0
  uint32_t sets;          // S_t
  uint32_t set_base;      // global id of set 0
  int32_t slot_base;      // global id of slot 0 (= set_base * ways)
  int32_t dim;
  int32_t dtype;          // 0 fp32, 1 fp16
  int32_t col;            // first output column
  int32_t lanes;          // lanes per row: 16 bytes of the row per lane
  uint32_t row_bytes;
  unsigned long long rps_magic, sets_magic;  // of the divisions by rows_per_set and sets (div_by)
  char *lines;            // device: cache lines of this table [sets*ways, row_bytes]
  float *slot_m;          // device: accumulators of the rows in those lines [sets*ways] (while a row is cached its
                          // accumulator lives here, next to 6 MB of its kind, instead of among those of all rows)
  char *host_w;           // pinned host rows [rows, row_bytes]
  float *host_m;          // host accumulators [rows]: read at create, written at flush
  bool flush_by_kernel;   // ... by launch_flush_state (else by a copy)
  float *dev_m;           // device: row-wise Adagrad accumulators of ALL rows of the table [rows]: current for
                          // the rows that are not in a cache line (commit moves them in and out with the row)
  // second-level cache (Section 5.3): sets2 = l2_factor * sets, so the second-level sets of the
  // rows of first-level set s are s, s + sets, s + 2 sets, ... and belong to that set alone
  uint32_t sets2;         // 0 = no second level for this table
  int32_t slot2_base;     // global id of second-level slot 0 of this table
  char *lines2;           // pinned host: second-level lines [sets2*ways, row_bytes]
  uint32_t *init_bits;    // device: deferred initialisation, one bit per row (1 = the row has a value); null = off
};

constexpr int32_t kRefusedBefore = 4;  // above any error of a batch's own

// Device-side scalars of one batch (one per batch buffer).
struct BatchCounters {
  int32_t n_uniq;     // distinct (table,row) of the batch
  int32_t n_touched;  // sets with at least one distinct row (+ pseudo sets of cacheless tables)
  int32_t n_ins;
  int32_t n_byp;
  int32_t n_heavy;    // entries of the heavy list (rows with more than kLongRun lookups, a hot row several times)
  int32_t err;        // 1 = bad offsets, 2 = index out of range, 0 = none; with kRefusedBefore: that of an earlier batch
  int32_t h_ranges;   // bag ranges the heavy rows' sums are split over in this batch
  int32_t n_mid;      // rows with 2..kLongRun lookups
  unsigned long long hits, evictions, hit_lookups;
  int32_t n_hchunks;  // (table, up to one workgroup's worth of heavy rows) chunks
  // second level: missed rows found there, victims moved down into it, rows it evicted to the
  // lower tier, victims that found no way and went to the lower tier directly
  int32_t l2_hits, l2_demotions, l2_evictions, l2_bypasses;
  // 1 = the sort payload of a lookup is (bag << within_bits) | position inside the bag, which spares
  // the gather of the bag ids after the sort; 0 = a bag is too long for that, the payload is the
  // lookup's position and the bag comes from bag_of_pos
  int32_t packed;
  int32_t n_long;     // rows with more than kLongRun lookups, one with several times kHeavySplit counted as often (what the caller is told)
};

// Arrays of one batch; three of these rotate: batch k+1 is prepared while batch k trains, and
// batch k's bypass list and overflow copies are still read by the commit of batch k+1 while
// batch k+2 is already being prepared.
struct BatchBuf {
  // per lookup
  uint32_t *loc;        // [N] location word of every lookup (kLoc* bits), input order
  int32_t *sorted_bag;  // [N] global bag id (t*B + b) of the i-th lookup in sorted order
  int32_t *bag_of_pos;  // [N] global bag id of lookup j (input order); only written when the sort payload
                        //     does not carry the bag (BatchCounters::packed == 0)
  float *inv_len;       // [T * batch] mean pooling: 1 / lookups of the bag (0 for an empty bag)
  bool mean;            // mean pooling instead of sum: forward and backward weigh by inv_len
  bool maxp;            // max pooling: forward records who supplied each maximum, backward sends the gradient there
  int32_t *argpos;      // [batch * sum_dim] max pooling: position inside its bag of the lookup that supplied the
                        //     maximum of each pooled element (-1 for an empty bag); null unless max pooling is set
  uint8_t *wins;        // [N * win_stride] max pooling: which elements of its (binary16) row a lookup supplied the maximum of,
                        //     input order: byte l for the elements of lane l, bit e for the lane's e-th; one array for all
                        //     batches (only the batch between its forward and its update has one)
  uint32_t *sorted_at;  // [N] max pooling, of the i-th lookup in sorted order: its position in input order (rows of a binary16
                        //     table) or inside its bag (fp32)
  uint32_t *uid_sorted; // [N] index of the distinct row of the i-th sorted lookup
  // per distinct row (ascending key)
  uint32_t *uniq_key;   // [N]
  int32_t *run_off;     // [N+1] first sorted position of each distinct row; run_off[U] = N
  int32_t *uniq_tab;    // [N] table of the distinct row
  int32_t *loc_u;       // [N] global slot id, or -2-j for the j-th bypassed row
  uint8_t *status;      // [N] Status
  int32_t *old_tag;     // [N] for inserts: row that was evicted, -1 if the entry was free
  // second level, per distinct row (null without one):
  int32_t *src2;        // [N] missed row: global second-level slot it was found in, -1 = not there
  int32_t *dst2;        // [N] insert with a victim: second-level slot the victim moves to, -1 = lower tier
  int32_t *evict2;      // [N] ... and the row that slot held (evicted to the lower tier), -1 = it was free
  uint2 *touched;       // [N] (global set id, first distinct row) of every touched set
  int32_t *ins_idx;     // [N] distinct-row indices of the inserts, ascending; per insert also:
  int32_t *ins_tab;     // [N]   its table
  int32_t *ins_slot;    // [N]   the global slot it takes
  int32_t *ins_old;     // [N]   the row evicted from that slot, -1 if it was free
  uint32_t *ins_key;    // [N]   its sort key
  uint32_t *vic_key;    // [N]   the sort key of the row evicted from that slot (the inserted row's if the entry was free)
  char **ins_src;       // [N]   where its row is fetched from (lower tier or second-level line)
  char **ins_dst;       // [N]   second level only: where its victim goes (second-level line or lower tier)
  char **l2v_src;       // [N]   second level only: line of the row the victim pushes out of the second
                        //       level (null = none), l2v_dst its row in the lower tier, l2v_key its sort key
  char **l2v_dst;
  uint32_t *l2v_key;
  uint32_t *ins_where;  // [N]   0 = fetch it from the backing tier; else a kWhere* code: the backing-tier
                        //       copy is stale, the current value is in HBM (see Staging::where)
  int32_t *byp_idx;     // [N] distinct-row indices of the bypasses, ascending; per bypass also:
  int32_t *byp_tab;     // [N]   its table
  uint32_t *byp_key;    // [N]   its sort key
  char **byp_src;       // [N]   its row in the backing tier
  uint32_t *byp_where;  // [N]   as ins_where
  uint8_t *byp_taken;   // [N]   1 = the next batch wants the row too and takes it over from the overflow copy in HBM, so
                        //       that copy need not go home: a newer one does, or the row's cache line
  char *ovf;            // [N * stride] HBM copies of the bypassed rows while their batch trains
  int32_t *mid_idx;     // [N/2 + 1] rows with 2..kLongRun lookups, in the order of the distinct rows (table order)
  int32_t *heavy;       // [N/32 + 1] rows with more lookups, same order, one entry per part of a row (heavy_parts)
  int32_t *heavy_sub;   // [N/32 + 1] per entry: part number | parts << 16
  int32_t *harrive;     // [N/32 + 1] per entry list position of a row's first part: parts whose sums are in (0 between batches)
  uint4 *hchunks;       // [N/kLongRun + T + 1] (table, first position in `heavy`, count, -)
  int32_t *hfirst;      // [T + 1] position of each table's first entry in the heavy list; hfirst[T] = number of entries
  int32_t *hperm;       // [N/32 + 1] the heavy list's positions, every table's entries ordered by lookups per entry
                        //     (descending, by power of two): lane groups that share a wavefront get rows of like length
  int32_t *hstart;      // [heavy rows * h_ranges] first sorted position of a heavy row in each bag range
  BatchCounters *cnt;   // device
  // host-side description
  const int64_t *d_indices;
  const int64_t *d_offsets;
  int32_t batch;
  int64_t n;
  int32_t k;
  int32_t prev_bi;      // buffer of the batch prefetched before this one, -1 = none
  hipStream_t link;     // the stream that its transfer, commit and write-back go to
  bool parks_prev;      // this batch's commit parks the overflow copies of the batch before it among its victims
};

// Scratch shared by all batches (only used inside the prefetch stage, which is serial).
struct SortScratch {
  uint2 *pairs[2];         // (sort key, payload) of every lookup
  uint32_t *slots;         // digit counts of the key generation's workgroups, then their sums (see SortShape)
  uint4 *tiles;            // the sort's tiles
  uint32_t *said;          // what its tiles say of each digit value
  unsigned long long *flags; //   and that they have said it
  unsigned long long *said_counts;  // [2 passes][4 words][kScanBlocks] counts of the compaction passes
  unsigned long long *tally;  // [3 * wavefronts of a compaction pass] (evictions, lookups that hit, late rows) per wave-
                              //     front of the last batch's status pass
  uint32_t *too_long;         // a bag of the batch does not fit the packed payload (0 between batches)
  uint32_t *stage_err;        // what the key generation finds wrong with the batch (0 between batches)
  int32_t *refused;           // error of the first batch that was refused, with kRefusedBefore (0: none): no batch behind it
                              //   does anything
  struct OneCtl *one;         // batches that one kernel takes through the stage (one_kernel_batch)
};

// Staging between the cache and the host link (one instance; the prefetch stage is serial).
//   in   : rows fetched ahead for the inserts of the batch being prefetched
//   out  : victims of the last two committed batches (by batch id parity): those of the
//          latest wait to be written back; a row evicted by batch k and wanted again by k+1
//          is taken from here instead of making the round trip over the link
struct Staging {
  char *in;            // [max_inserts * stride]
  char *out[2];        // [(max_inserts + max_parked) * stride] each
  char **wb_dst;       // [max_inserts] backing-tier row of each staged victim (null = none)
  uint32_t *wb_rb;     // [max_inserts] row bytes
  uint8_t *wb_skip[2]; // [max_inserts] by parity of the batch that parked the victim: 1 = the next batch
                       // takes the row straight back (from `out`), so it need not travel to the host
  int32_t *wb_n;       // [0] number of parked victim slots, [1] which `out` holds them (device), [2] workgroups of the
                       // transfer kernel that are done (0 between transfers)
  uint32_t *where;     // [key span] per sort key: where the row's value was the last time its backing-tier copy went
                       // stale (kWhereOverflow | j: bypassed row j of that batch, kWhereParked | i: its i-th victim; 0:
                       // never).  Entries are not taken out: one counts while the list it points into still belongs to
                       // a batch whose copies are on their way and holds this key there (StaleRows)
  uint32_t stride;     // bytes per staged row (widest row)
  int64_t max_inserts;
  int64_t max_parked;  // room behind the victims for the overflow copies parked with them (0: they are never parked)
};

// Second-level cache: tags and timestamps in HBM, lines in pinned host memory (TableMeta),
// and the staging of the rows it evicts: such a row is read into `out2` by the transfer of
// the batch that pushes it out and written to the lower tier by the next transfer, exactly
// like a first-level victim parked in Staging::out; its map code is kWhereParked | (max_inserts + i).
constexpr int kL2Sums = 64, kL2Line = 32;
static_assert(kL2Sums == kWave, "a lane each adds them up");
struct Level2 {
  bool on = false;
  int32_t factor = 0;
  int64_t total_slots2 = 0;
  int32_t *tags2 = nullptr, *ts2 = nullptr;
  int32_t *sums = nullptr;  // [kL2Sums * kL2Line] what the probe's wavefronts add to the batch's four counters, a line each
                            //   (0 between batches)
  char *out2[2] = {nullptr, nullptr};  // [max_inserts * stride] each, by batch parity
  char **wb2_dst = nullptr;            // [max_inserts] lower-tier row of each staged second-level victim
  const char *lines_lo = nullptr, *lines_hi = nullptr;  // address range of the second-level lines (pinned host memory)
};

// Emulation of a slower backing tier, for measurements only: the transfer kernel pauses after every row it
// reads from or writes to the backing tier proper (not the second-level lines).  0 pauses = off.
struct Throttle {
  int32_t pauses = 0;  // s_sleep instructions of the longest kind per backing-tier row
};

// Which backing-tier copies are stale when a batch is decided on, and where the rows' values are: the lists of the
// batches whose copies are still in HBM, against which an entry of Staging::where is checked.  A row that is in one of
// them has its newest entry there, because every batch enters its own rows and the lists of older batches run out first.
struct DeepBuf {  // one batch buffer of the pipeline several batches deep
  const BatchCounters *cnt;
  const uint32_t *byp_key;
};
struct StaleRows {
  uint32_t *where;
  uint32_t max_inserts;            // codes kWhereParked | (max_inserts + i): rows pushed out of the second level
  uint32_t own_code;               // kWhereOverflow, with the batch's buffer in the pipeline several batches deep
  uint8_t *wb_skip;                // of the victims the batch before parked: 1 = this batch takes the row back
  const BatchCounters *prev_cnt;   // the batch before (null: none since the start or the last flush): its victims, and
  const uint32_t *prev_vic_key;    //   in the one-deep pipeline the rows it bypassed
  const uint32_t *prev_byp_key;
  uint8_t *prev_byp_taken;
  char *const *prev_l2v_src;       // second level only: rows its victims pushed out of there
  const uint32_t *prev_l2v_key;
  const BatchCounters *pp_cnt;     // the batch before that one, when prev's commit parks the copies of its bypassed rows
  const uint32_t *pp_byp_key;      //   behind prev's victims (else null)
  const DeepBuf *deep;             // pipeline several batches deep: all batch buffers, and which of them hold a batch
  uint32_t live;                   //   that has not trained yet
};

// Running totals of the batches' counters: sum (hits, evictions, lookups that hit), n ([0] distinct rows, [1] inserts,
// [2] bypasses, [3] late rows) and, with a second level, l2 (its four counters).
struct Totals {
  BatchCounters *sum;
  unsigned long long *n, *l2;
  int32_t *l2_sums;
};

struct Geometry {
  int32_t T, ways;
  int32_t sum_dim;
  int32_t key_bits;     // bits of the largest sort key
  int32_t seg_bits;     // bits of the widest table's keys
  int32_t within_bits;  // bits left for the position inside the bag in a packed sort payload (0 = never packed)
  int32_t partial_stride;  // floats per partial-sum slot (widest row, padded to whole lanes)
  int64_t partial_slots;   // slots of the partial-sum buffer (heavy rows x bag ranges of a batch fit in)
  int32_t probe_min_windows = 0;  // the probe does not group touched sets while that leaves fewer windows than this (0: not set)
  int32_t heavy_target;    // (chunk, bag range) work items the heavy rows' tile kernel should have: the CUs free for it
  int32_t dtypes;          // storage types among the tables: 1 fp32, 2 binary16
  int32_t win_stride;      // lanes of the widest row; under max pooling the bytes of a lookup's record of the maxima it supplied
  uint32_t ovf_stride;     // bytes per overflow / staging slot (widest row)
  uint32_t total_sets;
  int64_t total_slots;
};

// Tables grouped by (storage type, lanes per row); forward and backward are launched once
// per class.  lanes = dim / elements-per-16-bytes rounded up to a power of two.
constexpr int kMaxClasses = 14;
struct ClassInfo {
  int n_classes;
  int cls_dtype[kMaxClasses];
  int cls_lanes[kMaxClasses];
  int cls_count[kMaxClasses];
  const int32_t *cls_tables[kMaxClasses];  // device: table ids of the class
  const int32_t *table_class;              // device: class of every table
};

// Batches of few lookups, which are bound by launches and by the latency of dependent kernels, not by bytes: their stage runs
// beside training behind the last commit (prefetch_behind_training), and the backward is one launch.
constexpr int64_t kSmallLookups = 524288, kSmallBags = 65536;
constexpr int kMaxSortPasses = 4;
constexpr int kScanBlocks = 2048;  // workgroups of a compaction pass, at most
inline bool small_batch(const Geometry &g, int64_t n, int32_t batch) {
  return n > 0 && n <= kSmallLookups && (int64_t)g.T * batch <= kSmallBags;
}

// Digits of the radix sort: pass p sorts by (key >> shift[p]) & mask[p].
struct DigitPlan {
  int passes;
  int shift[kMaxSortPasses];
  uint32_t mask[kMaxSortPasses];
};
inline DigitPlan digit_plan(int key_bits, int passes) {
  DigitPlan d{};
  d.passes = passes;
  int shift = 0;
  for (int p = 0; p < passes; p++) {
    const int w = (key_bits - shift + (passes - p) - 1) / (passes - p);  // balanced digit widths, the wider ones first
    d.shift[p] = shift;
    d.mask[p] = (1u << w) - 1u;
    shift += w;
  }
  return d;
}

// ---- the sort of a batch that goes through the stage a kernel a pass ----
// Bags are table-major, so a batch's keys arrive sorted by table.  Where the tables have enough lookups to fill tiles of their
// own, every table is a segment that is sorted by itself, by the bits of the widest table's keys: 32 tables of a million rows
// are two passes by 10 bits instead of three by 9, 8 and 8.  A pass is one kernel; what bounds it is the number of its tiles
// (latency of a tile's chain: keys, ranks, counts said and heard, output), so a tile has as many keys as leave enough of them to
// fill the chip.  Us a pass, tiles of 1024 / 2048 / 4096 / 8192 keys: 41 k lookups 7.0 / 8.8 / 9.7 / -, 90 k 8.4 / 11.7 / 13.5 / -,
// 262 k - / 15.0 / 16.2 / -, 818 k - / - / 18.6 / 22.3, 3.9 M - / - / 39.7 / 32.2, 7.9 M - / - / 70 / 55.6.
// Tiles of 1024 keys add up the counts of all the tiles before them, in one trip, the larger ones hear in two how far the sums have come
// (sort_pass_kernel).  The first is a hand-over shorter, but its reads grow with the square of a segment's tiles, and with the digit values.  Stage and
// training, us a step, a kernel that counts and one that writes / sums / all counts: tables that are one segment, by 8 bits, 40 tables of 2000
// lookups 156 / 166 / 153, 60 of 2000 168 / 164 / 156, 30 of 320 70 / 72 / 68; by 10 bits, 26 of 1700 103 / 106 / 104, one of 10 k 79 / 77 /
// 74, 40 k 94 / 96 / 93, 70 k 155 / 155 / 151, 100 k 164 / 160 / 165, 130 k 179 / 174 / 182; four and eight segments, 41 k and 120 k 103, 179 /
// 94, 159 / 92, 155.  All counts with tiles of 2048 keys, one segment by 10 bits: 130 k, 190 k, 260 k, 520 k 175, 184, 195, 245, by sums
// 174, 180, 187, 226.
// Digits of 10 bits at most: a tile hears the counts of every digit value from the key generation's slots and from the tiles before
// it, so a pass by 11 bits, which would spare keys of 21 and 22 bits one of three, takes more than it saves.  Us for the passes, two
// by 11 / three by 8, lookups of ten to 32 tables as one segment, 5 k, 15 k, 30 k, 60 k 22, 38, 48, 54 / 20, 25, 29, 32; of one table 8 k,
// 40 k, 130 k, 260 k, 520 k, 1 M 27, 50, 37, 40, 60, 67 / 24, 30, 32, 37, 48, 60; 10.5 M 240 / 192.  Two by 10 pay: 20-bit keys, 8 k, 40 k,
// 130 k, 260 k, 520 k, 1 M 18, 26, 27, 30, 42, 49 / 24, 30, 32, 36, 48, 60.
// (Digits of 8 bits with a kernel that counts, one that scans and one that writes to a pass: 3.9 M lookups of 23 bits 115 us, now
// 64; 7.9 M of 25 bits 207, now 111; 818 k 69, now 37.)
constexpr int kLutTables = 512;  // models with more tables read the descriptions from memory in the passes of the stage
constexpr int kSortThreads = 512;
constexpr int64_t kTiles1k = 131072, kTiles2k = 524288, kTiles4k = 2097152;  // lookups up to which tiles have 1024, 2048, 4096 keys
constexpr int64_t kTiles1kSegment = 65536;  // ... and lookups a segment up to which they have 1024, with the widest digits (more with narrower ones)
constexpr int kWidestDigit = 10;
constexpr int64_t kSegmentLookups = 2048;                                    // lookups a table, on average, from which tables are segments
constexpr int kSlotsHeard = 32;  // slots of a segment that the workgroups of the sort add up themselves
constexpr uint32_t kLastTile = 0x80000000u;
struct SortShape {
  DigitPlan digits;
  int rb;          // bits of the widest digit (8 at least)
  int segs, bags;  // segments, and the bags of one
  int items;       // keys of a thread
  int lanes;       // of the key generation that read a bag
  int slots;       // workgroups of the key generation for a segment, each with a slot for its counts of all digit values
  bool add_slots;  // they are added up by a kernel of their own
  int tiles;       // at most
  __host__ __device__ int tile() const { return kSortThreads * items; }
};
// lanes: 0, or what the batch would have with other lookups a bag
inline SortShape sort_shape(const Geometry &g, int64_t n, int32_t batch, int lanes = 0) {
  SortShape s{};
  s.segs = g.T > 1 && g.T <= kLutTables && n >= kSegmentLookups * g.T ? g.T : 1;
  s.bags = (int)((int64_t)g.T * batch / s.segs);
  const int bits = s.segs > 1 ? g.seg_bits : g.key_bits;
  const int passes = (bits + kWidestDigit - 1) / kWidestDigit;
  s.digits = digit_plan(bits, passes);
  s.rb = (bits + passes - 1) / passes;
  if (s.rb < 8) s.rb = 8;
  s.items = n <= kTiles1k && n << s.rb <= (kTiles1kSegment << kWidestDigit) * s.segs ? 2 : n <= kTiles2k ? 4 : n <= kTiles4k ? 8 : 16;
  // A bag has eight lanes, or one where bags have two lookups or fewer on average: seven of eight lanes had nothing to read, and the
  // rounds that this takes were what bounded the kernel.  The whole stage and the forward, us, with eight / one: 2.2 M bags of one lookup in
  // one table and in eight 304, 314 / 218, 229, 400 k in one 121 / 104, 200 k of two 111 / 102, 100 k of four 106 / 103, of eight 106 / 109;
  // 256 tables of 2112 bags of one, 512 of 8192 166, 630 / 139, 506.
  s.lanes = lanes ? lanes : n <= 2 * (int64_t)s.segs * s.bags ? 1 : 8;
  // A workgroup of the key generation takes 64 bags at a time (512, a lane each).  Up to four rounds of them are left to
  // kSlotsHeard workgroups, whose counts the sort can add up by itself; many more lookups are worth the addition's launch, 5 us.  Us for keys, addition and two
  // passes, 32 workgroups / one a round and the addition: 40 k lookups in 8000 bags 33 / 32, 21 k in 2100 25 / 25, 84 k 33 / 32, 96 k in
  // 2400 30 / 30, 128 k in 8000 37 / 32, 210 k in 2100 44 / 41, 242 k in 4756 44 / 38, 320 k in 8000 51 / 40; four tables, 252 k in 2100
  // bags of each 32 / 31, 280 k in 7000 40 / 36, less what one launch more takes the host.  So from 131072 lookups a segment on.
  // 1024 workgroups in all, or as many as have 256 lookups each: a workgroup writes some thousand counters, and with 32 for each of
  // 512 segments of 2112 lookups the counters were 134 MB for 9 MB of keys, which took 17 of 243 us.
  const int64_t round = 2 * 256 / s.lanes, rounds = (s.bags + round - 1) / round;
  int64_t most = n / ((int64_t)s.segs * 256);
  if (most > kSlotsHeard) most = kSlotsHeard;
  if (most < 1024 / s.segs) most = 1024 / s.segs;
  int64_t slots = rounds > kSlotsHeard && rounds < 4 * kSlotsHeard && n <= (int64_t)kTiles1k * s.segs ? kSlotsHeard : rounds;
  if (slots > most) slots = most;
  s.slots = (int)(slots < 1 ? 1 : slots);
  s.add_slots = s.slots > kSlotsHeard || (s.slots > 4 && n > 1000000);
  s.tiles = (int)((n + s.tile() - 1) / s.tile() + s.segs);
  return s;
}
// What the sort of any batch of at most `n` lookups in `batch` bags a table needs.
struct SortNeeds { int64_t said, tiles, slots; };  // words of tiles' counts, tiles, words of slots
inline SortNeeds sort_needs(const Geometry &g, int64_t n, int32_t batch) {
  SortNeeds r{1, 1, 1};
  // (a batch of fewer lookups can have more tiles or, as one segment, more workgroups, one of fewer bags more lanes and so workgroups)
  const int64_t steps[] = {n, kTiles1kSegment, kTiles1k, kTiles2k, kTiles4k, kSegmentLookups * g.T - 1};
  for (int64_t m : steps) {
    if (m > n || m < 1) continue;
    const SortShape s = sort_shape(g, m, batch, 8);
    const int64_t said = 2 * (int64_t)s.tiles << s.rb, slots = (int64_t)(s.slots + 1) * s.segs * (s.digits.passes << s.rb);
    if (said > r.said) r.said = said;
    if (s.tiles > r.tiles) r.tiles = s.tiles;
    if (slots > r.slots) r.slots = slots;
  }
  return r;
}

// Batches of very few lookups: one kernel takes them through the whole prefetch stage (tbe_one.hip), which spares six
// launches (22 us of host time).  4096 lookups are what one workgroup sorts in its LDS: with several tiles, passes of the sort as
// phases of the same kernel, one XCD's 32 CUs are no longer enough for the probe (4 tables of 100 k rows, 40960 lookups: 150 us
// a step instead of 127; 11 to 15 k lookups 1.04 to 1.26 times as long, 5 k equal).  Its one workgroup reads 512 bags at a time:
// 3853 lookups in 3380 bags took 238 instead of 217 us in two steps, a few hundred bags are faster.  Us a step with one kernel /
// with a kernel a pass, a third of the rows cached: beside training 500, 2000, 3000 and 4096 lookups 60, 68, 74, 90 / 94, 94, 94, 95; in a
// batch that the forward prefetches, where the host is idle, 52, 60, 68, 73 / 51, 58, 62, 63, no row cached 1000, 2000 and 4096 73, 101,
// 149 / 80, 102, 139.  (With a kernel a pass in nine instead of seven launches, between a model of 24 small kernels on either side, 2000
// and 4096 lookups 590, 595 / 616, 632: the host is busy, and the launches spared count.  So are the figures from here on.)  On one stream for everything the kernels are all that counts: 1000, 2000
// and 4096 lookups 54, 62, 74 / 59, 60, 72 (sets of one way 65, 76, 102 / 69, 73, 89).
// With a second level one XCD is short of wavefronts where the sets are few: 4096 lookups beside training in 625, 1250 and 1876
// sets 118, 107, 71 / 101, 97, 99, 3000 in 1250 sets 81 / 95, 2000 in 625 sets 80 / 82.  With more tables than the passes keep
// constants of in LDS its few workgroups look every lookup's table up in memory: beside training 500, 1000, 1200, 2000 and 3600
// lookups 71, 79, 69, 96, 99 / 88, 88, 94, 70, 97, on one stream 150, 500 and 1000 lookups 64, 66, 75 / 67, 63, 66.
constexpr int64_t kOneLookups = 4096, kOneBags = 2048;
constexpr int kOnePhases = 4;  // sorted lookups and distinct rows, probe, lists, end
constexpr int kOneItems = 4;   // items of the phase that writes the lists, at most

// Sets that a batch can touch, at most (all rows of a table without a cache count as one set).
inline int64_t sets_touched(const Geometry &g, int64_t n) {
  const int64_t sets = (int64_t)g.total_sets + g.T;
  return sets < n ? sets : n;
}
inline bool many_rows_a_set(const Geometry &g, int64_t n) { return 2 * n > 5 * sets_touched(g, n); }
// one_stream: the prefetch stream is the compute stream
inline bool one_kernel_batch(const Geometry &g, bool l2, bool one_stream, int64_t n, int32_t batch) {
  const int64_t most = g.T > kLutTables ? (one_stream ? 512 : 1536)
                       : one_stream ? 1024 : l2 && many_rows_a_set(g, n) ? 2048 : kOneLookups;
  return n > 0 && n <= most && (int64_t)g.T * batch <= kOneBags;
}

// Windows below which the probe groups no sets: what the caller has set, or the wavefronts that keep the chip busy -- of the
// one-kernel stage, those that it has (0: the kernel of its own, which has as many as there are windows).
inline int32_t probe_min_windows(const Geometry &g, int one_kernel_waves) {
  return g.probe_min_windows ? g.probe_min_windows : one_kernel_waves ? one_kernel_waves : 4096;
}

// Do transfer and commit follow the stage on its stream?  A stream of their own costs a record and a wait, 10 us of host time,
// of a step whose stage is one launch; on the stage's stream they hold the next batch's stage back, for as long as their rows
// take.  Us a step beside training, on the stage's stream / on their own / with a kernel a pass (which varies with the host): a
// third of the rows cached, 1000, 2000 and 4096 lookups 54, 65, 77 / 66, 67, 70 / 95, 88, 96, whatever the rows' width, and with a
// model of 24 small kernels on either side 554 / 583 / 600 (2000 lookups); no row cached, 2000, 3000 and 4096 rows of 256 bytes
// 83, 97, 115 / 73, 75, 80 / 107, 93, 102, 500, 1000, 2000 and 4096 rows of 1 KB 69, 90, 126, 188 / 67, 74, 92, 150 / 102, 110,
// 115, 173.  The probe of a second level with many rows a set takes its time as well: 500, 1000 and 2000 lookups in 32 sets 89, 103,
// 118 / 68, 79, 92 / 95, 96, 97, 1000 and 2000 in 313 sets 83, 97 / 72, 81 / 97, 98, 500 52 / 62 / 93, 1000 in 625 and 1876 sets
// 56, 57 / 64, 66 / 96, 98.
inline bool link_with_stage(const Geometry &g, bool l2, int64_t n, int32_t batch) {
  return one_kernel_batch(g, l2, false, n, batch) && (n <= 1024 || n * g.ovf_stride <= 512 << 10) && !(l2 && many_rows_a_set(g, n));
}

// Does a batch that a forward prefetches itself go to the compute stream, stage, transfer and commit, like the forward?  That
// spares the events (2 tables x 2000 rows, 16 bags, two steps: 190 us with them, 102 without).  But with the inputs ready such a
// stage need not wait for what the caller has given the compute stream between the last update and the forward, nor the
// transfer: on streams of their own they run beside it, which is worth the events once the transfer is long (never, when all rows
// are in a cache that holds them all).  Us a step, on the compute stream / on their own, with a copy of 256 MB before and after
// each update: no row cached, 16000 rows of 64 bytes 376 / 348, 16000, 32000 and 64000 of 256 bytes 455, 620, 862 / 421, 562, 787,
// 16000 of 1 KB 887 / 818, a third cached 330, 411, 1028 / 317, 404, 1018 (64 bytes 16000, 64000, 1 KB 64000); with four products of
// 4096 x 4096 x 4096 instead, no row cached, 1069, 1226, 1479 / 1080, 1215, 1376 (256 bytes, 16000, 32000, 64000), 1 KB 16000 and
// 64000 1544, 2836 / 1518, 2660, a third cached, 64 bytes 16000, 64000 991, 1071 / 1012, 1091; with nothing, a third cached,
// 16000 of 64 bytes, 16000 and 64000 of 1 KB 120, 353, 811 / 169, 408, 863.
constexpr int64_t kOwnLookups = 65536, kOwnBytes = 4 << 20;
inline bool on_compute_stream(const Geometry &g, bool inputs_ready, bool never_bypasses, int64_t n) {
  return n <= kOwnLookups && (!inputs_ready || never_bypasses || n * g.ovf_stride <= kOwnBytes);
}

// Does the write-back of the rows that such a batch bypassed go to the link stream all the same, beside what the caller gives the
// compute stream behind the update?  (The next batch waits for it.)  From where it would hold that up for more than half a
// millisecond, and not below, where the events cost more.  Inputs ordered, us a step, on the compute stream / on the link's: no
// row cached, with a copy of 256 MB before and after each update, 8, 16 and 64 MB of rows 606, 886, 2208 / 593, 856, 2130, with
// four products of 4096 x 4096 x 4096 1193, 1479, 2809 / 1208, 1493, 2829; a third cached, 16 MB 564, 1148 / 583, 1173.
constexpr int64_t kWriteBackBytes = 32 << 20;
inline bool write_back_beside(const Geometry &g, int64_t n) { return n * g.ovf_stride >= kWriteBackBytes; }

// Workgroups of the one-kernel stage: a wavefront for every set that the batch can touch and a thread for every lookup (the passes over
// lists), as far as 16 workgroups go, or 32 where a second level has many rows of a set to place.  Alone on one stream, us a
// step with 16 sets a workgroup / with 48 and none for the lists / with a kernel a pass: one table without a cache, 2000, 3000
// and 4096 lookups 72, 84, 97 / 79, 101, 123 / 81, 97, 102; a cache of 32 sets 86, 106 / 99, 144 / 94, 113 (2000, 4096);
// 313 sets with a second level, 500, 1000, 2000 lookups 50, 81, 96 / 52, 90, 153 / 67, 87, 98 (with 16 of them 115); sets by the
// thousand, 128 to 4096 lookups, equal (32 workgroups 2 to 4 % slower).  A batch of some dozen is soonest done by one workgroup,
// which hands over to itself: 48 lookups 40 / 42, 96 and 128 lookups in sets of 64 ways 54 / 47 and 58 / 46 with one / several.
constexpr int kOneThreads = 1024;
inline int one_stage_workgroups(const Geometry &g, bool l2, int64_t n) {
  const int64_t touched = sets_touched(g, n), waves = kOneThreads / kWave;
  if (n <= 4 * waves) return 1;
  const int64_t probe = (touched + waves - 1) / waves, lists = (n + kOneThreads - 1) / kOneThreads;
  const int64_t wgs = probe > lists ? probe : lists, most = l2 && n >= 4 * touched ? 32 : 16;
  return (int)(wgs < most ? wgs : most);
}

// What they share; all zero between launches.  A line for each word that many of them change.
struct OneCtl {
  struct alignas(128) Word { uint32_t n; };
  alignas(128) uint32_t chosen;  // 1 + the XCD that the stage runs on
  alignas(128) uint32_t left;    // workgroups that have ended
  alignas(128) uint32_t next;    // the next ticket
  alignas(128) uint32_t err;     // 1 = bad offsets, 2 = index out of range
  Word done[kOnePhases];         // items of every phase that are done
  unsigned long long said[2 * kOneItems];  // [2 words][kOneItems] counts of the pass that writes lists
};

// Sum and mean pooling, heavy rows of batches that are not among the largest: a workgroup for each of their entries in the heavy
// list, in the launch of the rest of the backward (up to kSmallLookups) or one behind it, instead of the tile kernel's launch, which
// reads the gradient rows of a bag range once for all heavy rows, in tiles, and the one that adds up its sums.  A tile is read
// whatever few heavy rows look at it, and a workgroup that reads a lookup's gradient row from L2 has no other to wait for.
// The backward alone, us, tile kernel / entries, one table of 50 k rows of 64 fp32, 32 lookups a bag, lookups by a power law, on a
// hundred rows, evenly on all: 65536 lookups 52, 31, 17 / 14, 11, 14; 524288 83, 67, 26 / 31, 21, 22; 2097152 159, 76, 97 / 97, 64, 97;
// rows of 256 fp32, 262144 103, 60, 50 / 43, 37, 44, 2097152 1197, 291, 367 / 398, 266, 367; rows of 8 fp32, all lookups on five rows
// 524288 279 / 18.  Eight tables, 2097152 lookups, 128 binary16: 156, 75, 120 / 119, 81, 120.  Behind the line the lookups' gradient rows
// at L2 cost more than the tiles: 7.9 M lookups on 32 x 1M rows of 128 binary16, whole backward, 463 / 536, 3.9 M on 16 x 500k 246 / 250.
// Tables of 100 to 3000 rows, which have all the lookups, one, four and sixteen of them, 8, 32 and 128 lookups a bag, 1, 1.5 and 2 M
// lookups, rows of 32 to 512 binary16 and of 64 and 128 fp32: entries take 0.15 to 1.0 times as long in ten of eleven such models, up to
// 1.4 times in the others, most of them with rows of 128 and 256 binary16 from 1.5 M on.  Which it is changes from table count to table
// count and from bag length to bag length (2 M, 128 binary16, one table of 100 rows, 8, 32, 128 a bag 192, 104, 84 / 180, 137, 77; four of
// 300 128, 77, 65 / 164, 94, 66; sixteen of 300 126, 76, 63 / 118, 68, 60), and a model with some larger tables beside the small ones is
// faster by entries throughout (1.2 to 1.5 times): no line between them.
constexpr int64_t kLongLookups = 2097152;
inline bool long_rows_in_rest(int64_t n) { return n <= kLongLookups; }
// Lookups of a heavy row from which it has one entry more: a workgroup's share, or what would hold up a lane group of the tile
// kernel.  Entries of 256 / 512 / 1024 lookups, 256 fp32, us: 8192 lookups on one row 14 / 19 / 28, 65536 on five 16 / 20 / 30, 524288 on
// one 106 / 69 / 55 (the sums of a row's entries are one workgroup's to add up).
inline int heavy_split(int64_t n, bool maxp) {
  return maxp || !long_rows_in_rest(n) ? kHeavySplit : n <= 32768 ? 256 : n <= 262144 ? 512 : 1024;
}

// ---- launchers (each enqueues on `s` and returns the HIP status of the launch) ----

// counters of the batch to zero, sort keys and payloads of its lookups into ss.pairs[0]
hipError_t launch_keygen(const TableMeta *tm, const Geometry &g, const BatchBuf &b, const SortScratch &ss, hipStream_t s);
hipError_t launch_sort(const TableMeta *tm, const Geometry &g, const BatchBuf &b, const SortScratch &ss, int *result_buf, hipStream_t s);
// lock: batches before the current one whose ways are locked like the current batch's own (0 in the one-deep pipeline)
hipError_t launch_dedup_probe(const TableMeta *tm, const Geometry &g, const BatchBuf &b, SortScratch &ss,
                              const uint2 *sorted, int32_t *tags, int32_t *ts, int32_t *freq, bool lfu, const Level2 &l2, int lock, const StaleRows &stale,
                              const Totals &totals, hipStream_t s);
// the whole stage of a batch for which one_kernel_batch holds
hipError_t launch_one_kernel_stage(const TableMeta *tm, const Geometry &g, const BatchBuf &b, const SortScratch &ss, int32_t *tags,
                              int32_t *ts, int32_t *freq, bool lfu, const Level2 &l2, int lock, const StaleRows &stale,
                              const Totals &totals, hipStream_t s);
// write back the staged victims and (b != null) fetch ahead the rows b's batch inserts
// Deferred initialisation on read (Section 5.4.2): a row of the backing tier has no value until it is
// first fetched; the fetch then makes it up instead of reading it.
struct DeferredInit {
  const TableMeta *tm = nullptr;  // device table descriptions (init_bits); null = off
  unsigned long long seed = 0;
  float std = 0.f;
};

// parked: slots parked for write-back, at most
hipError_t launch_transfer(const BatchBuf *b, int64_t parked, const Staging &st, const Level2 &l2, const DeferredInit &di,
                           const Throttle &th, int k, const uint32_t *rb_of_table,
                           unsigned long long *bytes_h2d, unsigned long long *bytes_d2h, hipStream_t s);
// prev_mode: what becomes of prev's overflow copies: kPrevKeep (nothing), kPrevWrite (to the backing tier now),
// kPrevPark (among this batch's parked victims: the next transfer writes them)
constexpr int kPrevKeep = 0, kPrevWrite = 1, kPrevPark = 2;
// deep: the pipeline is several batches deep -- rows whose current value is an overflow copy of a batch that may
// not have trained yet are left to launch_fixup
hipError_t launch_commit(const TableMeta *tm, const BatchBuf &b, const BatchBuf *prev, int prev_mode, const Staging &st,
                         const Level2 &l2, const uint32_t *rb_of_table, unsigned long long *bytes_d2h, bool deep,
                         hipStream_t s);
// Transfer and commit of a batch, with none in flight in front of it, in one launch (prev_mode: kPrevKeep)?  That spares a launch and
// the 2 us between two kernels of a chain that the forward waits for; but the transfer kernel's own workgroups keep the link busier.
// Us a step on the compute stream, two launches / one: no row cached, 1000 rows of 64 bytes to 1 KB 57 / 55, 4000 80..83 / 77..80,
// 16000 of 64 bytes, 256 bytes and 1 KB 140, 182, 453 / 129, 186, 455, 64000 334, 584, 2069 / 338, 603, 2080; a third cached, 16000
// and 64000 of 256 bytes 68, 94 / 67, 94.
constexpr int64_t kSwapLookups = 8192;
hipError_t launch_swap(const TableMeta *tm, const BatchBuf &b, const BatchBuf *prev, int64_t parked, const Staging &st, const Level2 &l2,
                       const DeferredInit &di, const Throttle &th, const uint32_t *rb_of_table, unsigned long long *bytes_h2d,
                       unsigned long long *bytes_d2h, hipStream_t s);
// ---- pipeline several batches deep (Section 5.7) ----
// The overflow copies of every batch buffer, by buffer number.
struct OverflowCopies {
  const char *of_buf[kMaxBatchBufs];
};
// before b's forward, on the compute stream (every earlier batch has trained): the rows of b whose current value
// was an overflow copy of an earlier batch when b's commit ran are copied from there to where b uses them, and
// the accumulators of those it inserted are taken over again
hipError_t launch_fixup(const TableMeta *tm, const BatchBuf &b, const OverflowCopies &oc, const Staging &st,
                        const uint32_t *rb_of_table, unsigned long long *n_copied, hipStream_t s);
// after the batch's backward: its bypassed rows go from their HBM copies to the backing tier
// parked: how many overflow copies of the batch before, at most, b's commit parked and no transfer has written yet: they go first
hipError_t launch_ovf_writeback(const BatchBuf &b, int64_t parked, const Staging &st, const uint32_t *rb_of_table,
                                unsigned long long *bytes_d2h, hipStream_t s);
hipError_t launch_flush(const TableMeta *tm, const Geometry &g, const int32_t *tags, const Level2 &l2,
                        unsigned long long *bytes_h2d, unsigned long long *bytes_d2h, hipStream_t s);
// after launch_flush: the counters of `buffers` batch buffers to pinned host memory, and the accumulators of the tables with flush_by_kernel (at most kFlushStateRows rows, pinned host array)
constexpr int64_t kFlushStateRows = 262144;  // a megabyte: what the copy engine moves in the time it takes to start
hipError_t launch_flush_state(const TableMeta *tm, const Geometry &g, const BatchCounters *counters, BatchCounters *host_counters,
                              int buffers, hipStream_t s);
hipError_t launch_forward_classes(const TableMeta *tm, const ClassInfo &ci, const Geometry &g, const BatchBuf &b,
                                  float *out, hipStream_t s);
// which: kBwdHeavy (tile kernel; under max pooling the hot rows, a workgroup each, and for rows narrower than 16 lanes all with
// more than kLongRun lookups), or any of kBwdCombine (sums of the tile kernel's partial sums + update; nothing under max
// pooling), kBwdSingle (rows with one lookup), kBwdShort (rows with 2..kLongRun lookups, under max pooling also the other long
// rows) in one launch
constexpr int kBwdHeavy = 1, kBwdCombine = 2, kBwdSingle = 4, kBwdShort = 8;
constexpr int kBwdLong = 16;  // (of the kernel, see long_rows_in_rest: the heavy rows, a workgroup for each entry, in the combine's place)
hipError_t launch_backward_classes(int which, const TableMeta *tm, const ClassInfo &ci, const Geometry &g,
                                   const BatchBuf &b, const float *grad_out, float *partials, float lr, float eps,
                                   hipStream_t s);

// ---- small device helpers ----

// Bag ranges of the heavy-row backward for a batch with n_hchunks (table, row group) chunks and n_heavy
// heavy rows: enough ranges for about target_items work items, no more than the partial-sum buffer
// (slot_capacity slots of one row each) holds.  A function of the batch alone, so the summation order is
// reproducible.
__host__ __device__ inline int heavy_ranges(int n_hchunks, int n_heavy, long long slot_capacity, int target_items) {
  if (n_hchunks < 1 || n_heavy < 1) return 1;
  long long r = target_items / n_hchunks;  // rounded down: one round of workgroups
  // With many chunks (a model of many tables, or tables with thousands of heavy rows) one round would leave each
  // workgroup a quarter of a batch or more to sweep alone: four rounds of shorter items then, which also evens out
  // what the tables differ in (heterogeneous model: tile kernel 6.5 -> 1.7 ms).
  if (r < kHeavyRounds) r = ((long long)kHeavyRounds * target_items + n_hchunks - 1) / n_hchunks;
  if (r > kHeavyMaxRanges) r = kHeavyMaxRanges;
  if (r > slot_capacity / n_heavy) r = slot_capacity / n_heavy;
  return r < 1 ? 1 : (int)r;
}

// Heavy rows a workgroup of the tile kernel takes at once, and bags per gradient tile, for rows of
// `lanes` lanes of 16 bytes (4 fp32 or 8 fp16 elements each).
__host__ __device__ inline int heavy_chunk_rows(int lanes, int dtype) { return kHeavyThreads / lanes * heavy_rows_per_group(dtype); }
// parts a heavy row of `len` lookups is split into
__host__ __device__ inline int heavy_parts(int len, int split) {
  const int p = (len + split - 1) / split, most = split < kHeavySplit ? 0x7FFF : kHeavyMaxParts;
  return p < 1 ? 1 : (p > most ? most : p);
}
// first bag of bag range `range` of R over a batch of B bags per table (the ranges are equal to within one bag, so
// that the workgroups of the tile kernel, one per (chunk, range), have equal shares of the lookups)
__host__ __device__ inline int heavy_range_first(int B, int R, int range) { return (int)((long long)B * range / R); }
__host__ __device__ inline int heavy_tile_bags(int lanes, int dtype) {
  return kHeavyTileBytes / (lanes * (dtype == 0 ? 4 : 8) * 4);
}

// Workgroups are handed to the 8 XCDs (each with an L2 of its own) round robin by their
// linear id.  These helpers turn that id into a position in the work so that every XCD
// owns one contiguous eighth of it and walks it front to back: work is ordered by table,
// so a table's rows and its slice of the output gradient are cached in one L2 instead of
// in all eight.  Only the placement changes; any mapping gives the same results.
constexpr int kXcds = 8;

// position of linear workgroup `id` of `n` when every workgroup is one unit of work
__device__ inline int xcd_block_position(int id, int n) {
  const int q = n / kXcds, rem = n % kXcds, x = id % kXcds;
  return x * q + (x < rem ? x : rem) + id / kXcds;
}

// [first, end) and step of a grid-stride loop over `n` units, `per_block` units per workgroup
// and pass, confined to the XCD's eighth; gridDim.x must be a multiple of kXcds
__device__ inline void xcd_span(int n, int per_block, int &first, int &end, int &step) {
  const int x = blockIdx.x % kXcds, nb = gridDim.x / kXcds;
  const int lo = (int)((int64_t)n * x / kXcds);
  end = (int)((int64_t)n * (x + 1) / kXcds);
  first = lo + (int)(blockIdx.x / kXcds) * per_block;
  step = nb * per_block;
}

// the same for a kernel whose workgroups are numbered `id` of `nblocks` (a multiple of kXcds)
__device__ inline void xcd_span_of(int id, int nblocks, int n, int per_block, int &first, int &end, int &step) {
  const int x = id % kXcds, nb = nblocks / kXcds;
  const int lo = (int)((int64_t)n * x / kXcds);
  end = (int)((int64_t)n * (x + 1) / kXcds);
  first = lo + (id / kXcds) * per_block;
  step = nb * per_block;
}

// ---- words through which the workgroups of one kernel tell each other their counts ----
// A word carries its own "said" bit, so that a reader needs nothing but the word: written and read by atomics at the scope
// of the whole GPU, which pass the XCDs' own L2s by.
__device__ inline void say(unsigned long long *p, unsigned long long v) {
  __hip_atomic_store(p, v | 1ull << 63, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class W>
__device__ inline W look(const W *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class W>
__device__ inline W hear(const W *p, W v) {  // v: what a first look found
  constexpr W kSaid = (W)1 << (sizeof(W) * 8 - 1);
  while (!(v & kSaid)) {
    __builtin_amdgcn_s_sleep(1);
    v = look(p);
  }
  return v & ~kSaid;
}
// How often a workgroup looks at what another one has yet to say before it counts that one's part itself: some 60 us.
#ifndef TBE_POLLS
#define TBE_POLLS 64
#endif
constexpr int kPolls = TBE_POLLS;

// The batch's counters as its stage finds them; err: of a batch before it that was refused.
__device__ inline void begin_counters(BatchCounters *c, int32_t err) {
  c->n_uniq = c->n_touched = c->n_ins = c->n_byp = c->n_heavy = c->n_long = 0;
  c->err = err;
  c->n_mid = c->n_hchunks = 0;
  c->h_ranges = 1;
  c->hits = c->evictions = c->hit_lookups = 0;
  c->l2_hits = c->l2_demotions = c->l2_evictions = c->l2_bypasses = 0;
  c->packed = 0;
}

// n / d for any 32-bit n, with m = ceil(2^64 / d) (0 stands for d = 1): exact, because m d exceeds 2^64 by less than d
__device__ inline uint32_t div_by(uint32_t n, unsigned long long m) { return m ? (uint32_t)__umul64hi((unsigned long long)n, m) : n; }
__host__ __device__ inline unsigned long long div_magic(uint32_t d) { return d > 1 ? ~0ull / d + 1ull : 0ull; }

__device__ inline uint32_t row_of_key(const TableMeta &m, uint32_t key) {
  uint32_t local = key - m.key_base;
  if (m.sets == 0) return local;
  uint32_t s = local / m.rows_per_set;
  return (local - s * m.rows_per_set) * m.sets + s;
}

}  // namespace tbe
