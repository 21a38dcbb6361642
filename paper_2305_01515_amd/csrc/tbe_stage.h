// Device code of the prefetch stage that its two forms share: a kernel a pass (tbe_sort.hip, tbe_cache.hip), and the one kernel
// that takes a batch of very few lookups through all passes (tbe_one.hip).
#pragma once
#include "tbe_internal.h"

namespace tbe {

// The thread's number, opaque: a loop over all passes of the stage would otherwise keep in registers what each derives from it.
__device__ inline int my_thread() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

typedef unsigned long long u64;

// What a pass scans: 2 N counters of 32 bits, two to a word (a pass's Op::V).
template <int N>
struct Counts {
  u64 w[N];
  __device__ Counts &operator+=(const Counts &o) {
#pragma unroll
    for (int i = 0; i < N; i++) w[i] += o.w[i];
    return *this;
  }
  __device__ Counts operator-(const Counts &o) const {
    Counts r{};
#pragma unroll
    for (int i = 0; i < N; i++) r.w[i] = w[i] - o.w[i];
    return r;
  }
  __device__ uint32_t lo(int i) const { return (uint32_t)w[i]; }
  __device__ uint32_t hi(int i) const { return (uint32_t)(w[i] >> 32); }
};

template <int N>
__device__ inline Counts<N> wave_incl_scan(Counts<N> v, int lane) {
  for (int d = 1; d < 64; d <<= 1) {
    Counts<N> o{};
#pragma unroll
    for (int i = 0; i < N; i++) o.w[i] = __shfl_up(v.w[i], d);
    if (lane >= d) v += o;
  }
  return v;
}

template <int N>
__device__ inline Counts<N> wave_total(Counts<N> v) {
  for (int d = 32; d >= 1; d >>= 1) {
    Counts<N> o{};
#pragma unroll
    for (int i = 0; i < N; i++) o.w[i] = __shfl_xor(v.w[i], d);
    v += o;
  }
  return v;
}

// elements per wavefront: n spread over all wavefronts, in whole steps
__device__ inline int scan_chunk(int n, int waves, int step) {
  const int steps = (n + step - 1) / step;
  return (steps + waves - 1) / waves * step;
}

// Per-table constants the passes need for every flagged element, copied to LDS by the workgroup (a look-up in the table
// descriptions in memory is a chain of dependent loads per element otherwise).
struct KeyLut {
  u64 rps_magic[kLutTables];
  uint32_t key_base[kLutTables], sets[kLutTables], set_base[kLutTables];
};
struct TableLut {
  u64 rps_magic[kLutTables], sets_magic[kLutTables];
  uint32_t key_base[kLutTables], sets[kLutTables], rows_per_set[kLutTables], row_bytes[kLutTables];
  char *host_w[kLutTables];
  char *lines2[kLutTables];
  int32_t slot2_base[kLutTables];
};

__device__ inline void fill_lut(KeyLut &l, const TableMeta *tm, int T) {
  for (int t = my_thread(); t < T && t < kLutTables; t += blockDim.x) {
    l.key_base[t] = tm[t].key_base; l.sets[t] = tm[t].sets; l.rps_magic[t] = tm[t].rps_magic;
    l.set_base[t] = tm[t].set_base;
  }
}
__device__ inline void fill_lut(TableLut &l, const TableMeta *tm, int T) {
  for (int t = my_thread(); t < T && t < kLutTables; t += blockDim.x) {
    l.key_base[t] = tm[t].key_base; l.sets[t] = tm[t].sets; l.rows_per_set[t] = tm[t].rows_per_set;
    l.rps_magic[t] = tm[t].rps_magic; l.sets_magic[t] = tm[t].sets_magic;
    l.row_bytes[t] = tm[t].row_bytes; l.host_w[t] = tm[t].host_w;
    l.lines2[t] = tm[t].lines2; l.slot2_base[t] = tm[t].slot2_base;
  }
}

// a wavefront's chunk [base, end), with `carry` flags before it
template <class Op>
__device__ __forceinline__ void write_chunk(const Op &op, int base, int end, int n, int lane, typename Op::V carry) {
  typedef typename Op::V V;
  constexpr int kScanItems = Op::kItems, kScanStep = kWave * kScanItems;
  for (int i0 = base + lane * kScanItems; i0 - lane * kScanItems < end; i0 += kScanStep) {
    V f[kScanItems] = {};
    V tsum{};
#pragma unroll
    for (int q = 0; q < kScanItems; q++) {
      if (i0 + q < end) f[q] = op.flag(i0 + q, n);
      tsum += f[q];
    }
    const V incl = wave_incl_scan(tsum, lane);
    V pre = carry;
    pre += incl - tsum;
#pragma unroll
    for (int q = 0; q < kScanItems; q++) {
      if (i0 + q < end) op.emit(i0 + q, n, pre, f[q]);
      pre += f[q];
    }
    V last{};
#pragma unroll
    for (int i = 0; i < (int)(sizeof(V) / sizeof(u64)); i++) last.w[i] = __shfl(incl.w[i], 63, 64);
    carry += last;
  }
}

// ---- pass 1 over the N sorted lookups: distinct rows, run starts, and the first row of every touched set ----
// Set heads are found here as well, from the keys of neighbouring rows (they were a count and emit pass of their own over
// the set ids of the distinct rows, written here for it).  Keys ascend along a lane's elements, so every lane keeps the
// constants of the table it is in and moves on when a key passes the table's last; the set number is a multiplication.
struct DedupArgs {
  const TableMeta *tm;
  int T;
  const int32_t *bag_of_pos;
  const BatchCounters *cnt;
  int within_bits;
  const int64_t *offsets;
  // what a payload says of a lookup in `bag`: its position in input order and inside the bag
  __device__ uint32_t position(uint32_t p, int32_t bag) const {
    return cnt->packed ? (uint32_t)offsets[bag] + (p & ((1u << within_bits) - 1u)) : p;
  }
  __device__ uint32_t within(uint32_t p, int32_t bag) const {
    return cnt->packed ? p & ((1u << within_bits) - 1u) : p - (uint32_t)offsets[bag];
  }
  uint32_t *sorted_at;       // max pooling only (else null): position of the lookup in input order or inside its bag, by the
  int dtypes;                //   table's storage type (see BatchBuf; Geometry::dtypes)
  u64 bags_magic;            // of the bags per table
  uint32_t *uid_sorted;
  int32_t *sorted_bag;
  uint32_t *uniq_key;
  int32_t *run_off;
  int32_t *uniq_tab;
  uint2 *touched;
};
// Args: DedupArgs, or a reference to it (what a method needs of it is then loaded there)
template <class Args, int ITEMS = 1>
struct DedupPass {
  static constexpr int kItems = ITEMS;
  typedef Counts<1> V;  // lo: distinct rows, hi: touched sets
  typedef KeyLut Lut;
  Args a;
  // the table this lane's keys are in
  mutable int t;
  mutable uint32_t base, last, set_base;  // keys base .. last
  mutable u64 magic;                      // of rows_per_set; sets == 0: not used
  mutable bool cached;
  mutable const KeyLut *lut;  // null: the model has too many tables for it
  __device__ bool prepare(KeyLut &l) const {
    lut = a.T <= kLutTables ? &l : nullptr;
    if (lut) fill_lut(l, a.tm, a.T);
    t = -1;
    last = 0;
    return lut != nullptr;
  }
  __device__ void enter_table(uint32_t k) const {  // last table with key_base <= k
    int lo = t < 0 ? 0 : t, hi = a.T - 1;
    uint32_t sets;
    if (lut) {
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (lut->key_base[mid] <= k) lo = mid; else hi = mid - 1;
      }
      base = lut->key_base[lo]; sets = lut->sets[lo]; magic = lut->rps_magic[lo]; set_base = lut->set_base[lo];
      last = lo + 1 < a.T ? lut->key_base[lo + 1] - 1u : 0xFFFFFFFFu;
    } else {
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (a.tm[mid].key_base <= k) lo = mid; else hi = mid - 1;
      }
      base = a.tm[lo].key_base; sets = a.tm[lo].sets; magic = a.tm[lo].rps_magic; set_base = a.tm[lo].set_base;
      last = lo + 1 < a.T ? a.tm[lo + 1].key_base - 1u : 0xFFFFFFFFu;
    }
    t = lo;
    cached = sets != 0;
  }
  // Is the lookup with key k, behind one with key `before`, the first of its row (bit 0), the row the first of its set (bit 1)?
  __device__ uint32_t head(bool first, uint32_t k, uint32_t before) const {
    if (!first && k == before) return 0u;
    if (t < 0 || k > last) enter_table(k);
    // rows of a table without a cache are one set
    return first || before < base || (cached && div_by(k - base, magic) != div_by(before - base, magic)) ? 3u : 1u;
  }
  __device__ V flag(int i, int) const {
    const uint32_t f = head(i == 0, a.key[i], i ? a.key[i - 1] : 0u);
    return V{{(f & 1u) | (u64)(f >> 1) << 32}};
  }
  __device__ uint32_t sorted_at(uint32_t p, int32_t bag) const {
    const bool inside = a.dtypes == 1 || (a.dtypes == 3 && a.tm[div_by((uint32_t)bag, a.bags_magic)].dtype == 0);
    return inside ? a.within(p, bag) : a.position(p, bag);
  }
  // distinct row u, whose first lookup is the i-th; set_head: the first of the v-th touched set
  __device__ void write_row(uint32_t k, int i, uint32_t u, bool set_head, uint32_t v) const {
    if (t < 0 || k < base || k > last) enter_table_of(k);  // (the lane's next element may lie in the next table)
    a.uniq_key[u] = k;
    a.run_off[u] = i;
    a.uniq_tab[u] = t;
    if (set_head) a.touched[v] = make_uint2(cached ? set_base + div_by(k - base, magic) : kNoSet, u);
  }
  __device__ void emit(int i, int, const V &pre, const V &f) const {
    const uint32_t u = pre.lo(0) + f.lo(0) - 1u;
    a.uid_sorted[i] = u;
    const uint32_t p = a.pos[i];
    const int32_t bag = a.bag_of(p);
    a.sorted_bag[i] = bag;
    if (a.sorted_at) a.sorted_at[i] = sorted_at(p, bag);
    if (f.lo(0)) write_row(a.key[i], i, u, f.hi(0) != 0, pre.hi(0));
  }
  __device__ void enter_table_of(uint32_t k) const {
    t = -1;
    enter_table(k);
  }
  __device__ void rewind() const { t = -1; }
  __device__ void wave_done(int, int) const {}
  __device__ void finish(BatchCounters *cnt, int n, const V &total) const {
    cnt->n_uniq = (int32_t)total.lo(0);
    cnt->n_touched = (int32_t)total.hi(0);
    a.run_off[total.lo(0)] = n;
  }
};

// The plan of the tile kernel, from the heavy list (in table order; first_of_table[t] = position of table t's first entry,
// first_of_table[T] = their number), by workgroups of the stage's last kernel:
//   - every workgroup adds up the chunks of all tables (a chunk: the rows one workgroup of the tile kernel takes,
//     heavy_chunk_rows of the table's lanes per row) and so knows the batch's number of bag ranges;
//   - workgroup t < T writes table t's chunks and orders its entries by lookups per entry, descending, in classes of powers
//     of two (entries of a class keep their order, so the result is a function of the batch alone): the tile kernel deals
//     the entries round its lane groups in this order, so the groups that share a wavefront -- which runs as long as its
//     busiest group -- get rows of like length;
//   - the others find, for every entry and bag range, the first sorted position of the entry's row whose bag lies in the
//     range (the row's lookups are sorted by bag), a thread per (entry, range).
// (As three kernels, the chunks by one workgroup and the order by one wavefront per table: 10 M rows of one table, 32 k
// bags, beside the transfer kernel: 4 + 35 + 21 us; as one kernel of workgroups of 512 threads 17 us.)
struct PlanArgs {
  const TableMeta *tm;
  int T, B;
  const int32_t *first_of_table, *heavy, *heavy_sub, *uniq_tab, *run_off, *sorted_bag;
  uint4 *hchunks;
  int32_t *hperm, *hstart;
  long long slot_capacity;
  int target_items;
};
constexpr int kPlanClasses = 32;
template <int THREADS>
struct PlanLds {
  int all[THREADS / kWave], before[THREADS / kWave];
  int base[THREADS / kWave][kPlanClasses];
};
template <int THREADS>
__device__ __forceinline__ void plan_heavy(int blk, int blocks, const PlanArgs &a, PlanLds<THREADS> &s, BatchCounters *cnt) {
  constexpr int kPlanThreads = THREADS, kWaves = kPlanThreads / kWave, kClasses = kPlanClasses;
  auto &s_all = s.all;
  auto &s_before = s.before;
  auto &s_base = s.base;
  const TableMeta *tm = a.tm;
  const int T = a.T, B = a.B, target_items = a.target_items;
  const long long slot_capacity = a.slot_capacity;
  const int32_t *first_of_table = a.first_of_table, *heavy = a.heavy, *heavy_sub = a.heavy_sub, *uniq_tab = a.uniq_tab,
                *run_off = a.run_off, *sorted_bag = a.sorted_bag;
  uint4 *hchunks = a.hchunks;
  int32_t *hperm = a.hperm, *hstart = a.hstart;
  const int tid = my_thread(), lane = tid & 63, wave = tid >> 6;
  const int n_heavy = cnt->n_heavy;
  int all = 0, before = 0;  // chunks of all tables, and of those before this workgroup's
  for (int t = tid; t < T; t += kPlanThreads) {
    const int per = heavy_chunk_rows(tm[t].lanes, tm[t].dtype);
    const int chunks = (first_of_table[t + 1] - first_of_table[t] + per - 1) / per;
    all += chunks;
    if (t < blk) before += chunks;
  }
  for (int d = 32; d >= 1; d >>= 1) { all += __shfl_xor(all, d); before += __shfl_xor(before, d); }
  if (lane == 0) { s_all[wave] = all; s_before[wave] = before; }
  if (tid < kClasses)
    for (int w = 0; w < kWaves; w++) s_base[w][tid] = 0;
  __syncthreads();
  all = before = 0;
  for (int w = 0; w < kWaves; w++) { all += s_all[w]; before += s_before[w]; }
  const int R = heavy_ranges(all, n_heavy, slot_capacity, target_items);
  if (blk == 0 && tid == 0) {
    cnt->n_hchunks = all;
    cnt->h_ranges = R;
  }
  if (blk >= T) {
    const int n = n_heavy * R;
    for (int x = (blk - T) * kPlanThreads + tid; x < n; x += (blocks - T) * kPlanThreads) {
      const int h = x / R, range = x % R;
      const int u = heavy[h];
      const int t = uniq_tab[u];
      const long long first_bag = (long long)t * B + heavy_range_first(B, R, range);
      int lo = run_off[u], hi = run_off[u + 1];
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (sorted_bag[mid] < first_bag) lo = mid + 1; else hi = mid;
      }
      hstart[x] = lo;
    }
    return;
  }
  const int t = blk;
  const int first = first_of_table[t], n = first_of_table[t + 1] - first;
  if (n == 0) return;
  const int per = heavy_chunk_rows(tm[t].lanes, tm[t].dtype);
  for (int c = tid; c * per < n; c += kPlanThreads)
    hchunks[before + c] = make_uint4((uint32_t)t, (uint32_t)(first + c * per), (uint32_t)min(per, n - c * per), 0u);
  auto klass = [&](int h) {  // 31 - floor(log2(lookups per entry)): longer entries first
    const int u = heavy[h];
    const int len = (run_off[u + 1] - run_off[u]) / (heavy_sub[h] >> 16);
    return __clz(len < 1 ? 1 : len);
  };
  // every wavefront takes a contiguous part of the entries: its counts per class, then the part's positions in order
  const int part = ((n + kWaves - 1) / kWaves + 63) / 64 * 64;
  const int p0 = min(n, wave * part), p1 = min(n, p0 + part);
  for (int i = p0 + lane; i < p1; i += kWave) atomicAdd(&s_base[wave][klass(first + i) & (kClasses - 1)], 1);
  __syncthreads();
  if (tid < kClasses) {  // counts to first positions: classes in order, inside a class the wavefronts in order
    int mine = 0;
    for (int w = 0; w < kWaves; w++) mine += s_base[w][tid];
    int incl = mine;
    for (int d = 1; d < kClasses; d <<= 1) {
      const int o = __shfl_up(incl, d, 64);
      if (tid >= d) incl += o;
    }
    int at = incl - mine;
    for (int w = 0; w < kWaves; w++) { const int c = s_base[w][tid]; s_base[w][tid] = at; at += c; }
  }
  __syncthreads();
  const uint64_t lt_mask = (1ull << lane) - 1ull;
  for (int i0 = p0; i0 < p1; i0 += kWave) {
    const bool valid = i0 + lane < p1;
    const int k = valid ? klass(first + i0 + lane) & (kClasses - 1) : 0;
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int bit = 0; bit < 5; bit++) {
      const bool on = (k >> bit) & 1;
      const uint64_t bal = __ballot(on);
      peers &= on ? bal : ~bal;
    }
    const int below = __popcll(peers & lt_mask);
    int at = 0;
    if (valid && below == 0) at = atomicAdd(&s_base[wave][k], __popcll(peers));
    at = __shfl(at, valid ? __ffsll((unsigned long long)peers) - 1 : lane);
    if (valid) hperm[first + at + below] = first + i0 + lane;
  }
}

// ---- pass 2 over the distinct rows after the probe: insert and bypass lists, the work lists of the backward by run
// length (see kLongRun; in the order of the distinct rows, i.e. in table order: the backward kernels give each XCD a
// contiguous part of a list), counters, and for every missed row
// whether its backing-tier copy is stale and where its value is instead.  The map that says so is read and written here,
// by the lane that handles the row; its entries are checked against the lists of the batches whose copies are on their
// way instead of being taken out again.  (With a pass of its own over the missed rows for the look-up and up to three
// for entering and taking out entries, four launches more: small configuration, six steps 1276 -> 1198 us; 16 x 500k
// resident rows, four steps 2773 -> 2731 us.  On the benchmark workload, where two thirds of the distinct rows miss, this pass
// itself takes 66 to 92 instead of 34 us alone and 114 instead of 38 beside the other streams, as a row's entry and the list that it
// points into are two dependent reads; the five kinds of launches that it took over were 128 us there.)
struct StatusArgs {
  const TableMeta *tm;
  int T;
  const uint8_t *status;
  const int32_t *run_off;
  const int32_t *old_tag;
  const uint32_t *uniq_key;
  const int32_t *uniq_tab;
  int32_t *ins_idx;
  int32_t *ins_tab;
  int32_t *ins_slot;
  int32_t *ins_old;
  uint32_t *ins_key;
  uint32_t *vic_key;
  char **ins_src;
  uint32_t *ins_where;
  int32_t *byp_idx;
  int32_t *byp_tab;
  uint32_t *byp_key;
  char **byp_src;
  uint32_t *byp_where;
  uint8_t *byp_taken;
  StaleRows stale;
  int32_t *loc_u;
  int32_t *mid_idx, *heavy, *heavy_sub, *first_of_table;
  // second level (all null without one)
  const int32_t *src2, *dst2, *evict2;
  char **ins_dst, **l2v_src, **l2v_dst;
  uint32_t *l2v_key;
  u64 *tally;
  int heavy_split;
};
template <class Args>
struct StatusPass {
  static constexpr int kItems = 1;
  typedef Counts<2> V;  // lo and hi of word 0: inserts, bypasses; of word 1: rows with 2..kLongRun lookups, heavy-list entries
  struct Lut : TableLut {};
  Args a;
  // per-thread tallies (the emit kernel keeps one Op copy per thread in registers); every wavefront leaves
  // its sums in `a.tally` (three words each), which the kernel that keeps the running totals adds up -- thousands
  // of atomic additions to one counter from all over the chip would take longer than the pass itself
  mutable unsigned int evs, late;
  mutable u64 hit_lookups;
  mutable const TableLut *lut;  // null: the model has too many tables for it
  __device__ bool prepare(TableLut &l) const {
    lut = a.T <= kLutTables ? &l : nullptr;
    if (lut) fill_lut(l, a.tm, a.T);
    return lut != nullptr;
  }
  struct TabView {
    u64 rps_magic, sets_magic;
    uint32_t key_base, sets, rows_per_set, row_bytes;
    char *host_w, *lines2;
    int32_t slot2_base;
    __device__ uint32_t row_of(uint32_t key) const {
      const uint32_t local = key - key_base;
      if (sets == 0) return local;
      const uint32_t s = div_by(local, rps_magic);
      return (local - s * rows_per_set) * sets + s;
    }
    __device__ uint32_t key_of(uint32_t row) const {
      if (sets == 0) return key_base + row;
      const uint32_t q = div_by(row, sets_magic);
      return key_base + (row - q * sets) * rows_per_set + q;
    }
  };
  __device__ TabView view(int t) const {
    if (lut)
      return TabView{lut->rps_magic[t], lut->sets_magic[t], lut->key_base[t], lut->sets[t], lut->rows_per_set[t], lut->row_bytes[t], lut->host_w[t], lut->lines2[t],
                     lut->slot2_base[t]};
    const TableMeta &m = a.tm[t];
    return TabView{m.rps_magic, m.sets_magic, m.key_base, m.sets, m.rows_per_set, m.row_bytes, m.host_w, m.lines2, m.slot2_base};
  }
  // Where the value of the missed row with this key is: 0 = in the backing tier, else the kWhere* code of an HBM copy
  // that is newer (the row is "late").  Says so to whoever would send that copy home.
  __device__ uint32_t current_place(uint32_t key) const {
    const uint32_t code = a.stale.where[key];
    if (code == 0u || !a.stale.prev_cnt) return 0u;
    if (code & kWhereOverflow) {
      if (a.stale.deep) {
        const uint32_t buf = (code >> kWhereBufShift) & (kMaxBatchBufs - 1), j = code & kWhereBufIndex;
        if (!(a.stale.live >> buf & 1u)) return 0u;
        const DeepBuf d = a.stale.deep[buf];  // (whose copy goes home all the same, right behind its batch's own backward)
        return (int)j < d.cnt->n_byp && d.byp_key[j] == key ? code : 0u;
      }
      const int j = (int)(code & kWhereIndex);
      if (j < a.stale.prev_cnt->n_byp && a.stale.prev_byp_key[j] == key) {
        a.stale.prev_byp_taken[j] = 1;  // that copy need not go home: this batch's does, or the row's cache line
        return code;
      }
      if (a.stale.pp_cnt && j < a.stale.pp_cnt->n_byp && a.stale.pp_byp_key[j] == key) {
        const uint32_t slot = (uint32_t)(a.stale.prev_cnt->n_ins + j);
        a.stale.wb_skip[slot] = 1;
        return kWhereParked | slot;
      }
      return 0u;
    }
    // a victim the batch before parked and this batch wants back skips the trip to the host
    const uint32_t i = code & kWhereIndex;
    const uint32_t n = (uint32_t)a.stale.prev_cnt->n_ins;
    bool there = i < n && a.stale.prev_vic_key[i] == key;
    if (a.stale.prev_l2v_src && i >= a.stale.max_inserts) {
      const uint32_t v = i - a.stale.max_inserts;
      there = v < n && a.stale.prev_l2v_src[v] && a.stale.prev_l2v_key[v] == key;
    }
    if (!there) return 0u;
    a.stale.wb_skip[i] = 1;
    return code;
  }
  __device__ V flag(int u, int) const {
    V f{};
    const uint8_t s = a.status[u];
    const int len = a.run_off[u + 1] - a.run_off[u];
    f.w[0] = s == ST_INSERT ? 1ull : s == ST_BYPASS ? (1ull << 32) : 0ull;
    f.w[1] = len > kLongRun ? (u64)heavy_parts(len, a.heavy_split) << 32 : len >= 2 ? 1ull : 0ull;
    return f;
  }
  __device__ void emit(int u, int, const V &pre, const V &f) const {
    const int t = a.uniq_tab[u];
    for (int x = u ? a.uniq_tab[u - 1] + 1 : 0; x <= t; x++) a.first_of_table[x] = (int32_t)pre.hi(1);
    if (f.lo(1)) a.mid_idx[pre.lo(1)] = u;
    const int parts = (int)f.hi(1);
    for (int q = 0; q < parts; q++) {  // a hot row is entered in several parts
      a.heavy[pre.hi(1) + q] = u;
      a.heavy_sub[pre.hi(1) + q] = q | (parts << 16);
    }
    if (f.lo(0)) {
      const uint32_t i = pre.lo(0);
      const uint32_t key = a.uniq_key[u];
      const TabView m = view(t);
      const uint32_t row = m.row_of(key);
      const int32_t old = a.old_tag[u];
      a.ins_idx[i] = u;
      a.ins_tab[i] = t;
      a.ins_slot[i] = a.loc_u[u];
      a.ins_old[i] = old;
      a.ins_key[i] = key;
      const uint32_t place = current_place(key);
      a.ins_where[i] = place;
      late += place != 0u;
      a.ins_src[i] = m.host_w + (size_t)row * m.row_bytes;
      if (a.src2) {  // second level: the row may come from there, the victim may go there
        const int32_t s2 = a.src2[u], d2 = a.dst2[u], e2 = a.evict2[u];
        if (s2 >= 0) a.ins_src[i] = m.lines2 + (size_t)(s2 - m.slot2_base) * m.row_bytes;
        char *dst = old >= 0 ? m.host_w + (size_t)old * m.row_bytes : nullptr;
        if (old >= 0 && d2 >= 0) dst = m.lines2 + (size_t)(d2 - m.slot2_base) * m.row_bytes;
        a.ins_dst[i] = dst;
        a.l2v_src[i] = e2 >= 0 ? dst : nullptr;  // the line the victim takes still holds the row it pushes out
        a.l2v_dst[i] = e2 >= 0 ? m.host_w + (size_t)e2 * m.row_bytes : nullptr;
        a.l2v_key[i] = e2 >= 0 ? m.key_of((uint32_t)e2) : 0u;
        if (e2 >= 0) a.stale.where[a.l2v_key[i]] = kWhereParked | (a.stale.max_inserts + i);  // staged behind the victims
      }
      // The victim's entry in the map.  No row of this batch is a victim of it, and no two of its rows have the same
      // victim, so every entry is read or written by one lane.
      uint32_t vk = key;
      if (old >= 0) {
        evs++;
        vk = m.key_of((uint32_t)old);
        a.stale.where[vk] = kWhereParked | i;
      }
      a.vic_key[i] = vk;
    } else if (f.hi(0)) {
      const uint32_t j = pre.hi(0);
      const uint32_t key = a.uniq_key[u];
      const TabView m = view(t);
      a.byp_idx[j] = u;
      a.byp_tab[j] = t;
      a.byp_key[j] = key;
      a.byp_src[j] = m.host_w + (size_t)m.row_of(key) * m.row_bytes;
      const uint32_t place = current_place(key);
      a.byp_where[j] = place;
      late += place != 0u;
      a.stale.where[key] = a.stale.own_code | j;
      a.byp_taken[j] = 0;
      if (a.src2 && a.src2[u] >= 0)  // lives in the second level: used in place
        a.byp_src[j] = m.lines2 + (size_t)(a.src2[u] - m.slot2_base) * m.row_bytes;
      a.loc_u[u] = -2 - (int32_t)j;  // the row is served from the j-th overflow slot
    } else if (a.status[u] == ST_HIT) {
      hit_lookups += (u64)(a.run_off[u + 1] - a.run_off[u]);
    }
  }
  __device__ void rewind() const {}
  __device__ void wave_done(int lane, int w) const {
    u64 e = evs, l = hit_lookups;
    unsigned int lt = late;
    for (int d = 32; d >= 1; d >>= 1) {
      e += __shfl_xor(e, d);
      l += __shfl_xor(l, d);
      lt += __shfl_xor(lt, d);
    }
    if (lane == 0) {
      a.tally[3 * w] = e;
      a.tally[3 * w + 1] = l;
      a.tally[3 * w + 2] = lt;
    }
  }
  __device__ void finish(BatchCounters *cnt, int n, const V &total) const {
    cnt->n_ins = (int32_t)total.lo(0);
    cnt->n_byp = (int32_t)total.hi(0);
    cnt->n_mid = (int32_t)total.lo(1);
    cnt->n_heavy = (int32_t)total.hi(1);
    for (int x = n > 0 ? a.uniq_tab[n - 1] + 1 : 0; x <= a.T; x++) a.first_of_table[x] = (int32_t)total.hi(1);
  }
};
typedef StatusPass<StatusArgs> StatusOp;

// --------------------------------------------------------------------------------------
// Probe + replacement.  A wavefront takes a window of consecutive touched sets -- as many as hold about a
// wavefront's width of distinct rows, at most kProbeSets -- and keeps the ways of all of them in LDS.
//   phase 1, a lane per distinct row over the whole window: a row that is found is a hit, its way is
//            stamped k and its count grows by the row's lookups in the batch;
//   phase 2, per set of the window that has a miss, lane w holding way w: the evictable ways are ranked by
//            (timestamp, way) -- LRU -- or by (count, timestamp, way) -- LFU; the j-th miss in ascending
//            row order takes the way of rank j (evicting what it held) and starts counting at its own
//            lookups; misses beyond the number of such ways bypass the cache.
// Rows of a set arrive in ascending order because the sort key is (set, row div S).
// A set's chain of dependent reads (set head -> table -> ways -> rows) is several memory round trips; with a
// cache as large as the tables a batch touches a million sets with two or three rows each, and one set per
// wavefront left the kernel waiting on that chain (0.67 ms for the benchmark shapes with every row resident).
// --------------------------------------------------------------------------------------
__device__ inline int32_t add_saturating(int32_t a, int32_t b) {  // a, b >= 0
  const uint32_t v = (uint32_t)a + (uint32_t)b;
  return v > 0x7FFFFFFFu ? 0x7FFFFFFF : (int32_t)v;
}

#ifndef TBE_PROBE_ROWS
#define TBE_PROBE_ROWS 64        // distinct rows a window aims for
#endif

struct ProbeArgs {
  const TableMeta *tm;
  int T, W;
  int32_t k, evictable_below, min_windows;
  const uint32_t *uniq_key;
  const int32_t *uniq_tab;
  const uint2 *touched;
  int32_t *tags, *ts, *freq;
  const int32_t *run_off;
  int32_t *loc_u;
  uint8_t *status;
  int32_t *old_tag, *tags2, *ts2;
  int l2_factor;
  int32_t *src2, *dst2, *evict2;
  int32_t *l2_sums;  // second level: its four counters, kL2Sums times, a line each (0 between batches)
};

// (Added to the batch's counters themselves by three thousand wavefronts, the additions were most of the probe: 4 x 500k rows, 327 k lookups 90 us, now 33.)

// What a wavefront keeps of its window of at most SETS sets, and as many ways as 32 a set make (a set of 64 ways fits two).
template <bool L2, int SETS>
struct ProbeLds {
  static_assert(SETS >= 2 && SETS <= 32, "a window's sets with a miss are a 32-bit mask");
  static constexpr int kWays = 32 * SETS;
  // ways of set i of the window at [i * (W + 1), i * (W + 1) + W): the odd stride keeps lanes that scan
  // different sets on different banks
  int32_t w_tag[kWays + SETS], w_ts[kWays + SETS], w_freq[kWays + SETS];
  int32_t h_u0[SETS + 1], h_tab[SETS], h_slot0[SETS];
  uint32_t h_key0[SETS], h_sets[SETS], h_set[SETS];
  int32_t l_way[kWave];
  int32_t l_tag2[L2 ? kWave : 1], l_ts2[L2 ? kWave : 1], l_way2[L2 ? kWave : 1];
  int32_t v_row[L2 ? kWave : 1], v_u[L2 ? kWave : 1];
};

// What the lanes of a wavefront have written, each other's to read.
__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Wavefront `wave` of `waves`: every waves-th window.
template <bool LFU, bool L2, int SETS>
__device__ __forceinline__ void probe_windows(const ProbeArgs &a, ProbeLds<L2, SETS> &s, int wave, int waves, BatchCounters *cnt) {
  constexpr int kProbeSets = SETS, kProbeWays = ProbeLds<L2, SETS>::kWays;
  auto &w_tag = s.w_tag; auto &w_ts = s.w_ts; auto &w_freq = s.w_freq;
  auto &h_u0 = s.h_u0; auto &h_tab = s.h_tab; auto &h_slot0 = s.h_slot0;
  auto &h_key0 = s.h_key0; auto &h_sets = s.h_sets; auto &h_set = s.h_set;
  auto &l_way = s.l_way; auto &l_tag2 = s.l_tag2; auto &l_ts2 = s.l_ts2; auto &l_way2 = s.l_way2;
  auto &v_row = s.v_row; auto &v_u = s.v_u;
  const TableMeta *tm = a.tm;
  const int W = a.W, l2_factor = a.l2_factor;
  const int32_t k = a.k, evictable_below = a.evictable_below, min_windows = a.min_windows;
  const uint32_t *uniq_key = a.uniq_key;
  const int32_t *uniq_tab = a.uniq_tab, *run_off = a.run_off;
  const uint2 *touched = a.touched;
  int32_t *tags = a.tags, *ts = a.ts, *freq = a.freq, *loc_u = a.loc_u, *old_tag = a.old_tag, *tags2 = a.tags2, *ts2 = a.ts2,
          *src2 = a.src2, *dst2 = a.dst2, *evict2 = a.evict2;
  uint8_t *status = a.status;
  int n_l2hit = 0, n_l2dem = 0, n_l2ev = 0, n_l2byp = 0;  // this lane's share of the second-level counters
  const int lane = my_thread() & (kWave - 1);
  const int n_touched = cnt->n_touched, n_uniq = cnt->n_uniq;
  const uint64_t lt_mask = (1ull << lane) - 1ull;
  const int WP = W + 1;
  int ns = n_uniq > 0 ? (int)(((long long)TBE_PROBE_ROWS * n_touched + n_uniq - 1) / n_uniq) : 1;
  int ns_max = kProbeWays / W < kProbeSets ? kProbeWays / W : kProbeSets;
  if (ns_max > n_touched / min_windows) ns_max = n_touched / min_windows;  // few sets: a wavefront each
  ns = ns > ns_max ? ns_max : ns;
  ns = ns < 1 ? 1 : ns;
  for (long long v0 = (long long)wave * ns; v0 < n_touched; v0 += (long long)waves * ns) {
    const int nv = n_touched - v0 < ns ? (int)(n_touched - v0) : ns;
    wave_sync();
    if (lane <= nv) {
      const long long v = v0 + lane;
      uint2 head = make_uint2(kNoSet, (uint32_t)n_uniq);
      if (v < n_touched) head = touched[v];
      h_u0[lane] = (int)head.y;
      if (lane < nv) {
        if (head.x == kNoSet) {  // rows of tables without a cache
          h_slot0[lane] = -1;
        } else {
          const int t = uniq_tab[head.y];
          const TableMeta &m = tm[t];
          const uint32_t set = head.x - m.set_base;
          h_tab[lane] = t;
          h_slot0[lane] = (int)head.x * W;  // global slot id of way 0 (set_base * W == slot_base)
          h_set[lane] = set;
          h_sets[lane] = m.sets;
          h_key0[lane] = m.key_base + set * m.rows_per_set;
        }
      }
    }
    wave_sync();
    const int U0 = h_u0[0], U1 = h_u0[nv];
    for (int e = lane; e < nv * W; e += kWave) {
      const int si = e / W, w = e - si * W;
      const int s0 = h_slot0[si];
      if (s0 >= 0) {
        w_tag[si * WP + w] = tags[s0 + w];
        w_ts[si * WP + w] = ts[s0 + w];
        w_freq[si * WP + w] = freq[s0 + w];
      }
    }
    wave_sync();
    // phase 1: hits, a lane per distinct row of the window
    uint32_t miss_sets = 0;
    for (int c = U0; c < U1; c += kWave) {
      const int u = c + lane;
      if (u < U1) {
        int si = 0;
        for (int i = 1; i < nv; i++) si += h_u0[i] <= u ? 1 : 0;
        const int s0 = h_slot0[si];
        if (L2) src2[u] = dst2[u] = evict2[u] = -1;
        if (s0 < 0) {
          loc_u[u] = -1;
          status[u] = ST_BYPASS;
        } else {
          const int32_t row = (int32_t)((uniq_key[u] - h_key0[si]) * h_sets[si] + h_set[si]);
          const int base = si * WP;
          int hit = -1;
          for (int w = 0; w < W; w++)
            if (w_tag[base + w] == row) hit = w;
          if (hit >= 0) {
            w_ts[base + hit] = k;
            w_freq[base + hit] = add_saturating(w_freq[base + hit], run_off[u + 1] - run_off[u]);
            loc_u[u] = s0 + hit;
            status[u] = ST_HIT;
          } else {
            status[u] = ST_MISS;
            miss_sets |= 1u << si;
          }
        }
      }
    }
    for (int d = 32; d >= 1; d >>= 1) miss_sets |= __shfl_xor(miss_sets, d);
    const uint32_t new_tags = miss_sets;  // only a miss changes a set's tags
    wave_sync();
    while (miss_sets) {  // the same in every lane
      const int si = __ffs(miss_sets) - 1;
      miss_sets &= miss_sets - 1;
      const int base = si * WP;
      int32_t *l_tag = w_tag + base, *l_ts = w_ts + base, *l_freq = w_freq + base;
      const int u0 = h_u0[si], u1 = h_u0[si + 1];
      const int slot0 = h_slot0[si];
      const TableMeta &m = tm[h_tab[si]];
      const uint32_t set = h_set[si], key0 = h_key0[si];
      // phase 2: rank the evictable ways
      const int32_t my_ts = lane < W ? l_ts[lane] : 0x7FFFFFFF;
      // evictable: free ways (-1) and ways stamped before evictable_below = max(k - lock, 1): the ways of this batch
      // and, in a pipeline `lock` batches deep, of the batches that may still be waiting for their training
      const bool cand = lane < W && my_ts < evictable_below;
      const int32_t my_freq = lane < W ? l_freq[lane] : 0;
      int rank = 0;
      for (int w = 0; w < W; w++) {
        const int32_t tw = l_ts[w];
        if (tw >= evictable_below) continue;
        bool first = tw < my_ts || (tw == my_ts && w < lane);
        if (LFU) {
          const int32_t fw = l_freq[w];
          first = fw < my_freq || (fw == my_freq && first);
        }
        if (first) rank++;
      }
      const int n_cand = __popcll(__ballot(cand));
      wave_sync();
      if (cand) l_way[rank] = lane;
      wave_sync();
      int before = 0;
      for (int c = u0; c < u1; c += kWave) {
        const int u = c + lane;
        const bool miss = u < u1 && status[u] == ST_MISS;
        const uint64_t mb = __ballot(miss);
        if (miss) {
          const int j = before + __popcll(mb & lt_mask);
          if (j < n_cand) {
            const int way = l_way[j];
            old_tag[u] = l_tag[way];
            l_tag[way] = (int32_t)((uniq_key[u] - key0) * m.sets + set);
            l_ts[way] = k;
            l_freq[way] = run_off[u + 1] - run_off[u];
            loc_u[u] = slot0 + way;
            status[u] = ST_INSERT;
          } else {
            loc_u[u] = -1;
            status[u] = ST_BYPASS;
          }
        }
        before += __popcll(mb);
      }
      wave_sync();
      if (L2) {
        // ---- second level (exclusive): the rows this set missed are looked up there, then the
        // rows this set evicted move down.  sets2 = l2_factor * sets, so a row r of this set
        // belongs to second-level set  set + sets * ((r div sets) mod l2_factor)  and no other
        // first-level set shares it: this wavefront owns all of them.
        int n_v = 0;  // the victims of this set: at most W, one per lane
        for (int c = u0; c < u1; c += kWave) {
          const int u = c + lane;
          const bool valid = u < u1;
          const bool isv = valid && status[u] == ST_INSERT && old_tag[u] >= 0;
          const uint64_t vm = __ballot(isv);
          if (isv) {
            const int p = n_v + __popcll(vm & lt_mask);
            v_row[p] = old_tag[u];
            v_u[p] = u;
          }
          n_v += __popcll(vm);
        }
        wave_sync();
        const int32_t my_v = lane < n_v ? v_row[lane] : -1;
        const int my_vset = my_v >= 0 ? (int)(((uint32_t)my_v / m.sets) % (uint32_t)l2_factor) : -1;
        for (int j = 0; j < l2_factor; j++) {
          const int slot20 = m.slot2_base + (int)(set + (uint32_t)j * m.sets) * W;
          l_tag2[lane] = lane < W ? tags2[slot20 + lane] : -2;
          l_ts2[lane] = lane < W ? ts2[slot20 + lane] : 0x7FFFFFFF;
          wave_sync();
          // (A) missed rows of this second-level set: found and inserted above -> moves up, its entry
          // becomes free; found but bypassed above -> stays, used in place, stamped k
          for (int c = u0; c < u1; c += kWave) {
            const int u = c + lane;
            const uint32_t q = u < u1 ? uniq_key[u] - key0 : 0u;  // row div sets
            const bool mine = u < u1 && status[u] != ST_HIT && (int)(q % (uint32_t)l2_factor) == j;
            const int32_t row = mine ? (int32_t)(q * m.sets + set) : -3;
            int hw = -1;
            for (int w = 0; w < W; w++)
              if (l_tag2[w] == row) hw = w;
            if (hw >= 0) {
              src2[u] = slot20 + hw;
              if (status[u] == ST_INSERT) { l_tag2[hw] = -1; l_ts2[hw] = -1; } else l_ts2[hw] = k;
              n_l2hit++;
            }
          }
          wave_sync();
          // (B) victims of this second-level set in ascending row order take the ways older than
          // k - 1 in order of (timestamp, way); entries of this batch and the one before stay
          const bool vmine = my_vset == j;
          int vrank = 0;
          for (int w = 0; w < n_v; w++) {
            const int32_t o = v_row[w];
            if ((int)(((uint32_t)o / m.sets) % (uint32_t)l2_factor) == j && o < my_v) vrank++;
          }
          const int32_t my_ts2 = l_ts2[lane];
          const bool cand2 = lane < W && my_ts2 < k - 1;
          int rank2 = 0;
          for (int w = 0; w < W; w++) {
            const int32_t tw = l_ts2[w];
            if (tw < k - 1 && (tw < my_ts2 || (tw == my_ts2 && w < lane))) rank2++;
          }
          const int n_cand2 = __popcll(__ballot(cand2));
          if (cand2) l_way2[rank2] = lane;
          wave_sync();
          if (vmine) {
            if (vrank < n_cand2) {
              const int way = l_way2[vrank];
              const int32_t held = l_tag2[way];
              evict2[v_u[lane]] = held;
              dst2[v_u[lane]] = slot20 + way;
              l_tag2[way] = my_v;
              l_ts2[way] = k;
              n_l2dem++;
              if (held >= 0) n_l2ev++;
            } else {
              n_l2byp++;  // no way to take: the victim goes to the lower tier
            }
          }
          wave_sync();
          if (lane < W) {
            tags2[slot20 + lane] = l_tag2[lane];
            ts2[slot20 + lane] = l_ts2[lane];
          }
          wave_sync();
        }
      }
    }
    wave_sync();
    for (int e = lane; e < nv * W; e += kWave) {
      const int si = e / W, w = e - si * W;
      const int s0 = h_slot0[si];
      if (s0 >= 0) {
        if (new_tags >> si & 1u) tags[s0 + w] = w_tag[si * WP + w];
        ts[s0 + w] = w_ts[si * WP + w];
        freq[s0 + w] = w_freq[si * WP + w];
      }
    }
  }
  if (L2) {
    for (int d = 32; d >= 1; d >>= 1) {
      n_l2hit += __shfl_xor(n_l2hit, d); n_l2dem += __shfl_xor(n_l2dem, d);
      n_l2ev += __shfl_xor(n_l2ev, d); n_l2byp += __shfl_xor(n_l2byp, d);
    }
    if (lane == 0) {
      int32_t *l2 = a.l2_sums + wave % kL2Sums * kL2Line;
      if (n_l2hit) atomicAdd(l2, n_l2hit);
      if (n_l2dem) atomicAdd(l2 + 1, n_l2dem);
      if (n_l2ev) atomicAdd(l2 + 2, n_l2ev);
      if (n_l2byp) atomicAdd(l2 + 3, n_l2byp);
    }
  }
}

// Completes the batch's counters -- evictions, lookups that hit and late rows from the per-wavefront sums of the status pass,
// hits as what is left of the distinct rows -- and adds them to the running totals.  By one workgroup.
// heavy_sub, split: the heavy list's parts and what makes one; a row counts as often as it would be entered by kHeavySplit.
template <int THREADS>
struct TotalsLds {
  u64 e[THREADS / kWave], l[THREADS / kWave], t[THREADS / kWave];
  int longs;
};
template <int THREADS>
__device__ __forceinline__ void add_totals(BatchCounters *c, const Totals &t, const u64 *tally, int tally_waves, const int32_t *heavy_sub,
                                           int split, TotalsLds<THREADS> &s) {
  constexpr int kFinalThreads = THREADS;
  auto &s_e = s.e; auto &s_l = s.l; auto &s_t = s.t;
  const int n_heavy = c->n_heavy, per = kHeavySplit / split;
  if (threadIdx.x == 0) s.longs = 0;
  u64 e = 0, l = 0, late = 0;
#pragma unroll 4
  for (int w = threadIdx.x; w < tally_waves; w += kFinalThreads) { e += tally[3 * w]; l += tally[3 * w + 1]; late += tally[3 * w + 2]; }
  for (int d = 32; d >= 1; d >>= 1) { e += __shfl_xor(e, d); l += __shfl_xor(l, d); late += __shfl_xor(late, d); }
  if ((threadIdx.x & 63) == 0) { s_e[threadIdx.x >> 6] = e; s_l[threadIdx.x >> 6] = l; s_t[threadIdx.x >> 6] = late; }
  __syncthreads();
  if (per > 1 && n_heavy) {
    int longs = 0;
    for (int h0 = threadIdx.x; h0 < n_heavy; h0 += 8 * kFinalThreads) {
      int sub[8];
#pragma unroll
      for (int q = 0; q < 8; q++) sub[q] = h0 + q * kFinalThreads < n_heavy ? heavy_sub[h0 + q * kFinalThreads] : 1;
#pragma unroll
      for (int q = 0; q < 8; q++) {
        const int parts = ((sub[q] >> 16) + per - 1) / per;
        if (!(sub[q] & 0xFFFF)) longs += parts < kHeavyMaxParts ? parts : kHeavyMaxParts;
      }
    }
    if (longs) atomicAdd(&s.longs, longs);
    __syncthreads();
  }
  if (t.l2 && threadIdx.x < kL2Sums) {  // (one wavefront)
    int32_t *p = t.l2_sums + threadIdx.x * kL2Line;
    int4 v = *(int4 *)p;
    *(int4 *)p = make_int4(0, 0, 0, 0);
    for (int d = 32; d >= 1; d >>= 1) {
      v.x += __shfl_xor(v.x, d);
      v.y += __shfl_xor(v.y, d);
      v.z += __shfl_xor(v.z, d);
      v.w += __shfl_xor(v.w, d);
    }
    if (threadIdx.x == 0) {
      c->l2_hits = v.x;
      c->l2_demotions = v.y;
      c->l2_evictions = v.z;
      c->l2_bypasses = v.w;
    }
  }
  if (threadIdx.x != 0) return;
  e = l = late = 0;
  for (int w = 0; w < kFinalThreads / 64; w++) { e += s_e[w]; l += s_l[w]; late += s_t[w]; }
  c->n_long = per > 1 ? s.longs : n_heavy;
  c->hits = (u64)(c->n_uniq - c->n_ins - c->n_byp);
  c->evictions = e;
  c->hit_lookups = l;
  t.sum->hits += c->hits;
  t.sum->evictions += e;
  t.sum->hit_lookups += l;
  t.n[0] += (u64)c->n_uniq;
  t.n[1] += (u64)c->n_ins;
  t.n[2] += (u64)c->n_byp;
  t.n[3] += late;
  if (t.l2) {
    t.l2[0] += (u64)c->l2_hits;
    t.l2[1] += (u64)c->l2_demotions;
    t.l2[2] += (u64)c->l2_evictions;
    t.l2[3] += (u64)c->l2_bypasses;
  }
}

// What the passes of the stage work on, of one batch.
inline DedupArgs dedup_of(const TableMeta *tm, const Geometry &g, const BatchBuf &b) {
  return DedupArgs{tm, g.T, b.bag_of_pos, b.cnt, g.within_bits, b.d_offsets,
                 b.maxp ? b.sorted_at : nullptr, g.dtypes, div_magic((uint32_t)b.batch), b.uid_sorted, b.sorted_bag, b.uniq_key, b.run_off,
                 b.uniq_tab, b.touched};
}
inline ProbeArgs probe_of(const TableMeta *tm, const Geometry &g, const BatchBuf &b, int32_t *tags, int32_t *ts, int32_t *freq,
                          const Level2 &l2, int lock) {
  return ProbeArgs{tm, g.T, g.ways, b.k, b.k - lock > 1 ? b.k - lock : 1, probe_min_windows(g, 0), b.uniq_key, b.uniq_tab, b.touched,
                   tags, ts, freq, b.run_off, b.loc_u, b.status, b.old_tag, l2.tags2, l2.ts2, l2.factor,
                   l2.on ? b.src2 : nullptr, l2.on ? b.dst2 : nullptr, l2.on ? b.evict2 : nullptr, l2.sums};
}
inline StatusArgs status_of(const TableMeta *tm, const Geometry &g, const BatchBuf &b, const Level2 &l2, const StaleRows &stale, u64 *tally) {
  return StatusArgs{tm, g.T, b.status, b.run_off, b.old_tag, b.uniq_key, b.uniq_tab, b.ins_idx, b.ins_tab, b.ins_slot,
                  b.ins_old, b.ins_key, b.vic_key, b.ins_src, b.ins_where,
                  b.byp_idx, b.byp_tab, b.byp_key, b.byp_src, b.byp_where, b.byp_taken, stale, b.loc_u, b.mid_idx, b.heavy, b.heavy_sub, b.hfirst,
                  l2.on ? b.src2 : nullptr, l2.on ? b.dst2 : nullptr, l2.on ? b.evict2 : nullptr,
                  l2.on ? b.ins_dst : nullptr, l2.on ? b.l2v_src : nullptr, l2.on ? b.l2v_dst : nullptr,
                  l2.on ? b.l2v_key : nullptr, tally, heavy_split(b.n, b.maxp)};
}
inline PlanArgs plan_of(const TableMeta *tm, const Geometry &g, const BatchBuf &b) {
  return PlanArgs{tm, g.T, b.batch, b.hfirst, b.heavy, b.heavy_sub, b.uniq_tab, b.run_off, b.sorted_bag, b.hchunks, b.hperm, b.hstart,
                  (long long)g.partial_slots, g.heavy_target};
}

}  // namespace tbe
