// The prefetch stage of a small batch -- keys, sort, distinct rows, probe, lists, location words -- as one kernel.
//
// Such a stage is bound by launches (a launch is 4 us of host time with this many arguments) and by the latency of its
// dependent passes, not by bytes.  Here every pass is a phase
// of one launch, and the phases hand their results over through the L2 of one XCD: all workgroups that take part run on the
// XCD of the first one to begin (the others leave at once), so that what one has written another reads in the cache that they
// share.  Measured with 40960 words turned round per phase, us a phase: 16 workgroups of 1024 threads of one XCD 1.9 (1.2
// without the waves' invalidation of their L1), kernels of their own 2.2; workgroups of all XCDs, which have to write their
// L2 back and invalidate it at every hand-over, 5.4 to 6.7 with 32 to 128 of 512 threads.
//
// Work items go out by tickets, phase after phase: a workgroup takes the next one when it has done the one before, and waits
// until all items of the phase in front are done (in the phase that writes lists also for the counts of the items before its
// own).  So an item waits only for items with earlier tickets, and every one of
// those is in the hands of a workgroup that runs: every wait ends whatever else is on the GPU, and however many workgroups
// take part -- one is enough.
//
// The first phase is one workgroup's: a batch's keys fit its LDS, and three sort passes there take 5 us (119 lookups) to 14
// (3662), where as launches they took 21.  The whole stage, us on the GPU: 119 lookups 30, 3028 lookups 52; as nine launches
// 35 and 50 in the kernels alone and 2 between each two, but 37 us of host time instead of 4.  Two steps of 2 tables x 2000
// rows, 16 bags, no prefetching ahead: 251 -> 192 us; drawn models of 117 to 3028 lookups a batch 1.06 to 1.36 times as fast.
#include "tbe_stage.h"

namespace tbe {

constexpr int kOneWaves = kOneThreads / kWave;
constexpr int kOneProbeSets = 4;  // of a wavefront's window: 16 wavefronts' worth of ways fit 64 KB
constexpr int kKeygenLanes = 8;   // lanes per bag: 64-byte reads of the bag's indices
constexpr int kSortItems = kOneLookups / kOneThreads;
constexpr int kRadix = 256;
constexpr int kTileBits = 12;  // the sort's payload: the lookup's position in the low bits, its bag above
static_assert(kOneLookups == 1ll << kTileBits && kOneBags <= 1ll << (32 - kTileBits), "the payload holds both");
static_assert(kOneLookups % kOneThreads == 0, "a whole number of keys per thread");
static_assert(kOneLookups == kOneItems * kOneThreads && kOneItems <= kOneThreads, "the list pass: an element per thread, a thread hears one item");

struct OneStage {
  const TableMeta *tm;
  int T, B, n;
  const int64_t *indices, *offsets;
  uint32_t *sorted_pos;
  float *inv_len;             // null: not mean pooling
  DigitPlan digits;
  OneCtl *ctl;
  int32_t *refused;
  DedupArgs dedup;            // (its keys and payloads are not used)
  ProbeArgs probe;
  StatusArgs status;
  Totals totals;
  const u64 *tally;
  const uint32_t *uid_sorted;
  const int32_t *loc_u, *run_off;
  uint32_t *loc;
  BatchCounters *cnt;
  int probe_items, list_items, loc_items;
  int first[kOnePhases + 1];  // first ticket of every phase; behind the last one their number
};

// The pass over the sorted lookups, whose keys and payloads are in LDS.
struct TileDedupArgs {
  typedef __attribute__((address_space(3))) uint32_t *LdsWords;
  const TableMeta *tm;
  int T;
  LdsWords key, pos;
  const int64_t *offsets;
  uint32_t *sorted_at;
  int dtypes;
  u64 bags_magic;
  uint32_t *uid_sorted;
  int32_t *sorted_bag;
  uint32_t *uniq_key;
  int32_t *run_off;
  int32_t *uniq_tab;
  uint2 *touched;
  __device__ int32_t bag_of(uint32_t p) const { return (int32_t)(p >> kTileBits); }
  __device__ uint32_t position(uint32_t p, int32_t) const { return p & ((uint32_t)kOneLookups - 1u); }
  __device__ uint32_t within(uint32_t p, int32_t bag) const { return position(p, bag) - (uint32_t)offsets[bag]; }
};
typedef DedupPass<TileDedupArgs, kSortItems> TileDedup;
typedef StatusPass<const StatusArgs &> OneStatus;

template <class Op>
struct ListLds {
  typename Op::Lut lut;
  typename Op::V wave[kOneWaves], before[kOneWaves];
};
struct TileLds {
  uint32_t keys[kOneLookups], vals[kOneLookups];
  uint32_t cnt[kOneWaves][kRadix];
  uint32_t dstart[kRadix];
  uint32_t wtot[kRadix / kWave];
  uint32_t err, refused;
  ListLds<TileDedup> list;
};
template <bool L2>
union OneLds {
  TileLds tile;
  ListLds<OneStatus> status;
  ProbeLds<L2, kOneProbeSets> probe[kOneWaves];
  TotalsLds<kOneThreads> totals;
};

__device__ inline uint32_t word_of(const uint32_t *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline uint32_t add_to(uint32_t *p, uint32_t v) { return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// The batch's bags, 8 lanes each: put(position, sort key, bag) for every lookup, refuse(code) for what makes the batch one to
// refuse.  Four bags of a lane group are under way at a time: each is a chain of three reads (offsets, table, indices).
template <class Refuse, class Put>
__device__ __forceinline__ void keys_of_bags(const OneStage &a, Refuse refuse, Put put) {
  const int tid = my_thread();
  const int nb = a.T * a.B;
  const int sub = tid % kKeygenLanes;
  constexpr int kBags = kOneThreads / kKeygenLanes, K = 4;
  for (int bag0 = tid / kKeygenLanes; bag0 < nb; bag0 += K * kBags) {
    int lo[K], hi[K];
    int64_t r[K][2];
#pragma unroll
    for (int q = 0; q < K; q++) {
      const int bag = bag0 + q * kBags;
      lo[q] = hi[q] = 0;
      if (bag < nb) {
        const int64_t l = a.offsets[bag], h = a.offsets[bag + 1];
        if (l < 0 || h > a.n || l > h || (bag == 0 && l != 0) || (bag == nb - 1 && h != a.n)) {
          if (sub == 0) refuse(1 /* -TBE_EINVAL */);
        } else {
          lo[q] = (int)l;
          hi[q] = (int)h;
        }
        if (a.inv_len && sub == 0) a.inv_len[bag] = h > l ? 1.0f / (float)(h - l) : 0.0f;
      }
    }
#pragma unroll
    for (int q = 0; q < K; q++)
#pragma unroll
      for (int x = 0; x < 2; x++) {
        const int j = lo[q] + sub + x * kKeygenLanes;
        r[q][x] = j < hi[q] ? a.indices[j] : 0;
      }
#pragma unroll
    for (int q = 0; q < K; q++) {
      if (lo[q] + sub >= hi[q]) continue;
      const int bag = bag0 + q * kBags;
      const TableMeta &m = a.tm[bag / a.B];
      const int64_t rows = m.rows;
      const uint32_t key_base = m.key_base, sets = m.sets, rows_per_set = m.rows_per_set;
      const u64 sets_magic = m.sets_magic;
      for (int j = lo[q] + sub, x = 0; j < hi[q]; j += kKeygenLanes, x++) {
        int64_t row = x == 0 ? r[q][0] : x == 1 ? r[q][1] : a.indices[j];
        if (row < 0 || row >= rows) {
          refuse(2 /* -TBE_ERANGE */);
          row = 0;
        }
        const uint32_t d = div_by((uint32_t)row, sets_magic);
        put(j, sets ? key_base + ((uint32_t)row - d * sets) * rows_per_set + d : key_base + (uint32_t)row, bag);
      }
    }
  }
}

// Stable rank of every key of a wavefront's among those of its digit, and the wavefront's count of each digit in `cnt`.
__device__ __forceinline__ void rank_keys(const uint32_t (&key)[kSortItems], uint32_t (&rank)[kSortItems], uint32_t *cnt, int seg, int n,
                                          int lane, int shift, uint32_t mask) {
  const uint64_t lt_mask = (1ull << lane) - 1ull;
#pragma unroll
  for (int q = 0; q < kSortItems; q++) {
    rank[q] = 0;
    if (seg + q * kWave >= n) continue;  // the same in all lanes
    const bool valid = seg + q * kWave + lane < n;
    const uint32_t d = (key[q] >> shift) & mask;
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int bit = 0; bit < 8; bit++) {
      const bool on = (d >> bit) & 1u;
      const uint64_t bal = __ballot(on);
      peers &= on ? bal : ~bal;
    }
    const uint32_t below = __popcll(peers & lt_mask);
    uint32_t prev = 0;
    if (valid && below == 0) prev = atomicAdd(&cnt[d], (uint32_t)__popcll(peers));
    const int leader = valid ? (__ffsll((unsigned long long)peers) - 1) : lane;
    prev = __shfl(prev, leader);
    rank[q] = prev + below;
  }
}

__device__ inline void digit_of_pass(const DigitPlan &d, int pass, int &shift, uint32_t &mask) {
  shift = 0;
  mask = 0;
#pragma unroll
  for (int p = 0; p < kMaxSortPasses; p++)
    if (p == pass) { shift = d.shift[p]; mask = d.mask[p]; }
}

// A pass that writes lists (see the skeleton in tbe_cache.hip): an item counts the flags of its elements, kItems a thread, says
// its sums, adds up those of the items before it and writes; the last one knows the totals.
template <class Op>
__device__ __forceinline__ void list_phase(Op op, ListLds<Op> &s, int n, int blk, int items, u64 *said, BatchCounters *cnt) {
  typedef typename Op::V V;
  constexpr int kWords = sizeof(V) / sizeof(u64);
  if (op.prepare(s.lut)) __syncthreads();
  constexpr int kScanItems = Op::kItems;
  const int tid = my_thread(), lane = tid & 63, wave = tid >> 6;
  const int i0 = ((blk * kOneWaves + wave) * kWave + lane) * kScanItems;
  V mine{}, f[kScanItems] = {};
#pragma unroll
  for (int q = 0; q < kScanItems; q++)
    if (i0 + q < n) {
      f[q] = op.flag(i0 + q, n);
      mine += f[q];
    }
  const V of_lane = mine;
  mine = wave_total(mine);
  if (lane == 0) s.wave[wave] = mine;
  __syncthreads();
  V own{}, carry{};
  for (int w = 0; w < kOneWaves; w++) {
    own += s.wave[w];
    if (w < wave) carry += s.wave[w];
  }
  if (items > 1) {
    if (tid < kWords) say(said + tid * kOneItems + blk, tid == 0 ? own.w[0] : own.w[kWords - 1]);
    V before{};
    if (tid < blk) {  // an item before this one per thread
      V v{};
#pragma unroll
      for (int i = 0; i < kWords; i++) v.w[i] = look(said + i * kOneItems + tid);
#pragma unroll
      for (int i = 0; i < kWords; i++) before.w[i] = hear(said + i * kOneItems + tid, v.w[i]);
    }
    before = wave_total(before);
    if (lane == 0) s.before[wave] = before;
    __syncthreads();
    before = V{};
    for (int w = 0; w < kOneWaves; w++) before += s.before[w];
    carry += before;
    own += before;  // the last item's is the total
  }
  carry += wave_incl_scan(of_lane, lane) - of_lane;
#pragma unroll
  for (int q = 0; q < kScanItems; q++) {
    if (i0 + q < n) op.emit(i0 + q, n, carry, f[q]);
    carry += f[q];
  }
  op.wave_done(lane, blk * kOneWaves + wave);
  if (blk == items - 1 && tid == 0) op.finish(cnt, n, own);
}

// Keys, sort and distinct rows, by one workgroup, in LDS from the indices to the lists.
__device__ __forceinline__ void tile_phase(const OneStage &a, TileLds &s) {
  const int tid = my_thread(), lane = tid & 63, wave = tid >> 6;
  const int n = a.n;
  if (tid == 0) {
    begin_counters(a.cnt, 0);
    s.err = 0;
    s.refused = word_of((const uint32_t *)a.refused);
  }
  __syncthreads();
  keys_of_bags(a, [&](int code) { atomicMax(&s.err, (uint32_t)code); }, [&](int j, uint32_t key, int bag) {
    s.keys[j] = key;
    s.vals[j] = (uint32_t)bag << kTileBits | (uint32_t)j;
  });
  __syncthreads();
  if (s.err || s.refused) {
    if (tid == 0) atomicMax(&a.ctl->err, s.err);
    return;
  }
  const int waves = (n + kWave * kSortItems - 1) / (kWave * kSortItems);  // that have keys
  const int seg = wave * (kWave * kSortItems);
  for (int pass = 0; pass < a.digits.passes; pass++) {
    int shift;
    uint32_t mask;
    digit_of_pass(a.digits, pass, shift, mask);
    uint32_t key[kSortItems], val[kSortItems], rank[kSortItems];
#pragma unroll
    for (int q = 0; q < kSortItems; q++) {
      const int i = seg + q * kWave + lane;
      key[q] = i < n ? s.keys[i] : 0u;
      val[q] = i < n ? s.vals[i] : 0u;
    }
    for (int i = tid; i < waves * kRadix; i += kOneThreads) (&s.cnt[0][0])[i] = 0;
    __syncthreads();
    rank_keys(key, rank, s.cnt[wave], seg, n, lane, shift, mask);
    __syncthreads();
    uint32_t total = 0, incl = 0;
    if (tid < kRadix) {
      for (int w = 0; w < waves; w++) {
        const uint32_t c = s.cnt[w][tid];
        s.cnt[w][tid] = total;
        total += c;
      }
      incl = total;
      for (int dd = 1; dd < 64; dd <<= 1) {
        const uint32_t o = __shfl_up(incl, dd);
        if (lane >= dd) incl += o;
      }
      if (lane == 63) s.wtot[wave] = incl;
    }
    __syncthreads();
    if (tid < kRadix) {
      uint32_t wb = 0;
      for (int w = 0; w < wave; w++) wb += s.wtot[w];
      s.dstart[tid] = wb + incl - total;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kSortItems; q++) {
      if (seg + q * kWave + lane < n) {
        const uint32_t d = (key[q] >> shift) & mask;
        const uint32_t p = s.dstart[d] + s.cnt[wave][d] + rank[q];
        s.keys[p] = key[q];
        s.vals[p] = val[q];
      }
    }
    __syncthreads();
  }
  for (int i = tid; i < n; i += kOneThreads) a.sorted_pos[i] = s.vals[i] & ((uint32_t)kOneLookups - 1u);
  typedef TileDedupArgs::LdsWords LdsWords;
  const DedupArgs &d = a.dedup;
  list_phase(TileDedup{TileDedupArgs{d.tm, d.T, (LdsWords)s.keys, (LdsWords)s.vals, d.offsets, d.sorted_at, d.dtypes, d.bags_magic,
                                     d.uid_sorted, d.sorted_bag, d.uniq_key, d.run_off, d.uniq_tab, d.touched}},
             s.list, n, 0, 1, nullptr, a.cnt);
}

// The lookups' location words in input order.
__device__ __forceinline__ void locations(const OneStage &a, int item, int items) {
  for (int i = item * kOneThreads + my_thread(); i < a.n; i += items * kOneThreads) {
    const uint32_t u = a.uid_sorted[i], p = a.sorted_pos[i];
    const int32_t lu = a.loc_u[u];
    uint32_t w = lu >= 0 ? (uint32_t)lu : (kLocOverflow | (uint32_t)(-2 - lu));
    if (a.run_off[u + 1] - a.run_off[u] == 1) w |= kLocSingle;
    a.loc[p] = w;
  }
}

// The end of the stage: the totals by its first item, the location words.  (Heavy rows need no plan, see long_rows_in_rest.)
template <bool L2>
__device__ __forceinline__ void end_phase(const OneStage &a, OneLds<L2> &s, int item, uint32_t err) {
  const int tid = my_thread();
  if (item == 0) {
    if (tid < 2 * kOneItems) a.ctl->said[tid] = 0ull;
    if (err == 0) {
      add_totals(a.cnt, a.totals, a.tally, a.list_items * kOneWaves, a.status.heavy_sub, a.status.heavy_split, s.totals);
    } else if (tid == 0) {  // (what this batch's own fault is stays below that of a batch before it)
      a.cnt->err = (int32_t)err;
      if (*a.refused == 0) *a.refused = (int32_t)err | kRefusedBefore;  // (later items of this launch know of it from ctl->err)
    }
  } else {
    if (err == 0) locations(a, item - 1, a.loc_items);
  }
}

// Number of the XCD that the wavefront runs on (hardware register 20, XCC_ID, bits 0 to 3).
__device__ inline uint32_t my_xcd() { return __builtin_amdgcn_s_getreg((3 << 11) | 20); }

// The kernel's argument, in the memory that the launch put it in.  Opaque, so that what a phase needs of it is loaded there:
// the compiler would load all of it in front of the loop over the items, into five times as many scalar registers as there are.
__device__ inline const OneStage &stage_arg() {
  typedef const __attribute__((address_space(4))) OneStage *Arg;
  Arg p = (Arg)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const OneStage *)p;
}

template <bool LFU, bool L2>
__global__ __launch_bounds__(kOneThreads) void one_stage_kernel(OneStage) {
  __shared__ OneLds<L2> s;
  __shared__ uint32_t s_ticket, s_phase, s_err;
  const int tid = my_thread();
  const bool alone = gridDim.x == 1;
  if (tid == 0) {  // does this workgroup run on the XCD of the one that began first?
    uint32_t here = 1;
    if (!alone) {
      const OneStage &a = stage_arg();
      const uint32_t me = my_xcd() + 1;
      uint32_t v = word_of(&a.ctl->chosen);
      if (v == 0u && __hip_atomic_compare_exchange_strong(&a.ctl->chosen, &v, me, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) v = me;
      here = v == me;
    }
    s_ticket = here;
  }
  __syncthreads();
  const bool takes_part = s_ticket != 0;
  if (takes_part) {
    constexpr int kEnd = 3;
    int phase = -1;
    uint32_t ticket = 0;
    for (;;) {
      const OneStage &a = stage_arg();
      // Every store of this workgroup has reached the L2 before its item counts as done, and nothing that its CU's L1 holds
      // from before is read after the wait.
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      if (tid < kWave) {
        if (tid == 0) {
          uint32_t t = phase < 0 ? 0u : ticket + 1u;
          if (!alone) {
            if (phase >= 0) add_to(&a.ctl->done[phase].n, 1u);
            t = add_to(&a.ctl->next, 1u);
          }
          uint32_t p = 0, before = 0, from = 0;  // its phase, and the items of the phase in front
#pragma unroll
          for (int q = 1; q <= kOnePhases; q++)
            if (t >= (uint32_t)a.first[q]) {
              p = q;
              before = (uint32_t)a.first[q] - from;
              from = (uint32_t)a.first[q];
            }
          if (!alone && p > 0 && p <= kEnd)
            while (word_of(&a.ctl->done[p - 1].n) < before) __builtin_amdgcn_s_sleep(1);
          s_ticket = t;
          s_phase = p;
          s_err = p > 0 ? max(word_of(&a.ctl->err), word_of((const uint32_t *)a.refused)) : 0u;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      }
      __syncthreads();
      ticket = s_ticket;
      phase = (int)s_phase;
      const uint32_t err = s_err;
      if (phase > kEnd) break;
      int item = (int)ticket;
#pragma unroll
      for (int q = 1; q <= kEnd; q++)
        if (q == phase) item = (int)ticket - a.first[q];
      __syncthreads();  // (the words above are read by all before the next hand-over writes them)
      if (phase == 0) {
        tile_phase(stage_arg(), s.tile);
      } else if (phase == kEnd) {
        end_phase(stage_arg(), s, item, err);
      } else if (err) {
        // this batch, or one before it, is refused: nothing is done
      } else if (phase == 1) {
        const OneStage &a = stage_arg();
        const int wave = my_thread() / kWave;
        probe_windows<LFU, L2>(a.probe, s.probe[wave], item * kOneWaves + wave, a.probe_items * kOneWaves, a.cnt);
      } else {
        const OneStage &a = stage_arg();
        list_phase(OneStatus{a.status}, s.status, a.cnt->n_uniq, item, a.list_items, a.ctl->said, a.cnt);
      }
    }
  }
  // The last workgroup to leave puts the words back to zero: all others have read them for the last time.
  const OneStage &a = stage_arg();
  __syncthreads();
  if (tid == 0) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "agent");
    s_ticket = alone || add_to(&a.ctl->left, 1u) == gridDim.x - 1;
  }
  __syncthreads();
  if (s_ticket && tid < kOnePhases + 4) {
    uint32_t *w = tid < kOnePhases ? &a.ctl->done[tid].n : tid == kOnePhases ? &a.ctl->chosen : tid == kOnePhases + 1 ? &a.ctl->left
                  : tid == kOnePhases + 2 ? &a.ctl->next : &a.ctl->err;
    (void)__hip_atomic_exchange(w, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

hipError_t launch_one_kernel_stage(const TableMeta *tm, const Geometry &g, const BatchBuf &b, const SortScratch &ss, int32_t *tags,
                              int32_t *ts, int32_t *freq, bool lfu, const Level2 &l2, int lock, const StaleRows &stale,
                              const Totals &totals, hipStream_t s) {
  const int n = (int)b.n;
  OneStage a{};
  a.tm = tm;
  a.T = g.T;
  a.B = b.batch;
  a.n = n;
  a.indices = b.d_indices;
  a.offsets = b.d_offsets;
  a.inv_len = b.mean ? b.inv_len : nullptr;
  a.digits = digit_plan(g.key_bits, (g.key_bits + 7) / 8);
  a.ctl = ss.one;
  a.refused = ss.refused;
  a.dedup = dedup_of(tm, g, b);
  a.probe = probe_of(tm, g, b, tags, ts, freq, l2, lock);
  a.status = status_of(tm, g, b, l2, stale, ss.tally);
  a.totals = totals;
  a.tally = ss.tally;
  a.sorted_pos = (uint32_t *)ss.pairs[0];
  a.uid_sorted = b.uid_sorted;
  a.loc_u = b.loc_u;
  a.run_off = b.run_off;
  a.loc = b.loc;
  a.cnt = b.cnt;
  const int wgs = one_stage_workgroups(g, l2.on, n);
  a.probe_items = wgs;
  a.probe.min_windows = probe_min_windows(g, wgs * kOneWaves);
  a.list_items = (n + kOneThreads - 1) / kOneThreads;
  a.loc_items = a.list_items;
  static_assert(kOneLookups <= kLongLookups, "no plan of the heavy rows");
  const int items[kOnePhases] = {1, a.probe_items, a.list_items, 1 + a.loc_items};
  for (int p = 0; p < kOnePhases; p++) a.first[p + 1] = a.first[p] + items[p];
  auto kern = l2.on ? (lfu ? one_stage_kernel<true, true> : one_stage_kernel<false, true>)
                    : (lfu ? one_stage_kernel<true, false> : one_stage_kernel<false, false>);
  // workgroups are dealt round robin over the XCDs: as many as are wanted on each
  hipLaunchKernelGGL(kern, dim3(wgs == 1 ? 1 : wgs * kXcds), dim3(kOneThreads), 0, s, a);
  return hipGetLastError();
}

}  // namespace tbe
