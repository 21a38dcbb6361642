// Index dedup part 2 (run-length encoding of the sorted keys), the set-associative probe
// with LRU victim choice and miss-list compaction.  Paper Section 5.5: tag/state lookup
// (5.5.1, probe and grouping by destination) and cache algorithm (5.5.2), one-level cache.
#include "tbe_stage.h"

namespace tbe {

// --------------------------------------------------------------------------------------
// Generic flag -> exclusive prefix -> emit skeleton over n elements (n may live on the device): every workgroup counts the
// flags of its contiguous chunk, says its sums, adds up those of the workgroups before it and emits its elements in order; the
// last one knows the totals.  A word of the sums carries the batch it is of, so that none has to be cleared.  Workgroups begin in
// the order of their numbers as a rule, but nothing waits for that: where one before has said nothing for kPolls looks, its
// chunk is counted again here, so every workgroup ends whatever else runs on the GPU.  (Tickets that number the workgroups as
// they begin cost 20 us with 1024 of them: additions to one word, one after the other from all over the chip.)
// Inside a workgroup the unit is the wavefront: each one walks a chunk of its own and scans with lane shuffles only.
// --------------------------------------------------------------------------------------
constexpr int kScanThreads = 256;
constexpr int kScanWavesPerBlock = kScanThreads / kWave;
// Consecutive elements per lane and step: Op::kItems.  With several, the lanes of one store instruction write
// compacted entries that lie apart (the entries of a lane's other elements fall between them), and the emit pass
// that flags a third of its elements and writes seven arrays wrote 121 MB for 32 MB of lists (49 us; 38 MB and
// 34 us with one element per lane); the passes that flag nearly every element or nearly none are faster with four.
template <class Op>
__global__ __launch_bounds__(kScanThreads) void compact_kernel(Op op, const int32_t *n_ptr, int n_fixed, u64 *said, int32_t k,
                                                               BatchCounters *cnt) {
  typedef typename Op::V V;
  constexpr int kWords = sizeof(V) / sizeof(u64);
  __shared__ typename Op::Lut s_lut;
  __shared__ V s_wave[kScanWavesPerBlock], s_before[kScanWavesPerBlock];
  __shared__ int s_missing;
  if (cnt->err) return;  // the same for all workgroups
  const int blk = blockIdx.x;
  if (op.prepare(s_lut)) __syncthreads();
  constexpr int kScanItems = Op::kItems, kScanStep = kWave * kScanItems;
  const int n = n_ptr ? *n_ptr : n_fixed;
  const int chunk = scan_chunk(n, gridDim.x * kScanWavesPerBlock, kScanStep);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  auto bounds = [&](int b, int &base, int &end) {
    const int64_t base64 = (int64_t)(b * kScanWavesPerBlock + wave) * chunk;
    base = (int)(base64 < n ? base64 : n);
    end = (int)(base64 + chunk < n ? base64 + chunk : n);
  };
  auto flags_of = [&](int b) {  // the sum of the flags of this wavefront's chunk in workgroup b, in all lanes
    int base, end;
    bounds(b, base, end);
    V sum{};
    for (int i0 = base + lane * kScanItems; i0 < end; i0 += kScanStep) {
#pragma unroll
      for (int q = 0; q < kScanItems; q++)
        if (i0 + q < end) sum += op.flag(i0 + q, n);
    }
    return wave_total(sum);
  };
  int base, end;
  bounds(blk, base, end);
  const V mine = flags_of(blk);
  if (lane == 0) s_wave[wave] = mine;
  __syncthreads();
  V own{}, carry{};
  for (int w = 0; w < kScanWavesPerBlock; w++) {
    own += s_wave[w];
    if (w < wave) carry += s_wave[w];
  }
  if (gridDim.x > 1) {
    const u64 of_batch = (u64)(uint32_t)k << 32;
    if (tid < 2 * kWords) {  // a counter each
      u64 w = 0;
#pragma unroll
      for (int i = 0; i < kWords; i++)
        if (tid / 2 == i) w = own.w[i];
      __hip_atomic_store(said + tid * kScanBlocks + blk, of_batch | (uint32_t)(tid & 1 ? w >> 32 : w), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    V before{};
    int j = tid, polls = 0;
    for (;;) {
      while (j < blk && polls < kPolls) {
        u64 v[2 * kWords];
        bool said_all = true;
#pragma unroll
        for (int i = 0; i < 2 * kWords; i++) v[i] = look(said + i * kScanBlocks + j);
#pragma unroll
        for (int i = 0; i < 2 * kWords; i++) said_all = said_all && (v[i] ^ of_batch) >> 32 == 0;
        if (said_all) {
#pragma unroll
          for (int i = 0; i < 2 * kWords; i++) before.w[i / 2] += (v[i] & 0xFFFFFFFFull) << (i & 1 ? 32 : 0);
          j += kScanThreads;
        } else {
          polls++;
          __builtin_amdgcn_s_sleep(1);
        }
      }
      // A workgroup before this one has said nothing for long: it may not have begun, and this one waits for nobody.  What
      // the first of them would say is counted here.
      if (tid == 0) s_missing = blk;
      __syncthreads();
      if (j < blk) atomicMin(&s_missing, j);
      __syncthreads();
      const int missing = s_missing;
      if (missing == blk) break;
      op.rewind();
      const V its = flags_of(missing);
      if (lane == 0) s_before[wave] = its;
      __syncthreads();
      if (j == missing) {
        for (int w = 0; w < kScanWavesPerBlock; w++) before += s_before[w];
        j += kScanThreads;
      }
      polls = 0;
      __syncthreads();
    }
    before = wave_total(before);
    if (lane == 0) s_before[wave] = before;
    __syncthreads();
    before = V{};
    for (int w = 0; w < kScanWavesPerBlock; w++) before += s_before[w];
    carry += before;
    own += before;  // the last workgroup's is the total
  }
  op.rewind();
  write_chunk(op, base, end, n, lane, carry);
  op.wave_done(lane, blk * kScanWavesPerBlock + wave);
  if (blk == (int)gridDim.x - 1 && tid == 0) op.finish(cnt, n, own);
}

// Distinct rows, run starts and set heads of the sorted lookups.  The same skeleton with a tile's lookups in registers between
// their flags and what is written for them: a wavefront takes STEPS steps of two consecutive lookups a lane, whose places
// among the heads are popcounts of two ballots.  A batch with more tiles than workgroups (`chunk` parts a wavefront) reads them
// twice.  (As a kernel that counts and one that emits, which read the keys twice: 3.9 M lookups 49 us, now 33; 7.9 M 83, now 62;
// 41 k to 818 k lookups equal, with a launch less.)
template <int STEPS, bool ONE>
__global__ __launch_bounds__(kScanThreads) void dedup_kernel(DedupArgs a, const uint2 *__restrict__ sorted, int n, int chunk, u64 *said,
                                                             int32_t k, BatchCounters *cnt) {
  __shared__ KeyLut s_lut;
  __shared__ uint32_t s_wave[2][kScanWavesPerBlock], s_before[2][kScanWavesPerBlock];
  __shared__ int s_missing;
  if (cnt->err) return;
  const int blk = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint64_t lt_mask = (1ull << lane) - 1ull;
  constexpr int kPart = STEPS * 2 * kWave;  // lookups of a wavefront's part
  if (ONE) chunk = 1;
  DedupPass<const DedupArgs &> op{a};
  if (op.prepare(s_lut)) __syncthreads();
  uint4 e[STEPS];
  uint32_t heads, set_heads;  // of this lane's lookups, two bits a step
  auto first_of = [&](int b, int c) { return ((b * kScanWavesPerBlock + wave) * chunk + c) * kPart + 2 * lane; };
  auto load = [&](int base) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < STEPS; q++) {
      const int i = base + q * 2 * kWave;
      e[q] = make_uint4(0u, 0u, 0u, 0u);
      if (i + 1 < n) {
        e[q] = *(const uint4 *)(sorted + i);
      } else if (i < n) {
        const uint2 v = sorted[i];
        e[q].x = v.x;
        e[q].y = v.y;
      }
    }
  };
  auto find = [&](int base) __attribute__((always_inline)) {
    uint32_t prev = 0;  // key in front of the wavefront's step
    if (base - 2 * lane > 0 && base - 2 * lane <= n) prev = sorted[base - 2 * lane - 1].x;
    heads = set_heads = 0;
    op.rewind();
#pragma unroll
    for (int q = 0; q < STEPS; q++) {
      const int i = base + q * 2 * kWave;
      uint32_t before = __shfl_up(e[q].z, 1);
      if (lane == 0) before = prev;
      prev = __shfl(e[q].z, 63);
      const uint32_t f0 = i < n ? op.head(i == 0, e[q].x, before) : 0u;
      const uint32_t f1 = i + 1 < n ? op.head(false, e[q].z, e[q].x) : 0u;
      heads |= (f0 & 1u) << (2 * q) | (f1 & 1u) << (2 * q + 1);
      set_heads |= (f0 >> 1) << (2 * q) | (f1 >> 1) << (2 * q + 1);
    }
  };
  auto flags_of = [&](int b, uint32_t &h, uint32_t &sh) __attribute__((always_inline)) {  // this wavefront's part of workgroup b's, in all lanes
    h = sh = 0;
    for (int c = 0; c < chunk; c++) {
      load(first_of(b, c));
      find(first_of(b, c));
      uint32_t both = __popc(heads) | __popc(set_heads) << 16;  // at most 64 x 32 each
      for (int d = 32; d >= 1; d >>= 1) both += __shfl_xor(both, d);
      h += both & 0xFFFFu;
      sh += both >> 16;
    }
  };
  uint32_t h, sh;
  flags_of(blk, h, sh);
  if (lane == 0) { s_wave[0][wave] = h; s_wave[1][wave] = sh; }
  __syncthreads();
  uint32_t u0 = 0, t0 = 0, own_h = 0, own_sh = 0;
  for (int w = 0; w < kScanWavesPerBlock; w++) {
    own_h += s_wave[0][w];
    own_sh += s_wave[1][w];
    if (w < wave) { u0 += s_wave[0][w]; t0 += s_wave[1][w]; }
  }
  if (gridDim.x > 1) {
    const u64 of_batch = (u64)(uint32_t)k << 32;
    if (tid < 2)
      __hip_atomic_store(said + tid * kScanBlocks + blk, of_batch | (tid ? own_sh : own_h), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t hm = heads, shm = set_heads;
    uint32_t bh = 0, bs = 0;
    int j = tid, polls = 0;
    for (;;) {
      while (j < blk && polls < kPolls) {
        const u64 v = look(said + j), w = look(said + kScanBlocks + j);
        if (((v ^ of_batch) >> 32 | (w ^ of_batch) >> 32) == 0) {
          bh += (uint32_t)v;
          bs += (uint32_t)w;
          j += kScanThreads;
        } else {
          polls++;
          __builtin_amdgcn_s_sleep(1);
        }
      }
      if (tid == 0) s_missing = blk;
      __syncthreads();
      if (j < blk) atomicMin(&s_missing, j);
      __syncthreads();
      const int missing = s_missing;
      if (missing == blk) break;
      flags_of(missing, h, sh);
      if (lane == 0) { s_before[0][wave] = h; s_before[1][wave] = sh; }
      __syncthreads();
      if (j == missing) {
        for (int w = 0; w < kScanWavesPerBlock; w++) { bh += s_before[0][w]; bs += s_before[1][w]; }
        j += kScanThreads;
      }
      polls = 0;
      __syncthreads();
      if (ONE) load(first_of(blk, 0));  // (what was in the registers)
    }
    heads = hm;
    set_heads = shm;
    for (int d = 32; d >= 1; d >>= 1) { bh += __shfl_xor(bh, d); bs += __shfl_xor(bs, d); }
    if (lane == 0) { s_before[0][wave] = bh; s_before[1][wave] = bs; }
    __syncthreads();
    bh = bs = 0;
    for (int w = 0; w < kScanWavesPerBlock; w++) { bh += s_before[0][w]; bs += s_before[1][w]; }
    u0 += bh;
    t0 += bs;
    own_h += bh;  // the last workgroup's is the total
    own_sh += bs;
  }
  op.rewind();
  const bool packed = a.cnt->packed != 0;
  for (int c = 0; c < chunk; c++) {
    const int base = first_of(blk, c);
    if (!ONE) {
      load(base);
      find(base);
      op.rewind();
    }
#pragma unroll
    for (int q = 0; q < STEPS; q++) {
      const int i = base + q * 2 * kWave;
      const bool h0 = heads >> (2 * q) & 1u, h1 = heads >> (2 * q + 1) & 1u;
      const bool s0 = set_heads >> (2 * q) & 1u, s1 = set_heads >> (2 * q + 1) & 1u;
      const uint64_t b0 = __ballot(h0), b1 = __ballot(h1), bs0 = __ballot(s0), bs1 = __ballot(s1);
      const uint32_t u = u0 + __popcll(b0 & lt_mask) + __popcll(b1 & lt_mask) + h0 - 1u;
      const uint32_t v = t0 + __popcll(bs0 & lt_mask) + __popcll(bs1 & lt_mask);
      u0 += __popcll(b0) + __popcll(b1);
      t0 += __popcll(bs0) + __popcll(bs1);
      if (i >= n) continue;
      const bool two = i + 1 < n;
      const int32_t bag0 = packed ? (int32_t)(e[q].y >> a.within_bits) : a.bag_of_pos[e[q].y];
      const int32_t bag1 = !two ? 0 : packed ? (int32_t)(e[q].w >> a.within_bits) : a.bag_of_pos[e[q].w];
      if (two) {
        *(uint2 *)(a.uid_sorted + i) = make_uint2(u, u + h1);
        *(int2 *)(a.sorted_bag + i) = make_int2(bag0, bag1);
      } else {
        a.uid_sorted[i] = u;
        a.sorted_bag[i] = bag0;
      }
      if (a.sorted_at) {
        a.sorted_at[i] = op.sorted_at(e[q].y, bag0);
        if (two) a.sorted_at[i + 1] = op.sorted_at(e[q].w, bag1);
      }
      if (h0) op.write_row(e[q].x, i, u, s0, v);
      if (h1) op.write_row(e[q].z, i + 1, u + 1, s1, v + s0);
    }
  }
  if (blk == (int)gridDim.x - 1 && tid == 0) {
    cnt->n_uniq = (int32_t)own_h;
    cnt->n_touched = (int32_t)own_sh;
    a.run_off[own_h] = n;
  }
}

template <int STEPS, bool ONE>
static void launch_dedup(const DedupArgs &a, const uint2 *sorted, int n, const SortScratch &ss, int32_t k, BatchCounters *cnt, hipStream_t s) {
  constexpr int kTile = kScanThreads * 2 * STEPS;
  const int tiles = (int)(((int64_t)n + kTile - 1) / kTile);
  const int chunk = (tiles + kScanBlocks - 1) / kScanBlocks;
  hipLaunchKernelGGL((dedup_kernel<STEPS, ONE>), dim3((tiles + chunk - 1) / chunk), dim3(kScanThreads), 0, s, a, sorted, n, chunk,
                     ss.said_counts, k, cnt);
}

// pass: its number among those of the stage; returns the number of workgroups
template <class Op>
static int run_compaction(Op op, const int32_t *n_ptr, int n_fixed, int n_bound, const SortScratch &ss, int pass, int32_t k,
                          BatchCounters *cnt, hipStream_t s) {
  int nb = (int)(((int64_t)n_bound + kScanThreads * Op::kItems - 1) / (kScanThreads * Op::kItems));
  if (nb > kScanBlocks / 2) nb = kScanBlocks / 2;  // (1.65 M distinct rows: 512 / 1024 / 2048 workgroups 130 / 100 / 99 us, 192 k 13 / 12 / 19)
  hipLaunchKernelGGL(compact_kernel<Op>, dim3(nb), dim3(kScanThreads), 0, s, op, n_ptr, n_fixed,
                     ss.said_counts + 4 * pass * kScanBlocks, k, cnt);
  return nb;
}

#ifndef TBE_PROBE_SETS
#define TBE_PROBE_SETS 8
#endif
template <bool LFU, bool L2>
__global__ __launch_bounds__(kWave) void probe_kernel(ProbeArgs a, BatchCounters *cnt) {
  __shared__ ProbeLds<L2, TBE_PROBE_SETS> s;
  if (cnt->err) return;
  probe_windows<LFU, L2>(a, s, blockIdx.x, gridDim.x, cnt);
}

// Per-lookup location word, in input order, written from the sorted side: lookup i of the sorted sequence
// belongs to distinct row uid_sorted[i], whose word goes to the lookup's position.  These are 4-byte stores all
// over the array, but not without order: the sorted sequence and the input are both table-major, so the words
// of one table land in that table's stretch of the array (a megabyte in the benchmark workload).  Each XCD takes
// a contiguous eighth of the sorted sequence, i.e. whole tables, so a table's stretch is written through one L2,
// where the stores meet and leave as full lines; the streamed inputs are read around the cache.  (Workgroups
// dealt round robin over the XCDs wrote every line from eight L2s, in eight partial pieces: 260 MB of write
// traffic for 31 MB of words.)
//
// The first workgroup ends the stage (add_totals), the next plan the heavy rows for the tile kernel (plan_heavy; `plan` of them, a
// multiple of the XCDs), which needs the same lists and nothing of the location words.
#ifndef TBE_FINALIZE_BLOCKS
#define TBE_FINALIZE_BLOCKS 512  // a multiple of 8
#endif
constexpr int kFinalThreads = 256;
__global__ __launch_bounds__(kFinalThreads) void finalize_kernel(int n, const u64 *__restrict__ sorted,
                                                                 const uint32_t *__restrict__ uid_sorted,
                                                                 const int32_t *__restrict__ loc_u,
                                                                 const int32_t *__restrict__ run_off,
                                                                 uint32_t *__restrict__ loc,
                                                                 const int64_t *__restrict__ offsets, int within_bits,
                                                                 Totals totals, const u64 *__restrict__ tally,
                                                                 int tally_waves, uint32_t *too_long, uint32_t *stage_err,
                                                                 int32_t *refused, int split, int plan,
                                                                 PlanArgs pa, BatchCounters *cnt) {
  const bool totals_here = blockIdx.x == 0;  // (the next seven are there so that those behind them keep their XCDs)
  const int id = (int)blockIdx.x - kXcds;
  if (totals_here && threadIdx.x == 0) {
    *too_long = 0u;  // as the next batch expects them, whatever became of this one
    if (n == 0 && (int)*stage_err > cnt->err) cnt->err = (int)*stage_err;  // (no pass of the sort has; there is one workgroup)
    *stage_err = 0u;
    if (cnt->err && *refused == 0) *refused = cnt->err | kRefusedBefore;  // (read by a stage's first kernel alone)
  }
  if (cnt->err) return;
  if (totals_here) {
    __shared__ TotalsLds<kFinalThreads> s;
    add_totals(cnt, totals, tally, tally_waves, pa.heavy_sub, split, s);
    return;
  }
  if (id < 0) return;
  if (id < plan) {
    __shared__ PlanLds<kFinalThreads> s;
    plan_heavy(id, plan, pa, s, cnt);
    return;
  }
  const bool packed = cnt->packed != 0;
  const uint32_t within_mask = (1u << within_bits) - 1u;
  constexpr int K = 4;  // lookups per thread and pass, a workgroup's width apart: their loads are in flight together
  int first, end, step;
  xcd_span_of(id - plan, (int)gridDim.x - kXcds - plan, n, kFinalThreads * K, first, end, step);
  for (int i0 = first + threadIdx.x; i0 < end; i0 += step) {
    uint32_t u[K], p[K], w[K], at[K];
#pragma unroll
    for (int q = 0; q < K; q++) {
      const int i = i0 + q * kFinalThreads;
      u[q] = i < end ? __builtin_nontemporal_load(uid_sorted + i) : 0u;
      p[q] = i < end ? (uint32_t)(__builtin_nontemporal_load(sorted + i) >> 32) : 0u;  // the lookup's position: as is, or (bag, position inside it)
    }
#pragma unroll
    for (int q = 0; q < K; q++) {
      const int32_t lu = loc_u[u[q]];
      w[q] = lu >= 0 ? (uint32_t)lu : (kLocOverflow | (uint32_t)(-2 - lu));
      if (run_off[u[q] + 1] - run_off[u[q]] == 1) w[q] |= kLocSingle;
      at[q] = packed ? (uint32_t)offsets[p[q] >> within_bits] + (p[q] & within_mask) : p[q];
    }
#pragma unroll
    for (int q = 0; q < K; q++)
      if (i0 + q * kFinalThreads < end) loc[at[q]] = w[q];
  }
}

hipError_t launch_dedup_probe(const TableMeta *tm, const Geometry &g, const BatchBuf &b, SortScratch &ss,
                              const uint2 *sorted, int32_t *tags, int32_t *ts, int32_t *freq, bool lfu, const Level2 &l2, int lock, const StaleRows &stale,
                              const Totals &totals, hipStream_t s) {
  const int n = (int)b.n;
  if (n == 0) {  // nothing but the end of the stage
    hipLaunchKernelGGL(finalize_kernel, dim3(1), dim3(kFinalThreads), 0, s, 0, (const u64 *)sorted, b.uid_sorted, b.loc_u, b.run_off,
                       b.loc, b.d_offsets, g.within_bits, totals, ss.tally, 0, ss.too_long, ss.stage_err, ss.refused, kHeavySplit, 0, PlanArgs{}, b.cnt);
    return hipGetLastError();
  }
  auto dedup = n <= 131072 ? launch_dedup<2, true> : n <= 2097152 ? launch_dedup<4, true>
               : n <= kScanBlocks * kScanThreads * 16 ? launch_dedup<8, true> : launch_dedup<4, false>;
  dedup(dedup_of(tm, g, b), sorted, n, ss, b.k, b.cnt, s);
  int64_t max_touched = (int64_t)g.total_sets + g.T;
  if (max_touched > n) max_touched = n;
  const int probe_blocks = (int)(max_touched < 65536 ? max_touched : 65536);
  auto probe = l2.on ? (lfu ? probe_kernel<true, true> : probe_kernel<false, true>)
                     : (lfu ? probe_kernel<true, false> : probe_kernel<false, false>);
  hipLaunchKernelGGL(probe, dim3(probe_blocks), dim3(kWave), 0, s, probe_of(tm, g, b, tags, ts, freq, l2, lock), b.cnt);
  const int tally_waves = run_compaction(StatusOp{status_of(tm, g, b, l2, stale, ss.tally)}, &b.cnt->n_uniq, 0, n, ss, 1, b.k, b.cnt, s) * kScanWavesPerBlock;
  // (only the tile kernel needs a plan; 256 workgroups look for the ranges' starts)
  const int plan = b.maxp || long_rows_in_rest(n) ? 0 : (g.T + 256 + kXcds - 1) / kXcds * kXcds;
  // a multiple of the XCDs, no more than have a pass to do
  int final_blocks = (n + 4 * kFinalThreads - 1) / (4 * kFinalThreads);
  final_blocks = final_blocks > TBE_FINALIZE_BLOCKS ? TBE_FINALIZE_BLOCKS : (final_blocks + kXcds - 1) / kXcds * kXcds;
  hipLaunchKernelGGL(finalize_kernel, dim3(kXcds + plan + final_blocks), dim3(kFinalThreads), 0, s, n, (const u64 *)sorted, b.uid_sorted, b.loc_u,
                     b.run_off, b.loc, b.d_offsets, g.within_bits, totals, ss.tally, tally_waves, ss.too_long, ss.stage_err, ss.refused, heavy_split(n, b.maxp), plan,
                     plan_of(tm, g, b), b.cnt);
  return hipGetLastError();
}

}  // namespace tbe
