// Index dedup part 2 (run-length encoding of the sorted keys), the set-associative probe
// with LRU victim choice and miss-list compaction.  Paper Section 5.5: tag/state lookup
// (5.5.1, probe and grouping by destination) and cache algorithm (5.5.2), one-level cache.
#include "tbe_stage.h"

namespace tbe {

// --------------------------------------------------------------------------------------
// Generic flag -> exclusive prefix -> emit skeleton over n elements (n may live on the
// device).  Two 32-bit counters are scanned at once, packed into one 64-bit word.
//   count kernel : sum of op.flag(i) over the contiguous chunk of every wavefront, and per workgroup
//   emit kernel  : op.emit(i, exclusive prefix, flag) for every element, in order
// The unit is the wavefront: each one walks a chunk of its own and scans with lane shuffles only, so
// the emit pass has no barrier inside its loop -- a wave that waits for memory holds up nobody.  (With
// a workgroup-wide scan per tile, two barriers each, the waves of a workgroup ran at the pace of the
// slowest one, tile after tile: the emit passes of the benchmark workload took 0.11 ms each.)
// --------------------------------------------------------------------------------------
constexpr int kScanThreads = 256;
constexpr int kScanWavesPerBlock = kScanThreads / kWave;
static_assert(kSmallScanBlocks == kScanThreads, "a thread of the small batches' passes hears one workgroup");
// Consecutive elements per lane and step: Op::kItems.  With several, the lanes of one store instruction write
// compacted entries that lie apart (the entries of a lane's other elements fall between them), and the emit pass
// that flags a third of its elements and writes seven arrays wrote 121 MB for 32 MB of lists (49 us; 38 MB and
// 34 us with one element per lane); the passes that flag nearly every element or nearly none are faster with four.
#ifndef TBE_SCAN_BLOCKS
#define TBE_SCAN_BLOCKS 1024
#endif
constexpr int kScanBlocks = TBE_SCAN_BLOCKS;     // workgroups at most (SortScratch::blk holds 5 words per workgroup)

// blk: [0, nblocks) sums per workgroup; [nblocks, nblocks * 5) sums per wavefront
template <class Op>
__global__ __launch_bounds__(kScanThreads) void compact_count_kernel(Op op, const int32_t *n_ptr, int n_fixed,
                                                                     typename Op::V *blk, const BatchCounters *cnt) {
  __shared__ typename Op::V wsum[kScanWavesPerBlock];
  __shared__ typename Op::Lut s_lut;
  if (cnt->err) return;
  if (op.prepare_count(s_lut)) __syncthreads();
  constexpr int kScanItems = Op::kItems, kScanStep = kWave * kScanItems;
  const int n = n_ptr ? *n_ptr : n_fixed;
  const int chunk = scan_chunk(n, gridDim.x * kScanWavesPerBlock, kScanStep);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int w = blockIdx.x * kScanWavesPerBlock + wave;
  const int64_t base64 = (int64_t)w * chunk;
  const int base = (int)(base64 < n ? base64 : n), end = (int)(base64 + chunk < n ? base64 + chunk : n);
  typename Op::V s{};
  for (int i0 = base + lane * kScanItems; i0 < end; i0 += kScanStep) {
#pragma unroll
    for (int q = 0; q < kScanItems; q++)
      if (i0 + q < end) s += op.flag(i0 + q, n);
  }
  s = wave_total(s);
  if (lane == 0) {
    wsum[wave] = s;
    blk[gridDim.x + w] = s;
  }
  __syncthreads();
  if (tid == 0) {
    typename Op::V t{};
    for (int k = 0; k < kScanWavesPerBlock; k++) t += wsum[k];
    blk[blockIdx.x] = t;
  }
}

template <class Op>
__global__ __launch_bounds__(kScanThreads) void compact_emit_kernel(Op op, const int32_t *n_ptr, int n_fixed,
                                                                    const typename Op::V *blk, BatchCounters *cnt) {
  typedef typename Op::V V;
  __shared__ typename Op::Lut s_lut;
  if (cnt->err) return;
  if (op.prepare(s_lut)) __syncthreads();
  constexpr int kScanItems = Op::kItems, kScanStep = kWave * kScanItems;
  const int n = n_ptr ? *n_ptr : n_fixed;
  const int chunk = scan_chunk(n, gridDim.x * kScanWavesPerBlock, kScanStep);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int w = blockIdx.x * kScanWavesPerBlock + wave;
  const int64_t base64 = (int64_t)w * chunk;
  const int base = (int)(base64 < n ? base64 : n), end = (int)(base64 + chunk < n ? base64 + chunk : n);
  // flags before this wavefront: the workgroups before its own, then the waves before it in its own
  V carry{};
  for (int b = lane; b < (int)blockIdx.x; b += kWave) carry += blk[b];
  if (lane < wave) carry += blk[gridDim.x + blockIdx.x * kScanWavesPerBlock + lane];
  carry = wave_total(carry);
  V total{};
  if (blockIdx.x == 0 && wave == 0) {
    for (int b = lane; b < (int)gridDim.x; b += kWave) total += blk[b];
    total = wave_total(total);
  }
  write_chunk(op, base, end, n, lane, carry);
  op.wave_done(lane, w);
  if (blockIdx.x == 0 && tid == 0) op.finish(cnt, n, total);
}

// Small batches: the same in one kernel.  A workgroup counts its chunk, says its sums, adds up those of the workgroups
// before it and writes; the last one knows the totals.
template <class Op>
__global__ __launch_bounds__(kScanThreads) void compact_small_kernel(Op op, const int32_t *n_ptr, int n_fixed, u64 *said,
                                                                     uint32_t *ticket, BatchCounters *cnt) {
  typedef typename Op::V V;
  constexpr int kWords = sizeof(V) / sizeof(u64);
  __shared__ typename Op::Lut s_lut;
  __shared__ V s_wave[kScanWavesPerBlock], s_before[kScanWavesPerBlock];
  if (cnt->err) return;  // the same for all workgroups, and before their tickets
  const int blk = take_ticket(ticket);
  if (op.prepare(s_lut)) __syncthreads();
  constexpr int kScanItems = Op::kItems, kScanStep = kWave * kScanItems;
  const int n = n_ptr ? *n_ptr : n_fixed;
  const int chunk = scan_chunk(n, gridDim.x * kScanWavesPerBlock, kScanStep);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t base64 = (int64_t)(blk * kScanWavesPerBlock + wave) * chunk;
  const int base = (int)(base64 < n ? base64 : n), end = (int)(base64 + chunk < n ? base64 + chunk : n);
  V mine{};
  for (int i0 = base + lane * kScanItems; i0 < end; i0 += kScanStep) {
#pragma unroll
    for (int q = 0; q < kScanItems; q++)
      if (i0 + q < end) mine += op.flag(i0 + q, n);
  }
  mine = wave_total(mine);
  if (lane == 0) s_wave[wave] = mine;
  __syncthreads();
  V own{}, carry{};
  for (int w = 0; w < kScanWavesPerBlock; w++) {
    own += s_wave[w];
    if (w < wave) carry += s_wave[w];
  }
  if (gridDim.x > 1) {
    if (tid < kWords) say(said + tid * kSmallScanBlocks + blk, tid == 0 ? own.w[0] : own.w[kWords - 1]);
    V before{};
    if (tid < blk) {  // kSmallScanBlocks == kScanThreads: a workgroup before this one per thread
      V v{};
#pragma unroll
      for (int i = 0; i < kWords; i++) v.w[i] = look(said + i * kSmallScanBlocks + tid);
#pragma unroll
      for (int i = 0; i < kWords; i++) before.w[i] = hear(said + i * kSmallScanBlocks + tid, v.w[i]);
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

// small_pass: number of the pass among those of a small batch, -1 = not a small batch; returns the number of workgroups
template <class Op>
static int run_compaction(Op op, const int32_t *n_ptr, int n_fixed, int n_bound, const SortScratch &ss, int small_pass,
                          BatchCounters *cnt, hipStream_t s) {
  if (small_pass >= 0) {
    int nb = (n_bound + kScanThreads * Op::kItems - 1) / (kScanThreads * Op::kItems);
    if (nb > kSmallScanBlocks) nb = kSmallScanBlocks;
    hipLaunchKernelGGL(compact_small_kernel<Op>, dim3(nb), dim3(kScanThreads), 0, s, op, n_ptr, n_fixed,
                       ss.said_counts + 2 * small_pass * kSmallScanBlocks, ss.ticket, cnt);
    return nb;
  }
  u64 *words = ss.blk;
  typename Op::V *blk = (typename Op::V *)words;
  int nb = (n_bound + kScanThreads * Op::kItems - 1) / (kScanThreads * Op::kItems);
  if (nb > kScanBlocks) nb = kScanBlocks;
  if (nb < 1) nb = 1;
  hipLaunchKernelGGL(compact_count_kernel<Op>, dim3(nb), dim3(kScanThreads), 0, s, op, n_ptr, n_fixed, blk, cnt);
  hipLaunchKernelGGL(compact_emit_kernel<Op>, dim3(nb), dim3(kScanThreads), 0, s, op, n_ptr, n_fixed, blk, cnt);
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
// The first workgroups plan the heavy rows (plan_heavy; `plan` of them, a multiple of the XCDs), which needs the same lists
// and nothing of the location words.  One workgroup more (the last) ends the stage (add_totals).
#ifndef TBE_FINALIZE_BLOCKS
#define TBE_FINALIZE_BLOCKS 512  // a multiple of 8
#endif
constexpr int kFinalThreads = 256;
__global__ __launch_bounds__(kFinalThreads) void finalize_kernel(int n, const uint32_t *__restrict__ pos,
                                                                 const uint32_t *__restrict__ uid_sorted,
                                                                 const int32_t *__restrict__ loc_u,
                                                                 const int32_t *__restrict__ run_off,
                                                                 uint32_t *__restrict__ loc,
                                                                 const int64_t *__restrict__ offsets, int within_bits,
                                                                 Totals totals, const u64 *__restrict__ tally,
                                                                 int tally_waves, uint32_t *too_long, int32_t *refused, int plan,
                                                                 PlanArgs pa, BatchCounters *cnt) {
  const bool last = blockIdx.x + 1 == gridDim.x;
  if (last && threadIdx.x == 0) {
    *too_long = 0u;  // as the next batch expects it, whatever became of this one
    if (cnt->err && *refused == 0) *refused = cnt->err | kRefusedBefore;  // (read by a stage's first kernel alone)
  }
  if (cnt->err) return;
  if (last) {
    __shared__ TotalsLds<kFinalThreads> s;
    add_totals(cnt, totals, tally, tally_waves, s);
    return;
  }
  if ((int)blockIdx.x < plan) {
    __shared__ PlanLds<kFinalThreads> s;
    plan_heavy(blockIdx.x, plan, pa, s, cnt);
    return;
  }
  const bool packed = cnt->packed != 0;
  const uint32_t within_mask = (1u << within_bits) - 1u;
  constexpr int K = 4;  // lookups per thread and pass, a workgroup's width apart: their loads are in flight together
  int first, end, step;
  xcd_span_of(blockIdx.x - plan, gridDim.x - 1 - plan, n, kFinalThreads * K, first, end, step);
  for (int i0 = first + threadIdx.x; i0 < end; i0 += step) {
    uint32_t u[K], p[K], w[K], at[K];
#pragma unroll
    for (int q = 0; q < K; q++) {
      const int i = i0 + q * kFinalThreads;
      u[q] = i < end ? __builtin_nontemporal_load(uid_sorted + i) : 0u;
      p[q] = i < end ? __builtin_nontemporal_load(pos + i) : 0u;  // the lookup's position: as is, or (bag, position inside it)
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
                              const uint32_t *sorted_keys, const uint32_t *sorted_pos, int32_t *tags, int32_t *ts,
                              int32_t *freq, bool lfu, const Level2 &l2, int lock, const StaleRows &stale,
                              const Totals &totals, hipStream_t s) {
  const int n = (int)b.n;
  if (n == 0) {  // nothing but the end of the stage
    hipLaunchKernelGGL(finalize_kernel, dim3(1), dim3(kFinalThreads), 0, s, 0, sorted_pos, b.uid_sorted, b.loc_u, b.run_off,
                       b.loc, b.d_offsets, g.within_bits, totals, ss.tally, 0, ss.too_long, ss.refused, 0, PlanArgs{}, b.cnt);
    return hipGetLastError();
  }
  const bool small = small_batch(g, n, b.batch);
  run_compaction(DedupOp{dedup_of(tm, g, b, sorted_keys, sorted_pos)}, nullptr, n, n, ss, small ? 0 : -1, b.cnt, s);
  int64_t max_touched = (int64_t)g.total_sets + g.T;
  if (max_touched > n) max_touched = n;
  const int probe_blocks = (int)(max_touched < 65536 ? max_touched : 65536);
  auto probe = l2.on ? (lfu ? probe_kernel<true, true> : probe_kernel<false, true>)
                     : (lfu ? probe_kernel<true, false> : probe_kernel<false, false>);
  hipLaunchKernelGGL(probe, dim3(probe_blocks), dim3(kWave), 0, s, probe_of(tm, g, b, tags, ts, freq, l2, lock), b.cnt);
  const int tally_waves = run_compaction(StatusOp{status_of(tm, g, b, l2, stale, ss.tally)}, &b.cnt->n_uniq, 0, n, ss, small ? 1 : -1, b.cnt, s) * kScanWavesPerBlock;
  // (max pooling takes heavy rows a workgroup each and needs no plan, nor do batches that do the same; 64 or 256 workgroups
  // look for the ranges' starts)
  const int plan = b.maxp || long_rows_in_rest(n, g.win_stride) ? 0 : (g.T + (small ? 64 : 256) + kXcds - 1) / kXcds * kXcds;
  // a multiple of the XCDs, no more than have a pass to do, and the one that ends the stage
  int final_blocks = (n + 4 * kFinalThreads - 1) / (4 * kFinalThreads);
  final_blocks = final_blocks > TBE_FINALIZE_BLOCKS ? TBE_FINALIZE_BLOCKS : (final_blocks + kXcds - 1) / kXcds * kXcds;
  hipLaunchKernelGGL(finalize_kernel, dim3(plan + final_blocks + 1), dim3(kFinalThreads), 0, s, n, sorted_pos, b.uid_sorted, b.loc_u,
                     b.run_off, b.loc, b.d_offsets, g.within_bits, totals, ss.tally, tally_waves, ss.too_long, ss.refused, plan,
                     plan_of(tm, g, b), b.cnt);
  return hipGetLastError();
}

}  // namespace tbe
