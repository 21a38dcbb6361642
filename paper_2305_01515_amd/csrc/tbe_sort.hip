// Index dedup, part 1: sort keys for every lookup of a batch and a stable LSD radix sort
// of (key, position) pairs.  The paper does not describe this step; it serves the
// "group the indices" part of the tag/state lookup (Section 5.5.1) on a 64-wide machine.
#include "tbe_internal.h"

namespace tbe {

// --------------------------------------------------------------------------------------
// key generation: 8 lanes per bag, 64-byte coalesced reads of the bag's indices
// --------------------------------------------------------------------------------------
constexpr int kKeygenLanes = 8;

// First kernel of the stage: the batch's counters start at zero (workgroup 0), and every bag is looked at: does it fit the
// packed payload?  The answer is gathered in *too_long, which the stage's last kernel leaves at zero for the next batch, so
// that no launch has to come before this one.  It also clears the words in which the workgroups of a small batch's passes
// tell each other their counts.  Behind a batch that was refused every batch starts as refused, with that one's error (the
// host learns of it only when it synchronises, and until then issues more): every later kernel of the batch then returns at
// once, so tags, lines and copies stay as the last good batch left them, and a batch buffer that is used again still says so.
// (The key generation alone does not ask: a first load for every wavefront of it.  What it finds is below that error.)
__global__ __launch_bounds__(256) void begin_kernel(int64_t nb, const int64_t *__restrict__ offsets, int within_bits,
                                                    uint32_t *too_long, uint4 *said, int n_said, uint4 *said_counts,
                                                    int n_said_counts, const int32_t *refused, BatchCounters *cnt) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (int64_t i = gid; i < n_said + n_said_counts; i += (int64_t)gridDim.x * blockDim.x)
    (i < n_said ? said + i : said_counts + (i - n_said))[0] = make_uint4(0u, 0u, 0u, 0u);
  const int64_t bag = gid;
  if (bag == 0) begin_counters(cnt, *refused);
  const bool is = within_bits > 0 && bag < nb && offsets[bag + 1] - offsets[bag] > (1ll << within_bits);
  if (__ballot(is) && (threadIdx.x & 63) == 0) atomicOr(too_long, 1u);
}

// HIST (small batches): also counts the digits of every pass of the sort, in LDS, and adds them to the batch's totals, an
// addition to memory for every digit value that a workgroup has met; so a workgroup takes several lots of 32 bags.  (10 tables
// of 200 k rows, 3001 bags each, with 938 workgroups 21 us; four steps 612 us, with 256 / 128 / 64 workgroups 576 / 586 / 618.
// 4 tables, 4096 bags each, five steps: 981 us, 965 / 971 / 1007.)
constexpr int kSmallKeygenBlocks = 256;
template <bool HIST>
__global__ __launch_bounds__(256) void keygen_kernel(const TableMeta *__restrict__ tm, int T, int B, int64_t N, int64_t first_bag,
                                                     const int64_t *__restrict__ indices,
                                                     const int64_t *__restrict__ offsets, uint32_t *__restrict__ keys,
                                                     uint32_t *__restrict__ vals, int32_t *__restrict__ bag_of_pos,
                                                     float *__restrict__ inv_len, int within_bits,
                                                     const uint32_t *__restrict__ too_long, DigitPlan digits,
                                                     uint32_t *digit_totals, BatchCounters *cnt) {
  __shared__ uint32_t s_hist[HIST ? kMaxSortPasses * 256 : 1];
  if constexpr (HIST) {
    for (int i = threadIdx.x; i < kMaxSortPasses * 256; i += 256) s_hist[i] = 0;
    __syncthreads();
  }
  const int64_t nb = (int64_t)T * B;
  const bool packed = within_bits > 0 && *too_long == 0u;
  if (blockIdx.x == 0 && threadIdx.x == 0) cnt->packed = packed ? 1 : 0;
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int sub = (int)(gid % kKeygenLanes);
  auto keys_of_bag = [&](int64_t bag) {
    const int64_t lo = offsets[bag], hi = offsets[bag + 1];
    bool bad = lo < 0 || hi > N || lo > hi;
    if (bag == 0 && lo != 0) bad = true;
    if (bag == nb - 1 && hi != N) bad = true;
    if (bad) {
      if (sub == 0) atomicMax(&cnt->err, 1 /* -TBE_EINVAL */);
      return;
    }
    // mean pooling (Section 2.1.1): a lookup of a bag of L lookups weighs 1/L
    if (inv_len && sub == 0) inv_len[bag] = hi > lo ? 1.0f / (float)(hi - lo) : 0.0f;
    const int t = (int)(bag / B);
    const TableMeta m = tm[t];
    // two indices per lane and step, both requested before either is used (the loop is bound by the latency
    // of these reads: a bag has a few dozen lookups, so a lane makes only a few steps)
    auto emit = [&](int64_t j, int64_t r) {
      if (r < 0 || r >= m.rows) {
        atomicMax(&cnt->err, 2 /* -TBE_ERANGE */);
        r = 0;
      }
      const uint32_t key = key_of_row(m, (uint32_t)r);
      keys[j] = key;
      if (packed) {
        vals[j] = ((uint32_t)bag << within_bits) | (uint32_t)(j - lo);
      } else {
        vals[j] = (uint32_t)j;
        bag_of_pos[j] = (int32_t)bag;
      }
      if constexpr (HIST)
        for (int p = 0; p < digits.passes; p++) atomicAdd(&s_hist[p * 256 + ((key >> digits.shift[p]) & digits.mask[p])], 1u);
    };
    for (int64_t j = lo + sub; j < hi; j += 2 * kKeygenLanes) {
      const bool second = j + kKeygenLanes < hi;
      const int64_t r0 = indices[j];
      const int64_t r1 = second ? indices[j + kKeygenLanes] : 0;
      emit(j, r0);
      if (second) emit(j + kKeygenLanes, r1);
    }
  };
  const int64_t bag0 = first_bag + gid / kKeygenLanes;
  if constexpr (!HIST) {
    if (bag0 < nb) keys_of_bag(bag0);
  } else {
    for (int64_t bag = bag0; bag < nb; bag += (int64_t)gridDim.x * (256 / kKeygenLanes)) keys_of_bag(bag);
    __syncthreads();
    for (int i = threadIdx.x; i < digits.passes * 256; i += 256)
      if (s_hist[i]) atomicAdd(&digit_totals[i], s_hist[i]);
  }
}

// Passes of the sort by digits of at most 8 bits.
static int byte_passes(int key_bits) { return (key_bits + 7) / 8; }

hipError_t launch_keygen(const TableMeta *tm, const Geometry &g, const BatchBuf &b, const SortScratch &ss, hipStream_t s) {
  const int64_t nb = (int64_t)g.T * b.batch;
  const bool small = small_batch(g, b.n, b.batch);
  const DigitPlan digits = digit_plan(g.key_bits, byte_passes(g.key_bits));
  int n_said = 0, n_counts = 0;  // 16-byte pieces of the words to clear
  if (small) {
    const int blocks = small_sort_blocks(b.n);
    n_said = 64 * (kMaxSortPasses + (blocks > 1 ? digits.passes * blocks : 0));
    n_counts = 4 * kSmallScanBlocks / 2;
  }
  const int64_t threads0 = nb > n_said / 4 ? nb : n_said / 4;
  hipLaunchKernelGGL(begin_kernel, dim3((unsigned)(threads0 > 256 ? (threads0 + 255) / 256 : 1)), dim3(256), 0, s, nb,
                     b.d_offsets, g.within_bits, ss.too_long, (uint4 *)ss.said, n_said, (uint4 *)ss.said_counts, n_counts,
                     ss.refused, b.cnt);
  constexpr int64_t kBags = 1ll << 27;  // a launch holds fewer than 2^32 threads
  for (int64_t first = 0; first < nb; first += kBags) {
    const int64_t threads = (nb - first < kBags ? nb - first : kBags) * kKeygenLanes;
    const int64_t blocks = (threads + 255) / 256;
    hipLaunchKernelGGL((small ? keygen_kernel<true> : keygen_kernel<false>), dim3((unsigned)(small && blocks > kSmallKeygenBlocks ? kSmallKeygenBlocks : blocks)), dim3(256), 0, s,
                       tm, g.T, b.batch, b.n, first, b.d_indices, b.d_offsets, ss.keys[0], ss.vals[0], b.bag_of_pos,
                       b.mean ? b.inv_len : nullptr, g.within_bits, ss.too_long, digits, ss.said, b.cnt);
  }
  return hipGetLastError();
}

// --------------------------------------------------------------------------------------
// LSD radix sort, digits of up to 8 bits (9 where that saves a pass), three kernels per pass:
//   upsweep   : per-block digit histogram of the block's contiguous chunk
//   scan      : per digit, exclusive scan of its counts over the blocks, and digit totals
//   downsweep : the block walks its chunk tile by tile; inside a tile every wave ranks
//               its keys with ballot matching (stable), the tile is ordered by digit in
//               LDS and written out so that neighbouring lanes hit neighbouring addresses
// --------------------------------------------------------------------------------------
constexpr int kSortTile = 4096;        // keys of a tile
constexpr int kMaxRadix = 512;         // a pass sorts by a digit of up to 9 bits; one thread per digit value
constexpr int kMaxSortBlocks = 1024;
constexpr int kUpsweepKeys = 4;  // keys a thread of the counting pass has in flight (8 and 16: no faster)

template <int RB>
__global__ __launch_bounds__(1 << RB) void sort_upsweep_kernel(const uint32_t *__restrict__ keys, int n, int shift,
                                                               uint32_t mask, int chunk, uint32_t *__restrict__ hist) {
  constexpr int kRadix = 1 << RB, kSortThreads = kRadix;
  __shared__ uint32_t h[kRadix];
  const int tid = threadIdx.x;
  h[tid] = 0;
  __syncthreads();
  const int base = blockIdx.x * chunk;
  const int end = min(n, base + chunk);
  // Several keys per thread and step, their loads in flight together.  After the first pass equal keys lie side
  // by side, and a power-law batch has keys with thousands of copies: a wavefront whose 64 keys share one digit
  // adds them with one atomic instead of 64 to the same LDS word.
  for (int i0 = base; i0 < end; i0 += kUpsweepKeys * kSortThreads) {
    uint32_t k[kUpsweepKeys];
#pragma unroll
    for (int q = 0; q < kUpsweepKeys; q++) {
      const int i = i0 + q * kSortThreads + tid;
      k[q] = i < end ? keys[i] : 0u;
    }
#pragma unroll
    for (int q = 0; q < kUpsweepKeys; q++) {
      const bool valid = i0 + q * kSortThreads + tid < end;
      const uint32_t d = valid ? (k[q] >> shift) & mask : 0xFFFFFFFFu;
      const uint32_t d0 = __shfl(d, 0, 64);
      if (__all(d == d0)) {
        if ((tid & 63) == 0 && valid) atomicAdd(&h[d0], 64u);
      } else if (valid) {
        atomicAdd(&h[d], 1u);
      }
    }
  }
  __syncthreads();
  hist[tid * gridDim.x + blockIdx.x] = h[tid];
}

// One block per digit: exclusive scan, over the sort blocks, of that digit's counts (in
// place) and the digit's total.  nb <= kMaxSortBlocks.
__global__ __launch_bounds__(256) void sort_scan_kernel(uint32_t *hist, int nb, uint32_t *digit_total) {
  // 256 threads with four counts each (not one thread per count): a workgroup of 1024 threads waits for
  // half a CU's wave slots at once, which took this small kernel 60 to 80 us instead of 5 whenever the
  // other streams' kernels kept the CUs busy
  constexpr int kPer = kMaxSortBlocks / 256;
  __shared__ uint32_t wsum[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint32_t *row = hist + (size_t)blockIdx.x * nb;
  uint32_t v[kPer], mine = 0;
#pragma unroll
  for (int q = 0; q < kPer; q++) {
    const int i = tid * kPer + q;
    v[q] = i < nb ? row[i] : 0u;
    mine += v[q];
  }
  uint32_t incl = mine;
  for (int d = 1; d < 64; d <<= 1) {
    uint32_t o = __shfl_up(incl, d);
    if (lane >= d) incl += o;
  }
  if (lane == 63) wsum[wave] = incl;
  __syncthreads();
  uint32_t wb = 0;
  for (int w = 0; w < wave; w++) wb += wsum[w];
  uint32_t pre = wb + incl - mine;
#pragma unroll
  for (int q = 0; q < kPer; q++) {
    const int i = tid * kPer + q;
    if (i < nb) row[i] = pre;
    pre += v[q];
  }
  if (tid == 255) digit_total[blockIdx.x] = wb + incl;
}

template <int RB>
__global__ __launch_bounds__(1 << RB) void sort_downsweep_kernel(
    const uint32_t *__restrict__ keys_in, const uint32_t *__restrict__ vals_in, uint32_t *__restrict__ keys_out,
    uint32_t *__restrict__ vals_out, int n, int shift, uint32_t mask, int chunk, const uint32_t *__restrict__ hist,
    const uint32_t *__restrict__ digit_total) {
  constexpr int kRadix = 1 << RB, kSortThreads = kRadix, kWaves = kSortThreads / kWave;
  // keys per thread and tile; the 9-bit pass with 4, 6, 12, 16 keys per thread: 77, 69, 68, 71 us against 62
  constexpr int kSortItems = RB == 9 ? 8 : 16;
  constexpr int kTile = kSortThreads * kSortItems;  // 4096 either way; a block's chunk is a multiple of it
  __shared__ uint32_t s_keys[kTile];
  __shared__ uint32_t s_vals[kTile];
  __shared__ uint32_t s_cnt[kWaves][kRadix];  // per wave and digit: count, later exclusive prefix over waves
  __shared__ uint32_t s_dstart[kRadix];       // first tile-sorted position of each digit
  __shared__ uint32_t s_gbase[kRadix];        // next global output position of each digit for this block
  __shared__ uint32_t s_wtot[kWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint64_t lt_mask = (1ull << lane) - 1ull;
  const int block_base = blockIdx.x * chunk;
  const int block_end = min(n, block_base + chunk);
  {  // first output position of digit tid for this block: digits before it + blocks before this one
    const uint32_t tot = digit_total[tid];
    uint32_t incl = tot;
    for (int dd = 1; dd < 64; dd <<= 1) {
      uint32_t o = __shfl_up(incl, dd);
      if (lane >= dd) incl += o;
    }
    if (lane == 63) s_wtot[wave] = incl;
    __syncthreads();
    uint32_t wb = 0;
    for (int w = 0; w < wave; w++) wb += s_wtot[w];
    s_gbase[tid] = wb + incl - tot + hist[tid * gridDim.x + blockIdx.x];
    __syncthreads();
  }

  for (int tile = block_base; tile < block_end; tile += kTile) {
    for (int w = 0; w < kWaves; w++) s_cnt[w][tid] = 0;
    __syncthreads();
    uint32_t key[kSortItems], val[kSortItems], rank[kSortItems];
    const int seg = tile + wave * (kWave * kSortItems);
#pragma unroll
    for (int q = 0; q < kSortItems; q++) {
      const int i = seg + q * kWave + lane;
      const bool valid = i < block_end;
      key[q] = valid ? keys_in[i] : 0xFFFFFFFFu;
      val[q] = valid ? vals_in[i] : 0u;
    }
#pragma unroll
    for (int q = 0; q < kSortItems; q++) {
      const int i = seg + q * kWave + lane;
      const bool valid = i < block_end;
      const uint32_t d = (key[q] >> shift) & mask;
      uint64_t peers = __ballot(valid);
#pragma unroll
      for (int bit = 0; bit < RB; bit++) {
        const bool on = (d >> bit) & 1u;
        const uint64_t bal = __ballot(on);
        peers &= on ? bal : ~bal;
      }
      const uint32_t below = __popcll(peers & lt_mask);
      uint32_t prev = 0;
      if (valid && below == 0) prev = atomicAdd(&s_cnt[wave][d], (uint32_t)__popcll(peers));
      const int leader = valid ? (__ffsll((unsigned long long)peers) - 1) : lane;
      prev = __shfl(prev, leader);
      rank[q] = prev + below;
    }
    __syncthreads();
    // thread tid owns digit tid: totals, prefix over waves, start of the digit in the tile
    uint32_t total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; w++) {
      const uint32_t c = s_cnt[w][tid];
      s_cnt[w][tid] = total;
      total += c;
    }
    uint32_t incl = total;
    for (int dd = 1; dd < 64; dd <<= 1) {
      uint32_t o = __shfl_up(incl, dd);
      if (lane >= dd) incl += o;
    }
    if (lane == 63) s_wtot[wave] = incl;
    __syncthreads();
    uint32_t wb = 0;
    for (int w = 0; w < wave; w++) wb += s_wtot[w];
    const uint32_t dstart = wb + incl - total;
    s_dstart[tid] = dstart;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kSortItems; q++) {
      const int i = seg + q * kWave + lane;
      if (i < block_end) {
        const uint32_t d = (key[q] >> shift) & mask;
        const uint32_t p = s_dstart[d] + s_cnt[wave][d] + rank[q];
        s_keys[p] = key[q];
        s_vals[p] = val[q];
      }
    }
    __syncthreads();
    const int tile_n = min(kTile, block_end - tile);
    for (int p = tid; p < tile_n; p += kSortThreads) {
      const uint32_t k = s_keys[p];
      const uint32_t d = (k >> shift) & mask;
      const uint32_t gpos = s_gbase[d] + ((uint32_t)p - s_dstart[d]);
      keys_out[gpos] = k;
      vals_out[gpos] = s_vals[p];
    }
    __syncthreads();
    s_gbase[tid] += total;
    __syncthreads();
  }
}

// Small batches: a pass is one kernel.  The digits' totals are known from the key generation; a workgroup ranks its tile as
// above, says its digit counts, adds up those of the workgroups before it (the two halves of its threads every other one,
// eight requested at a time) and writes the tile out.  A batch that fits one workgroup is sorted through all passes in its
// LDS by one launch.
template <int ITEMS>
__global__ __launch_bounds__(kSmallSortThreads) void sort_small_kernel(
    const uint32_t *__restrict__ keys_in, const uint32_t *__restrict__ vals_in, uint32_t *__restrict__ keys_out,
    uint32_t *__restrict__ vals_out, int n, DigitPlan digits, int pass0, int pass1,
    const uint32_t *__restrict__ digit_totals, uint32_t *counts, uint32_t *ticket, const BatchCounters *cnt) {
  constexpr int kRadix = 256, kWaves = kSmallSortThreads / kWave, kTile = kSmallSortThreads * ITEMS;
  __shared__ uint32_t s_keys[kTile];
  __shared__ uint32_t s_vals[kTile];
  __shared__ uint32_t s_cnt[kWaves][kRadix];  // per wave and digit: count, later exclusive prefix over waves
  __shared__ uint32_t s_dstart[kRadix];       // first tile-sorted position of each digit
  __shared__ uint32_t s_gbase[2][kRadix];     // first output position of each digit for this workgroup
  __shared__ uint32_t s_wtot[2][4];
  if (cnt->err) return;  // the keys need not be whole; the same for all workgroups, and before their tickets
  const int blk = take_ticket(ticket);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint64_t lt_mask = (1ull << lane) - 1ull;
  const int tile = blk * kTile;
  const int tile_n = min(n - tile, kTile);
  const int seg = wave * (kWave * ITEMS);
  uint32_t key[ITEMS], val[ITEMS], rank[ITEMS];
#pragma unroll
  for (int q = 0; q < ITEMS; q++) {
    const int i = seg + q * kWave + lane;
    key[q] = i < tile_n ? keys_in[tile + i] : 0xFFFFFFFFu;
    val[q] = i < tile_n ? vals_in[tile + i] : 0u;
  }
  for (int pass = pass0; pass < pass1; pass++) {
    const int shift = digits.shift[pass];
    const uint32_t mask = digits.mask[pass];
    for (int i = tid; i < kWaves * kRadix; i += kSmallSortThreads) (&s_cnt[0][0])[i] = 0;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < ITEMS; q++) {
      const bool valid = seg + q * kWave + lane < tile_n;
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
      if (valid && below == 0) prev = atomicAdd(&s_cnt[wave][d], (uint32_t)__popcll(peers));
      const int leader = valid ? (__ffsll((unsigned long long)peers) - 1) : lane;
      prev = __shfl(prev, leader);
      rank[q] = prev + below;
    }
    __syncthreads();
    // thread tid < 256 owns digit tid: totals, prefix over waves, start of the digit in the tile and in the output
    uint32_t total = 0, incl = 0, all = 0, all_incl = 0;
    if (tid < kRadix) {
#pragma unroll
      for (int w = 0; w < kWaves; w++) {
        const uint32_t c = s_cnt[w][tid];
        s_cnt[w][tid] = total;
        total += c;
      }
      if (gridDim.x > 1) say(&counts[((size_t)pass * gridDim.x + blk) * kRadix + tid], total);
      all = gridDim.x > 1 ? digit_totals[pass * kRadix + tid] : total;
      incl = total;
      all_incl = all;
      for (int dd = 1; dd < 64; dd <<= 1) {
        const uint32_t o = __shfl_up(incl, dd), oa = __shfl_up(all_incl, dd);
        if (lane >= dd) { incl += o; all_incl += oa; }
      }
      if (lane == 63) { s_wtot[0][wave] = incl; s_wtot[1][wave] = all_incl; }
    }
    {  // the digit's keys in the workgroups before this one
      const int d = tid & (kRadix - 1), half = tid >> 8;
      const uint32_t *p = counts + (size_t)pass * gridDim.x * kRadix + d;
      constexpr int K = 8;
      uint32_t before = 0;
      for (int j = half; j < blk; j += 2 * K) {
        uint32_t v[K];
#pragma unroll
        for (int q = 0; q < K; q++) v[q] = j + 2 * q < blk ? look(p + (size_t)(j + 2 * q) * kRadix) : 0u;
#pragma unroll
        for (int q = 0; q < K; q++)
          if (j + 2 * q < blk) before += hear(p + (size_t)(j + 2 * q) * kRadix, v[q]);
      }
      s_gbase[half][d] = before;
    }
    __syncthreads();
    if (tid < kRadix) {
      uint32_t wb = 0, wa = 0;
      for (int w = 0; w < wave; w++) { wb += s_wtot[0][w]; wa += s_wtot[1][w]; }
      s_dstart[tid] = wb + incl - total;
      s_gbase[0][tid] += s_gbase[1][tid] + wa + all_incl - all;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < ITEMS; q++) {
      if (seg + q * kWave + lane < tile_n) {
        const uint32_t d = (key[q] >> shift) & mask;
        const uint32_t p = s_dstart[d] + s_cnt[wave][d] + rank[q];
        s_keys[p] = key[q];
        s_vals[p] = val[q];
      }
    }
    __syncthreads();
    if (pass + 1 < pass1) {  // one workgroup: the next pass takes the tile from LDS
#pragma unroll
      for (int q = 0; q < ITEMS; q++) {
        const int i = seg + q * kWave + lane;
        key[q] = i < tile_n ? s_keys[i] : 0xFFFFFFFFu;
        val[q] = i < tile_n ? s_vals[i] : 0u;
      }
    } else {
      for (int p = tid; p < tile_n; p += kSmallSortThreads) {
        const uint32_t k = s_keys[p];
        const uint32_t d = (k >> shift) & mask;
        const uint32_t gpos = gridDim.x > 1 ? s_gbase[0][d] + ((uint32_t)p - s_dstart[d]) : (uint32_t)p;
        keys_out[gpos] = k;
        vals_out[gpos] = s_vals[p];
      }
    }
  }
}

static hipError_t launch_sort_small(const Geometry &g, const BatchBuf &b, SortScratch &ss, int *result_buf, hipStream_t s) {
  const DigitPlan digits = digit_plan(g.key_bits, byte_passes(g.key_bits));
  const int blocks = small_sort_blocks(b.n);
  auto kern = small_sort_items(b.n) == 4 ? sort_small_kernel<4> : sort_small_kernel<8>;
  uint32_t *counts = ss.said + kMaxSortPasses * 256;
  int cur = 0;
  for (int p = 0; p < digits.passes; p = blocks == 1 ? digits.passes : p + 1) {
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(kSmallSortThreads), 0, s, ss.keys[cur], ss.vals[cur], ss.keys[cur ^ 1],
                       ss.vals[cur ^ 1], (int)b.n, digits, p, blocks == 1 ? digits.passes : p + 1, ss.said, counts, ss.ticket,
                       b.cnt);
    cur ^= 1;
  }
  *result_buf = cur;
  return hipGetLastError();
}

// Sorts ss.keys[0]/vals[0] (n pairs) by the low g.key_bits bits; *result_buf tells which of
// the two buffers holds the result.
hipError_t launch_sort(const Geometry &g, const BatchBuf &b, SortScratch &ss, int *result_buf, hipStream_t s) {
  const int64_t n = b.n;
  *result_buf = 0;
  if (n <= 1) return hipSuccess;
  if (small_batch(g, n, b.batch)) return launch_sort_small(g, b, ss, result_buf, s);
  // 8-bit digits, except that keys of 25 to 27 bits (32 tables of a million rows make 25) take three passes, some of
  // them by a 9-bit digit, instead of four
  const DigitPlan digits = digit_plan(g.key_bits, (g.key_bits >= 25 && g.key_bits <= 27) ? 3 : byte_passes(g.key_bits));
  const int64_t tiles = (n + kSortTile - 1) / kSortTile;
  const int blocks = (int)(tiles < kMaxSortBlocks ? tiles : kMaxSortBlocks);
  const int64_t tiles_per_block = (tiles + blocks - 1) / blocks;
  const int chunk = (int)(tiles_per_block * kSortTile);
  const int used_blocks = (int)((n + chunk - 1) / chunk);
  int cur = 0;
  uint32_t *digit_total = ss.hist + kMaxRadix * kMaxSortBlocks;
  for (int p = 0; p < digits.passes; p++) {
    const int shift = digits.shift[p];
    const uint32_t mask = digits.mask[p];
    if (mask > 255u) {
      hipLaunchKernelGGL(sort_upsweep_kernel<9>, dim3(used_blocks), dim3(512), 0, s, ss.keys[cur], (int)n, shift, mask,
                         chunk, ss.hist);
      hipLaunchKernelGGL(sort_scan_kernel, dim3(512), dim3(256), 0, s, ss.hist, used_blocks, digit_total);
      hipLaunchKernelGGL(sort_downsweep_kernel<9>, dim3(used_blocks), dim3(512), 0, s, ss.keys[cur], ss.vals[cur],
                         ss.keys[cur ^ 1], ss.vals[cur ^ 1], (int)n, shift, mask, chunk, ss.hist, digit_total);
    } else {
      hipLaunchKernelGGL(sort_upsweep_kernel<8>, dim3(used_blocks), dim3(256), 0, s, ss.keys[cur], (int)n, shift, mask,
                         chunk, ss.hist);
      hipLaunchKernelGGL(sort_scan_kernel, dim3(256), dim3(256), 0, s, ss.hist, used_blocks, digit_total);
      hipLaunchKernelGGL(sort_downsweep_kernel<8>, dim3(used_blocks), dim3(256), 0, s, ss.keys[cur], ss.vals[cur],
                         ss.keys[cur ^ 1], ss.vals[cur ^ 1], (int)n, shift, mask, chunk, ss.hist, digit_total);
    }
    cur ^= 1;
  }
  *result_buf = cur;
  return hipGetLastError();
}

}  // namespace tbe
