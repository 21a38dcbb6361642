// Index dedup, part 1: sort keys for every lookup of a batch and a stable LSD radix sort
// of (key, position) pairs.  The paper does not describe this step; it serves the
// "group the indices" part of the tag/state lookup (Section 5.5.1) on a 64-wide machine.
#include "tbe_internal.h"

namespace tbe {

typedef unsigned long long u64;

// --------------------------------------------------------------------------------------
// key generation: 8 lanes per bag, 64-byte coalesced reads of the bag's indices; short bags a lane each (SortShape::lanes)
// --------------------------------------------------------------------------------------
constexpr int kKeygenThreads = 256;

// First kernel of the stage where a bag may be too long for the packed payload, which only the offsets tell: it looks at every
// bag and gathers the answer in *too_long, which the stage's last kernel leaves at zero for the next batch.
__global__ __launch_bounds__(256) void begin_kernel(int64_t nb, const int64_t *__restrict__ offsets, int within_bits,
                                                    uint32_t *too_long) {
  const int64_t bag = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool is = bag < nb && offsets[bag + 1] - offsets[bag] > (1ll << within_bits);
  if (__ballot(is) && (threadIdx.x & 63) == 0) atomicOr(too_long, 1u);
}

struct KeygenArgs {
  const TableMeta *tm;
  int B, nb;
  int64_t N;
  const int64_t *indices, *offsets;
  uint2 *pairs;
  int32_t *bag_of_pos;
  float *inv_len;            // null: not mean pooling
  int within_bits;
  const uint32_t *too_long;  // null: no bag can be too long for the packed payload
  SortShape sh;
  uint32_t *slots;
  uint4 *tiles;
  const int32_t *refused;
  uint32_t *stage_err;
  BatchCounters *cnt;
};

// The tiles of the sort: (first position, end, segment, number inside its segment), with kLastTile on a segment's last one.
__device__ __forceinline__ void list_tiles(const KeygenArgs &a, int *s_first, int *s_wave) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int kPer = (kLutTables + kKeygenThreads - 1) / kKeygenThreads;
  const int tile = a.sh.tile();
  auto start_of = [&](int s) { return a.offsets[(int64_t)s * a.sh.bags]; };
  int nt[kPer], mine = 0;
#pragma unroll
  for (int q = 0; q < kPer; q++) {
    const int s = tid * kPer + q;
    int64_t len = s < a.sh.segs ? start_of(s + 1) - start_of(s) : 0;
    len = len < 0 ? 0 : len > a.N ? a.N : len;  // (of a batch that is refused)
    nt[q] = (int)((len + tile - 1) / tile);
    mine += nt[q];
  }
  int incl = mine;
  for (int d = 1; d < 64; d <<= 1) {
    const int o = __shfl_up(incl, d);
    if (lane >= d) incl += o;
  }
  if (lane == 63) s_wave[wave] = incl;
  __syncthreads();
  int at = incl - mine;
  for (int w = 0; w < wave; w++) at += s_wave[w];
#pragma unroll
  for (int q = 0; q < kPer; q++) {
    if (tid * kPer + q <= a.sh.segs) s_first[tid * kPer + q] = at;
    at += nt[q];
  }
  if (tid == kKeygenThreads - 1 && a.sh.segs == kPer * kKeygenThreads) s_first[a.sh.segs] = at;
  __syncthreads();
  const int total = s_first[a.sh.segs];
  for (int x = tid; x < a.sh.tiles; x += kKeygenThreads) {
    uint4 e = make_uint4(0u, 0u, 0u, 0u);
    if (x < total) {
      int lo = 0, hi = a.sh.segs - 1;  // last segment that begins at or before x
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (s_first[mid] <= x) lo = mid; else hi = mid - 1;
      }
      const int i = x - s_first[lo];
      const uint32_t end = (uint32_t)start_of(lo + 1), from = (uint32_t)start_of(lo) + (uint32_t)i * (uint32_t)tile;
      const bool last = x + 1 == s_first[lo + 1];
      e = make_uint4(from, last ? end : from + (uint32_t)tile, (uint32_t)lo | (last ? kLastTile : 0u), (uint32_t)i);
    }
    a.tiles[x] = e;
  }
}

// Workgroup (segment, g) takes the g-th part of the segment's bags, and counts the digits of every pass of the sort in LDS: its
// counts go to a slot of its own, whose sum over the segment the sort takes as the digits' totals (additions to totals in memory
// cost a third of a microsecond per ten thousand, and a workgroup has some thousand digit values).  The last workgroup lists
// the sort's tiles.  Workgroup 0 sets the batch's counters to zero; behind a batch that was refused every batch starts as
// refused, with that one's error (the host learns of it only when it synchronises, and until then issues more): every later
// kernel of the batch then returns at once, so tags, lines and copies stay as the last good batch left them, and a batch buffer
// that is used again still says so.  What is wrong with this batch is gathered in *stage_err, which the sort's first pass
// adds to the counters (a workgroup that finds a fault may run before workgroup 0).
//
// LANES: of a bag.  With one lane a bag, what a bag has beyond kLaneLookups is left to all lanes of the wavefront together, bag after
// bag, so that a long bag among short ones holds nobody up for longer than it does eight lanes.
constexpr int kLaneLookups = 16;
template <int LANES>
__global__ __launch_bounds__(kKeygenThreads) void keygen_kernel(KeygenArgs a) {
  extern __shared__ uint32_t s_hist[];
  __shared__ int s_wave[kKeygenThreads / kWave];
  const int words = a.sh.digits.passes << a.sh.rb;
  if (blockIdx.x + 1 == gridDim.x) {
    list_tiles(a, (int *)s_hist, s_wave);
    return;
  }
  for (int i = threadIdx.x; i < words; i += kKeygenThreads) s_hist[i] = 0;
  const bool packed = a.within_bits > 0 && (a.too_long == nullptr || *a.too_long == 0u);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    begin_counters(a.cnt, *a.refused);
    a.cnt->packed = packed ? 1 : 0;
  }
  __syncthreads();
  const int seg = blockIdx.x / a.sh.slots, part = blockIdx.x % a.sh.slots;
  const int first = seg * a.sh.bags + (int)((int64_t)a.sh.bags * part / a.sh.slots);
  const int end = seg * a.sh.bags + (int)((int64_t)a.sh.bags * (part + 1) / a.sh.slots);
  const int sub = threadIdx.x % LANES;
  constexpr int kBags = kKeygenThreads / LANES, K = 2, X = 4;  // two bags, four indices of each under way per lane
  const uint32_t key0 = a.sh.segs > 1 ? a.tm[seg].key_base : 0u;
  struct Keys {  // of a table (in registers: the stores could be to the descriptions for all that the compiler knows)
    int64_t rows;
    uint32_t key_base, sets, rows_per_set;
    u64 sets_magic;
  };
  auto keys_of = [&](int bag) __attribute__((always_inline)) {
    const TableMeta &m = a.tm[a.sh.segs > 1 ? seg : bag / a.B];
    return Keys{m.rows, m.key_base, m.sets, m.rows_per_set, m.sets_magic};
  };
  auto put = [&](const Keys m, int64_t row, int bag, int64_t bag_first, int64_t j) __attribute__((always_inline)) {
    if (row < 0 || row >= m.rows) {
      atomicMax(a.stage_err, 2u /* -TBE_ERANGE */);
      row = 0;
    }
    const uint32_t d = div_by((uint32_t)row, m.sets_magic);
    const uint32_t key = m.sets ? m.key_base + ((uint32_t)row - d * m.sets) * m.rows_per_set + d : m.key_base + (uint32_t)row;
    a.pairs[j] = make_uint2(key, packed ? ((uint32_t)bag << a.within_bits) | (uint32_t)(j - bag_first) : (uint32_t)j);
    if (!packed) a.bag_of_pos[j] = bag;
    for (int p = 0; p < a.sh.digits.passes; p++)
      atomicAdd(&s_hist[(p << a.sh.rb) + (((key - key0) >> a.sh.digits.shift[p]) & a.sh.digits.mask[p])], 1u);
  };
  for (int64_t bag0 = first + (int)threadIdx.x / LANES; bag0 < end; bag0 += K * kBags) {
    int64_t lo[K], hi[K], r[K][X];
#pragma unroll
    for (int q = 0; q < K; q++) {
      const int64_t bag = bag0 + q * kBags;
      lo[q] = hi[q] = 0;
      if (bag < end) {
        const int64_t l = a.offsets[bag], h = a.offsets[bag + 1];
        if (l < 0 || h > a.N || l > h || (bag == 0 && l != 0) || (bag == a.nb - 1 && h != a.N)) {
          if (sub == 0) atomicMax(a.stage_err, 1u /* -TBE_EINVAL */);
        } else {
          lo[q] = l;
          hi[q] = h;
          // mean pooling (Section 2.1.1): a lookup of a bag of L lookups weighs 1/L
          if (a.inv_len && sub == 0) a.inv_len[bag] = h > l ? 1.0f / (float)(h - l) : 0.0f;
        }
      }
    }
#pragma unroll
    for (int q = 0; q < K; q++)
#pragma unroll
      for (int x = 0; x < X; x++) {
        const int64_t j = lo[q] + sub + x * LANES;
        r[q][x] = j < hi[q] ? a.indices[j] : 0;
      }
#pragma unroll
    for (int q = 0; q < K; q++) {
      const int64_t mine = LANES > 1 || hi[q] - lo[q] < kLaneLookups ? hi[q] : lo[q] + kLaneLookups;
      if (lo[q] + sub < mine) {
        const int bag = (int)(bag0 + q * kBags);
        const Keys m = keys_of(bag);
        for (int64_t j0 = lo[q] + sub;;) {
#pragma unroll
          for (int x = 0; x < X; x++) {
            const int64_t j = j0 + x * LANES;
            if (j < mine) put(m, r[q][x], bag, lo[q], j);
          }
          j0 += X * LANES;
          if (j0 >= mine) break;
#pragma unroll
          for (int x = 0; x < X; x++) {
            const int64_t j = j0 + x * LANES;
            r[q][x] = j < mine ? a.indices[j] : 0;
          }
        }
      }
      if constexpr (LANES == 1) {
        const int lane = threadIdx.x & 63;
        const uint64_t here = __ballot(true);  // (the last round has fewer lanes)
        const int helpers = __popcll(here), rank = __popcll(here & ((1ull << lane) - 1ull));
        for (uint64_t todo = __ballot(mine < hi[q]); todo; todo &= todo - 1) {
          const int src = __ffsll((unsigned long long)todo) - 1;
          const int64_t l = __shfl(lo[q], src), h = __shfl(hi[q], src);
          const int bag = __shfl((int)(bag0 + q * kBags), src);
          const Keys m = keys_of(bag);
          for (int64_t j = l + kLaneLookups + rank; j < h; j += helpers) put(m, a.indices[j], bag, l, j);
        }
      }
    }
  }
  __syncthreads();
  uint32_t *slot = a.slots + (size_t)blockIdx.x * words;
  for (int i = threadIdx.x; i < words; i += kKeygenThreads) slot[i] = s_hist[i];
}

// A segment's slots added up, 64 digits a workgroup.
constexpr int kSlotParts = 16;
__global__ __launch_bounds__(64 * kSlotParts) void add_slots_kernel(const uint32_t *__restrict__ slots, int n_slots, int words,
                                                                    uint32_t *__restrict__ sums) {
  __shared__ uint32_t s_part[kSlotParts][64];
  const int lane = threadIdx.x & 63, part = threadIdx.x >> 6;
  const uint32_t *p = slots + (size_t)blockIdx.y * n_slots * words + blockIdx.x * 64 + lane;
  uint32_t sum = 0;
#pragma unroll 8
  for (int g = part; g < n_slots; g += kSlotParts) sum += p[(size_t)g * words];
  s_part[part][lane] = sum;
  __syncthreads();
  if (part == 0) {
    for (int q = 1; q < kSlotParts; q++) sum += s_part[q][lane];
    sums[(size_t)blockIdx.y * words + blockIdx.x * 64 + lane] = sum;
  }
}

hipError_t launch_keygen(const TableMeta *tm, const Geometry &g, const BatchBuf &b, const SortScratch &ss, hipStream_t s) {
  KeygenArgs a{};
  a.tm = tm;
  a.B = b.batch;
  a.nb = g.T * b.batch;
  a.N = b.n;
  a.indices = b.d_indices;
  a.offsets = b.d_offsets;
  a.pairs = ss.pairs[0];
  a.bag_of_pos = b.bag_of_pos;
  a.inv_len = b.mean ? b.inv_len : nullptr;
  a.within_bits = g.within_bits;
  a.sh = sort_shape(g, b.n, b.batch);
  a.slots = ss.slots;
  a.tiles = ss.tiles;
  a.refused = ss.refused;
  a.stage_err = ss.stage_err;
  a.cnt = b.cnt;
  if (g.within_bits > 0 && b.n > 1ll << g.within_bits) {
    a.too_long = ss.too_long;
    hipLaunchKernelGGL(begin_kernel, dim3((unsigned)(((int64_t)a.nb + 255) / 256)), dim3(256), 0, s, (int64_t)a.nb, b.d_offsets,
                       g.within_bits, ss.too_long);
  }
  const int words = a.sh.digits.passes << a.sh.rb;
  const int lds = 4 * (words > kLutTables + 1 ? words : kLutTables + 1);
  hipLaunchKernelGGL(a.sh.lanes == 1 ? keygen_kernel<1> : keygen_kernel<8>, dim3(a.sh.segs * a.sh.slots + 1), dim3(kKeygenThreads), lds, s, a);
  if (a.sh.add_slots)
    hipLaunchKernelGGL(add_slots_kernel, dim3(words / 64, a.sh.segs), dim3(64 * kSlotParts), 0, s, ss.slots, a.sh.slots, words,
                       ss.slots + (size_t)a.sh.segs * a.sh.slots * words);
  return hipGetLastError();
}

// --------------------------------------------------------------------------------------
// LSD radix sort of every segment's pairs, a kernel per pass.  A workgroup ranks its tile's keys with ballot matching (stable),
// says its counts of the digit values, orders the tile in LDS, adds up the counts of the segment's tiles before it and writes the
// tile out, so that neighbouring lanes hit neighbouring addresses.  The digits' totals are known from the key generation.
// Tiles of 1024 keys say their counts in words that carry batch and pass, and add up those of all the tiles before them; larger tiles,
// of which a segment may have many, also say the sum up to them, and hear only as far back as one that has said it (see SortShape).
// A tile waits only for tiles before it, and where one of them has said nothing for kPolls looks (its workgroup may not have
// begun) counts that tile itself, so every workgroup ends whatever else runs on the GPU.  Of the larger tiles one wavefront looks at
// flags, and the counts are read when they are there: with every thread looking at its digit values' own words until they had come,
// that traffic past the L2s was what bounded a pass (7.9 M lookups 65 us, now 56).
// --------------------------------------------------------------------------------------
struct SortPassArgs {
  const uint2 *in;
  uint2 *out;
  const uint4 *tiles;
  const uint32_t *slots;   // of this pass, [segments * slots][words]
  int n_slots, words;
  const TableMeta *tm;     // null: one segment, keys as they are
  int shift;
  uint32_t mask;
  uint32_t *said;          // [tiles][digit values] a tile's counts, from sums_at on the sums up to it
  size_t sums_at;
  u64 *flags;              // [tiles] batch and pass, and what the tile has said in it
  u64 epoch;               // of batch and pass
  const uint32_t *stage_err;
  BatchCounters *cnt;
};
constexpr u64 kSaidOwn = 1, kSaidSum = 2;
constexpr int kTagCount = 12;        // bits of a count in a word with batch and pass (34 bits)
constexpr u64 kTagged = 1ull << 63;  // set in all of them, and in no pair of counts or sums that a larger batch has left there
template <int RB, int ITEMS>
__global__ __launch_bounds__(kSortThreads) void sort_pass_kernel(SortPassArgs a) {
  constexpr int R = 1 << RB, kWords = R / 2;  // counts of two digit values to a word
  constexpr int kWaves = kSortThreads / kWave, kTile = kSortThreads * ITEMS;
  constexpr int D = 2;  // a thread's digit values: a word
  static_assert(kWords <= kSortThreads, "a word a thread");
  constexpr bool kDirect = ITEMS == 2;  // tiles add up the counts of all tiles before them
  static_assert(!kDirect || kTile < 1 << kTagCount, "a count has room in a tagged word");
  constexpr int kGroups = kSortThreads / kWords;  // of threads that add up what others have counted
  __shared__ union {
    uint32_t cnt[kWaves][kWords];  // per wavefront and digit value: count, later the first place of its keys in the tile
    uint2 pairs[kTile];
  } s;
  __shared__ uint32_t s_out[R];  // per digit value: what takes a place in the tile to one in the output
  __shared__ uint32_t s_wtot[2][kWaves];
  __shared__ uint2 s_part[kGroups][kWords];
  __shared__ int s_take;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int blk = blockIdx.x;
  const uint4 tile = a.tiles[blk];  // (requested together with the errors)
  {
    const int err = a.cnt->err, here = (int)*a.stage_err;
    if (err | here) {  // the keys need not be whole; the same for all threads: what thread 0 adds was `here` before
      if (blk == 0 && tid == 0 && here > err) a.cnt->err = here;
      return;
    }
  }
  if (tile.x >= tile.y) return;  // behind the last one
  const uint2 *in = a.in + tile.x;
  const int n = (int)(tile.y - tile.x), seg = (int)(tile.z & ~kLastTile);
  const uint32_t key0 = a.tm ? a.tm[seg].key_base : 0u;
  const uint64_t lt_mask = (1ull << lane) - 1ull;
  const int w0 = wave * (kWave * ITEMS) + lane;
  uint2 e[ITEMS];
  uint32_t place[ITEMS];
#pragma unroll
  for (int q = 0; q < ITEMS; q++) e[q] = w0 + q * kWave < n ? in[w0 + q * kWave] : make_uint2(0u, 0u);
  for (int i = tid; i < kWaves * kWords; i += kSortThreads) (&s.cnt[0][0])[i] = 0;
  if (tid == 0) s_take = 0;
  const int grp = tid / kWords, word = tid % kWords;
  {  // the segment's totals of two digit values, a share of the slots each group
    uint2 sum = make_uint2(0u, 0u);
    const uint32_t *p = a.slots + (size_t)seg * a.n_slots * a.words + word * D;
    for (int g = grp; g < a.n_slots; g += 8 * kGroups) {
      uint2 v[8];
#pragma unroll
      for (int q = 0; q < 8; q++) v[q] = g + q * kGroups < a.n_slots ? *(const uint2 *)(p + (size_t)(g + q * kGroups) * a.words) : make_uint2(0u, 0u);
#pragma unroll
      for (int q = 0; q < 8; q++) {
        sum.x += v[q].x;
        sum.y += v[q].y;
      }
    }
    s_part[grp][word] = sum;
  }
  __syncthreads();
  auto digit = [&](uint32_t key) { return ((key - key0) >> a.shift) & a.mask; };
#pragma unroll
  for (int q = 0; q < ITEMS; q++) {  // stable rank among the wavefront's keys of the digit value
    place[q] = 0;
    if (wave * (kWave * ITEMS) + q * kWave >= n) continue;  // the same in all lanes
    const bool valid = w0 + q * kWave < n;
    const uint32_t d = digit(e[q].x);
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int bit = 0; bit < RB; bit++) {
      const bool on = (d >> bit) & 1u;
      const uint64_t bal = __ballot(on);
      peers &= on ? bal : ~bal;
    }
    const uint32_t below = __popcll(peers & lt_mask);
    const int half = (int)(d & 1u) * 16;
    uint32_t prev = 0;
    if (valid && below == 0) prev = atomicAdd(&s.cnt[wave][d >> 1], (uint32_t)__popcll(peers) << half) >> half & 0xFFFFu;
    const int leader = valid ? (__ffsll((unsigned long long)peers) - 1) : lane;
    place[q] = __shfl(prev, leader) + below;
  }
  __syncthreads();
  const bool mine = tid < kWords;  // this thread has digit values
  uint32_t count[D] = {}, total[D] = {}, before[D] = {};
  // The tile's counts, or the sums up to it, for the tiles behind it, and the flag that says that they are there.  They are
  // written through to memory and have arrived when the flag is.
  auto say_counts = [&](const uint32_t (&c)[D], size_t at, u64 state) {
    if (mine)
      __hip_atomic_store((u64 *)(a.said + at + (size_t)blk * R + tid * D), c[0] | (u64)c[1] << 32, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) __hip_atomic_store(a.flags + blk, a.epoch << 2 | state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  if (mine) {
    uint32_t sum = 0;
#pragma unroll
    for (int w = 0; w < kWaves; w++) {
      const uint32_t c = s.cnt[w][tid];
      s.cnt[w][tid] = sum;
      sum += c;
    }
    count[0] = sum & 0xFFFFu;
    count[1] = sum >> 16;
  }
  const u64 tag = kTagged | a.epoch << 2 * kTagCount;
  if (!(tile.z & kLastTile)) {
    if constexpr (!kDirect) say_counts(count, tile.w ? 0 : a.sums_at, tile.w ? kSaidOwn : kSaidSum);
    else if (mine)
      __hip_atomic_store((u64 *)(a.said + (size_t)blk * R + tid * D), tag | count[1] << kTagCount | count[0], __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
  }
  if (mine)
#pragma unroll
    for (int q = 0; q < kGroups; q++) {
      total[0] += s_part[q][tid].x;
      total[1] += s_part[q][tid].y;
    }
  uint32_t out[D] = {};  // first place of the segment's keys of each digit value in the output, less that in the tile
  {  // exclusive prefix over the digit values, of the tile's counts and of the segment's
    uint32_t c = 0, t = 0;
#pragma unroll
    for (int x = 0; x < D; x++) { c += count[x]; t += total[x]; }
    uint32_t ci = c, ti = t;
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t oc = __shfl_up(ci, d), ot = __shfl_up(ti, d);
      if (lane >= d) { ci += oc; ti += ot; }
    }
    if (lane == 63) { s_wtot[0][wave] = ci; s_wtot[1][wave] = ti; }
    __syncthreads();
    uint32_t at = ci - c, to = tile.x - tile.w * (uint32_t)kTile + ti - t;  // (the segment begins tile.w tiles before this one)
    for (int w = 0; w < wave; w++) { at += s_wtot[0][w]; to += s_wtot[1][w]; }
    if (mine) {
      const uint32_t at1 = at + count[0];
#pragma unroll
      for (int w = 0; w < kWaves; w++) s.cnt[w][tid] += at | at1 << 16;
      out[0] = to - at;
      out[1] = to + total[0] - at1;
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < ITEMS; q++) {
    const uint32_t d = digit(e[q].x);
    place[q] += s.cnt[wave][d >> 1] >> ((d & 1u) * 16) & 0xFFFFu;
  }
  __syncthreads();  // the counts are no longer read: the pairs take their room
#pragma unroll
  for (int q = 0; q < ITEMS; q++)
    if (w0 + q * kWave < n) s.pairs[place[q]] = e[q];
  if constexpr (kDirect) {
    // The keys of these digit values in the segment's tiles before this one, a share of the tiles each group.
    uint2 sum = make_uint2(0u, 0u);
    bool silent = false;
    int polls = 0;
    for (int t0 = grp; t0 < (int)tile.w && !silent; t0 += 8 * kGroups) {
      for (;;) {
        const u64 *p = (const u64 *)(a.said + (size_t)(blk - 1 - t0) * R) + word;
        u64 v[8];
        bool all = true;
#pragma unroll
        for (int q = 0; q < 8; q++) v[q] = t0 + q * kGroups < (int)tile.w ? look(p - (size_t)q * kGroups * kWords) : tag;
#pragma unroll
        for (int q = 0; q < 8; q++) all = all && (v[q] ^ tag) >> 2 * kTagCount == 0;
        if (all) {
#pragma unroll
          for (int q = 0; q < 8; q++) {
            sum.x += (uint32_t)v[q] & ((1u << kTagCount) - 1u);
            sum.y += (uint32_t)(v[q] >> kTagCount) & ((1u << kTagCount) - 1u);
          }
          break;
        }
        silent = polls++ >= kPolls;
        if (silent) break;
        __builtin_amdgcn_s_sleep(1);
      }
    }
    if (silent) s_take = 1;
    s_part[grp][word] = sum;
    __syncthreads();
    if (s_take) {
      // A tile has said nothing for long: its workgroup may not have begun, and this one waits for nobody.  All are counted here.
      for (int i = tid; i < R; i += kSortThreads) s_out[i] = 0;
      __syncthreads();
      const uint2 *old = in - (size_t)tile.w * kTile;
      for (int i = tid; i < (int)tile.w * kTile; i += kSortThreads) atomicAdd(&s_out[digit(old[i].x)], 1u);
      __syncthreads();
      if (mine) {
        before[0] = s_out[tid * D];
        before[1] = s_out[tid * D + 1];
      }
    } else if (mine) {
#pragma unroll
      for (int q = 0; q < kGroups; q++) {
        before[0] += s_part[q][tid].x;
        before[1] += s_part[q][tid].y;
      }
    }
    __syncthreads();
  }
  // The keys of these digit values in the segment's tiles before this one: as many as have said their own counts, as far back
  // as one that has said the sum up to it (the segment's first says that at once).
  for (int done = kDirect ? (int)tile.w : 0; done < (int)tile.w;) {
    if (wave == 0) {
      int take = 0, how = 0;
      for (int polls = 0;; polls++) {
        const int back = done + lane + 1;
        const u64 f = back <= (int)tile.w ? look(a.flags + blk - back) : 0ull;
        const uint32_t state = f >> 2 == a.epoch ? (uint32_t)f & 3u : 0u;
        const uint64_t silent = __ballot(state == 0u);
        take = silent ? __ffsll((unsigned long long)silent) - 1 : kWave;
        const uint64_t sums = __ballot(state == kSaidSum) & (take == kWave ? ~0ull : (1ull << take) - 1ull);
        if (sums) {
          take = __ffsll((unsigned long long)sums);
          how = 1;
          break;
        }
        if (take == kWave) break;
        // A tile has said nothing for long: its workgroup may not have begun, and this one waits for nobody.  It is counted here.
        if (polls >= kPolls) {
          how = 2;
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
      if (lane == 0) s_take = take << 2 | how;
    }
    __syncthreads();
    const int take = s_take >> 2, how = s_take & 3;
    if (mine) {
      const uint32_t *p = a.said + ((size_t)blk - done - 1) * R + tid * D;
      for (int t0 = 0; t0 < take; t0 += 8) {
        u64 v[8];
#pragma unroll
        for (int q = 0; q < 8; q++) {
          const uint32_t *from = p - (size_t)(t0 + q) * R + (how == 1 && t0 + q + 1 == take ? a.sums_at : 0);
          v[q] = t0 + q < take ? look((const u64 *)from) : 0ull;
        }
#pragma unroll
        for (int q = 0; q < 8; q++) {
          before[0] += (uint32_t)v[q];
          before[1] += (uint32_t)(v[q] >> 32);
        }
      }
    }
    done = how == 1 ? (int)tile.w : done + take;
    if (how == 2) {
      done++;
      for (int i = tid; i < R; i += kSortThreads) s_out[i] = 0;
      __syncthreads();
      const uint2 *old = in - (size_t)done * kTile;
      for (int i = tid; i < kTile; i += kSortThreads) atomicAdd(&s_out[digit(old[i].x)], 1u);
      __syncthreads();
      if (mine)
#pragma unroll
        for (int x = 0; x < D; x++) before[x] += s_out[tid * D + x];
    }
    __syncthreads();
  }
  if (!kDirect && tile.w && !(tile.z & kLastTile)) {
#pragma unroll
    for (int x = 0; x < D; x++) count[x] += before[x];
    say_counts(count, a.sums_at, kSaidSum);
  }
  if (mine)
#pragma unroll
    for (int x = 0; x < D; x++) s_out[tid * D + x] = out[x] + before[x];
  __syncthreads();
  for (int p = tid; p < n; p += kSortThreads) {
    const uint2 v = s.pairs[p];
    a.out[s_out[digit(v.x)] + (uint32_t)p] = v;
  }
}

template <int RB>
static void (*sort_kernel_of(int items))(SortPassArgs) {
  return items == 2 ? sort_pass_kernel<RB, 2> : items == 4 ? sort_pass_kernel<RB, 4> : items == 8 ? sort_pass_kernel<RB, 8> : sort_pass_kernel<RB, 16>;
}

// Sorts ss.pairs[0] segment by segment; *result_buf tells which of the two buffers holds the result.
hipError_t launch_sort(const TableMeta *tm, const Geometry &g, const BatchBuf &b, const SortScratch &ss, int *result_buf, hipStream_t s) {
  *result_buf = 0;
  if (b.n == 0) return hipSuccess;
  const SortShape sh = sort_shape(g, b.n, b.batch);
  const int words = sh.digits.passes << sh.rb;
  auto kern = sh.rb == 8 ? sort_kernel_of<8>(sh.items) : sh.rb == 9 ? sort_kernel_of<9>(sh.items)
              : sort_kernel_of<10>(sh.items);
  SortPassArgs a{};
  a.tiles = ss.tiles;
  a.n_slots = sh.add_slots ? 1 : sh.slots;
  a.words = words;
  a.tm = sh.segs > 1 ? tm : nullptr;
  a.said = ss.said;
  a.sums_at = (size_t)sh.tiles << sh.rb;
  a.flags = ss.flags;
  a.stage_err = ss.stage_err;
  a.cnt = b.cnt;
  int cur = 0;
  for (int p = 0; p < sh.digits.passes; p++) {
    a.in = ss.pairs[cur];
    a.out = ss.pairs[cur ^ 1];
    a.slots = ss.slots + (sh.add_slots ? (size_t)sh.segs * sh.slots * words : 0) + ((size_t)p << sh.rb);
    a.shift = sh.digits.shift[p];
    a.mask = sh.digits.mask[p];
    a.epoch = (u64)b.k * kMaxSortPasses + p;
    hipLaunchKernelGGL(kern, dim3((unsigned)sh.tiles), dim3(kSortThreads), 0, s, a);
    cur ^= 1;
  }
  *result_buf = cur;
  return hipGetLastError();
}

}  // namespace tbe
