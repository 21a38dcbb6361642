// Data movement between the cache lines in HBM and the backing tier in pinned host memory
// (paper Section 5.5.3 data lookup/update, 5.5.4 data movement, one-level cache: missed rows
// are inserted from the lower tier, LRU rows are written back to it), arranged so that
// the host link works in both directions while the previous batch is still training
// (Section 5.7: prefetch ahead of training; Section 6.1: cache management overlapped with
// the computation of the batch before).
//
// For the batch being prefetched (k+1), with batch k possibly still training:
//   (the list pass of k+1, in the prefetch stage: a row wanted by k+1 whose backing-tier copy is being written in this very
//              window is "late".  A map over the sort keys says where its current value
//              is: in batch k's overflow copies (k bypassed it and trains on that copy)
//              or among the victims batch k parked (k evicted it).)
//   transfer : victims of batch k, parked in the staging area when k was committed, go to
//              the backing tier; at the same time the rows batch k+1 inserts or bypasses
//              are fetched into HBM, except the late ones.  Runs on the link stream, that of a
//              small batch on its stage's stream or the compute stream.
//   commit   : after batch k has trained: victims of k+1 move from their cache lines to
//              the staging area, the new rows move in; late rows are copied HBM to HBM from
//              where the map pointed.  Also writes batch k's overflow copies back.
// Host rows are reached through the pinned mapping, 16 bytes per lane, 4 to 16 lanes per row (TBE_BY_ROW_LANES).
#include <hip/hip_fp16.h>
#include "tbe_internal.h"

namespace tbe {

typedef unsigned long long u64;
// Runs CALL with `L` = the lanes that move a row, 16 bytes each: as many as the widest row of the model has pieces, 16
// at most.  Rows of at most 128 bytes used to leave half of their 16 lanes idle, and a wavefront had four of them under
// way instead of eight: swapping 241 k rows of 128 bytes with host memory 0.97 -> 0.93 ms (33 GB/s per direction; a
// kernel that does nothing else reaches 36.5 whatever the order of the rows: each is a request of its own on the link),
// their commit 0.050 -> 0.038 ms.  Wider rows keep a lane per piece: 256-byte rows by 8 lanes, two pieces each, have
// twice the bytes under way and take 6.2 instead of 5.2 ms per transfer of the benchmark workload; 128 to 512-byte
// rows mixed, by 8 lanes: 14.8 instead of 14.2 ms for four steps.
#define TBE_BY_ROW_LANES(STRIDE, CALL)                       \
  do {                                                       \
    if ((STRIDE) <= 64) { constexpr int L = 4; CALL; }       \
    else if ((STRIDE) <= 128) { constexpr int L = 8; CALL; } \
    else { constexpr int L = 16; CALL; }                     \
  } while (0)
constexpr int kLinkBlocks = 192;   // workgroups of the smaller kernels that write to the host link
constexpr int kLinkThreads = 1024;
constexpr int kSwapThreads = 256, kSwapBlocks = 192;
// Workgroups of `threads` for `rows` rows of `lanes` lanes, a row to each lane group, but no more than `most`: those of a small
// batch that find nothing to do cost it time to be dealt out (the commit of 119 lookups as 4096 workgroups 4.8 us, as two 3).
static int row_blocks(int64_t rows, int lanes, int threads, int most) {
  const int64_t want = (rows * lanes + threads - 1) / threads;
  return want < 1 ? 1 : want < most ? (int)want : most;
}

// ---- deferred initialisation: counter-based normal numbers of (seed, table, row, element) ----
// z = centred sum of twelve 16-bit uniforms (three 64-bit hashes per element, the finaliser of
// splitmix64), integer arithmetic up to one fp32 product -- the stored bits are the same
// wherever the definition is evaluated.
__device__ inline u64 mix64(u64 x) {
  x += 0x9E3779B97F4A7C15ull;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
  return x ^ (x >> 31);
}

__device__ inline u64 init_table_key(u64 seed, int t) { return mix64(seed ^ ((u64)(t + 1) * 0xD1342543DE82EF95ull)); }

__device__ inline float init_value(u64 table_key, uint32_t row, uint32_t e, float scale) {
  int32_t s = -12 * 65536;
#pragma unroll
  for (int j = 0; j < 3; j++) {
    const u64 h = mix64(table_key + (u64)row * 0x2545F4914F6CDD1Dull + (u64)e * 3u + (u64)j);
    s += 2 * (int32_t)((h & 0xFFFFu) + ((h >> 16) & 0xFFFFu) + ((h >> 32) & 0xFFFFu) + (h >> 48)) + 4;
  }
  float v = __fmul_rn((float)s, scale);
  // The fp32 product is the value; the fp16 table stores its rounding.  Without this barrier the
  // compiler folds product and conversion into one mixed-precision instruction that rounds once,
  // which differs from rounding the fp32 value wherever that value is an fp16 tie.
  asm volatile("" : "+v"(v));
  return v;
}

// the 16 bytes of row `row` that start at element e0 (4 fp32 or 8 fp16 values), std * z each
__device__ inline uint4 init_chunk(u64 table_key, uint32_t row, int dtype, uint32_t e0, float std) {
  const float scale = std * 0x1p-17f;  // exact
  if (dtype == 0)
    return make_uint4(__float_as_uint(init_value(table_key, row, e0, scale)),
                      __float_as_uint(init_value(table_key, row, e0 + 1, scale)),
                      __float_as_uint(init_value(table_key, row, e0 + 2, scale)),
                      __float_as_uint(init_value(table_key, row, e0 + 3, scale)));
  uint32_t w[4];
  for (int i = 0; i < 4; i++)
    w[i] = (uint32_t)__half_as_ushort(__float2half_rn(init_value(table_key, row, e0 + 2 * i, scale))) |
           ((uint32_t)__half_as_ushort(__float2half_rn(init_value(table_key, row, e0 + 2 * i + 1, scale))) << 16);
  return make_uint4(w[0], w[1], w[2], w[3]);
}

// Has row `row` of table m a value yet?  If not, it gets one now: lane 0 of the group marks the
// row and tells the others what the mark was before.
template <int L>
__device__ inline bool needs_init(const TableMeta &m, uint32_t row, int lig) {
  const uint32_t bit = 1u << (row & 31);
  uint32_t before = 0;
  if (lig == 0) before = atomicOr(m.init_bits + (row >> 5), bit);
  before = __shfl(before, 0, L);
  return (before & bit) == 0;
}

typedef uint32_t mv_u32x4 __attribute__((ext_vector_type(4)));
// A row on its way to host memory: non-temporal stores (the transfer of the benchmark workload
// 5.52 -> 5.36 ms; non-temporal loads from host memory change nothing).
template <int L>
__device__ inline void copy_row_to_host(char *dst, const char *src, uint32_t bytes, int lig) {
  for (uint32_t c = lig * 16; c < bytes; c += L * 16) {
    const mv_u32x4 v = *(const mv_u32x4 *)(src + c);
    __builtin_nontemporal_store(v, (mv_u32x4 *)(dst + c));
  }
}
template <int L>
__device__ inline void copy_row(char *dst, const char *src, uint32_t bytes, int lig) {
  for (uint32_t c = lig * 16; c < bytes; c += L * 16) *(uint4 *)(dst + c) = *(const uint4 *)(src + c);
}

// Rows between the host link and the staging areas: what transfer_kernel and swap_kernel share.
template <int L>
__device__ __forceinline__ void transfer_rows(const Staging &st, const BatchCounters *cnt, char *const *__restrict__ ins_src,
                                              const int32_t *__restrict__ ins_tab, const uint32_t *__restrict__ rb_of_table,
                                              const uint32_t *__restrict__ ins_where, char *const *__restrict__ byp_src,
                                              const int32_t *__restrict__ byp_tab, const uint32_t *__restrict__ byp_where,
                                              char *__restrict__ ovf, char *const *__restrict__ l2v_src,
                                              char *const *wb2_dst, char *out2_even, char *out2_odd, int k,
                                              const TableMeta *__restrict__ di_tm, u64 di_seed, float di_std,
                                              const uint32_t *__restrict__ ins_key, const uint32_t *__restrict__ byp_key,
                                              u64 *bytes_h2d, u64 *bytes_d2h, const char *l2_lo, const char *l2_hi,
                                              int pauses) {
  const int bid = blockIdx.x, n_blocks = gridDim.x;
  const int n_wb = *st.wb_n;
  const int n_ins = (cnt && cnt->err == 0) ? cnt->n_ins : 0;
  const int n_byp = (cnt && cnt->err == 0) ? cnt->n_byp : 0;
  // One pass of the loop fetches item i and writes back slot i.  When there are more slots to write
  // than items to fetch (the overflow copies parked behind the victims), the surplus is paired with
  // the first passes (slot i + n) instead of forming a tail of passes that only write: the link's two
  // directions stay busy together to the end.
  const int n = max((n_wb + 1) / 2, max(n_ins, n_byp));
  const int group = (bid * blockDim.x + threadIdx.x) / L;
  const int lig = threadIdx.x % L;
  const int n_groups = n_blocks * blockDim.x / L;
  u64 in_b = 0, out_b = 0;
  const int wpar = st.wb_n[1] & 1;
  // emulated slower tier: rows of this pass that the group moved to or from the backing tier proper
  int slow_rows = 0;
  auto in_backing = [&](const char *p) { return pauses > 0 && !(p >= l2_lo && p < l2_hi); };
  auto write_back = [&](int w) {
    if (w >= n_wb) return;
    char *dst = st.wb_dst[w];
    uint8_t *skip = st.wb_skip[wpar] + w;
    if (*skip) {  // the batch being prefetched takes this row back from the parked copy: the
      dst = nullptr;  // line stays dirty in HBM and is written back when it is evicted again
      if (lig == 0) *skip = 0;
    }
    if (dst) {
      const uint32_t wrb = st.wb_rb[w];
      copy_row_to_host<L>(dst, st.out[wpar] + (size_t)w * st.stride, wrb, lig);
      if (lig == 0) out_b += wrb;
      slow_rows += in_backing(dst);
    }
    if (wb2_dst) {  // second level: the row this victim pushed out of it goes to the lower tier
      char *dst2 = wb2_dst[w];
      uint8_t *skip2 = st.wb_skip[wpar] + st.max_inserts + w;
      if (dst2 && *skip2) {
        dst2 = nullptr;
        if (lig == 0) *skip2 = 0;
      }
      if (dst2) {
        const uint32_t wrb = st.wb_rb[w];
        copy_row_to_host<L>(dst2, (wpar ? out2_odd : out2_even) + (size_t)w * st.stride, wrb, lig);
        if (lig == 0) out_b += wrb;
        slow_rows += in_backing(dst2);
      }
    }
  };
  for (int i = group; i < n; i += n_groups) {
    // issue the host read first, then the write-back, so both directions are busy
    uint4 fresh[4];
    uint32_t rb = 0;
    bool fetch = false, made_up = false;
    if (i < n_ins) {
      fetch = ins_where[i] == 0;
      if (fetch) {
        const int t = ins_tab[i];
        rb = rb_of_table[t];
        if (di_tm) {  // deferred initialisation: a row read for the first time gets its value here
          const TableMeta &m = di_tm[t];
          const uint32_t row = row_of_key(m, ins_key[i]);
          made_up = needs_init<L>(m, row, lig);
          if (made_up) {
            const u64 tk = init_table_key(di_seed, t);
            const uint32_t esz = m.dtype == 0 ? 4u : 2u;
#pragma unroll
            for (int q = 0; q < 4; q++) {
              const uint32_t c = lig * 16 + q * L * 16;
              if (c < rb) fresh[q] = init_chunk(tk, row, m.dtype, c / esz, di_std);
            }
          }
        }
        if (!made_up) {
          const char *src = ins_src[i];
          slow_rows += in_backing(src);
#pragma unroll
          for (int q = 0; q < 4; q++) {
            const uint32_t c = lig * 16 + q * L * 16;
            if (c < rb) fresh[q] = *(const uint4 *)(src + c);
          }
        }
      }
    }
    write_back(i);
    write_back(i + n);  // the slots beyond the loop's length ride along with the first ones
    if (l2v_src && i < n_ins) {  // second level: the row an insert's victim pushes out is read while its
      const char *src = l2v_src[i];  // line still holds it (the victim is written there by the next transfer)
      if (src) {
        const uint32_t vrb = rb_of_table[ins_tab[i]];
        copy_row<L>(((k & 1) ? out2_odd : out2_even) + (size_t)i * st.stride, src, vrb, lig);
        if (lig == 0) in_b += vrb;
      }
    }
    if (fetch) {
      char *dst = st.in + (size_t)i * st.stride;
#pragma unroll
      for (int q = 0; q < 4; q++) {
        const uint32_t c = lig * 16 + q * L * 16;
        if (c < rb) *(uint4 *)(dst + c) = fresh[q];
      }
      if (lig == 0 && !made_up) in_b += rb;
    }
    if (i < n_byp && byp_where[i] == 0) {  // bypassed rows of this batch: HBM copy for its training
      const int t = byp_tab[i];
      const uint32_t brb = rb_of_table[t];
      bool fresh_row = false;
      if (di_tm) {
        const TableMeta &m = di_tm[t];
        const uint32_t row = row_of_key(m, byp_key[i]);
        fresh_row = needs_init<L>(m, row, lig);
        if (fresh_row) {
          const u64 tk = init_table_key(di_seed, t);
          const uint32_t esz = m.dtype == 0 ? 4u : 2u;
          for (uint32_t c = lig * 16; c < brb; c += L * 16)
            *(uint4 *)(ovf + (size_t)i * st.stride + c) = init_chunk(tk, row, m.dtype, c / esz, di_std);
        }
      }
      if (!fresh_row) {
        copy_row<L>(ovf + (size_t)i * st.stride, byp_src[i], brb, lig);
        if (lig == 0) in_b += brb;
        slow_rows += in_backing(byp_src[i]);
      }
    }
    if (pauses > 0) {  // the wavefront pauses once per backing-tier row its groups moved (a bounded delay: no wait on memory)
      int rows = 0;    // counted over the lanes still in the loop; a pass moves at most five rows per group
      for (int q = 1; q <= 5; q++) rows += __popcll(__ballot(lig == 0 && slow_rows >= q));
      for (int z = 0; z < rows * pauses; z++) __builtin_amdgcn_s_sleep(127);
      slow_rows = 0;
    }
  }
  for (int d = 32; d >= 1; d >>= 1) {
    in_b += __shfl_xor(in_b, d);
    out_b += __shfl_xor(out_b, d);
  }
  if ((threadIdx.x & 63) == 0) {
    if (in_b) atomicAdd(bytes_h2d, in_b);
    if (out_b) atomicAdd(bytes_d2h, out_b);
  }
}

template <int L>
__global__ __launch_bounds__(kLinkThreads) void transfer_kernel(Staging st, const BatchCounters *cnt,
                                                       char *const *__restrict__ ins_src,
                                                       const int32_t *__restrict__ ins_tab,
                                                       const uint32_t *__restrict__ rb_of_table,
                                                       const uint32_t *__restrict__ ins_where,
                                                       char *const *__restrict__ byp_src,
                                                       const int32_t *__restrict__ byp_tab,
                                                       const uint32_t *__restrict__ byp_where, char *__restrict__ ovf,
                                                       char *const *__restrict__ l2v_src,
                                                       char *const *__restrict__ wb2_dst, char *out2_even,
                                                       char *out2_odd, int k, const TableMeta *__restrict__ di_tm,
                                                       u64 di_seed, float di_std,
                                                       const uint32_t *__restrict__ ins_key,
                                                       const uint32_t *__restrict__ byp_key, u64 *bytes_h2d,
                                                       u64 *bytes_d2h, const char *l2_lo, const char *l2_hi,
                                                       int pauses) {
  // Waves that wait on the host link slow the memory accesses of every wave that shares their CU,
  // so this kernel keeps its CUs to itself: a workgroup of 16 wavefronts that claims 128 vector
  // registers per lane fills the register files of a CU's four SIMDs, and no wave of another
  // kernel is placed beside it (the clobber makes the compiler allocate up to v127).
  asm volatile("" ::: "v127");
  transfer_rows<L>(st, cnt, ins_src, ins_tab, rb_of_table, ins_where, byp_src, byp_tab, byp_where, ovf, l2v_src, wb2_dst,
                   out2_even, out2_odd, k, di_tm, di_seed, di_std, ins_key, byp_key, bytes_h2d, bytes_d2h, l2_lo, l2_hi,
                   pauses);
  // The last workgroup through empties the list of parked victims (every other one has read its length long before).
  __syncthreads();
  if (threadIdx.x == 0 && atomicInc((unsigned int *)&st.wb_n[2], gridDim.x - 1) == gridDim.x - 1) st.wb_n[0] = 0;
}

hipError_t launch_transfer(const BatchBuf *b, int64_t parked, const Staging &st, const Level2 &l2, const DeferredInit &di,
                           const Throttle &th, int k, const uint32_t *rb_of_table, u64 *bytes_h2d, u64 *bytes_d2h,
                           hipStream_t s) {
  // How many waves wait on the host link, and where, decides how the link and the HBM-bound kernels
  // of the other streams slow each other.  Measured on the benchmark workload (step / transfer
  // kernel / prefetch stage / forward kernel while the transfer runs, ms; alone the forward takes
  // 0.20 and the prefetch stage 0.94):
  //   192 workgroups of 256 threads on two XCDs, CUs shared with other kernels : 6.40 / 5.63 / 4.8 / 0.45
  //   512 such workgroups on two XCDs (they fill them)                         : 6.92 / 5.42 / 5.8 / 0.23
  //   32 workgroups of 1024 threads, a CU each (any XCD)                       : 7.44 / 6.66 / 1.7 / 0.25
  //   48                                                                       : 6.31 / 5.55 / 1.9 / 0.28
  //   64                                                                       : 6.29 / 5.56 / 2.0 / 0.30
  //   96                                                                       : 6.60 / 5.84 / 3.1 / 0.42
  // (with the overflow copies riding along, later: 40 CUs 5.81 ms per step, 48: 5.67, 56: 5.70, 64: 5.93, 72: 6.03)
  // The link needs about 750 waves; given CUs of their own (48 of 256) they leave the other
  // streams' kernels at 1.3 to 2 times their stand-alone time instead of 2.5 to 5 times.
  const int64_t passes = b && b->n > (parked + 1) / 2 ? b->n : (parked + 1) / 2;
  TBE_BY_ROW_LANES(st.stride, hipLaunchKernelGGL((transfer_kernel<L>), dim3(row_blocks(passes, L, kLinkThreads, kLinkCus)), dim3(kLinkThreads), 0, s, st, b ? b->cnt : nullptr,
                     b ? b->ins_src : nullptr, b ? b->ins_tab : nullptr, rb_of_table,
                     b ? b->ins_where : nullptr, b ? b->byp_src : nullptr, b ? b->byp_tab : nullptr,
                     b ? b->byp_where : nullptr, b ? b->ovf : nullptr, (b && l2.on) ? b->l2v_src : nullptr,
                     l2.on ? l2.wb2_dst : nullptr, l2.out2[0], l2.out2[1], k, b ? di.tm : nullptr, di.seed, di.std,
                     b ? b->ins_key : nullptr, b ? b->byp_key : nullptr, bytes_h2d, bytes_d2h, l2.lines_lo, l2.lines_hi,
                     th.pauses));
  return hipGetLastError();
}

// ---- pipeline several batches deep ----
template <int L>
__global__ __launch_bounds__(256) void fixup_kernel(const TableMeta *__restrict__ tm, const BatchCounters *cnt,
                                                    const int32_t *__restrict__ ins_tab,
                                                    const uint32_t *__restrict__ ins_where,
                                                    const int32_t *__restrict__ ins_slot,
                                                    const uint32_t *__restrict__ ins_key,
                                                    const int32_t *__restrict__ byp_tab,
                                                    const uint32_t *__restrict__ byp_where, char *__restrict__ ovf,
                                                    OverflowCopies oc, uint32_t stride,
                                                    const uint32_t *__restrict__ rb_of_table, u64 *n_copied) {
  if (cnt->err) return;
  const int n_ins = cnt->n_ins, n_byp = cnt->n_byp;
  const int group = (blockIdx.x * blockDim.x + threadIdx.x) / L;
  const int lig = threadIdx.x % L;
  const int n_groups = gridDim.x * blockDim.x / L;
  unsigned int copied = 0;
  for (int i = group; i < n_ins + n_byp; i += n_groups) {
    const bool ins = i < n_ins;
    const uint32_t code = ins ? ins_where[i] : byp_where[i - n_ins];
    if (!(code & kWhereOverflow)) continue;
    copied += lig == 0;
    const char *src = oc.of_buf[(code >> kWhereBufShift) & (kMaxBatchBufs - 1)] + (size_t)(code & kWhereBufIndex) * stride;
    if (ins) {
      const TableMeta &m = tm[ins_tab[i]];
      const int slot = ins_slot[i];
      copy_row<L>(m.lines + (size_t)(slot - m.slot_base) * m.row_bytes, src, m.row_bytes, lig);
      // the row's accumulator was updated among those of all rows while it trained as a bypassed row
      if (lig == 0) m.slot_m[slot - m.slot_base] = m.dev_m[row_of_key(m, ins_key[i])];
    } else {
      const int j = i - n_ins;
      copy_row<L>(ovf + (size_t)j * stride, src, rb_of_table[byp_tab[j]], lig);
    }
  }
  for (int d = 32; d >= 1; d >>= 1) copied += __shfl_xor(copied, d);
  if ((threadIdx.x & 63) == 0 && copied) atomicAdd(n_copied, (u64)copied);
}

hipError_t launch_fixup(const TableMeta *tm, const BatchBuf &b, const OverflowCopies &oc, const Staging &st,
                        const uint32_t *rb_of_table, u64 *n_copied, hipStream_t s) {
  if (b.n == 0) return hipSuccess;
  TBE_BY_ROW_LANES(st.stride, hipLaunchKernelGGL((fixup_kernel<L>), dim3(row_blocks(b.n, L, 256, 1024)), dim3(256), 0, s, tm, b.cnt, b.ins_tab, b.ins_where, b.ins_slot, b.ins_key,
                     b.byp_tab, b.byp_where, b.ovf, oc, st.stride, rb_of_table, n_copied));
  return hipGetLastError();
}

// The batch before (`prev`, may be absent) has trained when this runs, so a late row's
// current value is where its code says: prev's overflow copy or prev's parked victim, both
// still in HBM.  prev_mode says what becomes of prev's overflow rows: written back here (kPrevWrite), or
// parked behind this batch's victims for the next transfer to write them (kPrevPark): the link's
// write direction then carries them beside that transfer's fetches, which costs the transfer a
// hundredth of its time, instead of alone between two transfers.
template <bool DEEP, bool LIST, int L>
__device__ __forceinline__ void commit_rows(const TableMeta *__restrict__ tm, const Staging &st, const BatchCounters *cnt,
                                            const int32_t *__restrict__ ins_tab, const uint32_t *__restrict__ ins_where,
                                            const int32_t *__restrict__ ins_slot, const int32_t *__restrict__ ins_old,
                                            const int32_t *__restrict__ byp_tab, const uint32_t *__restrict__ byp_where,
                                            char *__restrict__ ovf, const BatchCounters *prev_cnt,
                                            char *const *__restrict__ prev_byp_src, const int32_t *__restrict__ prev_byp_tab,
                                            const uint8_t *__restrict__ prev_byp_taken, const char *__restrict__ prev_ovf,
                                            int wb_prev, int k, char *const *__restrict__ ins_dst,
                                            char *const *__restrict__ l2v_src, char *const *__restrict__ l2v_dst,
                                            char **wb2_dst, const char *__restrict__ out2_prev,
                                            const uint32_t *__restrict__ rb_of_table, const uint32_t *__restrict__ ins_key,
                                            u64 *bytes_d2h) {
  constexpr bool deep = DEEP;  // pipeline several batches deep (an instance of its own: the one-deep pipeline's commit
                               // is on the critical path of every step and keeps its code as it was)
  const uint32_t M = (uint32_t)st.max_inserts;  // map codes kWhereParked | (M + i): rows staged in out2
  const int n_prev = (prev_cnt && prev_cnt->err == 0) ? prev_cnt->n_byp : 0;
  const int group = (blockIdx.x * blockDim.x + threadIdx.x) / L;
  const int lig = threadIdx.x % L;
  const int n_groups = gridDim.x * blockDim.x / L;
  if (cnt->err) {
    // This batch is refused (bad offsets or an index out of range) and does nothing, and no batch behind it does
    // anything (SortScratch::refused).  The batch before it has trained on its overflow copies, though: they go home now,
    // whatever was planned for them, so that a flush leaves the backing tier with that batch's updates.
    if (wb_prev != kPrevKeep) {
      u64 b = 0;
      for (int j = group; j < n_prev; j += n_groups) {
        const uint32_t rb = rb_of_table[prev_byp_tab[j]];
        copy_row_to_host<L>(prev_byp_src[j], prev_ovf + (size_t)j * st.stride, rb, lig);
        if (lig == 0) b += rb;
      }
      for (int d = 32; d >= 1; d >>= 1) b += __shfl_xor(b, d);
      if ((threadIdx.x & 63) == 0 && b) atomicAdd(bytes_d2h, b);
    }
    return;
  }
  const int n_ins = cnt->n_ins, n_byp = cnt->n_byp;
  const int par = k & 1, ppar = par ^ 1;
  if (LIST && blockIdx.x == 0 && threadIdx.x == 0) {
    st.wb_n[0] = n_ins + (wb_prev == kPrevPark ? n_prev : 0);
    st.wb_n[1] = par;
  }
  u64 out_b = 0;
  // An overflow copy of the batch before that this batch takes over stays in HBM: its row goes home with this batch's
  // copy of it, or from its cache line.  Where sets are smaller than what a batch looks up in them the same rows bypass
  // batch after batch: heterogeneous model (60 tables, half of the distinct rows bypass), four steps 14.56 -> 11.21 ms;
  // 8 x 4M rows, batch 32768: 29.99 -> 29.05 ms; the benchmark workload, where 6 % bypass: 23.98 -> 23.86 ms.
  if (wb_prev == kPrevWrite)
    for (int j = group; j < n_prev; j += n_groups) {
      if (prev_byp_taken[j]) continue;
      const uint32_t rb = rb_of_table[prev_byp_tab[j]];
      copy_row_to_host<L>(prev_byp_src[j], prev_ovf + (size_t)j * st.stride, rb, lig);
      if (lig == 0) out_b += rb;
    }
  if (wb_prev == kPrevPark)
    for (int j = group; j < n_prev; j += n_groups) {
      const uint32_t rb = rb_of_table[prev_byp_tab[j]];
      const size_t slot = (size_t)n_ins + (size_t)j;
      const bool taken = prev_byp_taken[j] != 0;
      if (!taken) copy_row<L>(st.out[par] + slot * st.stride, prev_ovf + (size_t)j * st.stride, rb, lig);
      if (lig == 0) {
        st.wb_dst[slot] = taken ? nullptr : prev_byp_src[j];
        st.wb_rb[slot] = rb;
      }
    }
  for (int i = group; i < n_ins; i += n_groups) {
    const TableMeta &m = tm[ins_tab[i]];
    const int slot = ins_slot[i];
    const int32_t old = ins_old[i];
    const uint32_t code = ins_where[i];
    const uint32_t rb = m.row_bytes;
    char *line = m.lines + (size_t)(slot - m.slot_base) * rb;
    const uint32_t ix = code & kWhereIndex;
    // (deep pipeline: an overflow copy may belong to a batch that has not trained yet -- the line gets the staging
    //  slot's content for now and the value, with its accumulator, before this batch's forward: fixup_kernel)
    const char *src = (code == 0 || (deep && (code & kWhereOverflow))) ? st.in + (size_t)i * st.stride
                      : (code & kWhereOverflow) ? prev_ovf + (size_t)ix * st.stride
                      : (out2_prev && ix >= M)  ? out2_prev + (size_t)(ix - M) * st.stride
                                                : st.out[ppar] + (size_t)ix * st.stride;
    char *park = st.out[par] + (size_t)i * st.stride;
    // The accumulators move with the rows: the victim's back among those of all rows, the new row's to the
    // slot (a row is in a cache line or among the others, never both, so the two differ).  Both are requested
    // before the row is copied, so that they travel beside it.
    float *sm = m.slot_m + (slot - m.slot_base);
    float m_victim = 0.f, m_fresh = 0.f;
    if (lig == 0) {
      m_victim = *sm;
      m_fresh = m.dev_m[row_of_key(m, ins_key[i])];
    }
    for (uint32_t c = lig * 16; c < rb; c += L * 16) {
      // The staged row and the parked victim pass through once: read and written around the caches, so that
      // the forward that follows does not start behind half a gigabyte of dirty lines (commit 0.274 -> 0.253 ms,
      // the forward after it 0.198 -> 0.186 ms).  The line itself is about to be read: it is stored as usual.
      const mv_u32x4 fresh = __builtin_nontemporal_load((const mv_u32x4 *)(src + c));
      if (old >= 0) __builtin_nontemporal_store(*(const mv_u32x4 *)(line + c), (mv_u32x4 *)(park + c));
      *(mv_u32x4 *)(line + c) = fresh;
    }
    if (lig == 0) {
      st.wb_dst[i] = old < 0 ? nullptr : ins_dst ? ins_dst[i] : m.host_w + (size_t)old * rb;
      st.wb_rb[i] = rb;
      if (wb2_dst) wb2_dst[i] = l2v_src[i] ? l2v_dst[i] : nullptr;
      if (old >= 0) m.dev_m[old] = m_victim;
      *sm = m_fresh;
    }
  }
  for (int j = group; j < n_byp; j += n_groups) {  // late bypassed rows
    const uint32_t code = byp_where[j];
    if (code == 0 || (deep && (code & kWhereOverflow))) continue;
    const uint32_t ix = code & kWhereIndex;
    const char *src = (code & kWhereOverflow) ? prev_ovf + (size_t)ix * st.stride
                      : (out2_prev && ix >= M) ? out2_prev + (size_t)(ix - M) * st.stride
                                              : st.out[ppar] + (size_t)ix * st.stride;
    copy_row<L>(ovf + (size_t)j * st.stride, src, rb_of_table[byp_tab[j]], lig);
  }
  for (int d = 32; d >= 1; d >>= 1) out_b += __shfl_xor(out_b, d);
  if ((threadIdx.x & 63) == 0 && out_b) atomicAdd(bytes_d2h, out_b);
}

template <bool DEEP, int L>
__global__ __launch_bounds__(256) void commit_kernel(const TableMeta *__restrict__ tm, Staging st,
                                                     const BatchCounters *cnt, const int32_t *__restrict__ ins_tab,
                                                     const uint32_t *__restrict__ ins_where,
                                                     const int32_t *__restrict__ ins_slot,
                                                     const int32_t *__restrict__ ins_old,
                                                     const int32_t *__restrict__ byp_tab,
                                                     const uint32_t *__restrict__ byp_where, char *__restrict__ ovf,
                                                     const BatchCounters *prev_cnt,
                                                     char *const *__restrict__ prev_byp_src,
                                                     const int32_t *__restrict__ prev_byp_tab,
                                                     const uint8_t *__restrict__ prev_byp_taken,
                                                     const char *__restrict__ prev_ovf, int wb_prev, int k,
                                                     char *const *__restrict__ ins_dst,
                                                     char *const *__restrict__ l2v_src,
                                                     char *const *__restrict__ l2v_dst, char **wb2_dst,
                                                     const char *__restrict__ out2_prev,
                                                     const uint32_t *__restrict__ rb_of_table,
                                                     const uint32_t *__restrict__ ins_key, u64 *bytes_d2h) {
  commit_rows<DEEP, true, L>(tm, st, cnt, ins_tab, ins_where, ins_slot, ins_old, byp_tab, byp_where, ovf, prev_cnt,
                             prev_byp_src, prev_byp_tab, prev_byp_taken, prev_ovf, wb_prev, k, ins_dst, l2v_src, l2v_dst,
                             wb2_dst, out2_prev, rb_of_table, ins_key, bytes_d2h);
}

// Transfer and commit in one launch, for a batch that was prefetched with none in flight: its commit need not wait for an update.
// Small batches only, bound by the latency of one trip over the link and by launches: 92 lookups 62.5 -> 58.0 us a step, 18 and 51
// 48.5 -> 46.2 and 47.3 -> 45.0.  A lane group handles the same items in both parts, so what it fetched (st.in), the parked victim it wrote
// home and that victim's slot in the list are its own.  The groups need not wait for one another: the transfer part touches no cache
// line, reads the victims of the batch before (out[par ^ 1], which the commit part only reads), the list's slots i and i + n, n >=
// n_ins (the commit part writes slots i < n_ins, each after its group has read it), and the second level's lines, which no commit
// touches; rows pushed out of the second level go to out2[par], late ones come from out2[par ^ 1].  No workgroup of 1024 threads
// with a CU to itself: nothing of the library's runs beside it, and 192 of 256 threads are as many wavefronts.
template <int L>
__global__ __launch_bounds__(kSwapThreads) void swap_kernel(Staging st, const BatchCounters *cnt,
                                                            char *const *__restrict__ ins_src,
                                                            const int32_t *__restrict__ ins_tab,
                                                            const uint32_t *__restrict__ rb_of_table,
                                                            const uint32_t *__restrict__ ins_where,
                                                            char *const *__restrict__ byp_src,
                                                            const int32_t *__restrict__ byp_tab,
                                                            const uint32_t *__restrict__ byp_where, char *__restrict__ ovf,
                                                            char *const *__restrict__ l2v_src, char **wb2_dst,
                                                            char *out2_even, char *out2_odd, int k,
                                                            const TableMeta *__restrict__ di_tm, u64 di_seed, float di_std,
                                                            const uint32_t *__restrict__ ins_key,
                                                            const uint32_t *__restrict__ byp_key, u64 *bytes_h2d,
                                                            u64 *bytes_d2h, const char *l2_lo, const char *l2_hi, int pauses,
                                                            const TableMeta *__restrict__ tm,
                                                            const int32_t *__restrict__ ins_slot,
                                                            const int32_t *__restrict__ ins_old,
                                                            const char *__restrict__ prev_ovf,
                                                            char *const *__restrict__ ins_dst,
                                                            char *const *__restrict__ l2v_dst,
                                                            const char *__restrict__ out2_prev) {
  transfer_rows<L>(st, cnt, ins_src, ins_tab, rb_of_table, ins_where, byp_src, byp_tab, byp_where, ovf, l2v_src, wb2_dst,
                   out2_even, out2_odd, k, di_tm, di_seed, di_std, ins_key, byp_key, bytes_h2d, bytes_d2h, l2_lo, l2_hi,
                   pauses);
  commit_rows<false, false, L>(tm, st, cnt, ins_tab, ins_where, ins_slot, ins_old, byp_tab, byp_where, ovf, nullptr, nullptr,
                               nullptr, nullptr, prev_ovf, kPrevKeep, k, ins_dst, l2v_src, l2v_dst, wb2_dst, out2_prev,
                               rb_of_table, ins_key, bytes_d2h);
  // The last workgroup through leaves the list of this batch's victims (every other one has read the old one's length).
  __syncthreads();
  if (threadIdx.x == 0 && atomicInc((unsigned int *)&st.wb_n[2], gridDim.x - 1) == gridDim.x - 1) {
    st.wb_n[0] = cnt->err ? 0 : cnt->n_ins;
    if (!cnt->err) st.wb_n[1] = k & 1;
  }
}

template <int L>
__global__ __launch_bounds__(256) void ovf_writeback_kernel(Staging st, const BatchCounters *cnt,
                                                            char *const *__restrict__ byp_src,
                                                            const int32_t *__restrict__ byp_tab,
                                                            const char *__restrict__ ovf,
                                                            const uint32_t *__restrict__ rb_of_table, u64 *bytes_d2h) {
  if (cnt->err) return;
  const int n_byp = cnt->n_byp;
  const int group = (blockIdx.x * blockDim.x + threadIdx.x) / L;
  const int lig = threadIdx.x % L;
  const int n_groups = gridDim.x * blockDim.x / L;
  u64 out_b = 0;
  for (int j = group; j < n_byp; j += n_groups) {
    const uint32_t rb = rb_of_table[byp_tab[j]];
    copy_row_to_host<L>(byp_src[j], ovf + (size_t)j * st.stride, rb, lig);
    if (lig == 0) out_b += rb;
  }
  for (int d = 32; d >= 1; d >>= 1) out_b += __shfl_xor(out_b, d);
  if ((threadIdx.x & 63) == 0 && out_b) atomicAdd(bytes_d2h, out_b);
}

// The overflow copies that batch b's commit parked behind its victims (those of the batch before it, but for the ones that b
// took over, which are not parked), written to the backing tier ahead of their turn: b has trained with no batch prefetched
// behind it, and a bypassed row of a batch that has trained goes home without waiting for a batch that may never come.  Their
// slots are emptied, so the next transfer passes them by.  How many they are stands in the list's length, which only
// transfers and commits change, each behind the one before and this kernel between them, whatever their streams; the counters of the batch before are not read, because by now its buffer may be in use again (two
// batches prefetched before the next forward) with nothing that orders its first kernel behind this one.
template <int L>
__global__ __launch_bounds__(256) void parked_copies_writeback_kernel(Staging st, const BatchCounters *cnt, u64 *bytes_d2h) {
  if (cnt->err) return;
  const int base = cnt->n_ins, n = st.wb_n[0] - base;
  const char *out = st.out[st.wb_n[1] & 1];
  const int group = (blockIdx.x * blockDim.x + threadIdx.x) / L;
  const int lig = threadIdx.x % L;
  const int n_groups = gridDim.x * blockDim.x / L;
  u64 out_b = 0;
  for (int j = group; j < n; j += n_groups) {
    const size_t slot = (size_t)base + (size_t)j;
    char *dst = st.wb_dst[slot];
    if (dst) {
      const uint32_t rb = st.wb_rb[slot];
      copy_row_to_host<L>(dst, out + slot * st.stride, rb, lig);
      if (lig == 0) out_b += rb;
    }
  }
  __syncthreads();  // every lane of a group has read its slot's destination
  for (int j = group; j < n; j += n_groups)
    if (lig == 0) st.wb_dst[(size_t)base + (size_t)j] = nullptr;
  for (int d = 32; d >= 1; d >>= 1) out_b += __shfl_xor(out_b, d);
  if ((threadIdx.x & 63) == 0 && out_b) atomicAdd(bytes_d2h, out_b);
}

hipError_t launch_ovf_writeback(const BatchBuf &b, int64_t parked, const Staging &st, const uint32_t *rb_of_table, u64 *bytes_d2h,
                                hipStream_t s) {
  if (parked)
    TBE_BY_ROW_LANES(st.stride, hipLaunchKernelGGL((parked_copies_writeback_kernel<L>), dim3(row_blocks(parked, L, 256, kLinkBlocks)), dim3(256), 0, s, st, b.cnt, bytes_d2h));
  if (b.n == 0) return hipGetLastError();
  TBE_BY_ROW_LANES(st.stride, hipLaunchKernelGGL((ovf_writeback_kernel<L>), dim3(row_blocks(b.n, L, 256, kLinkBlocks)), dim3(256), 0, s, st, b.cnt, b.byp_src, b.byp_tab, b.ovf,
                     rb_of_table, bytes_d2h));
  return hipGetLastError();
}

hipError_t launch_commit(const TableMeta *tm, const BatchBuf &b, const BatchBuf *prev, int prev_mode, const Staging &st,
                         const Level2 &l2, const uint32_t *rb_of_table, u64 *bytes_d2h, bool deep, hipStream_t s) {
  const int64_t rows = prev && prev->n > b.n ? prev->n : b.n;
  TBE_BY_ROW_LANES(st.stride, hipLaunchKernelGGL((deep ? commit_kernel<true, L> : commit_kernel<false, L>), dim3(row_blocks(rows, L, 256, 4096)), dim3(256), 0, s, tm, st, b.cnt, b.ins_tab, b.ins_where, b.ins_slot,
                     b.ins_old, b.byp_tab, b.byp_where, b.ovf, prev ? prev->cnt : nullptr,
                     prev ? prev->byp_src : nullptr, prev ? prev->byp_tab : nullptr,
                     prev ? prev->byp_taken : nullptr, prev ? prev->ovf : nullptr,
                     prev ? prev_mode : kPrevKeep, b.k, l2.on ? b.ins_dst : nullptr, l2.on ? b.l2v_src : nullptr,
                     l2.on ? b.l2v_dst : nullptr, l2.on ? l2.wb2_dst : nullptr, l2.out2[(b.k & 1) ^ 1], rb_of_table,
                     b.ins_key, bytes_d2h));
  return hipGetLastError();
}

hipError_t launch_swap(const TableMeta *tm, const BatchBuf &b, const BatchBuf *prev, int64_t parked, const Staging &st, const Level2 &l2,
                       const DeferredInit &di, const Throttle &th, const uint32_t *rb_of_table, u64 *bytes_h2d, u64 *bytes_d2h,
                       hipStream_t s) {
  const int64_t passes = std::max(b.n, (parked + 1) / 2);
  TBE_BY_ROW_LANES(st.stride, hipLaunchKernelGGL((swap_kernel<L>), dim3(row_blocks(passes, L, kSwapThreads, kSwapBlocks)), dim3(kSwapThreads), 0, s, st, b.cnt, b.ins_src, b.ins_tab, rb_of_table, b.ins_where, b.byp_src, b.byp_tab, b.byp_where, b.ovf,
                     l2.on ? b.l2v_src : nullptr, l2.on ? l2.wb2_dst : nullptr, l2.out2[0], l2.out2[1], b.k, di.tm, di.seed,
                     di.std, b.ins_key, b.byp_key, bytes_h2d, bytes_d2h, l2.lines_lo, l2.lines_hi, th.pauses, tm, b.ins_slot,
                     b.ins_old, prev ? prev->ovf : nullptr, l2.on ? b.ins_dst : nullptr, l2.on ? b.l2v_dst : nullptr,
                     l2.out2[(b.k & 1) ^ 1]));
  return hipGetLastError();
}

// flush: every valid line goes to the backing tier, its accumulator to those of all rows (which the host code copies)
template <int L>
__global__ __launch_bounds__(256) void flush_kernel(const TableMeta *__restrict__ tm, int T, int64_t total_slots,
                                                    const int32_t *__restrict__ tags, u64 *bytes_d2h) {
  const int64_t group = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / L;
  const int lig = threadIdx.x % L;
  const int64_t n_groups = (int64_t)gridDim.x * blockDim.x / L;
  u64 out_b = 0;
  for (int64_t slot = group; slot < total_slots; slot += n_groups) {
    const int32_t row = tags[slot];
    if (row < 0) continue;
    int lo = 0, hi = T - 1;  // table owning this slot: last t with slot_base <= slot
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if ((int64_t)tm[mid].slot_base <= slot) lo = mid; else hi = mid - 1;
    }
    const TableMeta &m = tm[lo];
    copy_row_to_host<L>(m.host_w + (size_t)row * m.row_bytes, m.lines + (size_t)(slot - m.slot_base) * m.row_bytes, m.row_bytes, lig);
    if (lig == 0) {
      out_b += m.row_bytes;
      m.dev_m[row] = m.slot_m[slot - m.slot_base];  // the caller copies dev_m to the host; the line stays valid
    }
  }
  for (int d = 32; d >= 1; d >>= 1) out_b += __shfl_xor(out_b, d);
  if ((threadIdx.x & 63) == 0 && out_b) atomicAdd(bytes_d2h, out_b);
}

// flush of the second level: every valid line goes to its row in the lower tier (host to
// host through the GPU); the levels are exclusive, so no row is written twice
template <int L>
__global__ __launch_bounds__(256) void flush2_kernel(const TableMeta *__restrict__ tm, int T, int64_t total_slots2,
                                                     const int32_t *__restrict__ tags2, u64 *bytes_h2d,
                                                     u64 *bytes_d2h) {
  const int64_t group = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / L;
  const int lig = threadIdx.x % L;
  const int64_t n_groups = (int64_t)gridDim.x * blockDim.x / L;
  u64 b = 0;
  for (int64_t slot = group; slot < total_slots2; slot += n_groups) {
    const int32_t row = tags2[slot];
    if (row < 0) continue;
    int lo = 0, hi = T - 1;  // table owning this slot: last t with slot2_base <= slot
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if ((int64_t)tm[mid].slot2_base <= slot) lo = mid; else hi = mid - 1;
    }
    const TableMeta &m = tm[lo];
    copy_row<L>(m.host_w + (size_t)row * m.row_bytes, m.lines2 + (size_t)(slot - m.slot2_base) * m.row_bytes, m.row_bytes, lig);
    if (lig == 0) b += m.row_bytes;
  }
  for (int d = 32; d >= 1; d >>= 1) b += __shfl_xor(b, d);
  if ((threadIdx.x & 63) == 0 && b) {
    atomicAdd(bytes_h2d, b);
    atomicAdd(bytes_d2h, b);
  }
}

hipError_t launch_flush(const TableMeta *tm, const Geometry &g, const int32_t *tags, const Level2 &l2, u64 *bytes_h2d,
                        u64 *bytes_d2h, hipStream_t s) {
  if (g.total_slots)
    TBE_BY_ROW_LANES(g.ovf_stride, hipLaunchKernelGGL((flush_kernel<L>), dim3(1024), dim3(256), 0, s, tm, g.T, g.total_slots, tags, bytes_d2h));
  if (l2.on && l2.total_slots2)
    TBE_BY_ROW_LANES(g.ovf_stride, hipLaunchKernelGGL((flush2_kernel<L>), dim3(kLinkBlocks), dim3(256), 0, s, tm, g.T, l2.total_slots2, l2.tags2, bytes_h2d,
                       bytes_d2h));
  return hipGetLastError();
}

// flush: accumulators of the small tables to the host, a table per grid row (the arrays are aligned to floats only), and the
// batch buffers' counters, in which the host looks for errors once it has waited for the flush
__global__ __launch_bounds__(256) void flush_state_kernel(const TableMeta *__restrict__ tm, int T, const uint32_t *counters,
                                                          uint32_t *host_counters, int counter_words) {
  if (blockIdx.x == 0 && blockIdx.y == 0)
    for (int i = threadIdx.x; i < counter_words; i += blockDim.x) __builtin_nontemporal_store(counters[i], host_counters + i);
  for (int t = blockIdx.y; t < T; t += gridDim.y) {
    const TableMeta &m = tm[t];
    if (!m.flush_by_kernel) continue;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m.rows; i += (int64_t)gridDim.x * blockDim.x)
      __builtin_nontemporal_store(m.dev_m[i], m.host_m + i);
  }
}

hipError_t launch_flush_state(const TableMeta *tm, const Geometry &g, const BatchCounters *counters, BatchCounters *host_counters,
                              int buffers, hipStream_t s) {
  static_assert(sizeof(BatchCounters) % 4 == 0, "copied word by word");
  hipLaunchKernelGGL(flush_state_kernel, dim3(32, g.T < 1024 ? g.T : 1024), dim3(256), 0, s, tm, g.T,
                     (const uint32_t *)counters, (uint32_t *)host_counters, (int)(buffers * sizeof(BatchCounters) / 4));
  return hipGetLastError();
}

}  // namespace tbe
