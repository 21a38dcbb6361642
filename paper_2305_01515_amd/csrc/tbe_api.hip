// C ABI of libtbe: handle life cycle, the batch pipeline over up to three streams (compute, prefetch,
// host link), observation calls.
// Declarations and the contract of every call are in include/tbe.h.
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <deque>
#include <mutex>
#include <vector>

#include "../../include/tbe.h"
#include "tbe_internal.h"

using namespace tbe;

// Scratch memory of tbe_backward_update_static: the partial sums of the backward's longest rows, for callers
// that must not allocate.  One copy per GPU, at an address of its own, held until the process ends.  In host
// code the array's name is only a handle for hipGetSymbolAddress; kernels are given the address it returns.
constexpr size_t kStaticScratchBytes = (size_t)TBE_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

thread_local std::string g_create_error;

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices] = {};  // device address of `scratch` on every GPU the library has been used on

// Address of the current device's copy of `scratch` (looked up once per device, with that device current).
hipError_t static_scratch_of_current_device(void **out, int *device) {
  *out = nullptr;
  hipError_t e = hipGetDevice(device);
  if (e != hipSuccess) return e;
  if (*device < 0 || *device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[*device]) {
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[*device] = p;
  }
  *out = g_scratch_ptr[*device];
  return hipSuccess;
}

struct DevAlloc {  // everything hipMalloc'ed, freed together
  std::vector<void *> ptrs;
  char *pool = nullptr;  // the rest of the block that small pieces are cut from (a small handle is sixty of them, and
  size_t left = 0;       // an allocation of its own for each was most of the time of tbe_create)
  template <class P>
  hipError_t get(P **p, size_t bytes) {
    constexpr size_t kBlock = 1 << 20, kSmall = 1 << 16;
    void *v = nullptr;
    bytes = bytes ? (bytes + 255) & ~(size_t)255 : 256;
    if (bytes <= kSmall) {
      if (left < bytes) {
        hipError_t e = hipMalloc(&v, kBlock);
        if (e != hipSuccess) { *p = nullptr; return e; }
        ptrs.push_back(v);
        pool = (char *)v;
        left = kBlock;
      }
      *p = (P *)pool;
      pool += bytes;
      left -= bytes;
      return hipSuccess;
    }
    hipError_t e = hipMalloc(&v, bytes);
    if (e == hipSuccess) ptrs.push_back(v);
    *p = e == hipSuccess ? (P *)v : nullptr;
    return e;
  }
  void release() {
    for (void *p : ptrs) (void)hipFree(p);
    ptrs.clear();
    pool = nullptr;
    left = 0;
  }
};

}  // namespace

// Batch buffers rotate over three: the buffer of batch k is still read after k has trained
// (its bypass list by the commit of batch k+1) while batch k+2 is already being prefetched.
// A pipeline D batches deep (tbe_set_prefetch_depth) rotates over 2 D + 1: the overflow copies of batch k are
// read before the forward of every batch up to k + D, and batch k + 2 D + 1 may be prefetched once batch k + D
// has trained.
constexpr int kBatchBufs = 3;

struct tbe_ctx {
  Geometry g{};
  std::vector<TableMeta> tm;  // host copy
  TableMeta *d_tm = nullptr;
  ClassInfo ci{};
  DevAlloc mem;
  int32_t *tags = nullptr, *ts = nullptr, *freq = nullptr;
  int policy = TBE_POLICY_LRU;
  int pooling = TBE_POOL_SUM;
  DeferredInit di;              // deferred initialisation on read (off unless enabled)
  Throttle throttle;            // emulated slower backing tier (off unless tbe_set_backing_throttle was called)
  uint32_t *init_bits = nullptr;
  size_t huge_slots = 0;        // (huge row, bag range) pairs a batch can have
  Level2 l2;                    // second-level cache (off unless tbe_enable_second_level was called)
  char *lines2 = nullptr;       // its lines: one pinned host allocation
  unsigned long long *d_l2tot = nullptr;  // running totals of the four second-level counters
  float *d_state = nullptr;   // row-wise Adagrad accumulators of all rows of all tables
  float *d_slot_m = nullptr;  // ... and of the rows in the cache lines, by slot
  float *partials = nullptr;  // segment sums of the backward's longest rows
  float *static_partials = nullptr;  // the same in the library's static scratch array on this handle's GPU
  int device = -1;                   // GPU the handle was created on
  char *lines = nullptr;
  BatchBuf buf[kMaxBatchBufs]{};
  int nbuf = kBatchBufs;        // batch buffers in use
  DeepBuf *d_deep = nullptr;    // deep pipeline: the batch buffers, for the look-up of rows whose backing-tier copy is stale
  int deep = 0;                 // 0: the one-deep pipeline; D >= 2: batches are fetched into the cache up to D ahead
  hipEvent_t ev_home[kMaxBatchBufs] = {};   // deep pipeline: the write-back of the buffer's bypassed rows
  bool home_recorded[kMaxBatchBufs] = {};
  SortScratch ss{};
  Staging st{};
  uint32_t *d_rb = nullptr;  // row bytes of every table
  int prev_buf = -1;         // buffer of the batch prefetched before the current one
  BatchCounters *counters = nullptr;      // of the batch buffers, one behind the other
  BatchCounters *host_counters = nullptr; // pinned host memory for a copy of them
  BatchCounters *d_total = nullptr;       // running totals of the per-batch counters
  unsigned long long *d_bytes = nullptr;  // [0] backing->cache, [1] cache->backing
  hipStream_t cs = nullptr, as = nullptr;  // compute / prefetch streams (caller's)
  hipStream_t ls = nullptr;                // host-link stream: transfer and commit (own, unless cs == as)
  bool own_ls = false;

  hipEvent_t ev_fwd = nullptr;  // the last forward launched ...
  int fwd_of = -1;              //   ... that recorded it: the batch's buffer
  int last_trained = -1;        // buffer of the batch whose backward recorded its event last
  bool unmarked = false;        // the compute stream has been given work of a batch since that left no event
  hipStream_t link_s = nullptr; // the stream that the last transfer went to, and what of the link comes behind it
  int64_t parked = 0;           // slots that the last commit parked for write-back, at most
  bool never_bypasses = true;   // every table has a way for each of its rows
  hipEvent_t ev_inputs = nullptr, ev_ready[kMaxBatchBufs] = {}, ev_trained[kMaxBatchBufs] = {}, ev_probed[kMaxBatchBufs] = {};
  int64_t flush_state_bytes = 0;
  bool inputs_ready = false;  // caller guarantees index / offset buffers are complete when tbe_prefetch is called
  int32_t max_batch = 0;
  int64_t max_lookups = 0;
  int32_t k = 0;
  // pipeline: buffers prefetched and waiting for forward (oldest first), the buffer that
  // was forwarded and waits for its update, and a buffer whose copies wait for that update
  int pend[kMaxBatchBufs] = {-1, -1};
  // batches accepted by tbe_prefetch further ahead than the pipeline runs: their work is issued, in order, as
  // soon as the batch before has been forwarded
  struct Queued { const int64_t *d_indices, *d_offsets; int32_t batch; int64_t n; };
  std::deque<Queued> queued;
  int depth = 1;                // batches tbe_prefetch accepts ahead of training (those beyond the next one are queued)
  int n_pend = 0;
  int current = -1;
  int deferred = -1;
  int last_buf = -1;
  int64_t total_lookups = 0;
  int sticky = 0;
  std::string err;
  // optional stage timing: (start, stop) event pairs per stage, in call order
  int profiling = 0;  // 0 off, 1 every bracket, 2 the whole-stage brackets only
  std::vector<std::pair<hipEvent_t, hipEvent_t>> prof[TBE_NUM_STAGES];
};

namespace {

int fail(tbe_ctx *h, int code, const std::string &msg) {
  if (h) h->err = msg; else g_create_error = msg;
  return code;
}

int hipfail(tbe_ctx *h, hipError_t e, const char *what) {
  (void)hipGetLastError();  // HIP keeps the error until it is read: the next launch check must not report it again
  return fail(h, e == hipErrorOutOfMemory ? TBE_ENOMEM : TBE_EHIP, std::string(what) + ": " + hipGetErrorString(e));
}

#define HIP_TRY(h, call)                                  \
  do {                                                    \
    hipError_t e__ = (call);                              \
    if (e__ != hipSuccess) return hipfail(h, e__, #call); \
  } while (0)

constexpr size_t kMaxProfiledCalls = 16384;

// Brackets the launches of one stage with timing events on the stream they go to.
struct StageTimer {
  tbe_ctx *h;
  hipStream_t s;
  hipEvent_t stop = nullptr;
  StageTimer(tbe_ctx *h_, int stage, hipStream_t s_) : h(h_), s(s_) {
    const bool inner = stage == TBE_STAGE_BACKWARD_HEAVY || stage == TBE_STAGE_BACKWARD_COMBINE ||
                       stage == TBE_STAGE_BACKWARD_SINGLE || stage == TBE_STAGE_BACKWARD_SHORT;
    if (!h->profiling || (inner && h->profiling == 2) || h->prof[stage].size() >= kMaxProfiledCalls) return;
    hipEvent_t a = nullptr, b = nullptr;
    if (hipEventCreate(&a) != hipSuccess || hipEventCreate(&b) != hipSuccess) { if (a) (void)hipEventDestroy(a); return; }
    (void)hipEventRecord(a, s);
    h->prof[stage].emplace_back(a, b);
    stop = b;
  }
  ~StageTimer() { if (stop) (void)hipEventRecord(stop, s); }
};

void drop_profile(tbe_ctx *h) {
  for (auto &v : h->prof) {
    for (auto &p : v) { (void)hipEventDestroy(p.first); (void)hipEventDestroy(p.second); }
    v.clear();
  }
}

int next_pow2(int v) { int p = 1; while (p < v) p <<= 1; return p; }

// Can a kernel write to these `bytes` of host memory at the address the host uses?  (Pinned memory: yes.  Pageable memory,
// and memory that was registered and mapped at another address: no.)
bool kernels_reach(const void *p, size_t bytes) {
  for (const char *q : {(const char *)p, (const char *)p + bytes - 1}) {
    hipPointerAttribute_t a{};
    const hipError_t e = hipPointerGetAttributes(&a, q);
    (void)hipGetLastError();  // (an error, for pageable memory, on some versions)
    if (e != hipSuccess || a.type != hipMemoryTypeHost || a.devicePointer != (const void *)q) return false;
  }
  return true;
}

__global__ void stream_pin_kernel() {}

int alloc_batchbuf(tbe_ctx *h, BatchBuf &b, int64_t n) {
  const size_t N = (size_t)std::max<int64_t>(n, 1);
  HIP_TRY(h, h->mem.get(&b.loc, 4 * N));
  HIP_TRY(h, h->mem.get(&b.sorted_bag, 4 * N));
  HIP_TRY(h, h->mem.get(&b.bag_of_pos, 4 * N));
  HIP_TRY(h, h->mem.get(&b.inv_len, 4 * (size_t)h->g.T * (size_t)h->max_batch));
  HIP_TRY(h, h->mem.get(&b.uid_sorted, 4 * N));
  HIP_TRY(h, h->mem.get(&b.uniq_key, 4 * N));
  HIP_TRY(h, h->mem.get(&b.run_off, 4 * (N + 1)));
  HIP_TRY(h, h->mem.get(&b.uniq_tab, 4 * N));
  HIP_TRY(h, h->mem.get(&b.loc_u, 4 * N));
  HIP_TRY(h, h->mem.get(&b.status, N));
  HIP_TRY(h, h->mem.get(&b.old_tag, 4 * N));
  HIP_TRY(h, h->mem.get(&b.touched, 8 * N));
  HIP_TRY(h, h->mem.get(&b.ins_idx, 4 * N));
  HIP_TRY(h, h->mem.get(&b.ins_tab, 4 * N));
  HIP_TRY(h, h->mem.get(&b.ins_slot, 4 * N));
  HIP_TRY(h, h->mem.get(&b.ins_old, 4 * N));
  HIP_TRY(h, h->mem.get(&b.ins_key, 4 * N));
  HIP_TRY(h, h->mem.get(&b.vic_key, 4 * N));
  HIP_TRY(h, h->mem.get(&b.ins_src, 8 * N));
  HIP_TRY(h, h->mem.get(&b.ins_where, 4 * N));
  HIP_TRY(h, h->mem.get(&b.byp_idx, 4 * N));
  HIP_TRY(h, h->mem.get(&b.byp_tab, 4 * N));
  HIP_TRY(h, h->mem.get(&b.byp_key, 4 * N));
  HIP_TRY(h, h->mem.get(&b.byp_src, 8 * N));
  HIP_TRY(h, h->mem.get(&b.byp_where, 4 * N));
  HIP_TRY(h, h->mem.get(&b.byp_taken, N));
  HIP_TRY(h, h->mem.get(&b.ovf, N * (size_t)h->g.ovf_stride));
  HIP_TRY(h, h->mem.get(&b.mid_idx, 4 * (N / 2 + 1)));
  HIP_TRY(h, h->mem.get(&b.heavy, 4 * (N / 32 + 1)));  // entries: N / 65 at most (a row of len > 64 has ceil(len / 256) at most, no more than len / 65)
  HIP_TRY(h, h->mem.get(&b.heavy_sub, 4 * (N / 32 + 1)));
  HIP_TRY(h, h->mem.get(&b.harrive, 4 * (N / 32 + 1)));
  HIP_TRY(h, hipMemset(b.harrive, 0, 4 * (N / 32 + 1)));
  HIP_TRY(h, h->mem.get(&b.hchunks, 16 * (N / 32 + (size_t)h->g.T + 1)));
  HIP_TRY(h, h->mem.get(&b.hfirst, 4 * ((size_t)h->g.T + 1)));
  HIP_TRY(h, h->mem.get(&b.hperm, 4 * (N / 32 + 1)));
  HIP_TRY(h, h->mem.get(&b.hstart, 4 * (h->huge_slots + 1)));
  b.cnt = h->counters + (&b - h->buf);
  return TBE_OK;
}

// What max pooling needs beside that: who supplied each maximum, by element and by lookup, and the lookups' positions by
// sorted order.  Whatever of it the buffer does not have yet: the mode and the prefetch depth, which adds buffers, can be set
// in any order and more than once, and an allocation that failed can be tried again.
int alloc_max_records(tbe_ctx *h, BatchBuf &b) {
  const size_t N = (size_t)std::max<int64_t>(h->max_lookups, 1);
  if (!b.argpos) HIP_TRY(h, h->mem.get(&b.argpos, 4 * (size_t)h->max_batch * (size_t)h->g.sum_dim));
  // One array for all buffers: the forward writes it, the update of the same batch reads it, both on the compute stream, and no
  // other batch is forwarded in between.  It lies in the partial sums' memory, which this mode does not use: with an array of
  // its own in every buffer a handle took up to 192 bytes more per lookup than before there were such records.
  b.wins = (uint8_t *)h->partials;
  if (!b.sorted_at) HIP_TRY(h, h->mem.get(&b.sorted_at, 4 * N));
  return TBE_OK;
}

int device_error_code(int e) { return e == 0 ? 0 : (e & ~kRefusedBefore) == 1 ? TBE_EINVAL : TBE_ERANGE; }

// After a synchronisation: pick up errors the device recorded (`all`: the batch buffers' counters as they are now).
int take_device_errors(tbe_ctx *h, const BatchCounters *all) {
  for (int i = 0; i < h->nbuf; i++) {
    const BatchCounters &c = all[i];
    if (c.err && !h->sticky) {
      h->sticky = device_error_code(c.err);
      h->err = h->sticky == TBE_EINVAL ? "offsets are not a non-decreasing partition of [0, num_lookups]"
                          : "an index is outside its table";
    }
  }
  return h->sticky;
}

int collect_device_errors(tbe_ctx *h) {
  BatchCounters all[kMaxBatchBufs];
  HIP_TRY(h, hipMemcpy(all, h->counters, sizeof(BatchCounters) * (size_t)h->nbuf, hipMemcpyDeviceToHost));
  return take_device_errors(h, all);
}

int sync_all(tbe_ctx *h) {
  HIP_TRY(h, hipStreamSynchronize(h->as));
  HIP_TRY(h, hipStreamSynchronize(h->ls));
  HIP_TRY(h, hipStreamSynchronize(h->cs));
  return TBE_OK;
}

// Stream `to` goes on behind what `from` has been given so far.
int order_after(tbe_ctx *h, hipStream_t from, hipStream_t to) {
  HIP_TRY(h, hipEventRecord(h->ev_inputs, from));
  HIP_TRY(h, hipStreamWaitEvent(to, h->ev_inputs, 0));
  return TBE_OK;
}

// The transfer of batch `b`, whose stage stream `s` has been given, on b.link.  Write-back of the previous batch's victims and
// fetch-ahead of this batch's rows share the host link; neither touches a cache line, so a batch in flight is not disturbed.
// `swap`: its commit in the same launch (enqueue_commit then has nothing to launch).
int enqueue_transfer(tbe_ctx *h, const BatchBuf &b, int bi, hipStream_t s, bool swap = false) {
  if (b.link != s) {  // (covers the transfers that `s` has had)
    HIP_TRY(h, hipEventRecord(h->ev_probed[bi], s));
    HIP_TRY(h, hipStreamWaitEvent(b.link, h->ev_probed[bi], 0));
  } else if (s == h->as && h->link_s == h->ls && h->ls != s) {
    const int rc = order_after(h, h->ls, s);
    if (rc) return rc;
  }
  h->link_s = b.link;
  if (swap) {
    HIP_TRY(h, launch_swap(h->d_tm, b, b.prev_bi >= 0 ? &h->buf[b.prev_bi] : nullptr, h->parked, h->st, h->l2, h->di, h->throttle,
                           h->d_rb, h->d_bytes, h->d_bytes + 1, b.link));
    return TBE_OK;
  }
  StageTimer tm_(h, TBE_STAGE_FILL, b.link);
  HIP_TRY(h, launch_transfer(&b, h->parked, h->st, h->l2, h->di, h->throttle, b.k, h->d_rb, h->d_bytes, h->d_bytes + 1, b.link));
  return TBE_OK;
}

// Victims of batch `bi` to the staging area, its new rows into the cache lines; then the
// batch is ready for forward.  Must follow the update of the batch before it.
int enqueue_commit(tbe_ctx *h, int bi, bool wb_prev, bool swapped = false) {
  BatchBuf &b = h->buf[bi];
  const int64_t prev_n = b.prev_bi >= 0 ? h->buf[b.prev_bi].n : 0;
  if (!swapped) {
    StageTimer tm_(h, TBE_STAGE_COMMIT, b.link);
    const int prev_mode = !wb_prev ? kPrevKeep : b.parks_prev ? kPrevPark : kPrevWrite;
    HIP_TRY(h, launch_commit(h->d_tm, b, b.prev_bi >= 0 ? &h->buf[b.prev_bi] : nullptr, prev_mode, h->st, h->l2, h->d_rb,
                             h->d_bytes + 1, false, b.link));
  }
  h->parked = b.n + (prev_n > 0 ? prev_n : 0);
  if (b.link != h->cs) HIP_TRY(h, hipEventRecord(h->ev_ready[bi], b.link));
  return TBE_OK;
}

// What batch `b` (buffer bi) finds of the rows whose backing-tier copy is stale.
StaleRows stale_rows(const tbe_ctx *h, const BatchBuf &b, int bi) {
  StaleRows r{};
  r.where = h->st.where;
  r.max_inserts = (uint32_t)h->st.max_inserts;
  r.own_code = kWhereOverflow | (h->deep ? (uint32_t)bi << kWhereBufShift : 0u);
  r.wb_skip = h->st.wb_skip[(b.k - 1) & 1];
  if (h->prev_buf < 0) return r;
  const BatchBuf &prev = h->buf[h->prev_buf];
  r.prev_cnt = prev.cnt;
  r.prev_vic_key = prev.vic_key;
  r.prev_byp_key = prev.byp_key;
  r.prev_byp_taken = prev.byp_taken;
  if (h->l2.on) {
    r.prev_l2v_src = prev.l2v_src;
    r.prev_l2v_key = prev.l2v_key;
  }
  if (prev.parks_prev && prev.prev_bi >= 0) {
    r.pp_cnt = h->buf[prev.prev_bi].cnt;
    r.pp_byp_key = h->buf[prev.prev_bi].byp_key;
  }
  if (h->deep) {
    r.deep = h->d_deep;
    for (int i = 0; i < h->n_pend; i++) r.live |= 1u << h->pend[i];
    if (h->current >= 0) r.live |= 1u << h->current;
  }
  return r;
}

// The prefetch stage of batch `b` (buffer bi).
hipError_t launch_stage(tbe_ctx *h, const BatchBuf &b, int bi, hipStream_t s) {
  const bool lfu = h->policy == TBE_POLICY_LFU;
  const StaleRows stale = stale_rows(h, b, bi);
  const Totals totals{h->d_total, h->d_bytes + 2, h->l2.on ? h->d_l2tot : nullptr, h->l2.sums};
  if (one_kernel_batch(h->g, h->l2.on, h->as == h->cs, b.n, b.batch))
    return launch_one_kernel_stage(h->d_tm, h->g, b, h->ss, h->tags, h->ts, h->freq, lfu, h->l2, h->deep, stale, totals, s);
  hipError_t e = launch_keygen(h->d_tm, h->g, b, h->ss, s);
  int res = 0;
  if (e == hipSuccess) e = launch_sort(h->d_tm, h->g, b, h->ss, &res, s);
  if (e != hipSuccess) return e;
  return launch_dedup_probe(h->d_tm, h->g, b, h->ss, h->ss.pairs[res], h->tags, h->ts, h->freq, lfu, h->l2,
                            h->deep, stale, totals, s);
}

// Pipeline several batches deep: the rows of `b` whose value was an overflow copy of a batch that had not trained when `b` was
// fetched are copied from there.
hipError_t fix_up(tbe_ctx *h, const BatchBuf &b) {
  OverflowCopies oc{};
  for (int x = 0; x < h->nbuf; x++) oc.of_buf[x] = h->buf[x].ovf;
  return launch_fixup(h->d_tm, b, oc, h->st, h->d_rb, h->d_bytes + 6, h->cs);
}

// The stream for the transfer and the commit of a batch that is prefetched beside training.  The link's own lets them run beside
// the next batch's stage; a few rows follow the stage on its stream.
hipStream_t link_stream(const tbe_ctx *h, int32_t batch, int64_t n) {
  return h->as != h->cs && link_with_stage(h->g, h->l2.on, n, batch) ? h->as : h->ls;
}

// The prefetch stream behind training.  The prefetch stage only decides on tags and timestamps, which training never reads;
// it follows all the same what the compute stream has been given so far, because the index buffers may have been produced
// there, or, if they are complete, the last forward or update.
// Training launched so far goes first: its kernels and this stage are all bound by HBM and slow each
// other down when they overlap, the model waits for training, and this stage has the whole transfer of
// the batch before it to finish in.  (Benchmark workload, this stage behind the last forward only, i.e.
// beside the backward: forward 0.27 ms, backward 0.78 ms, this stage 1.5 ms per step; behind both: see
// the design notes.  The step is bound by the host link either way.)
// The last of them on the compute stream is the forward of the batch in training, or the last update.
// A small batch's stage takes next to nothing of the memory system and its time is not hidden by a transfer: beside training it
// follows only what it needs, the commit of the batch in training or of the one that trained last.  That covers the readers of
// the buffer that it is about to put to use (three batches old, see do_prefetch) and the transfer that looked last at the skip
// flags it sets (those of the victims of two batches before it).
int prefetch_behind_training(tbe_ctx *h, bool small) {
  const bool marked = h->current >= 0 ? h->fwd_of == h->current : !h->unmarked;
  if (!h->inputs_ready || !marked) {
    h->unmarked = false;
    return order_after(h, h->cs, h->as);
  }
  const int beside = h->current >= 0 ? h->current : h->n_pend > 0 ? h->last_trained : -1;
  if (small && beside >= 0 && h->buf[beside].link != h->cs) HIP_TRY(h, hipStreamWaitEvent(h->as, h->ev_ready[beside], 0));
  else if (h->current >= 0) HIP_TRY(h, hipStreamWaitEvent(h->as, h->ev_fwd, 0));
  else if (h->last_trained >= 0) HIP_TRY(h, hipStreamWaitEvent(h->as, h->ev_trained[h->last_trained], 0));
  return TBE_OK;
}

// Pipeline several batches deep (Section 5.7): the batch is fetched into the cache as soon as it is decided on.
// The ways of the batches that may still wait for their training are locked (ts >= k - D), so its victims and
// the lines it fills are used by none of them and nothing waits for a backward -- except the rows whose current
// value is an overflow copy of such a batch: they are copied before this batch's forward (launch_fixup).
int do_prefetch_deep(tbe_ctx *h, const int64_t *d_indices, const int64_t *d_offsets, int32_t batch, int64_t n) {
  if (h->n_pend + (h->current >= 0 ? 1 : 0) > h->deep)
    return fail(h, TBE_EORDER, "prefetch: more batches would be ahead of training than the prefetch depth");
  const int bi = h->k % h->nbuf;
  BatchBuf &b = h->buf[bi];
  b.d_indices = d_indices; b.d_offsets = d_offsets; b.batch = batch; b.n = n; b.k = ++h->k;
  b.mean = h->pooling == TBE_POOL_MEAN;
  b.maxp = h->pooling == TBE_POOL_MAX;
  b.parks_prev = false;
  h->total_lookups += n;
  h->last_buf = bi;
  b.link = link_stream(h, batch, n);
  if (h->as != h->cs) {
    // the buffer last served batch k - (2 D + 1): every batch that read its overflow copies (up to k - D - 1) has
    // trained, and its bypassed rows have been written back
    int rc = prefetch_behind_training(h, false);
    if (rc) return rc;
    if (h->home_recorded[bi]) HIP_TRY(h, hipStreamWaitEvent(h->as, h->ev_home[bi], 0));
  }
  {
    StageTimer tm_(h, TBE_STAGE_PREFETCH, h->as);
    HIP_TRY(h, launch_stage(h, b, bi, h->as));
  }
  int rc = enqueue_transfer(h, b, bi, h->as);
  if (rc) return rc;
  b.prev_bi = h->prev_buf;
  h->prev_buf = bi;
  h->pend[h->n_pend++] = bi;
  {
    // the prefetch stream has waited for every backward launched so far, and the link stream for it, which covers the
    // batches whose lines this commit may overwrite: they were stamped before k - D
    StageTimer tm_(h, TBE_STAGE_COMMIT, b.link);
    HIP_TRY(h, launch_commit(h->d_tm, b, nullptr, kPrevKeep, h->st, h->l2, h->d_rb, h->d_bytes + 1, true, b.link));
  }
  h->parked = b.n;
  if (b.link != h->cs) HIP_TRY(h, hipEventRecord(h->ev_ready[bi], b.link));
  return TBE_OK;
}

// What the host can say about a batch.  (Lookups of no bag are bad offsets like others -- one offset cannot be 0 and n -- but
// the kernel that checks offsets does so bag by bag, so it would never see these.)
int check_batch(tbe_ctx *h, const int64_t *d_indices, const int64_t *d_offsets, int32_t batch, int64_t n) {
  if (!d_offsets || batch < 0 || n < 0 || (n > 0 && (!d_indices || batch == 0))) return fail(h, TBE_EINVAL, "prefetch: bad argument");
  if (batch > h->max_batch || n > h->max_lookups) return fail(h, TBE_ELIMIT, "prefetch: batch or lookups above the sizes given to tbe_create");
  // (a table's bags are one launch of the forward, a lane group each, and a launch holds fewer than 2^32 threads)
  if ((int64_t)batch * h->g.win_stride > (1ll << 32) - 256) return fail(h, TBE_ELIMIT, "prefetch: batch times the widest row's lanes reaches 2^32");
  return TBE_OK;
}

// own: a forward prefetches its batch itself.  With no other batch in flight nothing of the library's runs beside such a prefetch.
int do_prefetch(tbe_ctx *h, const int64_t *d_indices, const int64_t *d_offsets, int32_t batch, int64_t n, bool own = false) {
  int rc = check_batch(h, d_indices, d_offsets, batch, n);
  if (rc) return rc;
  if (h->deep) return do_prefetch_deep(h, d_indices, d_offsets, batch, n);
  if (h->n_pend + (h->current >= 0 ? 1 : 0) > 1) return fail(h, TBE_EORDER, "prefetch: more than one batch would be ahead of training");
  const int bi = h->k % kBatchBufs;  // free: at most the batch before this one is still in use
  BatchBuf &b = h->buf[bi];
  const bool in_flight = h->n_pend > 0 || h->current >= 0;
  b.d_indices = d_indices; b.d_offsets = d_offsets; b.batch = batch; b.n = n; b.k = ++h->k;
  b.mean = h->pooling == TBE_POOL_MEAN;
  b.maxp = h->pooling == TBE_POOL_MAX;
  // A batch prefetched while its predecessor is still in flight is committed right after that one's
  // update, and its commit then parks the predecessor's overflow copies for the next transfer.
  b.parks_prev = in_flight && h->prev_buf >= 0 && h->st.max_parked > 0 && !h->l2.on;
  h->total_lookups += n;
  h->last_buf = bi;
  own = own && !in_flight && on_compute_stream(h->g, h->inputs_ready, h->never_bypasses, n);
  hipStream_t stage_s = own ? h->cs : h->as;
  b.link = own ? h->cs : link_stream(h, batch, n);
  if (own && h->link_s != h->cs) {  // (all but the write-back behind the last update the forwards have waited for)
    rc = order_after(h, h->link_s, h->cs);
    if (rc) return rc;
  }
  if (stage_s != h->cs) {
    rc = prefetch_behind_training(h, small_batch(h->g, n, batch));
    if (rc) return rc;
    // This buffer (k - 3's, for batch k) is read by that batch's own kernels, by the list passes of k - 2 and k - 1 (this stream),
    // by the commit of batch k - 2 -- its bypass list, overflow copies and counters -- and, if batch k - 3 had no successor
    // when it had trained, by its write-back on the link stream, which that commit follows.  At most the batch before this
    // one is still in flight, so batch k - 2 has trained, behind its commit: what was waited for above covers them all.  (The
    // write-back of copies that commit(k - 2) parked runs behind the update of k - 2 and so is not covered: it reads nothing
    // of this buffer.)  (Each with a wait of its own, and both of the waits above: mean pooling, ragged, four steps 687
    // instead of 638 us, 8 x 500k rows under max pooling 1049 instead of 1028.)
  }
  {
    StageTimer tm_(h, TBE_STAGE_PREFETCH, stage_s);
    HIP_TRY(h, launch_stage(h, b, bi, stage_s));
  }
  b.prev_bi = h->prev_buf;
  const bool swap = !in_flight && !h->profiling && n <= kSwapLookups;
  rc = enqueue_transfer(h, b, bi, stage_s, swap);
  if (rc) return rc;
  h->prev_buf = bi;
  h->pend[h->n_pend++] = bi;
  if (in_flight) {
    h->deferred = bi;  // its cache lines may still be in use: commit after that batch's update
    return TBE_OK;
  }
  return enqueue_commit(h, bi, false, swap);
}

}  // namespace

extern "C" {

const char *tbe_last_error(tbe_handle h) { return h ? h->err.c_str() : g_create_error.c_str(); }

int tbe_host_alloc(void **h_ptr, size_t bytes) {
  if (!h_ptr) return TBE_EINVAL;
  hipError_t e = hipHostMalloc(h_ptr, bytes ? bytes : 16, hipHostMallocDefault);
  if (e != hipSuccess) { *h_ptr = nullptr; (void)hipGetLastError(); return TBE_ENOMEM; }
  return TBE_OK;
}

int tbe_host_free(void *h_ptr) { return hipHostFree(h_ptr) == hipSuccess ? TBE_OK : TBE_EHIP; }

int tbe_destroy(tbe_handle h) {
  if (!h) return TBE_EINVAL;
  (void)hipStreamSynchronize(h->as);
  (void)hipStreamSynchronize(h->ls);
  (void)hipStreamSynchronize(h->cs);
  if (h->own_ls) (void)hipStreamDestroy(h->ls);
  h->mem.release();
  if (h->lines2) (void)hipHostFree(h->lines2);
  if (h->host_counters) (void)hipHostFree(h->host_counters);
  drop_profile(h);
  if (h->ev_inputs) (void)hipEventDestroy(h->ev_inputs);
  if (h->ev_fwd) (void)hipEventDestroy(h->ev_fwd);
  for (int i = 0; i < kMaxBatchBufs; i++) {
    if (h->ev_ready[i]) (void)hipEventDestroy(h->ev_ready[i]);
    if (h->ev_trained[i]) (void)hipEventDestroy(h->ev_trained[i]);
    if (h->ev_probed[i]) (void)hipEventDestroy(h->ev_probed[i]);
    if (h->ev_home[i]) (void)hipEventDestroy(h->ev_home[i]);
  }
  delete h;
  return TBE_OK;
}

int tbe_create(tbe_handle *out, const tbe_table_spec *specs, int32_t num_tables, int32_t ways, int32_t max_batch,
               int64_t max_lookups, void *compute_stream, void *aux_stream) {
  if (!out) return fail(nullptr, TBE_EINVAL, "create: null output handle");
  *out = nullptr;
  if (!specs || num_tables <= 0) return fail(nullptr, TBE_EINVAL, "create: no tables");
  if (ways < 1 || ways > kWave) return fail(nullptr, TBE_EINVAL, "create: ways must be 1..64");
  if (max_batch < 1 || max_lookups < 1 || max_lookups > (1ll << 30))
    return fail(nullptr, TBE_EINVAL, "create: max_batch >= 1 and 1 <= max_lookups <= 2^30 required");
  if ((int64_t)num_tables * max_batch >= (1ll << 31)) return fail(nullptr, TBE_ELIMIT, "create: tables x batch too large");
  tbe_ctx *h = new (std::nothrow) tbe_ctx();
  if (!h) return fail(nullptr, TBE_ENOMEM, "create: host allocation failed");
  h->cs = (hipStream_t)compute_stream;
  h->as = (hipStream_t)aux_stream;
  h->ls = h->cs;
  h->link_s = h->cs;
  h->max_batch = max_batch;
  h->max_lookups = max_lookups;
  h->g.T = num_tables;
  h->g.ways = ways;
  h->tm.resize(num_tables);
  uint64_t key = 0, sets = 0;
  int64_t col = 0;
  size_t line_bytes = 0;
  std::vector<size_t> line_off(num_tables);
  std::vector<int> tclass(num_tables);
  for (int t = 0; t < num_tables; t++) {
    const tbe_table_spec &s = specs[t];
    TableMeta &m = h->tm[t];
    const int epl = s.dtype == TBE_FP32 ? 4 : 8;
    if ((s.dtype != TBE_FP32 && s.dtype != TBE_FP16) || s.rows < 1 || s.rows >= (1ll << 31) || s.dim < epl ||
        s.dim % epl || s.dim > 64 * epl || !s.host_weights || !s.host_state || s.cache_slots < 0) {
      delete h;
      return fail(nullptr, TBE_EINVAL, "create: bad table spec " + std::to_string(t));
    }
    m.rows = s.rows;
    m.dim = s.dim;
    m.dtype = s.dtype;
    m.row_bytes = (uint32_t)(s.dim * (s.dtype == TBE_FP32 ? 4 : 2));
    m.lanes = next_pow2(s.dim / epl);
    m.col = (int32_t)col;
    m.sets = (uint32_t)std::min<int64_t>(s.cache_slots / ways, (1ll << 31) / ways);
    m.rows_per_set = m.sets ? (uint32_t)((s.rows + m.sets - 1) / m.sets) : 0;
    m.rps_magic = div_magic(m.rows_per_set);
    m.sets_magic = div_magic(m.sets);
    m.key_base = (uint32_t)key;
    m.set_base = (uint32_t)sets;
    m.slot_base = (int32_t)(sets * ways);
    m.host_w = (char *)s.host_weights;
    m.host_m = s.host_state;
    key += m.sets ? (uint64_t)m.sets * m.rows_per_set : (uint64_t)s.rows;
    sets += m.sets;
    col += s.dim;
    line_off[t] = line_bytes;
    line_bytes += ((size_t)m.sets * ways * m.row_bytes + 255) & ~(size_t)255;
    if (m.sets == 0 || m.rows_per_set > (uint32_t)ways) h->never_bypasses = false;
    if (key > (1ull << 32) || sets * ways >= (1ull << 30) || col >= (1ll << 30)) {
      delete h;
      return fail(nullptr, TBE_ELIMIT, "create: key space, slot count or output width too large");
    }
    // class of the table
    int c = 0;
    for (; c < h->ci.n_classes; c++)
      if (h->ci.cls_dtype[c] == m.dtype && h->ci.cls_lanes[c] == m.lanes) break;
    if (c == h->ci.n_classes) {
      h->ci.cls_dtype[c] = m.dtype;
      h->ci.cls_lanes[c] = m.lanes;
      h->ci.cls_count[c] = 0;
      h->ci.n_classes++;
    }
    h->ci.cls_count[c]++;
    tclass[t] = c;
  }
  h->g.sum_dim = (int32_t)col;
  h->g.total_sets = (uint32_t)sets;
  h->g.total_slots = (int64_t)sets * ways;
  h->g.ovf_stride = 16;
  h->g.win_stride = 1;
  for (const TableMeta &m : h->tm) h->g.dtypes |= m.dtype == TBE_FP32 ? 1 : 2;
  for (const TableMeta &m : h->tm) h->g.win_stride = std::max(h->g.win_stride, m.lanes);
  for (const TableMeta &m : h->tm) h->g.ovf_stride = std::max(h->g.ovf_stride, m.row_bytes);
  h->g.key_bits = h->g.seg_bits = 1;
  for (const TableMeta &m : h->tm) {
    const uint64_t span = m.sets ? (uint64_t)m.sets * m.rows_per_set : (uint64_t)m.rows;
    while (h->g.seg_bits < 32 && (1ull << h->g.seg_bits) < span) h->g.seg_bits++;
  }
  while (h->g.key_bits < 32 && (1ull << h->g.key_bits) < key) h->g.key_bits++;
  {  // sort payload (bag, position inside the bag) when both fit 32 bits
    int bag_bits = 0;
    while ((1ll << bag_bits) < (int64_t)num_tables * max_batch) bag_bits++;
    h->g.within_bits = std::min(24, 32 - bag_bits);
    if (h->g.within_bits < 1) h->g.within_bits = 0;
  }

  auto bail = [&](int code) { tbe_destroy(h); return code; };
  auto hipbail = [&](hipError_t e, const char *what) {
    int code = hipfail(nullptr, e, what);
    tbe_destroy(h);
    return code;
  };
#define CREATE_TRY(call)                                  \
  do {                                                    \
    hipError_t e__ = (call);                              \
    if (e__ != hipSuccess) return hipbail(e__, #call);    \
  } while (0)

  const size_t slots = (size_t)h->g.total_slots;
  CREATE_TRY(h->mem.get(&h->lines, line_bytes));
  CREATE_TRY(h->mem.get(&h->tags, 4 * slots));
  CREATE_TRY(h->mem.get(&h->ts, 4 * slots));
  CREATE_TRY(h->mem.get(&h->freq, 4 * slots));
  if (slots) {
    CREATE_TRY(hipMemset(h->tags, 0xFF, 4 * slots));  // -1 = free
    CREATE_TRY(hipMemset(h->ts, 0xFF, 4 * slots));
    CREATE_TRY(hipMemset(h->freq, 0, 4 * slots));
  }
  {  // accumulators of all rows live in HBM; the host arrays give their initial values
    size_t total_rows = 0;
    for (int t = 0; t < num_tables; t++) total_rows += (size_t)h->tm[t].rows;
    CREATE_TRY(h->mem.get(&h->d_state, 4 * total_rows));
    size_t off = 0;
    for (int t = 0; t < num_tables; t++) {
      h->tm[t].dev_m = h->d_state + off;
      CREATE_TRY(hipMemcpy(h->tm[t].dev_m, h->tm[t].host_m, 4 * (size_t)h->tm[t].rows, hipMemcpyHostToDevice));
      off += (size_t)h->tm[t].rows;
    }
  }
  if (h->as != h->cs) {
    CREATE_TRY(hipStreamCreateWithFlags(&h->ls, hipStreamNonBlocking));
    h->own_ls = true;
  }
  CREATE_TRY(h->mem.get(&h->d_slot_m, 4 * slots));
  if (slots) CREATE_TRY(hipMemset(h->d_slot_m, 0, 4 * slots));
  for (int t = 0; t < num_tables; t++) {
    h->tm[t].lines = h->lines + line_off[t];
    h->tm[t].slot_m = h->d_slot_m + h->tm[t].slot_base;
    h->tm[t].flush_by_kernel = h->tm[t].rows <= kFlushStateRows && kernels_reach(h->tm[t].host_m, 4 * (size_t)h->tm[t].rows);
  }
  CREATE_TRY(h->mem.get(&h->d_tm, sizeof(TableMeta) * num_tables));
  CREATE_TRY(hipMemcpy(h->d_tm, h->tm.data(), sizeof(TableMeta) * num_tables, hipMemcpyHostToDevice));
  {  // class tables
    int32_t *d_tc = nullptr;
    CREATE_TRY(h->mem.get(&d_tc, 4 * (size_t)num_tables));
    CREATE_TRY(hipMemcpy(d_tc, tclass.data(), 4 * (size_t)num_tables, hipMemcpyHostToDevice));
    h->ci.table_class = d_tc;
    for (int c = 0; c < h->ci.n_classes; c++) {
      std::vector<int32_t> ids;
      for (int t = 0; t < num_tables; t++)
        if (tclass[t] == c) ids.push_back(t);
      int32_t *d_ids = nullptr;
      CREATE_TRY(h->mem.get(&d_ids, 4 * ids.size()));
      CREATE_TRY(hipMemcpy(d_ids, ids.data(), 4 * ids.size(), hipMemcpyHostToDevice));
      h->ci.cls_tables[c] = d_ids;
    }
  }
  // (heavy-list entry, bag range) pairs of a batch, one partial sum each: a batch has at most N / 65 entries (see alloc_batchbuf);
  // the number of ranges is chosen per batch so that the pairs fit (heavy_ranges)
  h->huge_slots = std::max<size_t>(4 * ((size_t)max_lookups / (kLongRun + 1) + 1), 32768);
  h->g.partial_slots = (int64_t)h->huge_slots;
  {
    int dev = 0, cus = 256;
    (void)hipGetDevice(&dev);
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) cus = 256;
    (void)hipGetLastError();
    // the transfer kernel keeps kLinkCus CUs to itself while it runs, which is most of the time when the link has
    // a stream of its own and rows miss (the same figure without such a stream: the split of the sums, and with
    // it their rounding, must not depend on how the streams are arranged)
    h->g.heavy_target = std::max(8, cus - kLinkCus);
  }
  CREATE_TRY(h->mem.get(&h->counters, sizeof(BatchCounters) * kMaxBatchBufs));
  CREATE_TRY(hipMemset(h->counters, 0, sizeof(BatchCounters) * kMaxBatchBufs));
  CREATE_TRY(hipHostMalloc((void **)&h->host_counters, sizeof(BatchCounters) * kMaxBatchBufs, hipHostMallocDefault));
  for (int i = 0; i < kBatchBufs; i++) {
    int rc = alloc_batchbuf(h, h->buf[i], max_lookups);
    if (rc) { g_create_error = h->err; return bail(rc); }
    CREATE_TRY(hipEventCreateWithFlags(&h->ev_ready[i], hipEventDisableTiming));
    CREATE_TRY(hipEventCreateWithFlags(&h->ev_trained[i], hipEventDisableTiming));
    CREATE_TRY(hipEventCreateWithFlags(&h->ev_probed[i], hipEventDisableTiming));
  }
  CREATE_TRY(hipEventCreateWithFlags(&h->ev_inputs, hipEventDisableTiming));
  CREATE_TRY(hipEventCreateWithFlags(&h->ev_fwd, hipEventDisableTiming));
  const size_t N = (size_t)max_lookups;
  for (int i = 0; i < 2; i++) {
    CREATE_TRY(h->mem.get(&h->ss.pairs[i], 8 * N));
  }
  {
    int widest = 0;
    for (const TableMeta &m : h->tm) widest = std::max(widest, m.lanes * (m.dtype == TBE_FP32 ? 4 : 8));
    h->g.partial_stride = widest;
    // (max pooling, which makes no partial sums, keeps the lookups' records there: at most as many bytes, but for 1/65 of them)
    CREATE_TRY(h->mem.get(&h->partials, std::max(4 * (size_t)widest * h->huge_slots, (size_t)h->g.win_stride * (size_t)max_lookups)));
  }
  {
    Staging &st = h->st;
    st.max_inserts = std::min<int64_t>(max_lookups, h->g.total_slots);
    st.stride = h->g.ovf_stride;
    std::vector<uint32_t> rb(num_tables);
    for (int t = 0; t < num_tables; t++) { rb[t] = h->tm[t].row_bytes; st.stride = std::max(st.stride, rb[t]); }
    const size_t M = (size_t)st.max_inserts;
    // room behind the victims for the overflow copies a commit parks with them (a batch bypasses at
    // most as many rows as it has lookups); none when the indices would not fit the map's codes
    st.max_parked = (M + (size_t)max_lookups <= (size_t)kWhereIndex) ? max_lookups : 0;
    const size_t P = M + (size_t)st.max_parked;
    CREATE_TRY(h->mem.get(&st.in, M * st.stride));
    for (int p2 = 0; p2 < 2; p2++) {
      CREATE_TRY(h->mem.get(&st.out[p2], P * st.stride));
      CREATE_TRY(h->mem.get(&st.wb_skip[p2], P));
      CREATE_TRY(hipMemset(st.wb_skip[p2], 0, P ? P : 1));
    }
    CREATE_TRY(h->mem.get(&st.wb_dst, 8 * P));
    CREATE_TRY(h->mem.get(&st.wb_rb, 4 * P));
    CREATE_TRY(h->mem.get(&st.wb_n, 16));
    CREATE_TRY(hipMemset(st.wb_n, 0, 16));
    CREATE_TRY(h->mem.get(&st.where, 4 * (size_t)key));
    CREATE_TRY(hipMemset(st.where, 0, 4 * (size_t)key));
    CREATE_TRY(h->mem.get(&h->d_rb, 4 * (size_t)num_tables));
    CREATE_TRY(hipMemcpy(h->d_rb, rb.data(), 4 * (size_t)num_tables, hipMemcpyHostToDevice));
  }
  {
    void *p = nullptr;
    CREATE_TRY(static_scratch_of_current_device(&p, &h->device));
    h->static_partials = (float *)p;
  }
  {
    const SortNeeds need = sort_needs(h->g, max_lookups, max_batch);
    CREATE_TRY(h->mem.get(&h->ss.slots, 4 * (size_t)need.slots));
    CREATE_TRY(h->mem.get(&h->ss.tiles, 16 * (size_t)need.tiles));
    CREATE_TRY(h->mem.get(&h->ss.said, 4 * (size_t)need.said));
    CREATE_TRY(hipMemset(h->ss.said, 0, 4 * (size_t)need.said));
    CREATE_TRY(h->mem.get(&h->ss.flags, 8 * (size_t)need.tiles));
    CREATE_TRY(hipMemset(h->ss.flags, 0, 8 * (size_t)need.tiles));
  }
  CREATE_TRY(h->mem.get(&h->ss.said_counts, 8 * 2 * 4 * (size_t)kScanBlocks));
  CREATE_TRY(hipMemset(h->ss.said_counts, 0, 8 * 2 * 4 * (size_t)kScanBlocks));
  CREATE_TRY(h->mem.get(&h->ss.tally, 8 * 3 * 4 * (size_t)kScanBlocks));
  CREATE_TRY(h->mem.get(&h->ss.too_long, 16));
  CREATE_TRY(hipMemset(h->ss.too_long, 0, 16));
  h->ss.refused = (int32_t *)h->ss.too_long + 2;
  h->ss.stage_err = h->ss.too_long + 3;
  CREATE_TRY(h->mem.get(&h->ss.one, sizeof(OneCtl)));
  CREATE_TRY(hipMemset(h->ss.one, 0, sizeof(OneCtl)));
  CREATE_TRY(h->mem.get(&h->d_total, sizeof(BatchCounters)));
  CREATE_TRY(hipMemset(h->d_total, 0, sizeof(BatchCounters)));
  CREATE_TRY(h->mem.get(&h->d_bytes, 8 * 8));
  CREATE_TRY(hipMemset(h->d_bytes, 0, 8 * 8));
  CREATE_TRY(hipDeviceSynchronize());
#undef CREATE_TRY
  *out = h;
  return TBE_OK;
}

// issue the work of queued batches as far as the pipeline takes them (one batch ahead of training)
static int pump_queue(tbe_ctx *h) {
  while (!h->queued.empty() && h->n_pend + (h->current >= 0 ? 1 : 0) <= 1) {
    const tbe_ctx::Queued q = h->queued.front();
    h->queued.pop_front();
    int rc = do_prefetch(h, q.d_indices, q.d_offsets, q.batch, q.n);
    if (rc) return rc;
  }
  return TBE_OK;
}

int tbe_prefetch(tbe_handle h, const int64_t *d_indices, const int64_t *d_offsets, int32_t batch, int64_t num_lookups) {
  if (!h) return TBE_EINVAL;
  if (h->sticky) return h->sticky;
  const int ahead = h->n_pend + (h->current >= 0 ? 1 : 0) + (int)h->queued.size();
  if (h->depth > 1 && (ahead > 1 || !h->queued.empty())) {  // beyond what runs now: keep it for later
    const int rc = check_batch(h, d_indices, d_offsets, batch, num_lookups);
    if (rc) return rc;
    if (ahead > h->depth) return fail(h, TBE_EORDER, "prefetch: more batches ahead of training than the queue takes");
    h->queued.push_back({d_indices, d_offsets, batch, num_lookups});
    return TBE_OK;
  }
  return do_prefetch(h, d_indices, d_offsets, batch, num_lookups);
}

int tbe_set_prefetch_depth(tbe_handle h, int32_t depth) {
  if (!h) return TBE_EINVAL;
  if (depth < 1 || 2 * depth + 1 > kMaxBatchBufs) return fail(h, TBE_EINVAL, "set_prefetch_depth: depth must be 1..7");
  if (h->k != 0) return fail(h, TBE_EORDER, "set_prefetch_depth: batches have been prefetched already");
  if (h->deep) return fail(h, TBE_EORDER, "set_prefetch_depth: already set");
  if (depth == 1) return TBE_OK;  // the pipeline as it is
  if (h->l2.on) return fail(h, TBE_EORDER, "set_prefetch_depth: not together with a second level");
  if (h->depth != 1) return fail(h, TBE_EORDER, "set_prefetch_depth: not together with a prefetch queue");
  if (h->max_lookups > (int64_t)kWhereBufIndex) return fail(h, TBE_ELIMIT, "set_prefetch_depth: max_lookups must be below 2^26");
  const int want = 2 * depth + 1;
  for (int i = h->nbuf; i < want; i++) {
    int rc = alloc_batchbuf(h, h->buf[i], h->max_lookups);
    if (rc) return rc;
    if (h->pooling == TBE_POOL_MAX && (rc = alloc_max_records(h, h->buf[i]))) return rc;
    HIP_TRY(h, hipEventCreateWithFlags(&h->ev_ready[i], hipEventDisableTiming));
    HIP_TRY(h, hipEventCreateWithFlags(&h->ev_trained[i], hipEventDisableTiming));
    HIP_TRY(h, hipEventCreateWithFlags(&h->ev_probed[i], hipEventDisableTiming));
    h->nbuf = i + 1;
  }
  for (int i = 0; i < want; i++) HIP_TRY(h, hipEventCreateWithFlags(&h->ev_home[i], hipEventDisableTiming));
  std::vector<DeepBuf> bufs(kMaxBatchBufs);
  for (int i = 0; i < want; i++) bufs[i] = DeepBuf{h->buf[i].cnt, h->buf[i].byp_key};
  HIP_TRY(h, h->mem.get(&h->d_deep, sizeof(DeepBuf) * kMaxBatchBufs));
  HIP_TRY(h, hipMemcpy(h->d_deep, bufs.data(), sizeof(DeepBuf) * kMaxBatchBufs, hipMemcpyHostToDevice));
  HIP_TRY(h, hipDeviceSynchronize());
  h->deep = depth;
  return TBE_OK;
}

int tbe_get_prefetch_depth(tbe_handle h, int32_t *depth, int64_t *rows_from_copies) {
  if (!h || !depth || !rows_from_copies) return TBE_EINVAL;
  int rc = sync_all(h);
  if (rc) return rc;
  unsigned long long n = 0;
  HIP_TRY(h, hipMemcpy(&n, h->d_bytes + 6, sizeof(n), hipMemcpyDeviceToHost));
  *depth = h->deep ? h->deep : 1;
  *rows_from_copies = (int64_t)n;
  return TBE_OK;
}

int tbe_set_prefetch_queue(tbe_handle h, int32_t depth) {
  if (!h) return TBE_EINVAL;
  if (h->deep) return fail(h, TBE_EORDER, "set_prefetch_queue: not together with a prefetch depth above one");
  if (depth < 1 || depth > 64) return fail(h, TBE_EINVAL, "set_prefetch_queue: length must be 1..64");
  if (!h->queued.empty()) return fail(h, TBE_EORDER, "set_prefetch_queue: batches are queued");
  h->depth = depth;
  return TBE_OK;
}

int tbe_forward(tbe_handle h, const int64_t *d_indices, const int64_t *d_offsets, int32_t batch, int64_t num_lookups,
                float *d_out) {
  if (!h) return TBE_EINVAL;
  if (h->sticky) return h->sticky;
  if (!d_out) return fail(h, TBE_EINVAL, "forward: null output");
  if (h->current >= 0) return fail(h, TBE_EORDER, "forward: the previous batch has not been updated");
  if (h->n_pend == 0 && !h->queued.empty()) {
    int rc = pump_queue(h);
    if (rc) return rc;
  }
  if (h->n_pend == 0) {
    int rc = do_prefetch(h, d_indices, d_offsets, batch, num_lookups, true);
    if (rc) return rc;
  }
  const int bi = h->pend[0];
  BatchBuf &b = h->buf[bi];
  if (b.d_indices != d_indices || b.d_offsets != d_offsets || b.batch != batch || b.n != num_lookups)
    return fail(h, TBE_EMISMATCH, "forward: buffers differ from the pending prefetch");
  if (h->deferred == bi) return fail(h, TBE_EORDER, "forward: the batch before this one has not been updated");
  for (int i = 1; i < h->n_pend; i++) h->pend[i - 1] = h->pend[i];
  h->n_pend--;
  if (b.link != h->cs) {
    HIP_TRY(h, hipStreamWaitEvent(h->cs, h->ev_ready[bi], 0));
    // A timing event recorded right after a wait for another stream is stamped before that wait is
    // over (measured: the forward's bracket began 0.15 ms before the commit it waits for had ended).
    // A kernel is held back by the wait, so an empty one in front of the bracket pins its beginning.
    if (h->profiling) hipLaunchKernelGGL(stream_pin_kernel, dim3(1), dim3(64), 0, h->cs);
  }
  if (h->deep) HIP_TRY(h, fix_up(h, b));
  {
    StageTimer tm_(h, TBE_STAGE_FORWARD, h->cs);
    HIP_TRY(h, launch_forward_classes(h->d_tm, h->ci, h->g, b, d_out, h->cs));
  }
  // An event that the next prefetch waits for if it comes before the update: not when one has come already and the pipeline
  // takes no more, nor when that prefetch has to wait for all of the stream.
  if (b.link != h->cs && h->inputs_ready && (h->deep || h->n_pend == 0)) {
    HIP_TRY(h, hipEventRecord(h->ev_fwd, h->cs));
    h->fwd_of = bi;
  } else {
    h->fwd_of = -1;
  }
  h->current = bi;
  return pump_queue(h);  // the next queued batch is prefetched while this one trains
}

// The backward of the forwarded batch with the partial sums of its longest rows in `partials`.
static int backward_update_with(tbe_ctx *h, const float *d_grad_out, float lr, float eps, float *partials) {
  if (h->sticky) return h->sticky;
  if (!d_grad_out) return fail(h, TBE_EINVAL, "backward_update: null gradient");
  if (h->current < 0) return fail(h, TBE_EORDER, "backward_update: no forwarded batch");
  const int bi = h->current;
  // The sections touch disjoint rows; the combine follows the heavy rows' kernel.  Small batches: everything in one launch for each
  // width of rows (under max pooling the hot rows' kernel in front of it; see long_rows_in_rest for sum and mean).  With more
  // lookups the rows with one and with 2..64 lookups first, the heavy rows' kernel, if there is one, and the combine last: 0.471 ms alone against 0.479 with the tile kernel first (it takes 0.124 instead of 0.134 ms when
  // it does not follow the forward), 0.627 against 0.635 ms beside the other streams.  (The heavy rows on a stream of their
  // own, beside the others: the tile kernel's workgroups need a CU to themselves each and waited for the others' waves to
  // drain -- 0.28 ms instead of 0.12 alone, the whole backward 0.51 ms instead of 0.48, and 0.72 instead of 0.65 ms beside
  // the other streams' work.)  With every section bracketed each has a launch of its own.
  {
    StageTimer all_(h, TBE_STAGE_BACKWARD, h->cs);
    auto run = [&](int which, int stage) -> int {
      StageTimer tm_(h, stage, h->cs);
      HIP_TRY(h, launch_backward_classes(which, h->d_tm, h->ci, h->g, h->buf[bi], d_grad_out, partials, lr, eps, h->cs));
      return TBE_OK;
    };
    int rc;
    if (h->profiling == 1)
      rc = (rc = run(kBwdSingle, TBE_STAGE_BACKWARD_SINGLE)) ? rc : (rc = run(kBwdShort, TBE_STAGE_BACKWARD_SHORT)) ? rc
           : (rc = run(kBwdHeavy, TBE_STAGE_BACKWARD_HEAVY)) ? rc : run(kBwdCombine, TBE_STAGE_BACKWARD_COMBINE);
    else if (h->buf[bi].n <= kSmallLookups)
      rc = (rc = run(kBwdHeavy, TBE_STAGE_BACKWARD_HEAVY)) ? rc
           : run(kBwdCombine | kBwdSingle | kBwdShort, TBE_STAGE_BACKWARD_SHORT);
    else
      rc = (rc = run(kBwdSingle | kBwdShort, TBE_STAGE_BACKWARD_SHORT)) ? rc : (rc = run(kBwdHeavy, TBE_STAGE_BACKWARD_HEAVY)) ? rc
           : run(kBwdCombine, TBE_STAGE_BACKWARD_COMBINE);
    if (rc) return rc;
  }
  h->current = -1;
  const BatchBuf &b = h->buf[bi];
  // What moves this batch's bypassed rows next waits for the update: the commit of the next batch, which also overwrites lines
  // that this batch used, if one is waiting, or a write-back of their own.  Either goes to the stream of the last transfer, so
  // that a later transfer finds all of them in front of it.  (The prefetch stream only decides on tags and timestamps, which
  // training never reads, so it does not wait here; a later prefetch does, for this event if the inputs are ready.)
  const bool write_back = h->deferred < 0 && !h->never_bypasses;
  const bool waited_for = h->deferred >= 0 || write_back || h->deep;
  hipStream_t next = h->link_s;
  if (write_back && next == h->cs && h->own_ls && write_back_beside(h->g, b.n)) next = h->link_s = h->ls;
  if (next != h->cs && (waited_for || h->inputs_ready)) {
    HIP_TRY(h, hipEventRecord(h->ev_trained[bi], h->cs));
    h->last_trained = bi;
    h->unmarked = false;
    if (waited_for) HIP_TRY(h, hipStreamWaitEvent(next, h->ev_trained[bi], 0));
  } else {
    h->unmarked = true;
  }
  // the rows this batch bypassed were trained on in HBM copies: back to the backing tier,
  // together with the commit of the next batch when that one is waiting
  if (h->deferred >= 0) {
    const int d = h->deferred;
    h->deferred = -1;
    int rc = enqueue_commit(h, d, true);
    return rc ? rc : pump_queue(h);
  }
  if (write_back) {
    // no batch has been prefetched after this one, so no transfer has run since its commit: the
    // overflow copies that commit parked (the previous batch's) go home, and this batch's
    HIP_TRY(h, launch_ovf_writeback(b, b.parks_prev && b.prev_bi >= 0 ? h->parked : 0, h->st, h->d_rb, h->d_bytes + 1, next));
    if (h->deep && next != h->cs) {  // the buffer is free once they are home
      HIP_TRY(h, hipEventRecord(h->ev_home[bi], next));
      h->home_recorded[bi] = true;
    }
  }
  return pump_queue(h);
}

int tbe_backward_update(tbe_handle h, const float *d_grad_out, float lr, float eps) {
  if (!h) return TBE_EINVAL;
  return backward_update_with(h, d_grad_out, lr, eps, h->partials);
}

// bytes of partial sums a batch of this handle can need at most
static size_t static_scratch_needed(const tbe_ctx *h) { return 4 * (size_t)h->g.partial_stride * h->huge_slots; }

int tbe_backward_update_static(tbe_handle h, const float *d_grad_out, float lr, float eps) {
  if (!h) return TBE_EINVAL;
  if (h->profiling) return fail(h, TBE_EORDER, "backward_update_static: stage timing is on (it creates events)");
  if (static_scratch_needed(h) > kStaticScratchBytes)
    return fail(h, TBE_ELIMIT, "backward_update_static: a batch of max_lookups could need " +
                                   std::to_string(static_scratch_needed(h)) + " bytes of partial sums, the static scratch holds " +
                                   std::to_string(kStaticScratchBytes));
  int dev = -1;
  HIP_TRY(h, hipGetDevice(&dev));
  if (dev != h->device || !h->static_partials)
    return fail(h, TBE_EORDER, "backward_update_static: the handle was created on another GPU than the current one");
  return backward_update_with(h, d_grad_out, lr, eps, h->static_partials);
}

int tbe_flush(tbe_handle h) {
  if (!h) return TBE_EINVAL;
  int rc = TBE_OK;
  if (h->n_pend == 0 && h->current < 0 && h->queued.empty()) {
    // Everything issued has been trained on.  The flush's kernels follow on the compute stream, behind the write-backs that
    // the last transfer's stream may still have (all else there, and on the prefetch stream, the forwards have waited for).
    if (h->link_s != h->cs && (rc = order_after(h, h->link_s, h->cs))) return rc;
  } else {
    if ((rc = sync_all(h))) return rc;
    // Allowed only after the device has refused a batch (bad offsets, index out of range): that batch and
    // any behind it do nothing and never will (the error sticks), so they are dropped here and the flush
    // brings the backing tier up to the last batch that trained.
    (void)collect_device_errors(h);
    if (!h->sticky) return fail(h, TBE_EORDER, "flush: a batch is still in flight");
    // Batches in front of the refused one may have been committed without training, and there is then a row whose value is in
    // their own copy alone: one that such a batch bypassed and took over from a parked victim, or from a copy of the batch
    // before it.  These copies go home here.  In the pipeline several batches deep some of their rows have yet to be copied
    // from the copies of earlier batches, into overflow copies or cache lines, which the forward would have done: in the order
    // of the batches, because one may take from the one before.
    for (int i = -1; i < h->n_pend; i++) {
      const int bi = i < 0 ? h->current : h->pend[i];
      if (bi < 0 || bi == h->deferred) continue;
      if (h->deep && i >= 0) HIP_TRY(h, fix_up(h, h->buf[bi]));
      HIP_TRY(h, launch_ovf_writeback(h->buf[bi], 0, h->st, h->d_rb, h->d_bytes + 1, h->cs));
    }
    h->n_pend = 0;
    h->current = -1;
    h->deferred = -1;
    h->queued.clear();
  }
  HIP_TRY(h, launch_transfer(nullptr, h->parked, h->st, h->l2, h->di, h->throttle, 0, h->d_rb, h->d_bytes, h->d_bytes + 1, h->cs));  // parked victims first
  // Every copy in the backing tier is current now: the next batch must not take any row for one on its way (it would
  // make the transfer skip a write-back that has already happened, and the request would hit a later batch's victim).
  h->prev_buf = -1;
  HIP_TRY(h, launch_flush(h->d_tm, h->g, h->tags, h->l2, h->d_bytes, h->d_bytes + 1, h->cs));  // also slot accumulators -> dev_m
  // A copy engine takes some 18 us per table, whatever its size, and 57 GB/s; a kernel writes all small tables' accumulators
  // in one launch (4 tables of 100 k rows: 29 instead of 72 us).  An array that is not pinned, which no kernel may write, is
  // copied whatever its size.
  HIP_TRY(h, launch_flush_state(h->d_tm, h->g, h->counters, h->host_counters, h->nbuf, h->cs));
  for (const TableMeta &m : h->tm) {
    if (!m.flush_by_kernel)
      HIP_TRY(h, hipMemcpyAsync(m.host_m, m.dev_m, 4 * (size_t)m.rows, hipMemcpyDeviceToHost, h->cs));
    h->flush_state_bytes += 4 * m.rows;
  }
  // (A checkpoint of 4 tables x 100 k rows after every other step: 508 us with the streams waited for in front of the flush's
  // kernels as well and the counters fetched by a copy of their own behind them, 485 so.)
  rc = sync_all(h);
  if (rc) return rc;
  return take_device_errors(h, h->host_counters);
}

int tbe_set_policy(tbe_handle h, int32_t policy) {
  if (!h) return TBE_EINVAL;
  if (policy != TBE_POLICY_LRU && policy != TBE_POLICY_LFU) return fail(h, TBE_EINVAL, "set_policy: unknown policy");
  if (h->k != 0) return fail(h, TBE_EORDER, "set_policy: batches have been prefetched already");
  h->policy = policy;
  return TBE_OK;
}

int tbe_set_backing_throttle(tbe_handle h, int64_t ns_per_row) {
  if (!h) return TBE_EINVAL;
  if (ns_per_row < 0 || ns_per_row > 100000000) return fail(h, TBE_EINVAL, "set_backing_throttle: 0 .. 1e8 ns per row");
  int khz = 0;
  if (hipDeviceGetAttribute(&khz, hipDeviceAttributeClockRate, h->device) != hipSuccess || khz < 1) khz = 2400000;
  (void)hipGetLastError();
  // one pause is s_sleep 127: about 127 x 64 clocks
  const double clocks = (double)ns_per_row * 1e-9 * (double)khz * 1e3;
  h->throttle.pauses = ns_per_row == 0 ? 0 : std::max(1, (int)(clocks / (127.0 * 64.0) + 0.5));
  return TBE_OK;
}

int tbe_set_probe_grouping(tbe_handle h, int32_t min_windows) {
  if (!h) return TBE_EINVAL;
  if (min_windows < 1 || min_windows > (1 << 30)) return fail(h, TBE_EINVAL, "set_probe_grouping: 1 .. 2^30 windows");
  h->g.probe_min_windows = min_windows;
  return TBE_OK;
}

int tbe_enable_second_level(tbe_handle h, int32_t factor) {
  if (!h) return TBE_EINVAL;
  if (factor < 1 || factor > 1024) return fail(h, TBE_EINVAL, "enable_second_level: factor must be 1..1024");
  if (h->k != 0) return fail(h, TBE_EORDER, "enable_second_level: batches have been prefetched already");
  if (h->l2.on) return fail(h, TBE_EORDER, "enable_second_level: already enabled");
  if (h->deep) return fail(h, TBE_EORDER, "enable_second_level: not together with a prefetch depth above one");
  if (h->st.max_inserts >= (1ll << 29)) return fail(h, TBE_ELIMIT, "enable_second_level: too many possible inserts per batch");
  int64_t slots2 = 0;
  size_t bytes2 = 0;
  for (TableMeta &m : h->tm) {
    if ((int64_t)m.sets * factor * h->g.ways + slots2 >= (1ll << 31)) return fail(h, TBE_ELIMIT, "enable_second_level: too many second-level slots");
    slots2 += (int64_t)m.sets * factor * h->g.ways;
    bytes2 += (size_t)m.sets * factor * h->g.ways * m.row_bytes;
  }
  if (slots2 == 0) return fail(h, TBE_EINVAL, "enable_second_level: no table has a first-level cache");
  if (h->lines2) (void)hipHostFree(h->lines2);  // of an earlier call that failed
  h->lines2 = nullptr;
  HIP_TRY(h, hipHostMalloc((void **)&h->lines2, bytes2, hipHostMallocDefault));
  h->l2.lines_lo = h->lines2;
  h->l2.lines_hi = h->lines2 + bytes2;
  Level2 &l2 = h->l2;
  const size_t M = (size_t)h->st.max_inserts;
  HIP_TRY(h, h->mem.get(&l2.tags2, 4 * (size_t)slots2));
  HIP_TRY(h, h->mem.get(&l2.ts2, 4 * (size_t)slots2));
  HIP_TRY(h, hipMemset(l2.tags2, 0xFF, 4 * (size_t)slots2));
  HIP_TRY(h, hipMemset(l2.ts2, 0xFF, 4 * (size_t)slots2));
  for (int p2 = 0; p2 < 2; p2++) {
    HIP_TRY(h, h->mem.get(&l2.out2[p2], M * h->st.stride));
    // the skip flags of the staged second-level victims follow those of the first-level ones (a larger array in place of the
    // one there is, never a smaller: if a later allocation fails the handle goes on with one level and its parked copies)
    const size_t flags = std::max(2 * M, M + (size_t)h->st.max_parked);
    uint8_t *skip = nullptr;
    HIP_TRY(h, h->mem.get(&skip, flags));
    HIP_TRY(h, hipMemset(skip, 0, flags ? flags : 1));
    h->st.wb_skip[p2] = skip;
  }
  HIP_TRY(h, h->mem.get(&l2.wb2_dst, 8 * M));
  HIP_TRY(h, hipMemset(l2.wb2_dst, 0, 8 * M ? 8 * M : 8));
  HIP_TRY(h, h->mem.get(&l2.sums, 4 * kL2Sums * kL2Line));
  HIP_TRY(h, hipMemset(l2.sums, 0, 4 * kL2Sums * kL2Line));
  HIP_TRY(h, h->mem.get(&h->d_l2tot, 8 * 4));
  HIP_TRY(h, hipMemset(h->d_l2tot, 0, 8 * 4));
  for (int i = 0; i < h->nbuf; i++) {
    BatchBuf &b = h->buf[i];
    const size_t N = (size_t)std::max<int64_t>(h->max_lookups, 1);
    HIP_TRY(h, h->mem.get(&b.src2, 4 * N));
    HIP_TRY(h, h->mem.get(&b.dst2, 4 * N));
    HIP_TRY(h, h->mem.get(&b.evict2, 4 * N));
    HIP_TRY(h, h->mem.get(&b.ins_dst, 8 * N));
    HIP_TRY(h, h->mem.get(&b.l2v_src, 8 * N));
    HIP_TRY(h, h->mem.get(&b.l2v_dst, 8 * N));
    HIP_TRY(h, h->mem.get(&b.l2v_key, 4 * N));
  }
  int64_t base = 0;
  size_t off = 0;
  for (TableMeta &m : h->tm) {
    m.sets2 = m.sets * (uint32_t)factor;
    m.slot2_base = (int32_t)base;
    m.lines2 = h->lines2 + off;
    base += (int64_t)m.sets2 * h->g.ways;
    off += (size_t)m.sets2 * h->g.ways * m.row_bytes;
  }
  HIP_TRY(h, hipMemcpy(h->d_tm, h->tm.data(), sizeof(TableMeta) * h->tm.size(), hipMemcpyHostToDevice));
  l2.factor = factor;
  l2.total_slots2 = slots2;
  l2.on = true;
  return TBE_OK;
}

int64_t tbe_num_sets2(tbe_handle h, int32_t table) {
  if (!h || table < 0 || table >= h->g.T) return TBE_EINVAL;
  return h->tm[table].sets2;
}

int tbe_export_second_level_state(tbe_handle h, int32_t table, int64_t *h_tags, int32_t *h_ts) {
  if (!h || table < 0 || table >= h->g.T || !h_tags || !h_ts) return TBE_EINVAL;
  int rc = sync_all(h);
  if (rc) return rc;
  const TableMeta &m = h->tm[table];
  const size_t n = (size_t)m.sets2 * h->g.ways;
  if (n == 0) return TBE_OK;
  std::vector<int32_t> tmp(n);
  HIP_TRY(h, hipMemcpy(tmp.data(), h->l2.tags2 + m.slot2_base, 4 * n, hipMemcpyDeviceToHost));
  for (size_t i = 0; i < n; i++) h_tags[i] = tmp[i];
  HIP_TRY(h, hipMemcpy(h_ts, h->l2.ts2 + m.slot2_base, 4 * n, hipMemcpyDeviceToHost));
  return TBE_OK;
}

int tbe_get_second_level_stats(tbe_handle h, int64_t *h_last4, int64_t *h_total4) {
  if (!h || !h_last4 || !h_total4) return TBE_EINVAL;
  for (int i = 0; i < 4; i++) h_last4[i] = h_total4[i] = 0;
  if (!h->l2.on) return TBE_OK;
  int rc = sync_all(h);
  if (rc) return rc;
  if (h->last_buf >= 0) {
    BatchCounters c;
    HIP_TRY(h, hipMemcpy(&c, h->buf[h->last_buf].cnt, sizeof(c), hipMemcpyDeviceToHost));
    h_last4[0] = c.l2_hits; h_last4[1] = c.l2_demotions; h_last4[2] = c.l2_evictions; h_last4[3] = c.l2_bypasses;
  }
  unsigned long long t[4];
  HIP_TRY(h, hipMemcpy(t, h->d_l2tot, sizeof(t), hipMemcpyDeviceToHost));
  for (int i = 0; i < 4; i++) h_total4[i] = (int64_t)t[i];
  return collect_device_errors(h);
}

int tbe_enable_deferred_init(tbe_handle h, uint64_t seed, float std) {
  if (!h) return TBE_EINVAL;
  if (!(std >= 0.f)) return fail(h, TBE_EINVAL, "enable_deferred_init: std must be >= 0");
  if (h->k != 0) return fail(h, TBE_EORDER, "enable_deferred_init: batches have been prefetched already");
  if (h->di.tm) return fail(h, TBE_EORDER, "enable_deferred_init: already enabled");
  size_t words = 0;
  for (const TableMeta &m : h->tm) words += ((size_t)m.rows + 31) / 32;
  HIP_TRY(h, h->mem.get(&h->init_bits, 4 * words));
  HIP_TRY(h, hipMemset(h->init_bits, 0, 4 * words));
  size_t off = 0;
  for (TableMeta &m : h->tm) {
    m.init_bits = h->init_bits + off;
    off += ((size_t)m.rows + 31) / 32;
  }
  HIP_TRY(h, hipMemcpy(h->d_tm, h->tm.data(), sizeof(TableMeta) * h->tm.size(), hipMemcpyHostToDevice));
  h->di.tm = h->d_tm;
  h->di.seed = seed;
  h->di.std = std;
  return TBE_OK;
}

int tbe_export_initialised(tbe_handle h, int32_t table, uint8_t *h_flags) {
  if (!h || table < 0 || table >= h->g.T || !h_flags) return TBE_EINVAL;
  if (!h->di.tm) return fail(h, TBE_EORDER, "export_initialised: deferred initialisation is not enabled");
  int rc = sync_all(h);
  if (rc) return rc;
  const TableMeta &m = h->tm[table];
  std::vector<uint32_t> w(((size_t)m.rows + 31) / 32);
  HIP_TRY(h, hipMemcpy(w.data(), m.init_bits, 4 * w.size(), hipMemcpyDeviceToHost));
  for (int64_t r = 0; r < m.rows; r++) h_flags[r] = (uint8_t)((w[(size_t)r >> 5] >> (r & 31)) & 1u);
  return TBE_OK;
}

int tbe_set_pooling(tbe_handle h, int32_t pooling) {
  if (!h) return TBE_EINVAL;
  if (pooling != TBE_POOL_SUM && pooling != TBE_POOL_MEAN && pooling != TBE_POOL_MAX)
    return fail(h, TBE_EINVAL, "set_pooling: unknown pooling mode");
  if (h->k != 0) return fail(h, TBE_EORDER, "set_pooling: batches have been prefetched already");
  if (pooling == TBE_POOL_MAX)
    for (int i = 0; i < h->nbuf; i++) {
      const int rc = alloc_max_records(h, h->buf[i]);
      if (rc) return rc;
    }
  h->pooling = pooling;
  return TBE_OK;
}

int tbe_export_argmax(tbe_handle h, int32_t *d_argmax) {
  if (!h || !d_argmax) return TBE_EINVAL;
  if (h->sticky) return h->sticky;
  if (h->pooling != TBE_POOL_MAX) return fail(h, TBE_EORDER, "export_argmax: the pooling mode is not max");
  if (h->current < 0) return fail(h, TBE_EORDER, "export_argmax: no forwarded batch waits for its update");
  const BatchBuf &b = h->buf[h->current];
  HIP_TRY(h, hipMemcpyAsync(d_argmax, b.argpos, 4 * (size_t)b.batch * (size_t)h->g.sum_dim, hipMemcpyDeviceToDevice, h->cs));
  return TBE_OK;
}

int tbe_set_inputs_ready(tbe_handle h, int32_t ready) {
  if (!h) return TBE_EINVAL;
  h->inputs_ready = ready != 0;
  return TBE_OK;
}

int tbe_set_profiling(tbe_handle h, int32_t enable) {
  if (!h) return TBE_EINVAL;
  int rc = sync_all(h);
  if (rc) return rc;
  drop_profile(h);
  h->profiling = enable == 2 ? 2 : (enable != 0 ? 1 : 0);
  return TBE_OK;
}

int64_t tbe_get_stage_times(tbe_handle h, int32_t stage, int64_t capacity, float *h_ms) {
  if (!h || stage < 0 || stage >= TBE_NUM_STAGES) return TBE_EINVAL;
  int rc = sync_all(h);
  if (rc) return rc;
  const auto &v = h->prof[stage];
  if (!h_ms) return (int64_t)v.size();
  if (capacity < (int64_t)v.size()) return fail(h, TBE_ELIMIT, "get_stage_times: capacity too small");
  for (size_t i = 0; i < v.size(); i++) HIP_TRY(h, hipEventElapsedTime(&h_ms[i], v[i].first, v[i].second));
  return (int64_t)v.size();
}

int64_t tbe_num_sets(tbe_handle h, int32_t table) {
  if (!h || table < 0 || table >= h->g.T) return TBE_EINVAL;
  return h->tm[table].sets;
}

int tbe_get_stats(tbe_handle h, tbe_stats *out) {
  if (!h || !out) return TBE_EINVAL;
  int rc = sync_all(h);
  if (rc) return rc;
  memset(out, 0, sizeof(*out));
  BatchCounters tot;
  unsigned long long b64[8];
  HIP_TRY(h, hipMemcpy(&tot, h->d_total, sizeof(tot), hipMemcpyDeviceToHost));
  HIP_TRY(h, hipMemcpy(b64, h->d_bytes, sizeof(b64), hipMemcpyDeviceToHost));
  if (h->last_buf >= 0) {
    BatchCounters c;
    HIP_TRY(h, hipMemcpy(&c, h->buf[h->last_buf].cnt, sizeof(c), hipMemcpyDeviceToHost));
    out->last.lookups = h->buf[h->last_buf].n;
    out->last.uniques = c.n_uniq;
    out->last.hits = (int64_t)c.hits;
    out->last.inserts = c.n_ins;
    out->last.bypasses = c.n_byp;
    out->last.evictions = (int64_t)c.evictions;
    out->last.hit_lookups = (int64_t)c.hit_lookups;
    out->last_long_rows = c.n_long;
  }
  out->total.lookups = h->total_lookups;
  out->total.uniques = (int64_t)b64[2];
  out->total.inserts = (int64_t)b64[3];
  out->total.bypasses = (int64_t)b64[4];
  out->total.hits = (int64_t)tot.hits;
  out->total.evictions = (int64_t)tot.evictions;
  out->total.hit_lookups = (int64_t)tot.hit_lookups;
  out->h2d_bytes = (int64_t)b64[0];
  out->d2h_bytes = (int64_t)b64[1] + h->flush_state_bytes;
  out->late_fetches = (int64_t)b64[5];
  out->batch_id = h->k;
  return collect_device_errors(h);
}

int tbe_export_cache_state(tbe_handle h, int32_t table, int64_t *h_tags, int32_t *h_ts) {
  if (!h || table < 0 || table >= h->g.T || !h_tags || !h_ts) return TBE_EINVAL;
  int rc = sync_all(h);
  if (rc) return rc;
  const TableMeta &m = h->tm[table];
  const size_t n = (size_t)m.sets * h->g.ways;
  if (n == 0) return TBE_OK;
  std::vector<int32_t> tmp(n);
  HIP_TRY(h, hipMemcpy(tmp.data(), h->tags + m.slot_base, 4 * n, hipMemcpyDeviceToHost));
  for (size_t i = 0; i < n; i++) h_tags[i] = tmp[i];
  HIP_TRY(h, hipMemcpy(h_ts, h->ts + m.slot_base, 4 * n, hipMemcpyDeviceToHost));
  return TBE_OK;
}

int tbe_export_cache_freq(tbe_handle h, int32_t table, int32_t *h_freq) {
  if (!h || table < 0 || table >= h->g.T || !h_freq) return TBE_EINVAL;
  int rc = sync_all(h);
  if (rc) return rc;
  const TableMeta &m = h->tm[table];
  const size_t n = (size_t)m.sets * h->g.ways;
  if (n == 0) return TBE_OK;
  HIP_TRY(h, hipMemcpy(h_freq, h->freq + m.slot_base, 4 * n, hipMemcpyDeviceToHost));
  return TBE_OK;
}

int tbe_import_cache_freq(tbe_handle h, int32_t table, const int32_t *h_freq) {
  if (!h || table < 0 || table >= h->g.T || !h_freq) return TBE_EINVAL;
  if (h->n_pend > 0 || h->current >= 0 || !h->queued.empty()) return fail(h, TBE_EORDER, "import_cache_freq: a batch is still in flight");
  int rc = sync_all(h);
  if (rc) return rc;
  const TableMeta &m = h->tm[table];
  const size_t n = (size_t)m.sets * h->g.ways;
  for (size_t i = 0; i < n; i++)
    if (h_freq[i] < 0) return fail(h, TBE_EINVAL, "import_cache_freq: negative count");
  if (n) HIP_TRY(h, hipMemcpy(h->freq + m.slot_base, h_freq, 4 * n, hipMemcpyHostToDevice));
  return TBE_OK;
}

int64_t tbe_export_batch_events(tbe_handle h, int32_t kind, int64_t capacity, int64_t *h_table, int64_t *h_row,
                                int64_t *h_slot, int64_t *h_old) {
  if (!h || kind < 0 || kind > 2) return TBE_EINVAL;
  if (h->last_buf < 0) return 0;
  int rc = sync_all(h);
  if (rc) return rc;
  const BatchBuf &b = h->buf[h->last_buf];
  BatchCounters c;
  HIP_TRY(h, hipMemcpy(&c, b.cnt, sizeof(c), hipMemcpyDeviceToHost));
  if (c.err) return device_error_code(c.err);
  const int64_t count = kind == 0 ? (int64_t)c.hits : kind == 1 ? c.n_ins : c.n_byp;
  if (!h_table || !h_row) return count;
  if (capacity < count) return fail(h, TBE_ELIMIT, "export_batch_events: capacity too small");
  const size_t U = (size_t)c.n_uniq;
  if (U == 0) return 0;
  std::vector<uint32_t> key(U);
  std::vector<uint8_t> st(U);
  std::vector<int32_t> loc(U), old(U);
  HIP_TRY(h, hipMemcpy(key.data(), b.uniq_key, 4 * U, hipMemcpyDeviceToHost));
  HIP_TRY(h, hipMemcpy(st.data(), b.status, U, hipMemcpyDeviceToHost));
  HIP_TRY(h, hipMemcpy(loc.data(), b.loc_u, 4 * U, hipMemcpyDeviceToHost));
  HIP_TRY(h, hipMemcpy(old.data(), b.old_tag, 4 * U, hipMemcpyDeviceToHost));
  const uint8_t want = kind == 0 ? ST_HIT : kind == 1 ? ST_INSERT : ST_BYPASS;
  int64_t n = 0;
  int t = 0;
  for (size_t u = 0; u < U; u++) {
    if (st[u] != want) continue;
    while (t + 1 < h->g.T && h->tm[t + 1].key_base <= key[u]) t++;
    const TableMeta &m = h->tm[t];
    const uint32_t local = key[u] - m.key_base;
    int64_t row = local;
    if (m.sets) {
      const uint32_t s = local / m.rows_per_set;
      row = (int64_t)(local - s * m.rows_per_set) * m.sets + s;
    }
    h_table[n] = t;
    h_row[n] = row;
    if (kind == 1 && h_slot) h_slot[n] = loc[u] - m.slot_base;
    if (kind == 1 && h_old) h_old[n] = old[u];
    n++;
  }
  return n;
}

}  // extern "C"
