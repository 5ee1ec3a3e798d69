// Host side of the C ABI declared in include/sfc.h: owns the device memory of one cache and
// enqueues the kernels of each step call on the caller's streams.  No call after
// sfc_cache_create allocates device memory or waits for the device, except the ones the header
// documents as synchronising.
//
// A step in flight is a StepCtx: the caller's buffers, the step's device counters, its grouping
// of positions, its victim list and its bypass region.  lookahead = L has L + 1 contexts.
// L = 0 runs the prepare on the main stream and the Host copies on the side stream (few of them on the
// main stream, see swap_on_main).  L >= 1 gives the prepare a stream of its own and the Host copies run on
// the side stream, so that the prepare of step t+L, the copies of the step before it and lookup / update of
// step t overlap (the paper's pipeline of Data-Loader, Host-Manager and GPU-Worker stages); a
// larger L means more contexts, i.e. a prepare need not wait for the most recent update.  The
// Prefetch comparison strategy keeps its prepare on the side stream, ahead of its copies.
// Streams are ordered by events only; the host never waits.
#include "../../include/sfc.h"

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "sfc_prepare_kernels.h"
#include "sfc_row_kernels.h"

using namespace sfc;

namespace {

thread_local std::string g_err;
std::mutex g_host_mu;
std::map<void*, int64_t> g_host_allocs;     // pieces handed out by sfc_host_alloc and still alive

int fail(int code, const char* what, hipError_t e = hipSuccess) {
  char buf[512];
  if (e != hipSuccess) snprintf(buf, sizeof buf, "%s: %s", what, hipGetErrorString(e));
  else snprintf(buf, sizeof buf, "%s", what);
  g_err = buf;
  return code;
}

#define HIPCHK(call)                                            \
  do {                                                          \
    hipError_t e_ = (call);                                     \
    if (e_ != hipSuccess) return fail(SFC_EHIP, #call, e_);     \
  } while (0)

// Scratch of sfc_segment_sum_static: lives in the code object, one copy per GPU that loads the
// library, held until the process ends.  In host code this name is only a handle for
// hipGetSymbolAddress; the address that kernels and copies use is scratch_ptr[device].
static __device__ __align__(256) unsigned char scratch[SFC_STATIC_SCRATCH_BYTES];
constexpr int kMaxDevices = 64;
void* scratch_ptr[kMaxDevices] = {};
std::mutex scratch_mu;

// The device address of `scratch` on the current device (looked up once per device).
int static_scratch(int device, void** out) {
  if (device < 0 || device >= kMaxDevices) return fail(SFC_EINVAL, "device number out of range");
  std::lock_guard<std::mutex> lk(scratch_mu);
  if (!scratch_ptr[device]) {
    void* p = nullptr;
    hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) return fail(SFC_EHIP, "hipGetSymbolAddress(scratch)", e);
    scratch_ptr[device] = p;
  }
  *out = scratch_ptr[device];
  return SFC_OK;
}

// Is stream s being captured?
bool capturing(hipStream_t s) {
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &cap) == hipSuccess) return cap != hipStreamCaptureStatusNone;
  (void)hipGetLastError();                      // (no answer is not an error of the call that asks)
  return true;
}

// The stream of a pipelined cache's prepares.  HIP puts the streams of a process on four hardware queues, and what stands
// behind a step's Host copies in a queue waits for hundreds of microseconds: with the prepares in the queue of the main or the
// side stream a step takes half as long again.  No call tells a stream's queue, so a few candidates are tried when the cache
// is created: a kernel that waits for a moment on the one stream, an empty one on the other.  us a step of one cache that
// is created behind 0 to 3 other streams, the first stream that comes / this way: 65536 x 39 ids of dim 32 with lookahead 2 501, 518,
// 737, 500 / 495, 498, 736, 496, 8192 x 26 of dim 128 164, 168, 127, 131 / 127, 163, 124, 122.  (In the two slow ones main and side stream
// share a queue, which this choice cannot change.  It is made once: a stream that is made later may still land in the queue.  One stream for
// all caches of a main stream: three caches in turn 456 to 704 us at 65536 x 39, 589 to 655 this way.)
__global__ void k_hold(long long ticks) {
  const long long t0 = wall_clock64();
  for (int i = 0; i < (1 << 16) && wall_clock64() - t0 < ticks; ++i) __builtin_amdgcn_s_sleep(8);
}
constexpr int kPrepTries = 4;                   // as many as there are hardware queues

// Does work of stream b run while stream a is busy?  (Both have nothing to do.)
bool side_by_side(hipStream_t a, hipStream_t b, hipEvent_t ea, hipEvent_t eb) {
  bool yes = false;
  for (int i = 0; i < 2 && !yes; ++i) {         // (the host may have been held up)
    hipLaunchKernelGGL(k_hold, dim3(1), dim3(64), 0, a, 6000LL);          // 60 us of a clock of 100 MHz
    if (hipEventRecord(ea, a) != hipSuccess) break;
    hipLaunchKernelGGL(k_hold, dim3(1), dim3(64), 0, b, 0LL);
    if (hipEventRecord(eb, b) != hipSuccess || hipEventSynchronize(eb) != hipSuccess) break;
    yes = hipEventQuery(ea) == hipErrorNotReady;
    if (hipEventSynchronize(ea) != hipSuccess) break;
  }
  (void)hipGetLastError();
  return yes;
}

hipError_t choose_prep_stream(hipStream_t main, hipStream_t side, hipStream_t* out) {
  hipStream_t s[kPrepTries] = {};
  hipEvent_t ea = nullptr, eb = nullptr;
  int n = 0, best = -1, most = -1;
  hipError_t e = hipEventCreateWithFlags(&ea, hipEventDisableTiming);
  if (e == hipSuccess) e = hipEventCreateWithFlags(&eb, hipEventDisableTiming);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_hold, dim3(1), dim3(64), 0, main, 0LL);          // its code is loaded
    e = hipStreamSynchronize(main);
  }
  // (a side stream that the caller has given work or is recording is left alone; asking whether it has work would end the recording)
  const bool ask_side = e == hipSuccess && !capturing(side) && hipStreamQuery(side) == hipSuccess;
  (void)hipGetLastError();
  while (e == hipSuccess && n < kPrepTries && most < 3) {
    if ((e = hipStreamCreateWithFlags(&s[n], hipStreamNonBlocking)) != hipSuccess) break;
    const int clear = 2 * side_by_side(main, s[n], ea, eb) + (!ask_side || side_by_side(side, s[n], ea, eb));
    if (clear > most) { most = clear; best = n; }
    ++n;
  }
  for (int i = 0; i < n; ++i)
    if (i != best) (void)hipStreamDestroy(s[i]);
  if (ea) (void)hipEventDestroy(ea);
  if (eb) (void)hipEventDestroy(eb);
  if (best < 0) return e;
  *out = s[best];
  return hipSuccess;
}

// life of a step context
enum State { FREE = 0, PREPARED = 1, FETCHED = 2 };
enum { P_PREPARE = 0, P_FETCH = 1, P_LOOKUP = 2, P_BACKWARD = 3, P_SEG_STREAM = 4, P_SEG_FINISH = 5,
       P_ADAGRAD = 6, P_N = 7 };

struct EventPair {
  hipEvent_t a, b;
  bool extra = false;   // adds to the time of its call but is not a call of its own
};

struct StepCtx {
  int state = FREE;
  int t = 0;                          // step number
  int64_t n_ids = 0, n_bags = 0;
  const int64_t* d_offsets = nullptr; // caller's buffers of this step
  int64_t* d_unique = nullptr;
  int32_t *d_inverse = nullptr, *d_slot = nullptr, *d_miss = nullptr;
  Ctr* ctr = nullptr;                 // device counters of this step
  int64_t* perm64 = nullptr;          // [max_ids] positions grouped by virtual id
  int64_t* grp = nullptr;             // [max_ids] per virtual id: (positions << 32) | start of its group
  int2* cold_pay = nullptr;           // [max_ids] per virtual id: the gradient rows of a cold group (-1 = none)
  int* pos_slot = nullptr;            // [max_ids] cache row of each position
  int* victim_slot = nullptr;         // [max_ids]
  int64_t* victim_id = nullptr;       // [max_ids]
  int* miss_row = nullptr;            // [max_ids] cache row of each miss (bypass rows already offset)
  int64_t* miss_id = nullptr;         // [max_ids] id of each miss
  int boff = 0;                       // bypass slot C + j lives at row C + boff + j
  hipEvent_t ev_prepared = nullptr;   // the step's prepare kernels have run (lookahead 0: all but the grouping pass)
  hipEvent_t ev_fetched = nullptr;    // the side-stream launch of the step's Host copies has run
  bool updated = false;               // backward_update has been enqueued for this step
  bool discarded = false;             // freed by sfc_discard: the step's copies may still be running
  bool copies_on_main = false;        // this step's copies run on the main stream
  bool told = false;                  // ev_prepared was completed by the grouping pass's own dispatch
  bool grouping_due = false;          // lookahead 0: the grouping pass goes out with sfc_fetch_misses (ungrouped: the rows of the positions)
  bool ungrouped = false;             // prepared without its grouping (see group_now)
  SortGeom sg{};                      // shape of the step's counting and grouping passes
  bool joined = false;                // the main stream is behind the side-stream launch of the step's copies
  // pipelined mode: the second launch of the Host copies, due on the main stream behind the
  // update of step main_after; bypass_from: see k_swap_rows (kIntMax: no older step was in flight)
  bool main_pending = false;
  int main_after = 0, bypass_from = kIntMax;
};

constexpr int kMaxCtx = 4;

}  // namespace

struct sfc_cache {
  sfc_config cfg{};
  int64_t C = 0, V = 0, max_ids = 0, max_bags = 0;
  int D = 0, d4 = 0, nctx = 1;
  hipStream_t st = nullptr, side = nullptr;     // main stream; stream of the Host copies
  hipStream_t prep = nullptr;                   // stream of the prepare kernels
  bool own_prep = false;                        // prep was created here (lookahead >= 1)
  hipEvent_t ev_tmp = nullptr;                  // cross-stream ordering inside one call
  // device memory
  float *cw = nullptr, *ca = nullptr;           // rows [(C + nctx * max_ids), D] and their optimizer state [.., S]
  int S = 0, s4 = 0;                            // floats / 16-byte chunks of optimizer state per row
  int64_t* slot_id = nullptr;                   // [C]
  int* stamp = nullptr;                         // [C]
  IdxEntry* index = nullptr; uint32_t hi = 0;   // cache index, hashed kind
  int* dmap = nullptr;                          // cache index, dense kind: [V] slot per id or -1 (else nullptr)
  int* hist = nullptr; int hist_len = 0;        // [max_steps + 2]
  // batch table [2*max_ids]: id and smallest position, 8 bytes per entry (16: see `wide`); vid per entry
  uint64_t* utab = nullptr; int* uvid = nullptr;
  bool wide = false;                            // entries of two words (WideTab)
  int* hslot = nullptr;                         // [max_ids]
  int* vid_hslot = nullptr;                     // [max_ids]
  int* blk_cnt = nullptr;                       // [max_ids / kPosChunk + 1]
  unsigned* first = nullptr;                    // [max_ids / 32 + ..] bit per position: first appearance of its id; zero between steps
  int *tile_lt = nullptr, *tile_eq = nullptr;   // [C / kPosChunk + 1]
  int* tile_miss = nullptr;                     // [max_ids / kVidTile + 1]
  // positions per virtual id [max_ids] and its copies for the lowest virtual ids [kHotRep, kHotBins] (zero between steps)
  int *cnt = nullptr, *cnt_rep = nullptr;
  int* cur_rep = nullptr;                       // [kHotRep, kHotBins] group cursors of the lowest virtual ids, one per copy
  int* n_unique = nullptr;                      // unique ids of the step whose unique passes ran last
  int* pos2bag = nullptr;                       // [max_ids] multi-hot: bag of each position
  int* vids = nullptr;                          // [max_ids] lookahead 0: virtual id of each position of an ungrouped step
  int64_t* bag_ends = nullptr;                  // [max_bags + 1] ... and its offsets
  int* tile_cnt = nullptr;                      // [max_ids / kVidTile + 1]
  int* tile_reuse = nullptr;                    // [max_ids / kVidTile + 1] deleted index entries reused per tile
  int* n_invalid = nullptr;                     // out-of-range positions of the step being prepared
  int* age_hist = nullptr;                      // [kAgeBins] hits of the step by age, zero between steps
  double* bp = nullptr; int* bp_vid = nullptr;  // [2 * blocks, D] edge partial sums of k_seg_stream, or the shares of k_update_groups
  int* share_ticket = nullptr;                  // [kMaxShares] shares that have arrived (k_update_groups), zero between steps
  float* gsum = nullptr;                        // [max_ids, D] common gradients of the step
  float* warm_sink = nullptr;                   // one float that k_warm_rows never writes
  HostRows host{};                              // device view of the Host table
  HostStatus* hstat = nullptr;                  // pinned status block (host view); d_hstat its device view
  HostStatus* d_hstat = nullptr;
  int reported_bad_step = 0;                    // last malformed-offsets step that sfc_check has returned
  int device = 0;                               // the GPU this cache lives on
  std::vector<void*> allocs;
  // steps
  StepCtx ctx[kMaxCtx];
  int t = 0;                                    // steps prepared so far
  bool updated_once = false;                    // an update has been enqueued: resident rows may differ from the Host table's
  int last_prepared = -1;                       // context of the most recent sfc_prepare
  int served = 0;                               // steps given up since a gradient came last, up to kServing
  bool recorded = false;                        // every batch is grouped by its prepare (see recording)
  // profiling
  int prof = 0;                                 // 0 off, 1 step calls, 2 also the kernels inside them
  std::vector<EventPair> pending[P_N], spare;
  double ms_sum[P_N] = {};
  int64_t calls[P_N] = {};
};

namespace {

template <typename T>
int dalloc(sfc_cache* c, T** p, int64_t n) {
  if (n < 1) n = 1;
  void* q = nullptr;
  hipError_t e = hipMalloc(&q, (size_t)n * sizeof(T));
  if (e != hipSuccess) return fail(SFC_ENOMEM, "hipMalloc", e);
  c->allocs.push_back(q);
  *p = (T*)q;
  return SFC_OK;
}

template <typename T>
void fill(hipStream_t s, T* p, int64_t n, T v) {
  if (n <= 0) return;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_fill<T>, dim3((unsigned)blocks), dim3(256), 0, s, p, n, v);
}

// bits that hold any position of a batch of n
int pos_bits(int64_t n) {
  int b = 1;
  while (b < 62 && ((int64_t)1 << b) < n) ++b;
  return b;
}

int grid_for(int64_t items, int per_block, int cap) {
  int64_t b = (items + per_block - 1) / per_block;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return (int)b;
}

bool prof_on(const sfc_cache* c, int which) { return c->prof >= (which > P_BACKWARD ? 2 : 1); }

int prof_begin(sfc_cache* c, int which, hipStream_t s, EventPair* ep) {
  if (!prof_on(c, which)) return SFC_OK;
  if (!c->spare.empty()) { *ep = c->spare.back(); c->spare.pop_back(); }
  else { HIPCHK(hipEventCreate(&ep->a)); HIPCHK(hipEventCreate(&ep->b)); }
  ep->extra = false;
  HIPCHK(hipEventRecord(ep->a, s));
  return SFC_OK;
}
// a pair of events for a timed launch (see LAUNCH_TIMED)
int prof_events(sfc_cache* c, EventPair* ep) {
  if (!c->spare.empty()) { *ep = c->spare.back(); c->spare.pop_back(); }
  else { HIPCHK(hipEventCreate(&ep->a)); HIPCHK(hipEventCreate(&ep->b)); }
  ep->extra = false;
  return SFC_OK;
}

// Launches a kernel; when profile entry `which` is on (and `timed`), the dispatch itself records
// the kernel's start and end in a pair of events, so the time read back is the kernel's own
// duration, as a profiler's kernel trace reports it, without the launch latency that a bracket
// of hipEventRecord calls around the launch would include.
#define LAUNCH_TIMED(c, which, timed, kernel, grid, block, s, ...) \
  LAUNCH_TIMED_X(c, which, timed, false, kernel, grid, block, s, __VA_ARGS__)
// extra: the kernel's time is added to the entry, but it is not a call of its own
#define LAUNCH_TIMED_X(c, which, timed, extra_, kernel, grid, block, s, ...)                     \
  do {                                                                                           \
    if ((timed) && prof_on(c, which)) {                                                          \
      EventPair ep_{};                                                                           \
      if (int rc_ = prof_events(c, &ep_)) return rc_;                                            \
      ep_.extra = (extra_);                                                                      \
      hipExtLaunchKernelGGL(kernel, grid, block, 0, s, ep_.a, ep_.b, 0, __VA_ARGS__);            \
      c->pending[which].push_back(ep_);                                                          \
    } else {                                                                                     \
      hipLaunchKernelGGL(kernel, grid, block, 0, s, __VA_ARGS__);                                \
    }                                                                                            \
  } while (0)

// Launches a kernel; with `tells` the dispatch itself completes the event.  A record behind the launch is a
// packet of its own: 6.6 us from launch to launch on the GPU against 4.0, and 1.1 us of host time.
// (What is recorded into a graph is a launch and an event of their own.)
#define LAUNCH_THEN(tells, event, kernel, grid, block, s, ...)                                   \
  do {                                                                                           \
    if (tells) hipExtLaunchKernelGGL(kernel, grid, block, 0, s, nullptr, event, 0, __VA_ARGS__); \
    else hipLaunchKernelGGL(kernel, grid, block, 0, s, __VA_ARGS__);                             \
  } while (0)
int prof_end(sfc_cache* c, int which, hipStream_t s, EventPair* ep) {
  if (!prof_on(c, which)) return SFC_OK;
  HIPCHK(hipEventRecord(ep->b, s));
  c->pending[which].push_back(*ep);
  return SFC_OK;
}
int prof_collect(sfc_cache* c) {
  for (int w = 0; w < P_N; ++w) {
    for (EventPair& ep : c->pending[w]) {
      float ms = 0.f;
      HIPCHK(hipEventSynchronize(ep.b));
      HIPCHK(hipEventElapsedTime(&ms, ep.a, ep.b));
      c->ms_sum[w] += ms;
      if (!ep.extra) c->calls[w] += 1;
      c->spare.push_back(ep);
    }
    c->pending[w].clear();
  }
  return SFC_OK;
}

// One read of pinned memory, no waiting: has a device-side consistency check fired?
int healthy(sfc_cache* c) {
  const volatile HostStatus* h = c->hstat;
  if (h && h->err) {
    // 1: a lookup walked the whole index, 2: so did an insert, 3: a victim was not in the index,
    // 4: more victims than the recency histogram promised
    char msg[128];
    snprintf(msg, sizeof msg, "cache manager state is inconsistent (device check %d at step %d)",
             h->err, h->err_step);
    return fail(SFC_ECORRUPT, msg);
  }
  return SFC_OK;
}

constexpr int64_t kBesidePlanMax = (int64_t)1 << 20;   // see plan_and_assign
constexpr int kGridCap = 2048;   // blocks of the grid-stride kernels whose size lives on the device
constexpr int kRebuildGrid = 2048; // blocks of the two launches that only work when the index is rebuilt

// The step that lookup / segment_sum / backward_update act on: the oldest one whose rows are (or
// are about to be) in place and that has not been updated yet.
StepCtx* training_ctx(sfc_cache* c) {
  StepCtx* best = nullptr;
  for (int k = 0; k < c->nctx; ++k) {
    StepCtx* x = &c->ctx[k];
    if (x->state == FETCHED && !x->updated && (!best || x->t < best->t))
      best = x;
  }
  return best;
}

// The copies are bound by the host link: with other kernels beside them (lookahead > 0) 32 blocks x 256
// lanes x 16 bytes in flight saturate it well enough, and a wider grid only slows those kernels.
constexpr int kSwapBlocks = 32;
// A step that moves hundreds of megabytes over the link (a miss-dominated workload) is bound by
// the link whatever else runs: there a wider grid is worth its disturbance of the other streams
// (128 blocks: 16.3 against 18.6 ms per step with 4e6 misses of 128 bytes per step).  With lookahead 0
// the copies have the GPU to themselves, and the wider grid is the faster one at every size (128 against
// 32 blocks: 20.6e3 misses of 960 bytes 532 / 590 us, 52.7e3 of 128 bytes 236 / 256, 58.2e3 of 256
// 394 / 412, 1.05e6 of 128 3749 / 4130; 64 blocks 541 / 250 / 408 / 3767, 256 blocks as 128).  The host
// cannot know a step's misses without waiting, so it goes by the latest count the device has
// published in the status block, which is a step or two old.
constexpr int kSwapBlocksWide = 128;
constexpr int64_t kSwapWideBytes = (int64_t)256 << 20;
// Lookahead 0: steps whose misses (judged as above) are at most this many bytes run their copies on
// the main stream (see swap_on_main): the way there and back took 33 us of GPU time and 20 us of host time between the
// prepare and the lookup, as much as 1 MiB each way takes on the link (a pass of 1024 x 39 ids with 0.88 MB
// of misses: 193 -> 147 us).
constexpr int64_t kSwapMainBytes = (int64_t)1 << 20;

// Misses of the latest step whose counters the device has published; -1: none yet.
int64_t recent_misses(const sfc_cache* c) {
  const uint64_t w = ((const volatile HostStatus*)c->hstat)->word[kStatMiss];
  return w ? (int64_t)(uint32_t)w : -1;
}

// Do this step's copies run on the main stream?  With lookahead 0 they stand between the prepare and the
// lookup of that stream, so a step that moves little stays there (kSwapMainBytes), but only while the side
// stream has nothing to do: what the caller has given that stream before sfc_fetch_misses comes before the
// copies.  (Asking takes the host half a microsecond; an event between the two streams in every step took a
// pass of 32 x 39 ids from 20 to 34 us or more, one of 1024 x 39 from 120 to 144.)
bool swap_on_main(sfc_cache* c) {
  if (c->nctx > 1) return false;
  if (c->side == c->st) return true;
  const int64_t recent = recent_misses(c);
  if (recent < 0 || recent * (c->d4 + c->s4) * 16 > kSwapMainBytes) return false;
  // (while the main stream is being captured the copies are recorded as a fork to the side stream: what that
  // stream is doing now says nothing about the time of the graph's launch)
  if (capturing(c->st)) return false;
  if (hipStreamQuery(c->side) == hipSuccess) return true;
  if (hipPeekAtLastError() == hipErrorNotReady) (void)hipGetLastError();
  return false;
}

// Have the victims to be written to the Host table?  Not while no update has ever been enqueued on this cache: every
// resident row is then as it was read.  (A graph may be launched when that has changed: what is recorded writes.)
bool writes_back(const sfc_cache* c) { return c->updated_once || capturing(c->st); }

ScatterArgs scatter_args(const sfc_cache* c, const StepCtx* x) {
  return ScatterArgs{x->d_inverse, x->d_offsets ? c->pos2bag : nullptr, (int)x->n_ids, x->grp, (int*)x->cold_pay, c->cur_rep,
                     x->sg.bins, x->sg.shift, x->sg.nrep, x->perm64, x->d_slot, x->pos_slot, (int)c->C, x->boff, (int)x->n_bags};
}

RowsArgs rows_args(const sfc_cache* c, const StepCtx* x) {
  return RowsArgs{x->d_inverse, x->d_slot, (int)x->n_ids, (int)c->C, x->boff, x->pos_slot};
}

// One launch of the Host<->cache copies of a step on stream s (see k_swap_rows for the two
// launches of pipelined mode).
int launch_swap(sfc_cache* c, StepCtx* x, hipStream_t s, int main_variant) {
  EventPair ep{};
  int rc;
  // the copies read the step's counters, miss list and victim list: its prepare comes first
  if (s != c->prep) HIPCHK(hipStreamWaitEvent(s, x->ev_prepared, 0));
  if ((rc = prof_begin(c, P_FETCH, s, &ep))) return rc;
  ep.extra = main_variant != 0;          // the second launch of a step: same call
  const int64_t recent_bytes = recent_misses(c) * (c->d4 + c->s4) * 16;
  const int swap_blocks = c->nctx == 1 || recent_bytes > kSwapWideBytes ? kSwapBlocksWide : kSwapBlocks;
  int blocks = grid_for(x->n_ids * (c->d4 + c->s4), 256, swap_blocks), staged_at = -1;
  // where victims are possible, and the copies have the side stream to themselves (see k_stage_victims)
  const bool write_back = writes_back(c);
  if (c->nctx == 1 && !x->copies_on_main && write_back && c->C > 0 && c->C < c->V && x->n_ids >= kSplitMin) {
    staged_at = (int)c->C + x->boff;
    blocks = kSplitWriters + kSplitReaders;
    hipLaunchKernelGGL(k_stage_victims, dim3(1024), dim3(256), 0, s, x->victim_slot, (float4*)c->cw,
                       (float4*)c->ca, (int)c->C, x->boff, c->d4, c->s4, (const Ctr*)x->ctr);
  }
  const bool tells = !main_variant && s != c->st;
  const SwapArgs args{x->miss_row, x->miss_id, x->victim_id, (float4*)c->cw, (float4*)c->ca, c->host, c->d4, c->s4,
                      (const Ctr*)x->ctr, x->bypass_from, main_variant, staged_at, write_back ? 1 : 0};
  if (x->grouping_due && x->ungrouped) {      // (copies on the main stream: see sfc_fetch_misses)
    x->grouping_due = false;
    hipLaunchKernelGGL(k_swap_pos_rows, dim3(blocks + (unsigned)((x->n_ids + 1023) / 1024)), dim3(256), 0, s, args, blocks,
                       rows_args(c, x));
  } else if (x->grouping_due) {
    x->grouping_due = false;
    hipLaunchKernelGGL(k_swap_scatter, dim3(blocks + x->sg.blocks), dim3(256), 0, s, args, blocks, scatter_args(c, x));
  } else {
    LAUNCH_THEN(tells && !prof_on(c, P_FETCH) && !capturing(s), x->ev_fetched, k_swap_rows, dim3(blocks), dim3(256), s, args);
  }
  HIPCHK(hipGetLastError());
  if ((rc = prof_end(c, P_FETCH, s, &ep))) return rc;
  if (main_variant) x->main_pending = false;
  else if (tells && (prof_on(c, P_FETCH) || capturing(s))) HIPCHK(hipEventRecord(x->ev_fetched, s));
  return SFC_OK;
}

// The main stream behind the side-stream launch of the step's copies (once per step: every
// cross-stream wait costs the host and the GPU microseconds).
int join_copies(sfc_cache* c, StepCtx* x) {
  if (!x->joined) HIPCHK(hipStreamWaitEvent(c->st, x->ev_fetched, 0));
  x->joined = true;
  return SFC_OK;
}

// Before main-stream work that reads the step's rows: both launches of its copies come first.
int rows_ready(sfc_cache* c, StepCtx* x) {
  int rc;
  if (x->main_pending && (rc = launch_swap(c, x, c->st, 1))) return rc;
  return join_copies(c, x);
}

// common[v] = segment sum of d_grad over the step's grouping: the stream, then the block-edge partials.
// bp / bp_vid: the block-edge partial sums and their virtual ids, 2 per block of the stream; timed:
// bracket the kernels with profiling events (which may have to be created).
// fused (sfc_backward_update with the Adagrad kernel): the stream passes over the cold groups and
// marks the groups it leaves as block-edge partials, and no finish kernel runs: the optimizer
// kernel chains the *n_slots partials itself.
int seg_launch(sfc_cache* c, StepCtx* x, const float* d_grad, float* d_common, double* bp,
               int* bp_vid, bool timed, bool fused, int* n_slots) {
  const int n = (int)x->n_ids;
  if (n_slots) *n_slots = 0;
  if (n <= 0) return SFC_OK;
  const SegGeom g = seg_geom(c->D, n);
  const int nblk = (g.waves + 3) / 4;
  auto kern = x->d_offsets ? (fused ? k_seg_stream<false, true> : k_seg_stream<false, false>)
                           : (fused ? k_seg_stream<true, true> : k_seg_stream<true, false>);
  LAUNCH_TIMED(c, P_SEG_STREAM, timed, kern, dim3(nblk), dim3(256), c->st, (const float4*)d_grad,
               (const int64_t*)x->perm64, n, c->d4, g.G, g.L, (float4*)d_common, bp, bp_vid,
               fused ? (int*)x->cold_pay : (int*)nullptr);
  if (n_slots) *n_slots = 2 * nblk;
  if (fused) return SFC_OK;
  LAUNCH_TIMED(c, P_SEG_FINISH, timed, k_seg_finish, dim3((unsigned)edge_blocks(2 * nblk, c->d4)), dim3(256), c->st,
               (const double*)bp, (const int*)bp_vid, 2 * nblk, c->d4, (float4*)d_common);
  return SFC_OK;
}

GroupArgs group_args(const sfc_cache* c, const StepCtx* x, bool grouped) {
  return GroupArgs{grouped ? c->cnt : nullptr, c->cnt_rep, c->cur_rep, x->sg.bins, x->sg.nrep, c->tile_cnt, x->grp,
                   x->cold_pay};
}

// The prepare's kernels behind the resolve: victims' plan (and sums and bags of the positions), victims' lists,
// slots of the misses.  (Called where the resolve has run on c->prep; group_positions follows.)
void plan_and_assign(sfc_cache* c, StepCtx* x) {
  hipStream_t s = c->prep;
  const int n = (int)x->n_ids;
  const SortGeom& sg = x->sg;
  // a cache that holds the whole table never evicts: there is a free slot for every id that is not resident
  const bool evicts = c->C < c->V;
  // Pipelined, the kernels of other streams hold the compute units, and blocks of 1024 threads wait for a whole one.
  // 2.56e6 ids, lookahead 2, ms per step, positions added up by kernels of 256 threads / beside the plan / with the
  // victims' count: 0.463 / 0.465 / 0.461 (k_plan and k_victim_count among the other streams' kernels 43 + 19 us beside
  // the plan, 18 + 30 otherwise).  Smaller batches have few such blocks (639e3 ids 0.283 / 0.277 / 0.277, 213e3 with
  // lookahead 1 137 us a pass beside the plan, 139 otherwise); in order 1024 x 39 ids take 102.0 us a pass beside the
  // plan, 102.6 otherwise.
  const bool beside_plan = !evicts || c->nctx == 1 || n < kBesidePlanMax;
  const int ft = beside_plan ? 1024 : 256;
  const FoldArgs fo{c->cnt, c->cnt_rep, sg.bins, sg.nrep, c->tile_cnt, x->ungrouped ? 0 : grid_for(n, ft, kFoldThreads / ft)};
  const BagArgs bags{x->d_offsets, (int)x->n_bags, n, c->pos2bag, x->ungrouped ? c->bag_ends : nullptr, 1};
  const int riders = fo.folds + (n > 0 && x->d_offsets ? (int)((x->n_bags + ft - 1) / ft) : 0);
  hipLaunchKernelGGL(k_plan, dim3(1 + (beside_plan ? riders : 0)), dim3(1024), 0, s, c->tile_miss, c->age_hist,
                     c->tile_reuse, c->hist, x->t, c->cfg.lookahead, (int)c->C, c->hi, c->dmap ? 1 : 0, x->ctr, fo, bags);
  if (evicts) {
    const int gs = grid_for(c->C, kPosChunk, kGridCap);
    hipLaunchKernelGGL(k_victim_count, dim3(gs + (beside_plan ? 0 : riders)), dim3(256), 0, s, c->stamp, c->tile_lt,
                       c->tile_eq, x->ctr, gs, fo, bags);
    hipLaunchKernelGGL(k_victim_write, dim3(gs), dim3(256), 0, s, c->stamp, c->slot_id, c->tile_lt,
                       c->tile_eq, x->victim_slot, x->victim_id, x->ctr, c->dmap, c->index, c->hi);
  }
  const int gv = grid_for(n, kVidTile, kGridCap);
  hipLaunchKernelGGL(k_assign_misses, dim3(gv), dim3(256), 0, s, x->d_unique, group_args(c, x, !x->ungrouped), c->tile_miss,
                     x->victim_slot, x->d_slot, x->d_miss, x->miss_row, x->miss_id, x->boff, c->slot_id,
                     c->stamp, c->index, c->hi, c->dmap, x->t, (int)c->C, c->tile_reuse, x->ctr);
}

// The grouping pass, on c->prep behind the above.  The Host copies need nothing of it: with lookahead 0
// sfc_fetch_misses launches it behind the event that lets the copies go, so that the way to the side stream
// (12 us) and this pass, beside the copies' first round trips, cost no time of their own.  (Not in the
// prepare with the event in front of it: the copies come behind what the caller gives the main stream
// between the two calls.)  Pipelined, the grouping is on the path of the next prepare and stays in its own.
// A step that is not grouped has the rows of its positions written down in its place.
int group_positions(sfc_cache* c, StepCtx* x, bool extra) {
  x->grouping_due = false;
  x->told = false;
  const int n = (int)x->n_ids;
  if (n <= 0) return SFC_OK;
  hipStream_t s = c->prep;
  const SortGeom& sg = x->sg;
  EventPair ep{};
  int rc;
  if (extra && (rc = prof_begin(c, P_PREPARE, s, &ep))) return rc;
  ep.extra = true;
  if (x->ungrouped) {
    hipLaunchKernelGGL(k_pos_rows, dim3((unsigned)((x->n_ids + 1023) / 1024)), dim3(256), 0, s, rows_args(c, x));
    return extra ? prof_end(c, P_PREPARE, s, &ep) : SFC_OK;
  }
  auto scat = sg.shift == 10 ? k_scatter<4, 256> : sg.shift == 12 ? k_scatter<8, 512> : k_scatter<8, 1024>;
  const int threads = sg.shift == 10 ? 256 : sg.shift == 12 ? 512 : 1024;
  // pipelined it is the last kernel of the prepare
  const bool tells = c->nctx > 1 && !capturing(s);
  LAUNCH_THEN(tells, x->ev_prepared, scat, dim3(sg.blocks), dim3(threads), s, scatter_args(c, x));
  x->told = tells;
  if (extra) return prof_end(c, P_PREPARE, s, &ep);
  return SFC_OK;
}

// Lookahead 0: a cache that has given up this many steps in a row without a gradient in between serves lookups, and
// its batches beyond the one-block prepare are prepared without the grouping of their positions, which the backward
// half alone reads: counts and ranks, sums, bags, starts of the groups and the grouping pass.  The rows of the positions,
// for the gather, are written down where the grouping pass would run.  A gradient that comes all the same (sfc_segment_sum,
// sfc_backward_update) has its step grouped first (group_now), and the following ones are grouped by their prepares again.
// Not while the stream is captured, and not once a gradient has been recorded: see recording.  Not with lookahead > 0: the
// grouping of one step would then run on the main stream, in scratch that the prepare of a later step is using on its own.
// us a pass looked up and given up, every row resident, grouped / not, and what the first sum takes longer when its step is grouped
// late (five launches): one-hot 8e3 ids of dim 16 32 / 29.5, 27; 50e3 of dim 32 38 / 33.5, 23; 639e3 of dim 16 86 / 65, 50;
// 2.56e6 of dim 32 215 / 161, 86; bags, 293e3 ids of dim 128 72 / 55, 35; 420e3 of dim 32 72 / 52, 38; 895e3 of dim 16 92 / 66, 53; 53e3,
// hashed, a third resident, 44 / 40, 38.  So a late grouping is paid back by 2 to 12 steps; behind 64, programs that validate on a
// few batches and train on have none, and one that trains on a single batch after each 65th loses half a microsecond a step.
// (The one-hot gather through the virtual id to the slot, without the rows written down: 639e3 63.5, 2.56e6 153; but it
// reads the caller's d_inverse and d_slot later than the grouping pass does.)
constexpr int kServing = 64;

// Called by what reads the groups of the positions: is it being recorded?  Then its graph may be launched behind
// any later prepare and reads the same arrays then; the host sees neither that nor that the steps it gives up have had a
// gradient.  So all further batches are grouped by their prepares.  (Those of the one-block prepare are in any case, and what is recorded with
// one of them fits no larger batch: the numbers of ids and bags are part of it.)
bool recording(sfc_cache* c, const StepCtx* x) {
  if (c->nctx > 1 || x->sg.bins == 0 || (c->recorded && !x->ungrouped) || !capturing(c->st)) return false;
  return c->recorded = true;
}

// What is only recorded has not run: the step stays as it is for the calls that follow, which do the same again if they come.
// And launched behind a later step it does nothing: these kernels go by the number in the step's counters.
// timed: its time is added to the prepare's (not where no events may be created, and not what is only recorded).
int group_now(sfc_cache* c, StepCtx* x, bool timed) {
  const bool later = recording(c, x);
  c->served = 0;
  if (!x->ungrouped) return SFC_OK;
  if (!later) x->ungrouped = false;
  hipStream_t s = c->st;                        // (lookahead 0: the prepares run here as well)
  EventPair ep{};
  int rc;
  timed = timed && !later;
  if (timed && (rc = prof_begin(c, P_PREPARE, s, &ep))) return rc;
  ep.extra = true;
  const int n = (int)x->n_ids;
  const SortGeom& sg = x->sg;
  const Ctr* const ctr = x->ctr;
  fill<int>(s, c->cnt, n, 0);
  // (all of it from what the prepare has kept: the caller's virtual ids and offsets may be gone; ranks where the table
  // entries were)
  const RankArgs rank{nullptr, nullptr, n, c->vids, c->cnt, c->cnt_rep, sg.nrep, c->hslot, nullptr};
  auto count = sg.shift == 10 ? k_count_late<1, 1024> : sg.shift == 12 ? k_count_late<8, 512> : k_count_late<8, 1024>;
  hipLaunchKernelGGL(count, dim3(sg.blocks), dim3(sg.shift == 12 ? 512 : 1024), 0, s, rank, ctr, x->t);
  const FoldArgs fo{c->cnt, c->cnt_rep, sg.bins, sg.nrep, c->tile_cnt, grid_for(n, 256, kFoldThreads / 256)};
  const BagArgs bags{c->bag_ends, (int)x->n_bags, n, c->pos2bag, nullptr, 0};
  hipLaunchKernelGGL(k_fold_late, dim3(fo.folds + (x->d_offsets ? (unsigned)((x->n_bags + 255) / 256) : 0u)), dim3(256), 0, s,
                     x->ctr, fo, bags, x->t);
  hipLaunchKernelGGL(k_starts_late, dim3(grid_for(n, kVidTile, kGridCap)), dim3(256), 0, s, group_args(c, x, true), ctr, x->t);
  auto scat = sg.shift == 10 ? k_scatter_late<4, 256> : sg.shift == 12 ? k_scatter_late<8, 512> : k_scatter_late<8, 1024>;
  ScatterArgs sc = scatter_args(c, x);
  sc.inverse = c->vids; sc.rank_slot = c->hslot;
  hipLaunchKernelGGL(scat, dim3(sg.blocks), dim3(sg.shift == 10 ? 256 : sg.shift == 12 ? 512 : 1024), 0, s, sc, ctr, x->t);
  return timed ? prof_end(c, P_PREPARE, s, &ep) : SFC_OK;
}

int sync_all(sfc_cache* c) {
  HIPCHK(hipStreamSynchronize(c->st));
  if (c->side != c->st) HIPCHK(hipStreamSynchronize(c->side));
  if (c->prep != c->st && c->prep != c->side) HIPCHK(hipStreamSynchronize(c->prep));
  return SFC_OK;
}

}  // namespace

extern "C" {

const char* sfc_strerror(int code) {
  switch (code) {
    case SFC_OK: return "ok";
    case SFC_EINVAL: return "invalid argument";
    case SFC_ESTATE: return "call out of order";
    case SFC_EHIP: return "HIP runtime error";
    case SFC_ENOMEM: return "out of memory";
    case SFC_ELIMIT: return "step limit reached";
    case SFC_ECORRUPT: return "cache manager state inconsistent";
    default: return "unknown error";
  }
}
const char* sfc_last_error(void) { return g_err.c_str(); }

void* sfc_host_alloc(int64_t bytes) {
  void* p = nullptr;
  if (bytes <= 0) return nullptr;
  {
    // several large pinned pieces at once have crashed the runtime at the next kernel launch
    // (see the header): refuse that layout instead of handing it out
    std::lock_guard<std::mutex> lk(g_host_mu);
    int64_t total = bytes;
    bool other_large = false;
    for (auto& kv : g_host_allocs) { total += kv.second; other_large |= kv.second >= SFC_HOST_ALLOC_LARGE_BYTES; }
    if (other_large && bytes >= SFC_HOST_ALLOC_LARGE_BYTES && total > SFC_HOST_ALLOC_MAX_BYTES) {
      fail(SFC_ENOMEM, "sfc_host_alloc: a second large pinned piece would take the total beyond "
                       "SFC_HOST_ALLOC_MAX_BYTES; allocate the table as one interleaved piece");
      return nullptr;
    }
  }
  if (hipHostMalloc(&p, (size_t)bytes, hipHostMallocMapped | hipHostMallocPortable) != hipSuccess) {
    (void)hipGetLastError();
    fail(SFC_ENOMEM, "hipHostMalloc failed");
    return nullptr;
  }
  std::lock_guard<std::mutex> lk(g_host_mu);
  g_host_allocs[p] = bytes;
  return p;
}
void sfc_host_free(void* p) {
  if (!p) return;
  { std::lock_guard<std::mutex> lk(g_host_mu); g_host_allocs.erase(p); }
  (void)hipHostFree(p);
}

void sfc_cache_destroy(sfc_cache* c) {
  if (!c) return;
  (void)hipStreamSynchronize(c->st);
  if (c->side != c->st) (void)hipStreamSynchronize(c->side);
  if (c->own_prep && c->prep) (void)hipStreamSynchronize(c->prep);
  for (int w = 0; w < P_N; ++w)
    for (EventPair& ep : c->pending[w]) { (void)hipEventDestroy(ep.a); (void)hipEventDestroy(ep.b); }
  for (EventPair& ep : c->spare) { (void)hipEventDestroy(ep.a); (void)hipEventDestroy(ep.b); }
  if (c->ev_tmp) (void)hipEventDestroy(c->ev_tmp);
  for (int k = 0; k < kMaxCtx; ++k) {
    if (c->ctx[k].ev_prepared) (void)hipEventDestroy(c->ctx[k].ev_prepared);
    if (c->ctx[k].ev_fetched) (void)hipEventDestroy(c->ctx[k].ev_fetched);
  }
  if (c->own_prep && c->prep) (void)hipStreamDestroy(c->prep);
  for (void* p : c->allocs) (void)hipFree(p);
  if (c->hstat) (void)hipHostFree(c->hstat);
  delete c;
}

int sfc_cache_create(const sfc_config* cfg, sfc_cache** out) {
  if (!cfg || !out) return fail(SFC_EINVAL, "null config or output pointer");
  *out = nullptr;
  if (cfg->capacity_rows < 0 || cfg->dim <= 0 || cfg->dim % 4 || cfg->dim > 256)
    return fail(SFC_EINVAL, "capacity_rows must be >= 0 and dim a multiple of 4 in [4, 256]");
  if (cfg->policy != SFC_POLICY_LRU_BATCH && cfg->policy != SFC_POLICY_PREFETCH)
    return fail(SFC_EINVAL, "unknown policy");
  if (cfg->policy == SFC_POLICY_PREFETCH && (cfg->capacity_rows != 0 || cfg->lookahead != 1))
    return fail(SFC_EINVAL, "the Prefetch strategy needs capacity_rows = 0 and lookahead = 1");
  if (cfg->max_ids_per_batch < 1 || cfg->max_bags_per_batch < 1 || cfg->host_rows < 1)
    return fail(SFC_EINVAL, "max_ids_per_batch, max_bags_per_batch and host_rows must be >= 1");
  if (cfg->lookahead < 0 || cfg->lookahead > 3) return fail(SFC_EINVAL, "lookahead must be 0, 1, 2 or 3");
  if (cfg->lookahead > 0 && (!cfg->side_stream || cfg->side_stream == cfg->stream))
    return fail(SFC_EINVAL, "lookahead > 0 needs a side_stream different from stream");
  const int64_t nctx = cfg->lookahead + 1;
  if (cfg->capacity_rows + nctx * cfg->max_ids_per_batch >= (int64_t)1 << 31 ||
      cfg->max_ids_per_batch >= (int64_t)1 << 30 || cfg->max_bags_per_batch >= (int64_t)1 << 31)
    return fail(SFC_EINVAL, "capacity_rows + (lookahead + 1) * max_ids_per_batch must stay below 2^31");
  if (!cfg->h_weights || !cfg->h_acc) return fail(SFC_EINVAL, "null host table");
  if (((uintptr_t)cfg->h_weights | (uintptr_t)cfg->h_acc) & 15)
    return fail(SFC_EINVAL, "host table must be 16-byte aligned");
  if (cfg->host_row_stride && (cfg->host_row_stride < cfg->dim || cfg->host_row_stride % 4))
    return fail(SFC_EINVAL, "host_row_stride must be 0 or a multiple of 4 that is >= dim");
  if (cfg->max_steps < 0) return fail(SFC_EINVAL, "max_steps must be >= 0");
  if (cfg->optimizer < SFC_OPT_ADAGRAD || cfg->optimizer > SFC_OPT_ROWWISE_ADAGRAD)
    return fail(SFC_EINVAL, "unknown optimizer");
  if (cfg->index_kind < SFC_INDEX_AUTO || cfg->index_kind > SFC_INDEX_DENSE)
    return fail(SFC_EINVAL, "unknown index_kind");
  const int S = cfg->optimizer == SFC_OPT_ADAM ? 2 * cfg->dim
              : cfg->optimizer == SFC_OPT_ROWWISE_ADAGRAD ? 4 : cfg->dim;
  if (cfg->host_state_stride && (cfg->host_state_stride < S || cfg->host_state_stride % 4))
    return fail(SFC_EINVAL, "host_state_stride must be 0 or a multiple of 4 that is >= the state size");
  if (cfg->optimizer == SFC_OPT_ADAM &&
      !(cfg->beta1 >= 0.0 && cfg->beta1 < 1.0 && cfg->beta2 >= 0.0 && cfg->beta2 < 1.0))
    return fail(SFC_EINVAL, "Adam needs 0 <= beta1, beta2 < 1");

  sfc_cache* c = new (std::nothrow) sfc_cache;
  if (!c) return fail(SFC_ENOMEM, "host allocation failed");
  c->cfg = *cfg;
  c->C = cfg->capacity_rows; c->V = cfg->host_rows; c->D = cfg->dim; c->d4 = cfg->dim / 4;
  c->S = S; c->s4 = S / 4;
  c->max_ids = cfg->max_ids_per_batch; c->max_bags = cfg->max_bags_per_batch;
  c->nctx = (int)nctx;
  c->st = (hipStream_t)cfg->stream;
  c->side = cfg->side_stream ? (hipStream_t)cfg->side_stream : c->st;
  c->hist_len = (cfg->max_steps ? cfg->max_steps : (1 << 20)) + 2;
  (void)hipGetDevice(&c->device);
  const bool dense = cfg->index_kind == SFC_INDEX_DENSE ||
                     (cfg->index_kind == SFC_INDEX_AUTO &&
                      cfg->host_rows * (int64_t)sizeof(int) <= SFC_DENSE_INDEX_MAX_BYTES);
  if (!dense) {
    // four entries per possible resident id keep probe sequences short (HBM is plentiful); two
    // where four would not fit a 32-bit entry number
    int64_t h = 4 * (c->C + c->max_ids);
    if (h > (int64_t)0xF0000000LL) h = 2 * (c->C + c->max_ids);
    c->hi = (uint32_t)h;
  }
  if (c->hi < 64) c->hi = 64;

  int rc = SFC_OK;
  hipError_t e;
  void* dp = nullptr;
  if ((e = hipHostGetDevicePointer(&dp, cfg->h_weights, 0)) != hipSuccess) {
    rc = fail(SFC_EINVAL, "h_weights is not pinned device-mapped host memory", e); goto bad;
  }
  c->host.w = (float4*)dp;
  if ((e = hipHostGetDevicePointer(&dp, cfg->h_acc, 0)) != hipSuccess) {
    rc = fail(SFC_EINVAL, "h_acc is not pinned device-mapped host memory", e); goto bad;
  }
  c->host.a = (float4*)dp;
  c->host.hs4 = (cfg->host_row_stride ? cfg->host_row_stride : cfg->dim) / 4;
  c->host.has4 = (cfg->host_state_stride ? cfg->host_state_stride : S) / 4;
  // lookahead 0: prepare on the main stream; otherwise on a stream of its own, beside the Host copies of the step
  // before (the Prefetch strategy: on the side stream, ahead of its copies).  One stream and no more: the streams of
  // a process share four hardware queues, and what stands behind a step's copies in one of them waits for hundreds
  // of microseconds.  A second stream, for the unique passes of 2^18 to 2^20 ids beside the rest of the previous prepare,
  // against this one, us a step of one cache / of three in turn: 300e3 ids of dim 16 with lookahead 1 135 -> 114 / 137 -> 108, 639e3
  // 335 -> 313 / 347 -> 325, with lookahead 2 272 -> 272 / 346 -> 326, hashed 277 -> 286 / 365 -> 341, 950e3 398 -> 404 / 466 -> 460;
  // 700e3 in bags of dim 32 145 -> 123 / 128 -> 129.  With caches of 1e6 rows of 1e7, lookahead 2: 639e3 152 -> 124, hashed 165 -> 125, 950e3
  // 404 -> 402 (three of four orders of creation; 545 -> 402 in the other).
  c->prep = cfg->lookahead == 0 ? c->st : c->side;
  if (cfg->lookahead >= 1 && cfg->policy != SFC_POLICY_PREFETCH) {
    if ((e = choose_prep_stream(c->st, c->side, &c->prep)) != hipSuccess) {
      c->prep = nullptr;
      rc = fail(SFC_EHIP, "hipStreamCreate", e); goto bad;
    }
    c->own_prep = true;
  }

  {
    void* hp = nullptr;
    if ((e = hipHostMalloc(&hp, sizeof(HostStatus), hipHostMallocMapped | hipHostMallocPortable)) != hipSuccess) {
      rc = fail(SFC_ENOMEM, "hipHostMalloc (status block)", e); goto bad;
    }
    c->hstat = (HostStatus*)hp;
    memset(c->hstat, 0, sizeof(HostStatus));
    if ((e = hipHostGetDevicePointer(&dp, hp, 0)) != hipSuccess) {
      rc = fail(SFC_EHIP, "hipHostGetDevicePointer (status block)", e); goto bad;
    }
    c->d_hstat = (HostStatus*)dp;
  }
  {
    const int64_t rows = c->C + nctx * c->max_ids;
    // the batch table of a step has max(2 * n_ids, 64) entries (see sfc_prepare)
    const int64_t hu = 2 * c->max_ids < 64 ? 64 : 2 * c->max_ids;
    if ((rc = dalloc(c, &c->cw, rows * c->D))) goto bad;
    if ((rc = dalloc(c, &c->ca, rows * c->S))) goto bad;
    if ((rc = dalloc(c, &c->slot_id, c->C))) goto bad;
    if ((rc = dalloc(c, &c->stamp, c->C))) goto bad;
    if ((rc = dalloc(c, &c->index, (int64_t)c->hi))) goto bad;
    if (dense && (rc = dalloc(c, &c->dmap, c->V))) goto bad;
    if ((rc = dalloc(c, &c->hist, (int64_t)c->hist_len))) goto bad;
    // a position of the largest batch and the largest tag (V) side by side in 64 bits, below all ones
    c->wide = (uint64_t)c->V >= (~0ull >> pos_bits(c->max_ids));
    if ((rc = dalloc(c, &c->utab, c->wide ? 2 * hu : hu))) goto bad;
    if ((rc = dalloc(c, &c->uvid, hu))) goto bad;
    if ((rc = dalloc(c, &c->hslot, c->max_ids))) goto bad;
    if ((rc = dalloc(c, &c->vid_hslot, c->max_ids))) goto bad;
    if ((rc = dalloc(c, &c->blk_cnt, c->max_ids / kPosChunk + 2))) goto bad;
    if ((rc = dalloc(c, &c->first, (c->max_ids / kPosChunk + 1) * (kPosChunk / 32)))) goto bad;
    if ((rc = dalloc(c, &c->tile_lt, c->C / kPosChunk + 2))) goto bad;
    if ((rc = dalloc(c, &c->tile_eq, c->C / kPosChunk + 2))) goto bad;
    if ((rc = dalloc(c, &c->tile_miss, c->max_ids / kVidTile + 2))) goto bad;
    if ((rc = dalloc(c, &c->cnt, c->max_ids))) goto bad;
    if ((rc = dalloc(c, &c->n_unique, 1))) goto bad;
    if ((rc = dalloc(c, &c->pos2bag, c->max_ids))) goto bad;
    if (nctx == 1 && ((rc = dalloc(c, &c->vids, c->max_ids)) || (rc = dalloc(c, &c->bag_ends, c->max_bags + 1)))) goto bad;
    if ((rc = dalloc(c, &c->tile_cnt, c->max_ids / kVidTile + 2))) goto bad;
    if ((rc = dalloc(c, &c->tile_reuse, c->max_ids / kVidTile + 2))) goto bad;
    if ((rc = dalloc(c, &c->age_hist, (int64_t)kAgeBins))) goto bad;
    if ((rc = dalloc(c, &c->n_invalid, 1))) goto bad;
    if ((rc = dalloc(c, &c->cnt_rep, (int64_t)kHotRep * kHotBins))) goto bad;
    if ((rc = dalloc(c, &c->cur_rep, (int64_t)kHotRep * kHotBins))) goto bad;
    {
      const int64_t nw = seg_geom(c->D, c->max_ids).waves + 8;
      const int64_t nwmax = nw > kSegTargetWaves + 8 ? nw : kSegTargetWaves + 8;
      if ((rc = dalloc(c, &c->bp, 2 * nwmax * c->D))) goto bad;
      if ((rc = dalloc(c, &c->bp_vid, 2 * nwmax))) goto bad;
    }
    if ((rc = dalloc(c, &c->share_ticket, (int64_t)kMaxShares))) goto bad;
    if ((rc = dalloc(c, &c->gsum, c->max_ids * c->D))) goto bad;
    if ((rc = dalloc(c, &c->warm_sink, 1))) goto bad;
    for (int k = 0; k < c->nctx; ++k) {
      StepCtx* x = &c->ctx[k];
      if ((rc = dalloc(c, &x->ctr, 1))) goto bad;
      if ((rc = dalloc(c, &x->perm64, c->max_ids))) goto bad;
      if ((rc = dalloc(c, &x->grp, c->max_ids))) goto bad;
      if ((rc = dalloc(c, &x->cold_pay, c->max_ids))) goto bad;
      if ((rc = dalloc(c, &x->pos_slot, c->max_ids))) goto bad;
      if ((rc = dalloc(c, &x->victim_slot, c->max_ids))) goto bad;
      if ((rc = dalloc(c, &x->victim_id, c->max_ids))) goto bad;
      if ((rc = dalloc(c, &x->miss_row, c->max_ids))) goto bad;
      if ((rc = dalloc(c, &x->miss_id, c->max_ids))) goto bad;
      x->boff = (int)(k * c->max_ids);
      if ((e = hipEventCreateWithFlags(&x->ev_prepared, hipEventDisableTiming)) != hipSuccess ||
          (e = hipEventCreateWithFlags(&x->ev_fetched, hipEventDisableTiming)) != hipSuccess) {
        rc = fail(SFC_EHIP, "hipEventCreate", e); goto bad;
      }
    }

    hipStream_t s = c->st;
    fill<int64_t>(s, c->slot_id, c->C, (int64_t)-1);
    fill<int>(s, c->stamp, c->C, 0);
    IdxEntry empty; empty.key = kEmpty; empty.slot = -1; empty.pad = 0;
    fill<IdxEntry>(s, c->index, (int64_t)c->hi, empty);
    if (dense) fill<int>(s, c->dmap, c->V, -1);
    fill<int>(s, c->hist, (int64_t)c->hist_len, 0);
    fill<int>(s, c->age_hist, (int64_t)kAgeBins, 0);
    fill<int>(s, c->n_invalid, 1, 0);
    fill<int>(s, c->cnt_rep, (int64_t)kHotRep * kHotBins, 0);
    fill<int>(s, c->n_unique, 1, 0);
    fill<int>(s, c->share_ticket, (int64_t)kMaxShares, 0);
    fill<int>(s, c->tile_reuse, c->max_ids / kVidTile + 2, 0);
    UEntry uempty; uempty.key = kEmpty; uempty.minpos = kIntMax; uempty.pad = 0;
    if (c->wide) fill<UEntry>(s, (UEntry*)c->utab, hu, uempty);
    else fill<uint64_t>(s, c->utab, hu, ~0ull);
    fill<unsigned>(s, c->first, (c->max_ids / kPosChunk + 1) * (kPosChunk / 32), 0u);
    Ctr z; memset(&z, 0, sizeof z); z.oldest = 1; z.hstat = c->d_hstat; z.dense = dense ? 1 : 0;
    for (int k = 0; k < c->nctx; ++k)
      if ((e = hipMemcpyAsync(c->ctx[k].ctr, &z, sizeof z, hipMemcpyHostToDevice, s)) != hipSuccess) {
        rc = fail(SFC_EHIP, "cache initialisation", e); goto bad;
      }
    if ((e = hipEventCreateWithFlags(&c->ev_tmp, hipEventDisableTiming)) != hipSuccess ||
        (e = hipStreamSynchronize(s)) != hipSuccess || (e = hipGetLastError()) != hipSuccess) {
      rc = fail(SFC_EHIP, "cache initialisation", e); goto bad;
    }
  }
  *out = c;
  return SFC_OK;
bad:
  sfc_cache_destroy(c);
  return rc;
}

int sfc_prepare(sfc_cache* c, const int64_t* d_ids, int64_t n_ids, const int64_t* d_offsets,
                int64_t n_bags, int64_t* d_unique_ids, int32_t* d_inverse, int32_t* d_slot,
                int32_t* d_miss_vids) {
  if (!c) return fail(SFC_EINVAL, "null cache");
  if (int hrc = healthy(c)) return hrc;
  if (n_ids < 0 || n_bags < 0 || n_ids > c->max_ids || n_bags > c->max_bags)
    return fail(SFC_EINVAL, "n_ids / n_bags out of range");
  if (!d_offsets && n_bags != n_ids) return fail(SFC_EINVAL, "one-hot input needs n_bags == n_ids");
  if (d_offsets && n_bags == 0 && n_ids > 0) return fail(SFC_EINVAL, "multi-hot input with ids but no bags");
  if ((n_ids > 0 && !d_ids) || !d_unique_ids || !d_inverse || !d_slot || !d_miss_vids)
    return fail(SFC_EINVAL, "null buffer");
  if (c->last_prepared >= 0 && c->ctx[c->last_prepared].state == PREPARED)
    return fail(SFC_ESTATE, "sfc_prepare twice without sfc_fetch_misses: missed rows would never arrive");
  if (c->t + 1 >= c->hist_len - 1) return fail(SFC_ELIMIT, "max_steps reached");

  StepCtx* x = nullptr;
  for (int k = 0; k < c->nctx; ++k)
    if (c->ctx[k].state == FREE) { x = &c->ctx[k]; break; }
  if (!x)
    return fail(SFC_ESTATE, "every step context holds a step that has not been updated: call "
                            "sfc_backward_update (or sfc_discard) first");
  StepCtx* prev = c->last_prepared >= 0 ? &c->ctx[c->last_prepared] : x;
  // a small batch is prepared by one block (k_small_prepare), all of it when that block can also choose
  // the victims
  const bool small = n_ids > 0 && n_ids <= kSmallIds && n_bags <= kSmallBags;
  const bool whole = small && c->dmap && (c->C >= c->V || c->C <= kSmallSlots);
  hipStream_t s = c->prep;
  if (s != c->st) {
    // the prepare stream must not overtake what the main stream has been given so far: the
    // producer of d_ids and the last update that read this context's buffers
    HIPCHK(hipEventRecord(c->ev_tmp, c->st));
    HIPCHK(hipStreamWaitEvent(s, c->ev_tmp, 0));
    // a context freed by sfc_discard: its copies may still be reading its lists
    if (x->discarded && s != c->side) HIPCHK(hipStreamWaitEvent(s, x->ev_fetched, 0));
  } else if (x->discarded && !x->joined) {
    // lookahead 0: a step that was given up without a lookup left nothing on the main stream that
    // waits for its copies, which may still be reading the lists that this prepare rewrites
    HIPCHK(hipStreamWaitEvent(s, x->ev_fetched, 0));
  }
  c->t += 1;
  x->t = c->t; x->state = PREPARED; x->updated = false; x->main_pending = false; x->discarded = false;
  x->n_ids = n_ids; x->n_bags = n_bags; x->d_offsets = d_offsets;
  x->d_unique = d_unique_ids; x->d_inverse = d_inverse; x->d_slot = d_slot; x->d_miss = d_miss_vids;
  c->last_prepared = (int)(x - c->ctx);
  x->ungrouped = c->nctx == 1 && !small && n_ids > 0 && c->served >= kServing && !c->recorded && !capturing(s);

  EventPair ep{};
  int rc;
  if ((rc = prof_begin(c, P_PREPARE, s, &ep))) return rc;
  const int n = (int)n_ids;
  uint32_t hu = (uint32_t)(2 * n_ids);
  if (hu < 64) hu = 64;                       // the batch table is empty between steps: any size works
  const int nchunk = (n + kPosChunk - 1) / kPosChunk;
  const SortGeom sg = x->sg = small ? small_geom(n) : sort_geom(n);
  // Hashed index: its rebuild, when due, by further blocks of the unique passes
  const bool rebuild_inside = !c->dmap && !small && n > 0;
  const int extra = rebuild_inside ? rebuild_blocks(c->C) : 0;
  // What the resolve (and with it the start of the step's counters) waits for is done by the time the unique
  // passes are: a dense index has no rebuild.  Otherwise both are kernels of their own.
  const bool start_inside = c->dmap || rebuild_inside;
  if (!small && n > 0) {
    const bool big = n >= kUniqBigFrom;
    const int chunk = big ? kUniqChunkBig : kUniqChunk, nub = (n + chunk - 1) / chunk;
    if (c->wide) {
      WideTab tab{(UEntry*)c->utab, 0, c->V};
      auto insert = big ? k_uniq_insert<WideTab, kUniqChunkBig> : k_uniq_insert<WideTab, kUniqChunk>;
      hipLaunchKernelGGL(insert, dim3(nub + extra), dim3(256), 0, s, d_ids, n, tab, hu, c->hslot,
                         c->first, c->n_invalid, nub, (const Ctr*)prev->ctr, c->index, c->hi);
    } else {
      PackedTab tab{c->utab, pos_bits(n), c->V};
      auto insert = big ? k_uniq_insert<PackedTab, kUniqChunkBig> : k_uniq_insert<PackedTab, kUniqChunk>;
      hipLaunchKernelGGL(insert, dim3(nub + extra), dim3(256), 0, s, d_ids, n, tab, hu, c->hslot,
                         c->first, c->n_invalid, nub, (const Ctr*)prev->ctr, c->index, c->hi);
    }
    const int* const counts = n > kCountMin ? c->blk_cnt : nullptr;
    if (counts)
      hipLaunchKernelGGL(k_uniq_count, dim3((nchunk + 3) / 4), dim3(256), 0, s, (const unsigned*)c->first,
                         nchunk, c->blk_cnt);
    hipLaunchKernelGGL(k_uniq_assign, dim3(nchunk + extra), dim3(256), 0, s, d_ids, c->V, c->hslot,
                       (const unsigned*)c->first, n, counts, d_unique_ids, c->uvid, c->vid_hslot, c->cnt, c->n_unique,
                       nchunk, x->ctr, x->t, (const Ctr*)prev->ctr, c->index, c->hi, (const int64_t*)c->slot_id);
  } else if (!small) {
    fill<int>(s, c->n_unique, 1, 0);
  }
  const RankArgs rank{c->hslot, c->uvid, n, d_inverse, x->ungrouped ? nullptr : c->cnt, c->cnt_rep, sg.nrep,
                      x->ungrouped ? c->vids : x->pos_slot, c->first};
  const ResolveArgs res{d_unique_ids, c->vid_hslot, c->utab, c->wide ? 1 : 0, c->index, c->hi, c->dmap, c->stamp,
                        c->hist, x->t, d_slot, c->tile_miss, c->age_hist, x->ctr,
                        start_inside ? (const Ctr*)prev->ctr : (const Ctr*)nullptr, (const int*)c->n_unique, c->n_invalid};
  auto rank_resolve = sg.shift == 10 ? k_rank_resolve<1, 1024> : sg.shift == 12 ? k_rank_resolve<8, 512>
                                                                              : k_rank_resolve<8, 1024>;
  const int rt = sg.shift == 12 ? 512 : 1024, nres = small ? 0 : grid_for(n, rt, kResolveThreads / rt);
  const int ncount = small || n == 0 ? 0 : sg.blocks;
  // from here on behind the whole prepare of the previous step: the step's counters start from
  // that step's, the index is rebuilt if its plan asked for it
  if (!start_inside) {
    hipLaunchKernelGGL(k_ctr_init, dim3(kRebuildGrid), dim3(256), 0, s, x->ctr, prev->ctr,
                       c->n_unique, c->n_invalid, c->index, c->hi, x->t);
    hipLaunchKernelGGL(k_index_refill, dim3(kRebuildGrid), dim3(256), 0, s, c->index, c->hi, c->slot_id, x->ctr);
  }
  if (small) {
    SmallArgs a;
    a.ids = d_ids; a.n = n; a.V = c->V; a.offsets = d_offsets; a.n_bags = (int)n_bags;
    a.unique_ids = d_unique_ids; a.inverse = d_inverse; a.slot = d_slot; a.miss_vids = d_miss_vids;
    a.index = c->index; a.hi = c->hi; a.dmap = c->dmap;
    a.stamp = c->stamp; a.slot_id = c->slot_id; a.hist = c->hist;
    a.t = x->t; a.lookahead = c->cfg.lookahead; a.C = (int)c->C; a.boff = x->boff;
    a.cnt = c->cnt; a.tile_miss = c->tile_miss; a.age_hist = c->age_hist;
    a.grp = x->grp; a.cold_pay = x->cold_pay; a.perm64 = x->perm64; a.pos_slot = x->pos_slot;
    a.victim_slot = x->victim_slot; a.victim_id = x->victim_id; a.miss_row = x->miss_row; a.miss_id = x->miss_id;
    a.ctr = x->ctr; a.prev = c->dmap ? prev->ctr : nullptr;
    auto kern = n <= 2048 ? (whole ? k_small_prepare<true, 2> : k_small_prepare<false, 2>)
              : n <= 4096 ? (whole ? k_small_prepare<true, 4> : k_small_prepare<false, 4>)
                          : (whole ? k_small_prepare<true, kSmallPer> : k_small_prepare<false, kSmallPer>);
    hipLaunchKernelGGL(kern, dim3(1), dim3(1024), 0, s, a);
  } else {
    hipLaunchKernelGGL(rank_resolve, dim3(nres + ncount), dim3(rt), 0, s, rank, res, nres);
  }
  x->grouping_due = !whole && c->nctx == 1;
  x->told = false;
  if (!whole) {
    plan_and_assign(c, x);
    if (c->nctx > 1 && (rc = group_positions(c, x, false))) return rc;
  }
  if (c->nctx > 1 && !x->told) HIPCHK(hipEventRecord(x->ev_prepared, s));
  HIPCHK(hipGetLastError());
  return prof_end(c, P_PREPARE, s, &ep);
}

int sfc_fetch_misses(sfc_cache* c) {
  if (!c) return fail(SFC_EINVAL, "null cache");
  if (int hrc = healthy(c)) return hrc;
  StepCtx* x = c->last_prepared >= 0 ? &c->ctx[c->last_prepared] : nullptr;
  if (!x || x->state != PREPARED) return fail(SFC_ESTATE, "sfc_fetch_misses needs a preceding sfc_prepare");
  // older steps whose update has not been enqueued yet: their bypass rows are not in the Host
  // table yet (k_swap_rows decides on the device which of its two launches does the work)
  x->main_pending = false; x->main_after = 0; x->bypass_from = kIntMax;
  for (int k = 0; k < c->nctx && c->cfg.policy != SFC_POLICY_PREFETCH; ++k) {
    StepCtx* o = &c->ctx[k];
    if (o == x || o->state != FETCHED || o->updated) continue;
    // (the steps in flight follow one another, so these are all steps from the smallest of the numbers on)
    const int from = o->t == x->t - 1 && o->main_pending ? o->bypass_from : o->t;
    if (from < x->bypass_from) x->bypass_from = from;
    if (o->t > x->main_after) x->main_after = o->t;
  }
  // everything the main stream has been given so far comes before the copies: older updates and their
  // second launches, what the caller enqueued behind the prepare (rows it writes into the Host table, say),
  // with lookahead 0 the prepare itself, which launch_swap then waits for by this event
  const bool on_main = x->copies_on_main = swap_on_main(c);
  if (!on_main && c->nctx > 1) {
    HIPCHK(hipEventRecord(c->ev_tmp, c->st));
    HIPCHK(hipStreamWaitEvent(c->side, c->ev_tmp, 0));
  } else if (!on_main) {
    HIPCHK(hipEventRecord(x->ev_prepared, c->st));
  }
  int rc;
  // (on the main stream the grouping pass of a small batch goes out with the copies)
  const bool with_copies = on_main && x->n_ids > 0 && (x->ungrouped || x->sg.shift == 10) && !prof_on(c, P_PREPARE);
  if (x->grouping_due && !with_copies && (rc = group_positions(c, x, true))) return rc;
  x->joined = on_main;
  if ((rc = launch_swap(c, x, on_main ? c->st : c->side, 0))) return rc;
  x->main_pending = x->main_after > 0;
  x->state = FETCHED;
  return SFC_OK;
}

int sfc_lookup(sfc_cache* c, float* d_out) {
  if (!c) return fail(SFC_EINVAL, "null cache");
  if (int hrc = healthy(c)) return hrc;
  StepCtx* x = training_ctx(c);
  if (!x) return fail(SFC_ESTATE, "sfc_lookup needs sfc_prepare and sfc_fetch_misses first");
  if (x->n_bags > 0 && !d_out) return fail(SFC_EINVAL, "null output");
  if ((uintptr_t)d_out & 15) return fail(SFC_EINVAL, "output must be 16-byte aligned");
  int rc;
  if ((rc = rows_ready(c, x))) return rc;
  hipStream_t s = c->st;
  const int64_t total = x->n_bags * c->d4;
  if (total > 0) {
    // the rows of the batch into the memory-side cache first (not for a small output; returns at once when
    // the rows are too many)
    if (total >= kWarmMinChunks)
      LAUNCH_TIMED_X(c, P_LOOKUP, true, true, k_warm_rows, dim3(grid_for(x->n_ids * c->d4, 2048, kWarmGrid)),
                     dim3(256), s, (const int*)x->d_slot, (const float4*)c->cw, c->d4, (int)c->C, x->boff,
                     (const Ctr*)x->ctr, c->warm_sink, (const int4*)x->pos_slot, (int)(x->n_ids / 4));
    if (!x->d_offsets) {
      const int d4 = c->d4, sh = (d4 & (d4 - 1)) == 0 ? __builtin_ctz(d4) : -1;
      const int bpb = lookup_rows_per_block(d4);
      LAUNCH_TIMED(c, P_LOOKUP, true, k_lookup_onehot,
                   dim3((unsigned)((x->n_bags + bpb - 1) / bpb)), dim3(256), s,
                   (const int*)x->pos_slot, (const float4*)c->cw, (float4*)d_out, (int)x->n_bags, d4, sh, bpb);
    } else {
      const int G = 64 / c->d4 > 0 ? 64 / c->d4 : 1;          // bags per wavefront
      const int64_t per_block = 4 * (int64_t)G;
      LAUNCH_TIMED(c, P_LOOKUP, true, k_lookup_bags,
                   dim3((unsigned)((x->n_bags + per_block - 1) / per_block)), dim3(256), s,
                   x->d_offsets, (const int*)x->pos_slot, (const float4*)c->cw, (float4*)d_out,
                   (int)x->n_bags, c->d4, G, x->n_ids);
    }
  }
  HIPCHK(hipGetLastError());
  return SFC_OK;
}

int sfc_segment_sum(sfc_cache* c, const float* d_grad, float* d_common_grad) {
  if (!c) return fail(SFC_EINVAL, "null cache");
  if (int hrc = healthy(c)) return hrc;
  StepCtx* x = training_ctx(c);
  if (!x) return fail(SFC_ESTATE, "sfc_segment_sum needs sfc_prepare and sfc_fetch_misses first");
  if ((x->n_bags > 0 && !d_grad) || !d_common_grad) return fail(SFC_EINVAL, "null buffer");
  if (((uintptr_t)d_grad | (uintptr_t)d_common_grad) & 15) return fail(SFC_EINVAL, "buffers must be 16-byte aligned");
  int rc;
  if ((rc = rows_ready(c, x)) || (rc = group_now(c, x, true))) return rc;
  if ((rc = seg_launch(c, x, d_grad, d_common_grad, c->bp, c->bp_vid, true, false, nullptr))) return rc;
  HIPCHK(hipGetLastError());
  return SFC_OK;
}

int sfc_segment_sum_static(sfc_cache* c, const float* d_grad, float* d_common_grad) {
  if (!c) return fail(SFC_EINVAL, "null cache");
  if (int hrc = healthy(c)) return hrc;
  StepCtx* x = training_ctx(c);
  if (!x) return fail(SFC_ESTATE, "sfc_segment_sum_static needs sfc_prepare and sfc_fetch_misses first");
  if ((x->n_bags > 0 && !d_grad) || !d_common_grad) return fail(SFC_EINVAL, "null buffer");
  if (((uintptr_t)d_grad | (uintptr_t)d_common_grad) & 15) return fail(SFC_EINVAL, "buffers must be 16-byte aligned");
  int dev = -1;
  HIPCHK(hipGetDevice(&dev));
  if (dev != c->device) return fail(SFC_EINVAL, "the cache lives on another device than the current one");
  // per block of the stream two fp64 rows and two virtual ids
  const SegGeom g = seg_geom(c->D, x->n_ids > 0 ? x->n_ids : 1);
  const int64_t nblk = (g.waves + 3) / 4;
  const int64_t sums = 2 * nblk * c->D * (int64_t)sizeof(double);
  const int64_t used = sums + 2 * nblk * (int64_t)sizeof(int);
  // what is refused goes by the batch's size alone (see the header), not by the spans that the stream takes;
  // `used` fits wherever that does
  const int64_t counted = seg_scratch_count(c->D, x->n_ids > 0 ? x->n_ids : 1);
  if (counted > (int64_t)SFC_STATIC_SCRATCH_BYTES || used > (int64_t)SFC_STATIC_SCRATCH_BYTES) {
    char msg[192];
    snprintf(msg, sizeof msg, "sfc_segment_sum_static: a batch of %lld ids of dim %d counts as %lld bytes of "
             "scratch, the fixed array holds %d", (long long)x->n_ids, c->D, (long long)counted,
             (int)SFC_STATIC_SCRATCH_BYTES);
    return fail(SFC_ELIMIT, msg);
  }
  void* base = nullptr;
  int rc;
  if ((rc = static_scratch(dev, &base))) return rc;
  // both launches of the step's copies must have been issued already: issuing the second one here
  // could create profiling events
  if (x->main_pending)
    return fail(SFC_ESTATE, "the step's rows are still due on the main stream: call sfc_lookup first");
  if ((rc = join_copies(c, x)) || (rc = group_now(c, x, false))) return rc;
  // every slot that k_seg_finish reads is written by k_seg_stream in the same call: nothing to clear
  double* bp = (double*)base;
  int* bp_vid = (int*)((unsigned char*)base + sums);
  if ((rc = seg_launch(c, x, d_grad, d_common_grad, bp, bp_vid, false, false, nullptr))) return rc;
  HIPCHK(hipGetLastError());
  return SFC_OK;
}

int sfc_backward_update(sfc_cache* c, const float* d_grad) {
  if (!c) return fail(SFC_EINVAL, "null cache");
  if (int hrc = healthy(c)) return hrc;
  StepCtx* x = training_ctx(c);
  if (!x) return fail(SFC_ESTATE, "sfc_backward_update needs sfc_prepare and sfc_fetch_misses first");
  if (x->n_bags > 0 && !d_grad) return fail(SFC_EINVAL, "null gradient");
  if ((uintptr_t)d_grad & 15) return fail(SFC_EINVAL, "gradient must be 16-byte aligned");
  int rc;
  if ((rc = rows_ready(c, x)) || (rc = group_now(c, x, true))) return rc;
  c->updated_once = true;
  hipStream_t s = c->st;
  EventPair ep{};
  if ((rc = prof_begin(c, P_BACKWARD, s, &ep))) return rc;
  int n_slots = 0;
  // the update kernel sums the cold groups and chains the block-edge partials itself (row-wise Adagrad: where the
  // lanes of a row share a wavefront)
  const bool rowwise = c->cfg.optimizer == SFC_OPT_ROWWISE_ADAGRAD;
  const bool fused = !rowwise || (c->d4 & (c->d4 - 1)) == 0;
  // a small batch in one kernel
  const bool groups = !rowwise && small_update(x->n_ids, c->d4);
  if (!groups && (rc = seg_launch(c, x, d_grad, c->gsum, c->bp, c->bp_vid, true, fused, &n_slots))) return rc;
  if (c->cfg.policy == SFC_POLICY_PREFETCH) {
    // the copies of a newer step issued so far read the Host table before this update writes it
    for (int k = 0; k < c->nctx; ++k) {
      StepCtx* y = &c->ctx[k];
      if (y != x && y->state == FETCHED && !y->updated && y->t > x->t)
        HIPCHK(hipStreamWaitEvent(s, y->ev_fetched, 0));
    }
  }
  const dim3 ug(grid_for(x->n_ids * c->d4, 1024, kGridCap));
  // the stream above passed over the cold groups and left the block-edge partials unchained:
  // the fused kernels sum both themselves (their first blocks chain the partials, a lane group per slot)
  const int n_edge = edge_blocks(n_slots, c->d4);
  const int shares = groups ? update_shares(x->n_ids, c->d4) : 0;
  const dim3 gg((unsigned)(shares + grid_for(x->n_ids, kGroupShort, kGroupBlocks)));
  if (c->cfg.optimizer == SFC_OPT_ADAGRAD && groups) {
    AdagradOp op;
    op.lr = c->cfg.lr; op.eps = c->cfg.eps;
    LAUNCH_TIMED(c, P_ADAGRAD, true, k_update_groups<AdagradOp>, gg, dim3(kGroupThreads), s, op, (const int64_t*)x->grp,
                 (const int64_t*)x->perm64, (const float4*)d_grad, (const int*)x->d_slot, (const int64_t*)x->d_unique,
                 (float4*)c->cw, (float4*)c->ca, c->host, (int)c->C, x->boff, c->d4, (const Ctr*)x->ctr, (int)x->n_ids,
                 shares, c->bp, c->share_ticket);
  } else if (c->cfg.optimizer == SFC_OPT_ADAGRAD) {
    auto kern = x->d_offsets ? k_adagrad_rows<false> : k_adagrad_rows<true>;
    LAUNCH_TIMED(c, P_ADAGRAD, true, kern, dim3(ug.x + (unsigned)n_edge), dim3(256), s, (const float4*)c->gsum,
                 (const int*)x->d_slot, (const int64_t*)x->d_unique, (float4*)c->cw, (float4*)c->ca,
                 c->host, (int)c->C, x->boff, c->cfg.lr, c->cfg.eps, c->d4, (const Ctr*)x->ctr,
                 (const int2*)x->cold_pay, (const float4*)d_grad, (const double*)c->bp,
                 (const int*)c->bp_vid, n_slots, n_edge);
  } else if (c->cfg.optimizer == SFC_OPT_ADAM) {
    // every constant derived from the decay rates is computed in double and rounded to fp32 once
    AdamArgs k;
    k.b1 = (float)c->cfg.beta1; k.c1 = (float)(1.0 - c->cfg.beta1);
    k.b2 = (float)c->cfg.beta2; k.c2 = (float)(1.0 - c->cfg.beta2);
    k.bc1 = (float)(1.0 - pow(c->cfg.beta1, (double)x->t));
    k.bc2 = (float)(1.0 - pow(c->cfg.beta2, (double)x->t));
    k.lr = c->cfg.lr; k.eps = c->cfg.eps;
    AdamOp op;
    op.k = k;
    auto kern = x->d_offsets ? k_adam_rows<false> : k_adam_rows<true>;
    if (groups)
      LAUNCH_TIMED(c, P_ADAGRAD, true, k_update_groups<AdamOp>, gg, dim3(kGroupThreads), s, op, (const int64_t*)x->grp,
                   (const int64_t*)x->perm64, (const float4*)d_grad, (const int*)x->d_slot, (const int64_t*)x->d_unique,
                   (float4*)c->cw, (float4*)c->ca, c->host, (int)c->C, x->boff, c->d4, (const Ctr*)x->ctr, (int)x->n_ids,
                   shares, c->bp, c->share_ticket);
    else LAUNCH_TIMED(c, P_ADAGRAD, true, kern, dim3(ug.x + (unsigned)n_edge), dim3(256), s, (const float4*)c->gsum,
                 (const int*)x->d_slot, (const int64_t*)x->d_unique, (float4*)c->cw, (float4*)c->ca,
                 c->host, (int)c->C, x->boff, k, c->d4, (const Ctr*)x->ctr,
                 (const int2*)x->cold_pay, (const float4*)d_grad, (const double*)c->bp,
                 (const int*)c->bp_vid, n_slots, n_edge);
  } else if (fused) {
    auto kern = x->d_offsets ? k_rowwise_adagrad_rows<false> : k_rowwise_adagrad_rows<true>;
    LAUNCH_TIMED(c, P_ADAGRAD, true, kern, dim3(ug.x + (unsigned)n_edge), dim3(256), s, (const float4*)c->gsum,
                 (const int*)x->d_slot, (const int64_t*)x->d_unique, (float4*)c->cw, (float4*)c->ca,
                 c->host, (int)c->C, x->boff, c->cfg.lr, c->cfg.eps, c->d4, (const Ctr*)x->ctr,
                 (const int2*)x->cold_pay, (const float4*)d_grad, (const double*)c->bp,
                 (const int*)c->bp_vid, n_slots, n_edge);
  } else {
    LAUNCH_TIMED(c, P_ADAGRAD, true, k_rowwise_adagrad_any, ug, dim3(256), s,
                 (const float4*)c->gsum, (const int*)x->d_slot, (const int64_t*)x->d_unique,
                 (float4*)c->cw, (float4*)c->ca, c->host, (int)c->C, x->boff, c->cfg.lr, c->cfg.eps,
                 c->d4, (const Ctr*)x->ctr);
  }
  HIPCHK(hipGetLastError());
  if ((rc = prof_end(c, P_BACKWARD, s, &ep))) return rc;
  x->updated = true;
  x->state = FREE;
  // second launches of the copies of newer steps that had to stay behind this update, oldest first
  for (int pass = 0; pass < c->nctx; ++pass) {
    StepCtx* y = nullptr;
    for (int k = 0; k < c->nctx; ++k) {
      StepCtx* z = &c->ctx[k];
      if (z->state == FETCHED && z->main_pending && z->main_after <= x->t && (!y || z->t < y->t)) y = z;
    }
    if (!y) break;
    if ((rc = launch_swap(c, y, s, 1))) return rc;
  }
  return SFC_OK;
}

int sfc_flush(sfc_cache* c) {
  if (!c) return fail(SFC_EINVAL, "null cache");
  for (int k = 0; k < c->nctx; ++k)
    if (c->ctx[k].state == PREPARED || (c->ctx[k].state == FETCHED && c->ctx[k].main_pending))
      return fail(SFC_ESTATE, "sfc_flush while a prepared step still waits for its rows");
  int rc = sync_all(c);
  if (rc) return rc;
  if (c->last_prepared < 0) return SFC_OK;
  hipLaunchKernelGGL(k_flush, dim3(grid_for(c->C * 2 * c->d4, 256, kGridCap)), dim3(256), 0, c->st,
                     c->slot_id, (const float4*)c->cw, (const float4*)c->ca, c->host, c->d4, c->s4,
                     c->ctx[c->last_prepared].ctr);
  HIPCHK(hipGetLastError());
  return sync_all(c);
}

int sfc_get_stats(sfc_cache* c, sfc_stats* h_out) {
  if (!c || !h_out) return fail(SFC_EINVAL, "null argument");
  int rc = sync_all(c);
  if (rc) return rc;
  memset(h_out, 0, sizeof *h_out);
  if (c->last_prepared < 0) return SFC_OK;
  Ctr h;
  HIPCHK(hipMemcpy(&h, c->ctx[c->last_prepared].ctr, sizeof h, hipMemcpyDeviceToHost));
  if (h.err) {
    char msg[96];
    snprintf(msg, sizeof msg, "cache manager state is inconsistent (device check %d)", h.err);
    return fail(SFC_ECORRUPT, msg);
  }
  const int64_t rowbytes = (int64_t)sizeof(float) * (c->D + c->S);
  h_out->n_unique = h.U; h_out->n_hit = h.n_hit; h_out->n_miss = h.M; h_out->n_evict = h.K;
  h_out->n_bypass = h.n_bypass; h_out->n_invalid = h.n_invalid;
  h_out->h2d_bytes = h.M * rowbytes;
  h_out->d2h_bytes = ((int64_t)h.K + h.n_bypass) * rowbytes;
  h_out->n_bad_offsets = h.bad_offsets;
  return SFC_OK;
}

int sfc_check(sfc_cache* c) {
  if (!c) return fail(SFC_EINVAL, "null cache");
  if (int hrc = healthy(c)) return hrc;
  const int bad = ((const volatile HostStatus*)c->hstat)->bad_offsets_step;
  if (bad > c->reported_bad_step) {
    c->reported_bad_step = bad;
    char msg[96];
    snprintf(msg, sizeof msg, "malformed bag offsets in step %d (most recent such step)", bad);
    return fail(SFC_EINVAL, msg);
  }
  return SFC_OK;
}

int sfc_peek_stats(sfc_cache* c, sfc_stats* h_out, int64_t* h_step) {
  if (!c || !h_out || !h_step) return fail(SFC_EINVAL, "null argument");
  const volatile HostStatus* h = c->hstat;
  memset(h_out, 0, sizeof *h_out);
  *h_step = 0;
  // all words of one step; the kernel that publishes stores them together, microseconds apart at most on the
  // link, thousands of reads here, so the limit is a time far beyond that
  std::chrono::steady_clock::time_point end{};
  for (int tries = 1;; ++tries) {
    if (tries % 1024 == 0) {
      const auto now = std::chrono::steady_clock::now();
      if (tries == 1024) end = now + std::chrono::milliseconds(100);
      else if (now > end) break;
    }
    uint64_t w[kStatWords];
    for (int i = 0; i < kStatWords; ++i) w[i] = h->word[i];
    bool whole = true;
    for (int i = 1; i < kStatWords; ++i) whole = whole && w[i] >> 32 == w[0] >> 32;
    if (!whole) continue;
    const auto count = [&](int i) { return (int64_t)(uint32_t)w[i]; };
    const int64_t rowbytes = (int64_t)sizeof(float) * (c->D + c->S);
    h_out->n_unique = count(kStatU); h_out->n_hit = count(kStatHit); h_out->n_miss = count(kStatMiss);
    h_out->n_evict = count(kStatEvict); h_out->n_bypass = count(kStatBypass);
    h_out->n_invalid = count(kStatInvalid); h_out->n_bad_offsets = count(kStatBadOffsets);
    h_out->h2d_bytes = h_out->n_miss * rowbytes;
    h_out->d2h_bytes = (h_out->n_evict + h_out->n_bypass) * rowbytes;
    *h_step = (int64_t)(w[0] >> 32);
    return SFC_OK;
  }
  return fail(SFC_EHIP, "status block kept changing");
}

int sfc_discard(sfc_cache* c) {
  if (!c) return fail(SFC_EINVAL, "null cache");
  StepCtx* x = training_ctx(c);
  if (!x) return fail(SFC_ESTATE, "no fetched step to give up");
  if (x->main_pending)
    return fail(SFC_ESTATE, "the step's copies wait for an older update: it cannot be given up yet");
  x->state = FREE;
  x->discarded = true;
  if (c->served < kServing) ++c->served;
  return SFC_OK;
}

int sfc_verify(sfc_cache* c, int64_t* h_bad) {
  if (!c || !h_bad) return fail(SFC_EINVAL, "null argument");
  for (int k = 0; k < c->nctx; ++k)
    if (c->ctx[k].state == PREPARED)
      return fail(SFC_ESTATE, "sfc_verify while a prepared step still waits for its rows");
  int rc = sync_all(c);
  if (rc) return rc;
  for (int k = 0; k < 4; ++k) h_bad[k] = 0;
  if (c->last_prepared < 0) return SFC_OK;
  int* recount = nullptr;
  unsigned long long* d_bad = nullptr;
  HIPCHK(hipMalloc((void**)&recount, (size_t)c->hist_len * sizeof(int)));
  if (hipMalloc((void**)&d_bad, 4 * sizeof(unsigned long long)) != hipSuccess) {
    (void)hipFree(recount);
    return fail(SFC_ENOMEM, "hipMalloc");
  }
  hipStream_t s = c->st;
  fill<int>(s, recount, (int64_t)c->hist_len, 0);
  fill<unsigned long long>(s, d_bad, 4, 0ull);
  Ctr* ctr = c->ctx[c->last_prepared].ctr;
  hipLaunchKernelGGL(k_verify_slots, dim3(grid_for(c->C, 256, kGridCap)), dim3(256), 0, s,
                     c->slot_id, c->stamp, c->index, c->hi, c->dmap, recount, c->hist_len, d_bad, ctr);
  if (c->dmap)
    hipLaunchKernelGGL(k_verify_dense, dim3(grid_for(c->V, 256, kGridCap)), dim3(256), 0, s,
                       c->dmap, c->V, c->slot_id, (int)c->C, d_bad);
  else
    hipLaunchKernelGGL(k_verify_entries, dim3(grid_for((int64_t)c->hi, 256, kGridCap)), dim3(256), 0, s,
                       c->index, c->hi, c->slot_id, (int)c->C, d_bad);
  hipLaunchKernelGGL(k_verify_hist, dim3(grid_for((int64_t)c->hist_len, 256, kGridCap)), dim3(256), 0, s,
                     c->hist, recount, c->hist_len, d_bad);
  unsigned long long hb[4] = {0, 0, 0, 0};
  hipError_t e = hipMemcpyAsync(hb, d_bad, sizeof hb, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  (void)hipFree(recount);
  (void)hipFree(d_bad);
  if (e != hipSuccess) return fail(SFC_EHIP, "sfc_verify", e);
  Ctr h;
  HIPCHK(hipMemcpy(&h, ctr, sizeof h, hipMemcpyDeviceToHost));
  h_bad[0] = (int64_t)hb[0]; h_bad[1] = (int64_t)hb[1]; h_bad[2] = (int64_t)hb[2];
  h_bad[3] = (int64_t)hb[3] - (int64_t)h.f;          // live entries against occupied slots
  if (h_bad[0] || h_bad[1] || h_bad[2] || h_bad[3]) {
    char msg[160];
    snprintf(msg, sizeof msg, "sfc_verify: %lld slots not findable, %lld stray entries, %lld histogram "
             "words off, %lld live entries beyond the occupied slots",
             (long long)h_bad[0], (long long)h_bad[1], (long long)h_bad[2], (long long)h_bad[3]);
    return fail(SFC_ECORRUPT, msg);
  }
  return SFC_OK;
}

int sfc_cache_state(sfc_cache* c, int64_t* h_slot_id, int32_t* h_stamp, float* h_rows, float* h_acc) {
  if (!c) return fail(SFC_EINVAL, "null cache");
  int rc = sync_all(c);
  if (rc) return rc;
  if (c->C == 0) return SFC_OK;
  const size_t rows = (size_t)c->C * c->D * sizeof(float);
  if (h_slot_id) HIPCHK(hipMemcpy(h_slot_id, c->slot_id, (size_t)c->C * sizeof(int64_t), hipMemcpyDeviceToHost));
  if (h_stamp) HIPCHK(hipMemcpy(h_stamp, c->stamp, (size_t)c->C * sizeof(int32_t), hipMemcpyDeviceToHost));
  if (h_rows) HIPCHK(hipMemcpy(h_rows, c->cw, rows, hipMemcpyDeviceToHost));
  if (h_acc) HIPCHK(hipMemcpy(h_acc, c->ca, (size_t)c->C * c->S * sizeof(float), hipMemcpyDeviceToHost));
  return SFC_OK;
}

int sfc_profile_enable(sfc_cache* c, int32_t level) {
  if (!c) return fail(SFC_EINVAL, "null cache");
  c->prof = level < 0 ? 0 : (level > 2 ? 2 : level);
  return SFC_OK;
}

int sfc_profile_read(sfc_cache* c, int32_t which, double* h_ms_sum, int64_t* h_calls) {
  if (!c || which < 0 || which >= P_N || !h_ms_sum || !h_calls) return fail(SFC_EINVAL, "bad argument");
  int rc = sync_all(c);
  if (rc) return rc;
  if ((rc = prof_collect(c))) return rc;
  *h_ms_sum = c->ms_sum[which];
  *h_calls = c->calls[which];
  c->ms_sum[which] = 0;
  c->calls[which] = 0;
  return SFC_OK;
}

}  // extern "C"
