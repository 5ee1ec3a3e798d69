// Row-moving kernels: Host<->cache copies, the forward gather, the gradient segment-sum and
// the optimizer updates (Adagrad, Adam, row-wise Adagrad).  A row is D fp32 = D/4 chunks of 16 bytes; consecutive lanes take
// consecutive chunks, so a wavefront moves 1 KiB of contiguous output per instruction and a
// 128-byte row (D = 32) is one request of 8 lanes.
#pragma once
#include "sfc_device.h"
#include "sfc_prepare_kernels.h"

namespace sfc {

typedef float vf4 __attribute__((ext_vector_type(4)));

// streaming (non-temporal) 16-byte accesses for data that is touched once per step
__device__ __forceinline__ float4 ld_stream(const float4* p) {
  const vf4 v = __builtin_nontemporal_load(reinterpret_cast<const vf4*>(p));
  return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void st_stream(float4* p, float4 v) {
  vf4 x; x.x = v.x; x.y = v.y; x.z = v.z; x.w = v.w;
  __builtin_nontemporal_store(x, reinterpret_cast<vf4*>(p));
}
// kStream: the datum is read once per step (streamed); otherwise it is read again by other lanes
// later in the same kernel and should stay cached
template <bool kStream>
__device__ __forceinline__ float4 ld_row(const float4* p) { return kStream ? ld_stream(p) : *p; }
template <bool kStream>
__device__ __forceinline__ void st_row(float4* p, float4 v) { if (kStream) st_stream(p, v); else *p = v; }

// ---------------------------------------------------------------------------------------------
// Host link (Algorithm 1 lines 5-6).  The Host table is pinned, device-mapped memory; the kernels
// read / write it directly, 16 bytes per lane.  A row moves as (D + S)/4 chunks: its weights, then
// its S floats of optimizer state; hs4 / has4 are the Host row strides in 16-byte units.  When the
// caller interleaves the two Host arrays (h_acc = h_weights + D, both strides D + S) the lanes of
// a row touch one contiguous 4*(D+S)-byte block of Host memory, which the link moves measurably
// faster than two separate blocks (55 vs 41 GB/s Host->device for D = S = 32).
// The k-th miss takes the slot of the k-th victim (both lists are in ascending order of the
// assignment), so one lane group does both directions for that slot: it loads the victim's row
// from HBM and the missed row from Host, then stores each on the other side.  Reads and writes
// cross the link at the same time instead of one after the other.
//
// Pipelined steps: a row that bypassed the cache in an older step still in flight reaches the
// Host table only with that step's update, so this step's copies must then run behind it.  The
// host cannot know whether that happened without waiting, so it launches the kernel twice: once
// on the side stream right away and once on the main stream behind the older steps' updates; the
// device counters decide which of the two launches does the work (on_main below), the other one
// returns at once.  Bypass rows of step `bypass_from` or a later one send the copies to the main launch: the
// oldest step in flight when they were issued, or, where the previous step's main launch was still due
// then, that step's own bypass_from (these copies come behind those).  Both launches go by the step's own
// counters, which its prepare has completed: an older step's context is prepared anew while they are due.
// ---------------------------------------------------------------------------------------------
struct HostRows {
  float4* w;      // device view of h_weights
  float4* a;      // device view of h_acc (the optimizer state, s4 chunks per row)
  int64_t hs4;    // row stride of w in float4
  int64_t has4;   // row stride of a in float4
};

// Reads and writes of the link in separate blocks.  A lane that does both waits for its read, then writes,
// and with few rounds per lane the lanes of the whole grid do so in step: the link idles in turn one way
// and the other.  So with lookahead 0, and where the misses are many enough to matter (kSplitMin) and few
// enough that the rounds have not drifted apart, the victims' rows are first copied beside the step's bypass
// rows in HBM (k_stage_victims; the region has a row for every id of the batch, and victims + bypass rows are
// at most its misses); then kSplitWriters blocks carry them to the Host while the other blocks read the
// missed rows into their slots.  Copies alone, staging included, against one lane doing both, us: 128-byte
// rows 59e3 240 / 271, 99e3 380 / 407, 137e3 526 / 546, 194e3 732 / 743, 250e3 932 / 932, 377e3 1385 / 1350;
// 512-byte rows 18e3 234 / 264, 57e3 693 / 695, 93e3 1100 / 1112, 172e3 2005 / 1996, 212e3 2470 / 2457;
// 960-byte rows 17.5e3 445 / 460, 46e3 1109 / 1120, 86e3 2015 / 2012, 144e3 3354 / 3337; 6.9e3 of 256 bytes
// 67 / 65.  So the upper end is both a number of rows (kSplitMax) and of bytes (kSplitMaxBytes).
// What is in flight on the link decides the rest, and more is not better: a pass of 16384 x 39 / 65536 x 39 / 5003 x
// 39 with Adam, us, with kSplitFly 1 for the reads 375 / 694 / 648, 2 378 / 698 / 645, 4 382 / 702 / 654, 8 398 / 733 /
// 690, 2 both ways 377 / 696 / 640; 24 writers 379 / 700 / 643, 40 377 / 697 / 647; 192 readers (4 in flight) 394 /
// 719 / 668, 256 442 / 813 / 797; all writers on one XCD 457 / 847 / 885, on two 419 / 795 / 803.  A link that reads
// and writes rows at random at once reaches 70 to 76 GB/s both ways together for 128-byte rows (its reads alone 40),
// 88 for 256 bytes, 84 for 960, 97 for the copy engines on large blocks; the order of the rows changes nothing.
// The staging goes beside the grouping pass, not in front of it: copies that start before that pass has ended hold
// up its writes (37 -> 332 us at 65536 x 39) and are held up (368 -> 422).
constexpr int kSplitMin = 1 << 14;
constexpr int kSplitMax = 1 << 18;
constexpr unsigned kSplitMaxBytes = 64u << 20;
constexpr int kSplitWriters = 32, kSplitReaders = 128, kSplitFly = 2;
// M misses, K victims, both loaded together (one after the other they cost the copies 2 us); w2: 16-byte chunks
// of a row and its state
__device__ __forceinline__ bool split_swap(int M, int K, int w2) {
  return (M >= kSplitMin) & (M <= kSplitMax) & ((uint64_t)M * (unsigned)w2 <= kSplitMaxBytes / 16) & (K > 0);
}

__global__ __launch_bounds__(256) void k_stage_victims(const int* __restrict__ victim_slot,
                                                        float4* __restrict__ cw, float4* __restrict__ ca,
                                                        int C, int boff, int d4, int s4, const Ctr* ctr) {
  const int M = ctr->M, K = ctr->K;
  if (!split_swap(M, K, d4 + s4)) return;
  const unsigned w2 = (unsigned)(d4 + s4), total = (unsigned)K * w2;    // at most kSplitMaxBytes / 16
  const int64_t row0 = (int64_t)C + boff + ctr->n_bypass;
  for (unsigned i = blockIdx.x * 256 + threadIdx.x; i < total; i += gridDim.x * 256) {
    const unsigned k = i / w2;
    const int c = (int)(i - k * w2);
    const int64_t from = victim_slot[k], to = row0 + k;
    if (c < d4) cw[to * d4 + c] = cw[from * d4 + c];
    else ca[to * s4 + (c - d4)] = ca[from * s4 + (c - d4)];
  }
}

// One direction: rows list[k] (k < count) of the Host table and rows row(k) of the cache, kSplitFly chunks
// of a lane in flight.
template <bool kToHost, class Row>
__device__ __forceinline__ void link_rows(const int64_t* __restrict__ list, Row row, int count, float4* cw,
                                          float4* ca, const HostRows& h, int d4, int s4, int blk, int nblk) {
  const unsigned w2 = (unsigned)(d4 + s4), total = (unsigned)count * w2, stride = (unsigned)nblk * 256;
  for (unsigned i0 = (unsigned)blk * 256 + threadIdx.x; i0 < total; i0 += kSplitFly * stride) {
    int64_t at[kSplitFly], hat[kSplitFly];                  // chunk in the cache array, chunk in the Host array
    bool on[kSplitFly], state[kSplitFly];
    vf4 v[kSplitFly];
#pragma unroll
    for (int u = 0; u < kSplitFly; ++u) {
      const unsigned i = i0 + u * stride;
      on[u] = i < total;
      const unsigned k = on[u] ? i / w2 : 0;
      const int c = on[u] ? (int)(i - k * w2) : 0;
      state[u] = c >= d4;
      const int64_t id = list[k], r = row(k);
      at[u] = state[u] ? r * s4 + (c - d4) : r * d4 + c;
      hat[u] = state[u] ? id * h.has4 + (c - d4) : id * h.hs4 + c;
    }
#pragma unroll
    for (int u = 0; u < kSplitFly; ++u)
      if (on[u]) {
        const float4* const from = kToHost ? (state[u] ? ca : cw) : (state[u] ? h.a : h.w);
        v[u] = *reinterpret_cast<const vf4*>(&from[kToHost ? at[u] : hat[u]]);
      }
#pragma unroll
    for (int u = 0; u < kSplitFly; ++u)
      if (on[u]) {
        float4* const to = kToHost ? (state[u] ? h.a : h.w) : (state[u] ? ca : cw);
        *reinterpret_cast<vf4*>(&to[kToHost ? hat[u] : at[u]]) = v[u];
      }
  }
}

__device__ __forceinline__ void swap_rows(const int* __restrict__ miss_row, const int64_t* __restrict__ miss_id,
                                          const int64_t* __restrict__ victim_id, float4* __restrict__ cw,
                                          float4* __restrict__ ca, const HostRows& h, int d4, int s4, const Ctr* ctr,
                                          int bypass_from, int main_variant, int staged_at, int write_back, int blocks) {
  const bool on_main = ctr->last_bypass >= bypass_from;      // the same in both launches
  if (on_main != (main_variant != 0)) return;
  __builtin_amdgcn_s_setprio(3);            // few waves, long round trips: issue ahead of the kernels beside them
  // write_back 0: no row of the cache has ever been updated, so the victims are what the Host table holds
  // already (a cache that only serves lookups: 2e5 power-law ids of dim 32 over 1e6 rows with a cache of 1e5 243 -> 183 us a pass,
  // 4e4 of dim 64 with a cache of 5e4 174 -> 127)
  const int M = ctr->M, K = write_back ? ctr->K : 0;
  // staged_at >= 0: k_stage_victims has run, the victims' rows are at staged_at + the bypass rows
  if ((staged_at >= 0) & split_swap(M, K, d4 + s4)) {
    const int64_t row0 = (int64_t)staged_at + ctr->n_bypass;
    if (blockIdx.x < kSplitWriters)
      link_rows<true>(victim_id, [&](unsigned k) { return row0 + k; }, K, cw, ca, h, d4, s4, (int)blockIdx.x,
                      kSplitWriters);
    else
      link_rows<false>(miss_id, [&](unsigned k) { return (int64_t)miss_row[k]; }, M, cw, ca, h, d4, s4,
                       (int)blockIdx.x - kSplitWriters, blocks - kSplitWriters);
    return;
  }
  const int w2 = d4 + s4;                   // chunks of a row and of its optimizer state
  const int64_t total = (int64_t)M * w2;
  const int64_t stride = (int64_t)blocks * 256;
  // A thread's chunks are a serial chain, and with few blocks (see the launch) the chain is long:
  // the list entries of the next chunk are fetched while this chunk's Host read is in flight, so
  // that the chain is one Host round trip per chunk and nothing that waits on HBM.
  int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  int row = 0;
  int64_t id = 0, vic = 0;
  if (i < total) {
    const int k = (int)(i / w2);
    row = miss_row[k]; id = miss_id[k]; vic = k < K ? victim_id[k] : -1;
  }
  while (i < total) {
    const int k = (int)(i / w2);
    int c = (int)(i - (int64_t)k * w2);
    const bool acc = c >= d4;
    if (acc) c -= d4;
    float4* hb = acc ? h.a : h.w;
    float4* cb = acc ? ca : cw;
    const int64_t hst = acc ? h.has4 : h.hs4;
    const int cst = acc ? s4 : d4;
    const int64_t dst = (int64_t)row * cst + c;
    const float4 nv = hb[id * hst + c];
    const int64_t vnow = vic;
    const int64_t inext = i + stride;
    if (inext < total) {
      const int kn = (int)(inext / w2);
      row = miss_row[kn]; id = miss_id[kn]; vic = kn < K ? victim_id[kn] : -1;
    }
    if (vnow >= 0) hb[vnow * hst + c] = cb[dst];
    cb[dst] = nv;
    i = inext;
  }
}
struct SwapArgs {
  const int* miss_row; const int64_t *miss_id, *victim_id; float4 *cw, *ca; HostRows h; int d4, s4; const Ctr* ctr;
  int bypass_from, main_variant, staged_at, write_back;
};
__device__ __forceinline__ void swap_rows(const SwapArgs& a, int blocks) {
  swap_rows(a.miss_row, a.miss_id, a.victim_id, a.cw, a.ca, a.h, a.d4, a.s4, a.ctr, a.bypass_from, a.main_variant,
            a.staged_at, a.write_back, blocks);
}
__global__ __launch_bounds__(256) void k_swap_rows(const SwapArgs a) { swap_rows(a, (int)gridDim.x); }

// Copies on the main stream: the grouping pass of a batch below 2^18 ids, which they do not need, is further blocks of their
// launch (few misses: what both take is start-up and dependent round trips, 5.8 us of grouping and 35 of copies at 1024 x 39
// ids with bypass rows; a pass of those 102.0 -> 96.4 us).  From 2^18 ids on the grouping takes larger blocks.
__global__ __launch_bounds__(256) void k_swap_scatter(const SwapArgs a, int swap_blocks, const ScatterArgs b) {
  if ((int)blockIdx.x < swap_blocks) swap_rows(a, swap_blocks);
  else scatter_positions<4, 256>(b, (int)blockIdx.x - swap_blocks);
}

// The same for a batch that is not grouped: the rows of its positions.
__global__ __launch_bounds__(256) void k_swap_pos_rows(const SwapArgs a, int swap_blocks, const RowsArgs b) {
  if ((int)blockIdx.x < swap_blocks) swap_rows(a, swap_blocks);
  else rows_of_positions(b, (int)blockIdx.x - swap_blocks);
}

__global__ __launch_bounds__(256) void k_flush(const int64_t* __restrict__ slot_id,
                                                const float4* __restrict__ cw,
                                                const float4* __restrict__ ca, HostRows h, int d4,
                                                int s4, const Ctr* ctr) {
  const int w2 = d4 + s4;
  const int64_t total = (int64_t)ctr->f * w2;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
    const int64_t s = i / w2;
    int c = (int)(i - s * w2);
    const bool acc = c >= d4;
    if (acc) c -= d4;
    const int64_t id = slot_id[s];
    if (id < 0) continue;
    if (acc) h.a[id * h.has4 + c] = ca[s * s4 + c];
    else h.w[id * h.hs4 + c] = cw[s * d4 + c];
  }
}

// ---------------------------------------------------------------------------------------------
// Forward gather (Algorithm 1 lines 9 and 11 fused): out[b] = cache row of the slot of position b.
// pos_slot[p] = slot[inverse[p]] is written by the prepare step, so the gather is one level of
// indirection.  A block stages the slots of its bags in LDS with one coalesced load, then every
// thread has its 16-byte row chunks (up to eight) in flight before the first store; a
// wavefront's stores are 1 KiB contiguous and non-temporal: the output is consumed by the model,
// and keeping it out of L2 keeps the hot rows in (plain stores measured 50 % slower).
// What bounds it on MI355X: with the rows resident in the memory-side cache the kernel runs at
// the write rate of HBM (52-58 us for 327 MB); in the training loop the other kernels of the step
// have evicted them, the ~59 MB of row reads mix into the write stream and the same kernel takes
// 79-85 us, which is what k_warm_rows below is for.  Variants without LDS staging or with
// persistent blocks measured within +-5 % of this one under those conditions.
// ---------------------------------------------------------------------------------------------
constexpr int kLookupBags = 256;      // most rows a block of the one-hot gather takes
// Rows per block of the one-hot gather: 512 16-byte chunks, two per thread.  With the rows
// waiting in the memory-side cache (k_warm_rows) small blocks win: 62.6 us at the target
// configuration against 69.7 with 256 rows (2048 chunks) per block; 32 rows: 66.4.
inline int lookup_rows_per_block(int d4) {
  int b = 512 / d4;
  if (b < 16) b = 16;
  if (b > kLookupBags) b = kLookupBags;
  return b;
}

// Before the gather: every row the batch needs is read once, by a kernel that does nothing else.
// The gather is sensitive to the latency of its slowest row: each wavefront holds eight rows per
// lane group in flight and stores nothing until the last has arrived, and a row that comes from
// HBM between the kernel's own writes takes several times as long as one that is cached.  This
// kernel has all its loads in flight at once and nothing to wait for; the 30 MB it reads at the
// target configuration stay in the memory-side cache for the microseconds until the gather asks
// for them.  Measured there: 9.6 us of warming take the gather from 80 to 60 us.
// It only pays while the rows fit that cache with room to spare: beyond kWarmMaxBytes of rows
// (decided on the device from the step's unique count) the kernel returns at once.
constexpr int64_t kWarmMaxBytes = (int64_t)96 << 20;
// Below this many 16-byte chunks of output (32 MB) the gather alone is the faster one: it is over before its
// writes get in the way of its reads.  A pass with / without the warm kernel, us, where other work between the
// steps has pushed the rows out of the caches (one-hot: millions of chunks = those read = those written):
// 1.28 260.6 / 259.2, 2.56 288.1 / 286.8 updated and 244.2 / 245.7 looked up only, 5.11 362.6 / 364.9, 6.82
// 329.1 / 333.0; bags, millions read and written: 9.36, 1.70 295.5 / 290.9; 5.12, 1.70 292.0 / 288.5; 6.82, 3.41
// 321.5 / 325.3; 13.6, 6.82 423.9 / 434.5; 34.1, 13.6 574.7 / 588.6.  So what is written decides, also for bags.
// With rows that are still cached, which the host cannot know, the line would lie higher: 2.56 141 / 137,
// 6.82 173.2 / 168.1, 10.2 320.6 / 329.1; bags 6.82, 3.41 172 / 171; 13.6, 6.82 272 / 282.
constexpr int64_t kWarmMinChunks = (int64_t)1 << 21;
constexpr int kWarmGrid = 2048;

__global__ __launch_bounds__(256) void k_warm_rows(const int* __restrict__ slot,
                                                    const float4* __restrict__ cw, int d4, int C,
                                                    int boff, const Ctr* ctr, float* sink,
                                                    const int4* __restrict__ pos_slot4, int n4) {
  const int64_t total = (int64_t)ctr->U * d4;
  if (total * 16 > kWarmMaxBytes) return;
  const int64_t stride = (int64_t)gridDim.x * 256;
  float acc = 0.f;
  // the per-position slots as well: in a pipelined run they were written steps ago and have left
  // every cache, and each block of the gather starts with a load of them
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += stride) {
    const int4 q = pos_slot4[i];
    acc += (float)(q.x ^ q.y ^ q.z ^ q.w) * 1e-30f;
  }
  for (int64_t i0 = (int64_t)blockIdx.x * 256 + threadIdx.x; i0 < total; i0 += 8 * stride) {
    float4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int64_t i = i0 + u * stride;
      v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (i < total) {
        const int vrow = (int)(i / d4);
        int s = slot[vrow];
        if (s >= C) s += boff;
        if (s >= 0) v[u] = cw[(int64_t)s * d4 + (i - (int64_t)vrow * d4)];
      }
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) acc += v[u].x + v[u].y + v[u].z + v[u].w;
  }
  // the loads must not be optimised away; no finite sum of table values equals this
  if (acc == 1.2345678e30f) *sink = acc;
}

// d4 is a runtime value; when it is a power of two (sh >= 0) index math is shifts and masks
__device__ __forceinline__ void split_chunk(unsigned ch, int d4, int sh, unsigned& r, unsigned& c) {
  if (sh >= 0) { r = ch >> sh; c = ch & (unsigned)(d4 - 1); }
  else { r = ch / (unsigned)d4; c = ch - r * (unsigned)d4; }
}

__global__ __launch_bounds__(256) void k_lookup_onehot(const int* __restrict__ pos_slot,
                                                        const float4* __restrict__ cw,
                                                        float4* __restrict__ out, int n_bags,
                                                        int d4, int sh, int bpb) {
  __shared__ int ls[kLookupBags];
  const int b0 = (int)blockIdx.x * bpb;          // bpb <= kLookupBags = block size
  {
    const int b = b0 + (int)threadIdx.x;
    ls[threadIdx.x] = ((int)threadIdx.x < bpb && b < n_bags) ? pos_slot[b] : -1;
  }
  __syncthreads();
  int nb = n_bags - b0;
  if (nb > bpb) nb = bpb;
  const unsigned chunks = (unsigned)nb * (unsigned)d4;
  float4* dst = out + (int64_t)b0 * d4;
  for (unsigned base = 0; base < chunks; base += 256 * 8) {
    float4 v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const unsigned ch = base + k * 256 + threadIdx.x;
      v[k] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (ch < chunks) {
        unsigned r, c;
        split_chunk(ch, d4, sh, r, c);
        const int s = ls[r];
        if (s >= 0) v[k] = cw[(int64_t)s * d4 + c];
      }
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const unsigned ch = base + k * 256 + threadIdx.x;
      if (ch < chunks) st_stream(&dst[ch], v[k]);
    }
  }
}

// Multi-hot forward (sum pooling): out[b] = sum over the positions q of bag b of the cached row of
// position q, fp32 adds in bag order.  A row is d4 lanes of 16 bytes, so a wavefront holds
// G = 64 / d4 lane groups and each group owns one bag: its lanes read the bag's slots (one
// broadcast load per position), keep kBagUnroll row chunks in flight per lane and fetch the
// slots of the next kBagUnroll positions meanwhile, so that the chain offsets -> slot -> row is
// walked once per kBagUnroll rows instead of once per row.  The four bags of a wavefront are
// neighbours, so its stores are contiguous (G * d4 * 16 bytes) and non-temporal.
// Bags are short (1-20 ids in the benchmark's multi-hot configuration), so the lane groups of a
// wavefront finish at different times; the idle lanes cost nothing that matters here, the kernel
// is bound by the row traffic (every position reads a full row; only the rows that are hot
// enough to stay in an XCD's L2 are not fetched again).
// Malformed offsets are reported by the prepare step; here they only must not lead outside
// pos_slot, hence the clamp of both ends to [0, n_ids] (a start near 2^63 as it is would wrap round when
// the unrolled loop adds to it).  Positions are 32 bits from there on: with 64 the clamp cost 1 %.
#ifndef SFC_BAG_UNROLL
#define SFC_BAG_UNROLL 8
#endif
constexpr int kBagUnroll = SFC_BAG_UNROLL;

__global__ __launch_bounds__(256) void k_lookup_bags(const int64_t* __restrict__ offsets,
                                                      const int* __restrict__ pos_slot,
                                                      const float4* __restrict__ cw,
                                                      float4* __restrict__ out, int n_bags,
                                                      int d4, int G, int64_t n_ids) {
  const int lane = lane_id();
  const int g = lane / d4, c = lane - g * d4;
  const int64_t b = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * G + g;
  if (g >= G || b >= n_bags) return;
  const BagRange r = bag_range(offsets[b], offsets[b + 1], (int)n_ids);
  int q = r.lo;
  const int e = r.hi;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  int sl[kBagUnroll], sn[kBagUnroll];
#pragma unroll
  for (int k = 0; k < kBagUnroll; ++k) sl[k] = q + k < e ? pos_slot[q + k] : -1;
  for (; q < e; q += kBagUnroll) {
    float4 v[kBagUnroll];
#pragma unroll
    for (int k = 0; k < kBagUnroll; ++k) {
      v[k] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (sl[k] >= 0) v[k] = cw[(int64_t)sl[k] * d4 + c];
    }
#pragma unroll
    for (int k = 0; k < kBagUnroll; ++k) {
      const int qn = q + kBagUnroll + k;
      sn[k] = qn < e ? pos_slot[qn] : -1;
    }
#pragma unroll
    for (int k = 0; k < kBagUnroll; ++k) {
      acc.x += v[k].x; acc.y += v[k].y; acc.z += v[k].z; acc.w += v[k].w;
      sl[k] = sn[k];
    }
  }
  st_stream(&out[b * d4 + c], acc);
}

// ---------------------------------------------------------------------------------------------
// Gradient segment-sum (GPU-Worker / Backward): common[v] = sum of the grad rows of the positions
// with virtual id v.  Input: perm64, the batch's positions grouped by virtual id, entry =
// (vid << 32) | row of grad.  The kernel is a barrier-free stream over perm64:
//   - a row is D/4 lanes of 16 bytes, so a wavefront holds G = 64 / (D/4) lane groups; group g of
//     wavefront w owns the span of L consecutive entries starting at (w*G + g)*L;
//   - a group walks its span four entries at a time, the grad rows of the next four already in
//     flight, and sums runs of equal vid in fp64 registers.  A run that begins and ends inside
//     the span is complete when it closes: it is rounded to fp32 once and stored as row vid of
//     the common-gradient matrix;
//   - a run cut by the span's edge leaves an fp64 partial (head / tail).  The G groups of the
//     wavefront chain their partials through LDS once, at the end; runs cut by the wavefront's
//     edge are chained once more across the block's four wavefronts; what is cut by the
//     block's edge goes to bp[block][0 = head, 1 = tail] in HBM and k_seg_finish chains those.
// No atomics; the summation tree depends only on perm64, n and D.  perm64 itself lists a group's
// positions in the order the grouping pass ranked them, which its atomics decide, so the fp64 sum
// of a frequent id can differ in its last bits from run to run; rounded to fp32 once, the results
// of two runs are nearly always identical and never further apart than one unit in the last place
// of the sum (ids with at most kColdMax positions are added in a fixed order and are identical).
// A run that covers a whole span (wavefront) stores its sum in the head slot and a zero in the
// tail slot under the same vid, so equal vids are always adjacent in the partial lists.
//
// The Adagrad update is a separate kernel over the common-gradient matrix (k_adagrad_rows).
// Fusing it into the stream (update the cached row when its run closes) was measured slower on
// MI355X: the dependent chain entry -> slot -> cached row sits inside the streaming loop and
// the extra registers cost a wavefront of occupancy per SIMD, which outweighs the 60 MB of
// common-gradient traffic that fusion saves.
// ---------------------------------------------------------------------------------------------
#ifndef SFC_SEG_CHUNK
#define SFC_SEG_CHUNK 4
#endif
constexpr int kSegChunk = SFC_SEG_CHUNK;        // entries per group per loop iteration
// the stream never has more wavefronts than this: 48 per compute unit measured best at the target
// size (16: stream 82 us + finish 10; 48: 75 + 14; the finish pass grows with the number of blocks)
#ifndef SFC_SEG_WAVES
#define SFC_SEG_WAVES 48
#endif
constexpr int kSegTargetWaves = 256 * SFC_SEG_WAVES;

constexpr int kSegMinWaves = 2048;

struct SegGeom { int G, L, waves; };
// L is chosen so that the stream has about kSegTargetWaves wavefronts.
inline SegGeom seg_geom(int D, int64_t n) {
  SegGeom g;
  g.G = 64 / (D / 4);
  if (g.G < 1) g.G = 1;
  const int64_t target_waves = kSegTargetWaves;
  int64_t L = (n + g.G * target_waves - 1) / (g.G * target_waves);
  // never below 32 entries per span (fewer partial sums, fewer block edges for the kernel behind to
  // chain), except where that leaves the chip with fewer than kSegMinWaves wavefronts: then 16 or 8.
  // sfc_backward_update us with spans of 8 / 16 / 32, power-law ids: 40e3 positions of dim 16 29.7 / 30.3 / 31.9,
  // 200e3 of dim 16 34.6 / 34.4 / 38.6, 639e3 of dim 16 (32: 1248 wavefronts) 44.4 / 44.7 / 46.9, 200e3 of dim 64
  // (1562) 42.3 / 39.1 / 40.4, 195e3 of dim 80 (2031) 47.7 / 43.5 / 43.6, 639e3 of dim 32 (2496) 49.9 / 45.5 /
  // 46.0, 213e3 of dim 128 (3328) 57.0 / 55.5 / 50.2, 40e3 of dim 256 (1250) 45.3 / 40.5 / 40.6; all ids distinct:
  // 40e3 of dim 256 56.5 / 57.2 / 61.2, 639e3 of dim 16 45.5 / 47.5 / 51.7, 213e3 of dim 128 115.3 / 112.0 / 112.2.
  int64_t lmin = 32;
  while (lmin > 8 && n < g.G * lmin * kSegMinWaves) lmin /= 2;
  if (L < lmin) L = lmin;
  L = (L + kSegChunk - 1) / kSegChunk * kSegChunk;
  g.L = (int)L;
  g.waves = (int)((n + (int64_t)g.G * L - 1) / ((int64_t)g.G * L));
  return g;
}

// Bytes of scratch by which sfc_segment_sum_static accepts or refuses a batch: that of spans of 8 entries
// below 2^18 positions and 32 above.  The stream above mostly takes less; where it takes more (short rows,
// at most 794 624 bytes then) both are far from the limit.
inline int64_t seg_scratch_count(int D, int64_t n) {
  const int64_t G = 64 / (D / 4) < 1 ? 1 : 64 / (D / 4);
  int64_t L = (n + G * kSegTargetWaves - 1) / (G * kSegTargetWaves);
  const int64_t lmin = n < ((int64_t)1 << 18) ? 8 : 32;
  if (L < lmin) L = lmin;
  L = (L + kSegChunk - 1) / kSegChunk * kSegChunk;
  const int64_t blocks = ((n + G * L - 1) / (G * L) + 3) / 4;
  return 2 * blocks * (D * (int64_t)sizeof(double) + (int64_t)sizeof(int));
}

struct D4 { double x, y, z, w; };
__device__ __forceinline__ void d4_zero(D4& a) { a.x = a.y = a.z = a.w = 0.0; }
__device__ __forceinline__ void d4_add(D4& a, float4 v) {
  a.x += (double)v.x; a.y += (double)v.y; a.z += (double)v.z; a.w += (double)v.w;
}
__device__ __forceinline__ float4 d4_round(const D4& a) {
  return make_float4((float)a.x, (float)a.y, (float)a.z, (float)a.w);
}

// A list of partial slots (even = head of a span, odd = its tail; vid -1 = none): the sum of the run of
// equal vids that begins at slot j, four slots per step; end = the slot behind it.
__device__ __forceinline__ D4 slot_run_sum(int j, int nslots, const int* __restrict__ vids,
                                           const double* __restrict__ sums, int D, int c4, int& end) {
  D4 s; d4_zero(s);
  const int v = vids[j];
  bool on = true;
  end = j;
  for (int k = j; on && k < nslots; k += 4) {
    int vk[4];
    D4 x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int kk = k + u < nslots ? k + u : nslots - 1;
      vk[u] = k + u < nslots ? vids[kk] : -1;
      const double* q = &sums[kk * D + 4 * c4];
      x[u].x = q[0]; x[u].y = q[1]; x[u].z = q[2]; x[u].w = q[3];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      on = on && vk[u] == v;
      if (on) { s.x += x[u].x; s.y += x[u].y; s.z += x[u].z; s.w += x[u].w; ++end; }
    }
  }
  return s;
}

// Chains such a list of 2 * nspan slots, a lane group per span, all spans at once (one group that walked
// the whole list, a chain of dependent LDS reads at the end of every wavefront and block, made the stream
// 64.3 instead of 61.7 us at 2.56e6 positions of dim 32, 24.9 instead of 21.1 at 639e3 of dim 16).  A run begins at a tail,
// and belongs to the group of that span, or at slot 0, then it belongs to group 0.  A run that begins at
// a tail and ends at a head lies inside the list: it is complete and stored.  What is open at the left
// edge is returned as (bv0, b0) in group 0; what is open at the right edge as (bv1, b1) in the group
// that owns it (own1), if there is any (last_v >= 0); a run open at both edges has its sum in b0 and a
// zero in b1.
struct ChainEdges { int bv0, bv1, last_v; bool own1; D4 b0, b1; };
__device__ __forceinline__ void chain_slots(int span, int nspan, const int* __restrict__ vids,
                                            const double* __restrict__ sums, int D, int d4, int c4,
                                            float4* __restrict__ common, ChainEdges& e) {
  e.bv0 = -1; e.bv1 = -1; e.own1 = false;
  d4_zero(e.b0); d4_zero(e.b1);
  const int nslots = 2 * nspan;
  e.last_v = vids[nslots - 1];
  int end;
  const int v = vids[2 * span + 1];
  if (v >= 0 && vids[2 * span] != v) {
    const D4 s = slot_run_sum(2 * span + 1, nslots, vids, sums, D, c4, end);
    if (((end - 1) & 1) == 0) common[(int64_t)v * d4 + c4] = d4_round(s);
    else { e.bv1 = v; e.b1 = s; e.own1 = true; }
  }
  if (span == 0 && vids[0] >= 0) {
    e.bv0 = vids[0];
    e.b0 = slot_run_sum(0, nslots, vids, sums, D, c4, end);
    if (((end - 1) & 1) != 0) { e.bv1 = e.bv0; d4_zero(e.b1); e.own1 = true; }
  }
}

// kOneHot: every gradient row is read exactly once (one position per bag): streamed with
// non-temporal loads (measured 75 against 96 us at the target one-hot configuration).  Multi-hot: a
// bag's row is read once per position of the bag, from all over the grouping: plain loads, so that
// the caches keep what they can (358 against 410 us at the multi-hot configuration).
// kSkipCold: entries of cold groups (see kColdBit) are passed over, their gradient rows are not
// read: sfc_backward_update with the Adagrad kernel, which sums those groups itself.  An entry
// that is passed over acts as a separator (key -1): it ends the run before it and begins none.
template <bool kSkipCold>
__device__ __forceinline__ int entry_key(int64_t e) {
  return (kSkipCold && entry_cold(e)) ? -1 : entry_vid(e);
}

// kSegChunk consecutive grouping entries from q on (q is a multiple of kSegChunk, the array is
// 256-byte aligned), -1 for those at or beyond se: 16-byte loads of two entries where both exist.
__device__ __forceinline__ void load_entries(const int64_t* __restrict__ perm64, int64_t q,
                                             int64_t se, int64_t (&e)[kSegChunk]) {
  static_assert(kSegChunk % 2 == 0, "entries are loaded in pairs");
#pragma unroll
  for (int k = 0; k < kSegChunk; k += 2) {
    if (q + k + 1 < se) {
      const longlong2 v = *reinterpret_cast<const longlong2*>(&perm64[q + k]);
      e[k] = v.x; e[k + 1] = v.y;
    } else {
      e[k] = q + k < se ? perm64[q + k] : (int64_t)-1;
      e[k + 1] = -1;
    }
  }
}

template <bool kOneHot, bool kSkipCold>
__global__ __launch_bounds__(256) void k_seg_stream(const float4* __restrict__ grad,
                                                     const int64_t* __restrict__ perm64, int n,
                                                     int d4, int G, int L,
                                                     float4* __restrict__ common,
                                                     double* __restrict__ bp,
                                                     int* __restrict__ bp_vid,
                                                     int* __restrict__ edge_mark) {
  // per wavefront: [2G slots][D] doubles (2*G*D <= 512) and the slots' vids
  __shared__ double part[4][512];
  __shared__ int pvid[4][128];
  __shared__ int wvid[8];
  // [4 wavefronts][2][D] (8 * D <= 2048 doubles): reuses part once every wavefront has chained its
  // own slots, which keeps the block at 18 KB of LDS and the kernel register-limited
  double* const wpart = &part[0][0];
  const int lane = lane_id(), wib = (int)(threadIdx.x >> 6);
  const int wave = (int)blockIdx.x * 4 + wib;
  const int g = lane / d4, c4 = lane - g * d4;
  const int D = d4 * 4;
  const bool active = g < G;
  const int64_t sb = ((int64_t)wave * G + g) * L;           // span of this group: [sb, se)
  int64_t se = sb + L;
  if (se > n) se = n;
  const bool nonempty = active && sb < n;

  int cur = -1;           // vid of the open run
  bool begun = false;     // the open run began inside this span
  D4 acc; d4_zero(acc);
  int head_v = -1; D4 head_s; d4_zero(head_s);     // run that continues from before the span
  int tail_v = -1; D4 tail_s; d4_zero(tail_s);     // run that continues past the span

  if (nonempty) {
    const int prev_v = sb > 0 ? entry_key<kSkipCold>(perm64[sb - 1]) : -1;
    // software pipeline: pe / x = entries and grad rows of the chunk being processed (issued one
    // iteration earlier), pn = the next chunk's entries
    int64_t pe[kSegChunk], pn[kSegChunk];
    float4 x[kSegChunk];
    load_entries(perm64, sb, se, pe);
#pragma unroll
    for (int k = 0; k < kSegChunk; ++k) {
      x[k] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (pe[k] >= 0 && entry_key<kSkipCold>(pe[k]) >= 0)
        x[k] = ld_row<kOneHot>(&grad[(int64_t)(uint32_t)pe[k] * d4 + c4]);
    }
    load_entries(perm64, sb + kSegChunk, se, pn);
    cur = entry_key<kSkipCold>(pe[0]);
    begun = prev_v != cur;

    for (int64_t e = sb; e < se; e += kSegChunk) {
      // issue the next chunk's rows and the chunk after that's entries
      float4 xn[kSegChunk];
      int64_t pnn[kSegChunk];
#pragma unroll
      for (int k = 0; k < kSegChunk; ++k) {
        xn[k] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (pn[k] >= 0 && entry_key<kSkipCold>(pn[k]) >= 0)
          xn[k] = ld_row<kOneHot>(&grad[(int64_t)(uint32_t)pn[k] * d4 + c4]);
      }
      load_entries(perm64, e + 2 * kSegChunk, se, pnn);
#pragma unroll
      for (int k = 0; k < kSegChunk; ++k) {
        if (pe[k] >= 0) {
          const int v = entry_key<kSkipCold>(pe[k]);
          if (v != cur) {
            if (begun) { if (cur >= 0) common[(int64_t)cur * d4 + c4] = d4_round(acc); }
            else { head_v = cur; head_s = acc; }
            cur = v; begun = true; d4_zero(acc);
          }
          d4_add(acc, x[k]);
        }
      }
#pragma unroll
      for (int k = 0; k < kSegChunk; ++k) { pe[k] = pn[k]; pn[k] = pnn[k]; x[k] = xn[k]; }
    }
    // close the span: the open run either ends here or continues into the next span
    const int next_v = se < n ? entry_key<kSkipCold>(perm64[se]) : -1;
    if (next_v != cur || cur < 0) {
      if (begun) { if (cur >= 0) common[(int64_t)cur * d4 + c4] = d4_round(acc); }
      else { head_v = cur; head_s = acc; }
    } else if (begun) {
      tail_v = cur; tail_s = acc;
    } else {
      head_v = cur; head_s = acc; tail_v = cur;          // whole span: zero marker in the tail
    }
  }

  // chain the 2G partial slots of this wavefront (slot order = span order; even = head, odd = tail)
  if (active) {
    double* ph = &part[wib][(2 * g) * D + 4 * c4];
    ph[0] = head_s.x; ph[1] = head_s.y; ph[2] = head_s.z; ph[3] = head_s.w;
    ph += D;
    ph[0] = tail_s.x; ph[1] = tail_s.y; ph[2] = tail_s.z; ph[3] = tail_s.w;
    if (c4 == 0) { pvid[wib][2 * g] = head_v; pvid[wib][2 * g + 1] = tail_v; }
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  ChainEdges we;
  we.own1 = false; we.last_v = -1;
  if (active) chain_slots(g, G, pvid[wib], part[wib], D, d4, c4, common, we);
  __syncthreads();                       // every wavefront has read its part of `part`
  // the wavefront's own head / tail become slots 2*wib, 2*wib+1 of the block's chain
  if (lane < d4) {
    double* o0 = &wpart[(2 * wib) * D + 4 * c4];
    o0[0] = we.b0.x; o0[1] = we.b0.y; o0[2] = we.b0.z; o0[3] = we.b0.w;
    if (c4 == 0) { wvid[2 * wib] = we.bv0; if (we.last_v < 0) wvid[2 * wib + 1] = -1; }
  }
  if (we.own1) {
    double* o1 = &wpart[(2 * wib + 1) * D + 4 * c4];
    o1[0] = we.b1.x; o1[1] = we.b1.y; o1[2] = we.b1.z; o1[3] = we.b1.w;
    if (c4 == 0) wvid[2 * wib + 1] = we.bv1;
  }
  __syncthreads();
  if (lane < d4) {                       // one lane group per wavefront
    ChainEdges be;
    chain_slots(wib, 4, wvid, wpart, D, d4, c4, common, be);
    const int64_t o = (int64_t)blockIdx.x * 2;
    // a group cut by a block's edge: its sum is not in `common`, and the optimizer kernel that
    // chains the partials itself (k_adagrad_rows) must not take it from there (see kEdgeMark)
    if (wib == 0) {
      double* o0 = &bp[(o + 0) * D + 4 * c4];
      o0[0] = be.b0.x; o0[1] = be.b0.y; o0[2] = be.b0.z; o0[3] = be.b0.w;
      if (c4 == 0) {
        bp_vid[o] = be.bv0;
        if (be.last_v < 0) bp_vid[o + 1] = -1;
        if (edge_mark && be.bv0 >= 0) edge_mark[2 * be.bv0] = kEdgeMark;
      }
    }
    if (be.own1) {
      double* o1 = &bp[(o + 1) * D + 4 * c4];
      o1[0] = be.b1.x; o1[1] = be.b1.y; o1[2] = be.b1.z; o1[3] = be.b1.w;
      if (c4 == 0) {
        bp_vid[o + 1] = be.bv1;
        if (edge_mark) edge_mark[2 * be.bv1] = kEdgeMark;
      }
    }
  }
}

// The block-edge partials: slot j = 2 * block + (0 head | 1 tail); equal vids are adjacent and a long
// group (the hottest id spans hundreds of blocks) is one long run of slots.
// One run, by a whole block: true (for the whole block) when j is the first slot of its run; then v is
// the run's virtual id and the threads tid < d4 hold its fp64 sum, chunk tid of the row, in s.  The lane
// groups sum the run's partials in a strided, fixed order, eight rows in flight, and combine in a tree.
__device__ __forceinline__ bool edge_run_sum(const double* __restrict__ bp,
                                             const int* __restrict__ bp_vid, int nslots, int d4,
                                             int j, int& v, D4& s) {
  __shared__ double red[256 * 4];
  __shared__ int s_first[4];
  v = bp_vid[j];
  if (v < 0 || (j > 0 && bp_vid[j - 1] == v)) return false;     // not the first slot of its run
  // the run's end, 1024 slots per round: all loads in flight, the first that differs ends it
  const int tid = (int)threadIdx.x;
  int end = j;
  for (int base = j;; base += 1024) {
    int first = base + 1024;
#pragma unroll
    for (int u = 3; u >= 0; --u) {
      const int k0 = base + u * 256 + (tid & ~63), k = k0 + (tid & 63);
      const uint64_t off = __ballot(!(k < nslots && bp_vid[k] == v));
      if (off) first = k0 + __builtin_ctzll(off);
    }
    if ((tid & 63) == 0) s_first[tid >> 6] = first;
    __syncthreads();
    end = s_first[0];
#pragma unroll
    for (int w = 1; w < 4; ++w) end = s_first[w] < end ? s_first[w] : end;
    __syncthreads();
    if (end < base + 1024) break;                          // at the latest where the slots end
  }
  const int D = d4 * 4;
  const int groups = 256 / d4, g = tid / d4, c4 = tid - g * d4;
  double s0 = 0., s1 = 0., s2 = 0., s3 = 0.;
  // Behind the first slot only heads (even slots) count: a tail inside the run is that of a block which
  // lies in the run from edge to edge, and its sum is in its head.  One compute unit reads all of it, and
  // that is what the longest run costs.
  const int e0 = j + (j & 1), ne = (end - e0 + 1) >> 1;
  if (g < groups) {
    const double* q = bp + 4 * c4;
    if (g == 0 && (j & 1)) { const double* x = q + (int64_t)j * D; s0 = x[0]; s1 = x[1]; s2 = x[2]; s3 = x[3]; }
    for (int k = g; k < ne; k += 8 * groups) {
      double x[8][4];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int kk = k + u * groups < ne ? k + u * groups : ne - 1;
#pragma unroll
        for (int i = 0; i < 4; ++i) x[u][i] = q[(int64_t)(e0 + 2 * kk) * D + i];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (k + u * groups < ne) { s0 += x[u][0]; s1 += x[u][1]; s2 += x[u][2]; s3 += x[u][3]; }
    }
  }
  double* r = &red[tid * 4];
  r[0] = s0; r[1] = s1; r[2] = s2; r[3] = s3;
  int o = 1;
  while (o < groups) o <<= 1;
  for (o >>= 1; o > 0; o >>= 1) {
    __syncthreads();
    if (g < o && g + o < groups) {
      const double* q = r + o * d4 * 4;
      r[0] += q[0]; r[1] += q[1]; r[2] += q[2]; r[3] += q[3];
    }
  }
  s.x = r[0]; s.y = r[1]; s.z = r[2]; s.w = r[3];
  return true;
}

// Every run, by edge_blocks() blocks: a lane group per slot.  Nearly all runs are two slots long (the tail
// of one stream block and the head of the next): a group that finds the first slot of a run of at most
// kEdgeShort slots adds them up itself, in slot order.  The few long runs (an id with thousands of
// positions spans many stream blocks) are summed by the whole block.  Their first slots lie more than
// kEdgeShort slots apart, and a block takes no more slots than that, so it meets at most one of them.
// emit(v, c4, sum): chunk c4 of the summed row of virtual id v, rounded to fp32.
// What bounds it is dependent loads and barriers, so the slots around one are loaded together and a long
// run ends in a tree.  As a kernel of its own, us, one block per slot / 4 * (64 / d4) slots per block, their
// long runs one after the other / this way: 2.56e6 positions of dim 32 9.6 / 9.1 / 7.3, 2e6 of dim 4 9.9 / 27.8 /
// 5.5, 200e3 of dim 16 4.6 / 11.2 / 5.5, 40e3 of dim 64 4.6 / 6.7 / 5.9, 213e3 of dim 128 18.3 / 6.2 / 6.1.  In front
// of the optimizer kernel's rows (whole kernel): 19.0 -> 16.8, 33.2 -> 7.3 and 14.1 -> 7.0 for the first three.
constexpr int kEdgeShort = 8;
inline __host__ __device__ int edge_slots(int d4) {
  const int groups = 4 * (64 / d4 > 0 ? 64 / d4 : 1);
  return groups < kEdgeShort ? groups : kEdgeShort;
}
inline int edge_blocks(int nslots, int d4) {
  const int per_block = edge_slots(d4);
  return (nslots + per_block - 1) / per_block;
}

template <class Emit>
__device__ __forceinline__ void edge_block(const double* __restrict__ bp, const int* __restrict__ bp_vid,
                                           int nslots, int d4, int blk, Emit emit) {
  __shared__ int long_at;                                  // first slot of the block's long run
  if (threadIdx.x == 0) long_at = -1;
  __syncthreads();
  const int lane = lane_id(), G = 64 / d4 > 0 ? 64 / d4 : 1;
  const int g = lane / d4, c4 = lane - g * d4;
  const int i = (int)(threadIdx.x >> 6) * G + g, per_block = edge_slots(d4);
  const int j = blk * per_block + i;
  if (g < G && i < per_block && j < nslots) {
    // the slots around, all in flight: a run of two is found in one round trip, not slot by slot
    int vs[kEdgeShort + 1];
    const int before = j > 0 ? bp_vid[j - 1] : -1;
#pragma unroll
    for (int u = 0; u <= kEdgeShort; ++u) vs[u] = j + u < nslots ? bp_vid[j + u] : -1;
    const int v = vs[0];
    if (v >= 0 && before != v) {                          // first slot of its run
      int len = 1;
#pragma unroll
      for (int u = 1; u <= kEdgeShort; ++u) len += len == u && vs[u] == v;
      if (len > kEdgeShort) {
        if (c4 == 0) long_at = j;
      } else {
        const int D = d4 * 4;
        double s0 = 0., s1 = 0., s2 = 0., s3 = 0.;
        for (int k = 0; k < len; ++k) {
          const double* q = bp + (int64_t)(j + k) * D + 4 * c4;
          s0 += q[0]; s1 += q[1]; s2 += q[2]; s3 += q[3];
        }
        emit(v, c4, make_float4((float)s0, (float)s1, (float)s2, (float)s3));
      }
    }
  }
  __syncthreads();
  if (long_at < 0) return;
  int v;
  D4 s;
  const bool first = edge_run_sum(bp, bp_vid, nslots, d4, long_at, v, s);
  if (first && (int)threadIdx.x < d4) emit(v, (int)threadIdx.x, d4_round(s));
}

__global__ __launch_bounds__(256) void k_seg_finish(const double* __restrict__ bp,
                                                     const int* __restrict__ bp_vid, int nslots,
                                                     int d4, float4* __restrict__ common) {
  edge_block(bp, bp_vid, nslots, d4, (int)blockIdx.x,
             [&](int v, int c4, float4 g) { common[(int64_t)v * d4 + c4] = g; });
}

// ---------------------------------------------------------------------------------------------
// Sparse Adagrad (Algorithm 1 line 14), once per unique row:
//   acc += g*g ; w -= lr * g / (sqrt(acc) + eps)
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ void adagrad1(float& w, float& a, float g, float lr, float eps) {
  a = a + g * g;
  w = w - lr * g / (sqrtf(a) + eps);
}
__device__ __forceinline__ void adagrad4v(float4& w, float4& a, float4 g, float lr, float eps) {
  adagrad1(w.x, a.x, g.x, lr, eps);
  adagrad1(w.y, a.y, g.y, lr, eps);
  adagrad1(w.z, a.z, g.z, lr, eps);
  adagrad1(w.w, a.w, g.w, lr, eps);
}

// The update kernels touch every row of the batch once.  When those rows (weights, state, summed
// gradient; read and written) exceed what the memory-side cache holds, keeping them cached only
// evicts what the next kernel could have used: they are then moved with non-temporal accesses
// (multi-hot configuration, 1.4e6 rows of 256 bytes: 305 against 400 us).  Below that size plain
// accesses are as fast or a little faster (target configuration: 32 us either way).
constexpr int64_t kStreamRowsBytes = (int64_t)256 << 20;
__device__ __forceinline__ bool stream_rows(int U, int d4, int s4) {
  return (int64_t)U * (3 * d4 + 2 * s4) * 16 > kStreamRowsBytes;
}

// ---------------------------------------------------------------------------------------------
// Adam (Experiment settings: the paper's optimizer), lazily on the rows of the batch, with the
// batch number t in the bias corrections bc = 1 - beta^t (computed by the host in double):
//   m = b1*m + c1*g ; v = b2*v + c2*g*g ; w -= lr * (m/bc1) / (sqrt(v/bc2) + eps)
// The state of a row is 2*d4 chunks: first moments, then second moments.
// ---------------------------------------------------------------------------------------------
struct AdamArgs {
  float b1, c1, b2, c2;   // beta1, 1-beta1, beta2, 1-beta2
  float bc1, bc2, lr, eps;
};
__device__ __forceinline__ void adam1(float& w, float& m, float& v, float g, const AdamArgs& k) {
  m = k.b1 * m + k.c1 * g;
  v = k.b2 * v + k.c2 * (g * g);
  const float mhat = m / k.bc1, vhat = v / k.bc2;
  w = w - k.lr * mhat / (sqrtf(vhat) + k.eps);
}

// The two element-wise optimizers as policies of one row kernel: kParts state chunks travel with
// each 16-byte chunk of a row (part p of chunk c of a row lies at row * kParts * d4 + p * d4 + c),
// kRows rows are in flight per thread.
struct AdagradOp {
  static constexpr int kParts = 1;
  static constexpr int kRows = 3;      // four cost a wavefront of occupancy: 33 against 28.5 us
  float lr, eps;
  __device__ __forceinline__ void apply(float4& w, float4 (&st)[1], float4 g) const {
    adagrad4v(w, st[0], g, lr, eps);
  }
};
struct AdamOp {
  static constexpr int kParts = 2;
  static constexpr int kRows = 2;
  AdamArgs k;
  __device__ __forceinline__ void apply(float4& w, float4 (&st)[2], float4 g) const {
    adam1(w.x, st[0].x, st[1].x, g.x, k);
    adam1(w.y, st[0].y, st[1].y, g.y, k);
    adam1(w.z, st[0].z, st[1].z, g.z, k);
    adam1(w.w, st[0].w, st[1].w, g.w, k);
  }
};

// The update over the rows of a batch (one row per virtual id), Op::kRows rows per thread in flight.
// A bypass row (slot >= C: a miss that found no cache slot) is also written to the Host table
// here: it lives for this step only.
// The gradient of a cold row (see kColdBit) is summed here from its at most kColdMax gradient rows
// (cold_pay[v] = their numbers, -1 = none; both -1 = not a cold row), in fp64, lower gradient row
// first (so the sum does not depend on the order in which the grouping pass happened to rank the
// group's positions); a row marked kEdgeMark is left to the block that chains its partials; every
// other row takes its sum from the common-gradient matrix.  kOneHot: a gradient row is read once
// per step.
template <class Op, bool kStream, bool kOneHot>
__device__ __forceinline__ void update_rows(const Op& op, const float4* __restrict__ common,
                                            const int* __restrict__ slot,
                                            const int64_t* __restrict__ unique_ids,
                                            float4* __restrict__ cw, float4* __restrict__ cs,
                                            const HostRows& h, int C, int boff, int d4, int U,
                                            const int2* __restrict__ cold_pay,
                                            const float4* __restrict__ grad, int blk, int nblk) {
  static_assert(kColdMax == 2, "the gather path below takes two gradient rows");
  constexpr int kR = Op::kRows, kP = Op::kParts;
  const int64_t total = (int64_t)U * d4;
  const int64_t stride = (int64_t)nblk * 256;
  for (int64_t i0 = (int64_t)blk * 256 + threadIdx.x; i0 < total; i0 += kR * stride) {
    float4 g[kR], w[kR], st[kR][kP], x1[kR];
    int64_t r[kR], rs[kR];
    int sl[kR], vrow[kR], cc[kR];
    int2 cp[kR];
    // two levels of indirection, kR rows in flight at each: slot and cold rows of the row, then
    // its weights, state and gradient (one row of the common matrix, or its own one or two rows)
#pragma unroll
    for (int u = 0; u < kR; ++u) {
      const int64_t i = i0 + u * stride;
      r[u] = -1; sl[u] = -1; cp[u] = make_int2(-1, -1);
      if (i < total) {
        vrow[u] = (int)(i / d4); cc[u] = (int)(i - (int64_t)vrow[u] * d4);
        sl[u] = slot[vrow[u]];
        cp[u] = cold_pay[vrow[u]];
      }
    }
#pragma unroll
    for (int u = 0; u < kR; ++u) {
      x1[u] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (cp[u].x == kEdgeMark) continue;     // updated by the block that chains its partials
      if (sl[u] < 0) continue;
      const int64_t row = sl[u] >= C ? sl[u] + boff : sl[u];
      r[u] = row * d4 + cc[u];
      rs[u] = row * (kP * d4) + cc[u];
      w[u] = ld_row<kStream>(&cw[r[u]]);
#pragma unroll
      for (int p = 0; p < kP; ++p) st[u][p] = ld_row<kStream>(&cs[rs[u] + p * d4]);
      if (cp[u].x >= 0) {
        // lower gradient row first
        const bool two = cp[u].y >= 0;
        const int q0 = two && cp[u].y < cp[u].x ? cp[u].y : cp[u].x;
        const int q1 = two && cp[u].y < cp[u].x ? cp[u].x : cp[u].y;
        g[u] = ld_row<kOneHot>(&grad[(int64_t)q0 * d4 + cc[u]]);
        if (two) x1[u] = ld_row<kOneHot>(&grad[(int64_t)q1 * d4 + cc[u]]);
      } else {
        g[u] = ld_row<kStream>(&common[(int64_t)vrow[u] * d4 + cc[u]]);
      }
    }
#pragma unroll
    for (int u = 0; u < kR; ++u)
      if (cp[u].x >= 0 && cp[u].y >= 0) {
        g[u].x = (float)((double)g[u].x + (double)x1[u].x);
        g[u].y = (float)((double)g[u].y + (double)x1[u].y);
        g[u].z = (float)((double)g[u].z + (double)x1[u].z);
        g[u].w = (float)((double)g[u].w + (double)x1[u].w);
      }
#pragma unroll
    for (int u = 0; u < kR; ++u)
      if (r[u] >= 0) {
        op.apply(w[u], st[u], g[u]);
        st_row<kStream>(&cw[r[u]], w[u]);
#pragma unroll
        for (int p = 0; p < kP; ++p) st_row<kStream>(&cs[rs[u] + p * d4], st[u][p]);
        if (sl[u] >= C) {
          const int64_t id = unique_ids[vrow[u]];
          h.w[id * h.hs4 + cc[u]] = w[u];
#pragma unroll
          for (int p = 0; p < kP; ++p) h.a[id * h.has4 + p * d4 + cc[u]] = st[u][p];
        }
      }
  }
}

// One update of row v, chunk c4 of it, with the summed gradient g (lanes c4 < d4 of a lane group).
template <class Op>
__device__ __forceinline__ void update_one_row(const Op& op, int v, int c4, float4 g,
                                               const int* __restrict__ slot,
                                               const int64_t* __restrict__ unique_ids,
                                               float4* __restrict__ cw, float4* __restrict__ cs,
                                               const HostRows& h, int C, int boff, int d4) {
  constexpr int kP = Op::kParts;
  const int sl = slot[v];
  if (sl < 0) return;
  const int64_t row = sl >= C ? sl + boff : sl;
  const int64_t r = row * d4 + c4, rs = row * (kP * d4) + c4;
  float4 w = cw[r], st[kP];
#pragma unroll
  for (int p = 0; p < kP; ++p) st[p] = cs[rs + p * d4];
  op.apply(w, st, g);
  cw[r] = w;
#pragma unroll
  for (int p = 0; p < kP; ++p) cs[rs + p * d4] = st[p];
  if (sl >= C) {
    const int64_t id = unique_ids[v];
    h.w[id * h.hs4 + c4] = w;
#pragma unroll
    for (int p = 0; p < kP; ++p) h.a[id * h.has4 + p * d4 + c4] = st[p];
  }
}

// Cold rows are summed here (the stream that ran before passed over them), and so are the groups
// that the stream left as block-edge partials: the first blocks of the grid do what k_seg_finish
// does and update the rows they have summed at once; the other blocks walk the rows and pass
// over the marked ones (kEdgeMark).  The two parts share nothing and wait for nothing: the chain of
// dependent loads that sums a run (ten microseconds as a kernel of its own) runs beside the row
// stream instead of before it.

template <class Op, bool kOneHot>
__device__ __forceinline__ void update_kernel(const Op& op, const float4* __restrict__ common,
                                              const int* __restrict__ slot,
                                              const int64_t* __restrict__ unique_ids,
                                              float4* __restrict__ cw, float4* __restrict__ cs,
                                              const HostRows& h, int C, int boff, int d4,
                                              const Ctr* ctr, const int2* __restrict__ cold_pay,
                                              const float4* __restrict__ grad,
                                              const double* __restrict__ bp,
                                              const int* __restrict__ bp_vid, int nslots,
                                              int nedge) {
  if ((int)blockIdx.x < nedge) {
    edge_block(bp, bp_vid, nslots, d4, (int)blockIdx.x, [&](int v, int c4, float4 g) {
      update_one_row(op, v, c4, g, slot, unique_ids, cw, cs, h, C, boff, d4);
    });
    return;
  }
  const int U = ctr->U;
  // Few rows for the grid (the host does not know their number): every thread that works takes
  // Op::kRows of them at once, the other blocks return; spread over all blocks there was one row in
  // flight per thread and two rounds of blocks.  132e3 rows of dim 16 23.5 -> 20.6 us, 200e3 of dim 32
  // 28.4 -> 26.7.
  const int64_t total = (int64_t)U * d4;
  const int64_t most = (total + 256 * Op::kRows - 1) / (256 * Op::kRows);
  const int blk = (int)blockIdx.x - nedge;
  int nblk = (int)gridDim.x - nedge;
  if (nblk > most) nblk = (int)most;
  if (blk >= nblk) return;
  if (stream_rows(U, d4, Op::kParts * d4))
    update_rows<Op, true, kOneHot>(op, common, slot, unique_ids, cw, cs, h, C, boff, d4, U, cold_pay, grad, blk, nblk);
  else
    update_rows<Op, false, kOneHot>(op, common, slot, unique_ids, cw, cs, h, C, boff, d4, U, cold_pay, grad, blk, nblk);
}

// Four wavefronts per SIMD: with the registers of five or six the kernel is slower (31.1 and 36.4 us
// against 29.1 at the target configuration: fewer loads in flight per wavefront, and more
// wavefronts evicting each other's lines).
template <bool kOneHot>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4)))
void k_adagrad_rows(
    const float4* __restrict__ common, const int* __restrict__ slot,
    const int64_t* __restrict__ unique_ids, float4* __restrict__ cw, float4* __restrict__ ca,
    HostRows h, int C, int boff, float lr, float eps, int d4, const Ctr* ctr,
    const int2* __restrict__ cold_pay, const float4* __restrict__ grad,
    const double* __restrict__ bp, const int* __restrict__ bp_vid, int nslots, int nedge) {
  AdagradOp op;
  op.lr = lr; op.eps = eps;
  update_kernel<AdagradOp, kOneHot>(op, common, slot, unique_ids, cw, ca, h, C, boff, d4, ctr, cold_pay,
                                    grad, bp, bp_vid, nslots, nedge);
}

template <bool kOneHot>
__global__ __launch_bounds__(256) void k_adam_rows(
    const float4* __restrict__ common, const int* __restrict__ slot,
    const int64_t* __restrict__ unique_ids, float4* __restrict__ cw, float4* __restrict__ cs,
    HostRows h, int C, int boff, AdamArgs k, int d4, const Ctr* ctr,
    const int2* __restrict__ cold_pay, const float4* __restrict__ grad,
    const double* __restrict__ bp, const int* __restrict__ bp_vid, int nslots, int nedge) {
  AdamOp op;
  op.k = k;
  update_kernel<AdamOp, kOneHot>(op, common, slot, unique_ids, cw, cs, h, C, boff, d4, ctr, cold_pay,
                                 grad, bp, bp_vid, nslots, nedge);
}

// ---------------------------------------------------------------------------------------------
// The whole update of a small batch (small_update), one launch: a lane group per virtual id
// reads the id's group, sums its gradient rows in fp64 in the order of the grouping and updates the row.
// Nothing here is many bytes; the stream and the row kernel took their time in start-up, chains of
// partial sums and the dependent loads of two kernels.  An id with more than kGroupShort positions is left to
// the whole block, its lane groups each a strided share in fixed order, combined in a tree; there is a block per
// kGroupShort positions, at most kGroupBlocks of them, and a block's ids lie as far apart as the grid allows, because the
// frequent ids of a batch are among its first ones (with a block's worth of lane groups per block, 100 ids of 12 to 50
// positions each came to one or two blocks, one after the other: 278 us at 5000 positions of dim 16, 9 this way).
// One compute unit loads gradient rows at 130 GB/s.  So from kSplitChunks on (320 KiB, 2.5 us of one block) a very
// frequent id is summed by further blocks, a share of the grouping each; the last to arrive adds up their sums in the
// order of the shares (2 us for the way through memory, so shares of 64 KiB, and an id takes more than two).
// sfc_backward_update us, stream and row kernel / one block per id / this way, power-law ids, half of the positions one
// id, all of them one id: 5000 positions of dim 16 (not split) 15.9 / 10.9, 15.6 / 12.6, 16.6 / 12.8; 10240 of dim 16
// 19.8 / 14.1 / 13.9, 17.8 / 15.5 / 11.9, 16.9 / 18.4 / 12.5; 5000 of dim 32 16.7 / 12.2 / 11.0, 15.1 / 14.7 / 11.7, 15.2 /
// 17.3 / 12.5; 2048 of dim 80 15.3 / 12.1 / 11.0, 14.5 / 14.4 / 11.3, 14.4 / 18.2 / 13.2; 1250 of dim 128 15.4 / 11.8 / 10.6,
// 13.8 / 13.9 / 11.0, 14.1 / 17.0 / 13.2; 640 of dim 256 14.9 / 12.0 / 10.4, 13.6 / 14.2 / 10.9, 13.6 / 17.0 / 12.3; 16384 of
// dim 4 (not split) 27.8 / 14.5, 29.1 / 12.3, 29.0 / 12.4.  All distinct 12.1 to 17 by the stream and the row kernel, 6.2 to 10
// this way.  The limit on the size lies where a batch of one id stops being faster on wide rows; beyond it, the same three
// inputs, two kernels / this way: 1536 of dim 128 14.8 / 11.2, 13.7 / 11.9, 13.7 / 13.7; 2048 of dim 128 15.3 / 11.3, 13.9 /
// 12.6, 13.9 / 14.8; 3276 of dim 80 15.9 / 11.8, 14.6 / 12.7, 14.4 / 15.1; 1000 of dim 256 13.9 / 11.2, 13.6 / 12.0, 13.5 / 14.5;
// 8192 of dim 32 17.2 / 13.7, 15.8 / 12.9, 15.5 / 14.1.
// ---------------------------------------------------------------------------------------------
constexpr int64_t kSmallUpdate = 1 << 14, kSmallUpdateChunks = 40 << 10;      // positions; 16-byte chunks of their rows
inline bool small_update(int64_t n, int d4) { return n > 0 && n <= kSmallUpdate && n * d4 <= kSmallUpdateChunks; }
constexpr int kGroupShort = 16;
constexpr int kGroupBlocks = 512;            // lane groups for kSmallUpdate ids of the narrowest rows
constexpr int kGroupThreads = 1024;
inline __host__ __device__ int update_groups(int d4) { return kGroupThreads / 64 * (64 / d4 > 0 ? 64 / d4 : 1); }
// A split batch: its grouping is cut into shares of update_share(d4) positions, and an id with more than two shares'
// worth of positions is summed by the blocks of its shares.
constexpr int kShareChunks = 4096, kSplitChunks = 20 << 10, kMaxShares = 16;
inline __host__ __device__ int update_share(int d4) { return kShareChunks / d4; }
inline int update_shares(int64_t n, int d4) {
  return n * d4 > kSplitChunks ? (int)((n + update_share(d4) - 1) / update_share(d4)) : 0;
}

template <class Op>
__global__ __launch_bounds__(kGroupThreads) void k_update_groups(
    const Op op, const int64_t* __restrict__ grp, const int64_t* __restrict__ perm64,
    const float4* __restrict__ grad, const int* __restrict__ slot, const int64_t* __restrict__ unique_ids,
    float4* __restrict__ cw, float4* __restrict__ cs, HostRows h, int C, int boff, int d4, const Ctr* ctr,
    int n, int shares, double* part, int* ticket) {
  constexpr int kP = Op::kParts, kFly = 8;
  __shared__ double red[kGroupThreads * 4];
  __shared__ int long_v[kGroupThreads], n_long;
  if (threadIdx.x == 0) n_long = 0;
  __syncthreads();
  const int U = ctr->U, groups = update_groups(d4), G = groups / (kGroupThreads / 64);
  const int lane = lane_id(), g = lane / d4, c4 = lane - g * d4;
  const int gi = (int)(threadIdx.x >> 6) * G + g;         // this lane group among the block's
  const bool active = g < G;
  const int share = update_share(d4), split_from = shares > 0 ? 2 * share : kIntMax;

  // the row of virtual id `id` with the sum s: weights and state are on their way before the sum is there
  auto apply = [&](int id, int sl, float4 w, float4 (&st)[kP], const D4& s) {
    const int64_t row = sl >= C ? sl + boff : sl;
    op.apply(w, st, d4_round(s));
    cw[row * d4 + c4] = w;
#pragma unroll
    for (int p = 0; p < kP; ++p) cs[row * (kP * d4) + p * d4 + c4] = st[p];
    if (sl >= C) {
      const int64_t host = unique_ids[id];
      h.w[host * h.hs4 + c4] = w;
#pragma unroll
      for (int p = 0; p < kP; ++p) h.a[host * h.has4 + p * d4 + c4] = st[p];
    }
  };
  auto load_row = [&](int sl, float4& w, float4 (&st)[kP]) {
    const int64_t row = sl >= C ? sl + boff : sl;
    w = cw[row * d4 + c4];
#pragma unroll
    for (int p = 0; p < kP; ++p) st[p] = cs[row * (kP * d4) + p * d4 + c4];
  };
  // entries first, first + step, ... below end
  auto add_rows = [&](D4& s, int first, int end, int step) {
    int64_t e[kFly];
#pragma unroll
    for (int u = 0; u < kFly; ++u) e[u] = first + u * step < end ? perm64[first + u * step] : (int64_t)-1;
    for (int q = first; q < end; q += kFly * step) {
      float4 x[kFly];
      int64_t en[kFly];
#pragma unroll
      for (int u = 0; u < kFly; ++u)
        if (e[u] >= 0) x[u] = grad[(int64_t)(uint32_t)e[u] * d4 + c4];
#pragma unroll
      for (int u = 0; u < kFly; ++u) {                    // the next round's entries meanwhile
        const int qn = q + (kFly + u) * step;
        en[u] = qn < end ? perm64[qn] : (int64_t)-1;
      }
#pragma unroll
      for (int u = 0; u < kFly; ++u) {
        if (e[u] >= 0) d4_add(s, x[u]);
        e[u] = en[u];
      }
    }
  };

  // the sum of the rows of entries [first, end) by the whole block; the result is the first lane group's
  auto block_rows = [&](int first, int end) {
    D4 s; d4_zero(s);
    if (active) add_rows(s, first + gi, end, groups);
    double* const r = &red[(gi * d4 + c4) * 4];           // (groups * d4 <= kGroupThreads)
    if (active) { r[0] = s.x; r[1] = s.y; r[2] = s.z; r[3] = s.w; }
    int o = 1;
    while (o < groups) o <<= 1;
    for (o >>= 1; o > 0; o >>= 1) {
      __syncthreads();
      if (active && gi < o && gi + o < groups) {
        const double* q = r + o * d4 * 4;
        r[0] += q[0]; r[1] += q[1]; r[2] += q[2]; r[3] += q[3];
      }
    }
    if (active) { s.x = r[0]; s.y = r[1]; s.z = r[2]; s.w = r[3]; }
    return s;
  };

  // A share's block: at most the first and the last group of its positions are split ones (a group with more
  // positions than a share that meets it covers one of its ends).  Whoever brings in the last share of an id adds
  // the shares up, in order, and updates the row.
  if ((int)blockIdx.x < shares) {
    const int lo = (int)blockIdx.x * share, hi = lo + share < n ? lo + share : n;
    const int v0 = entry_vid(perm64[lo]), v1 = entry_vid(perm64[hi - 1]);
    for (int which = 0; which < (v0 == v1 ? 1 : 2); ++which) {
      const int v = which ? v1 : v0, sl = slot[v];
      const int64_t gr = grp[v];
      const int cnt = (int)(gr >> 32), start = (int)gr;
      if (cnt <= split_from || sl < 0) continue;
      const D4 s = block_rows(start > lo ? start : lo, start + cnt < hi ? start + cnt : hi);
      if (gi == 0 && active) {
        double* const p = &part[((2 * (int)blockIdx.x + which) * d4 + c4) * 4];
        __hip_atomic_store(p, s.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(p + 1, s.y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(p + 2, s.z, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(p + 3, s.w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __threadfence();
      }
      __syncthreads();
      const int j0 = start / share, nj = (start + cnt - 1) / share - j0 + 1;
      if (threadIdx.x == 0) {
        n_long = atomicAdd(&ticket[j0], 1) == nj - 1;
        if (n_long) atomicExch(&ticket[j0], 0);            // for the next batch
        __threadfence();
      }
      __syncthreads();
      if (n_long && gi == 0 && active) {
        float4 w, st[kP];
        load_row(sl, w, st);
        D4 sum; d4_zero(sum);
        for (int j = 0; j < nj; ++j) {
          const int at = 2 * (j0 + j) + (j == 0 && start != j0 * share ? 1 : 0);
          double* const p = &part[(at * d4 + c4) * 4];
          sum.x += __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          sum.y += __hip_atomic_load(p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          sum.z += __hip_atomic_load(p + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          sum.w += __hip_atomic_load(p + 3, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        apply(v, sl, w, st, sum);
      }
      __syncthreads();
    }
    return;
  }

  const int blk = (int)blockIdx.x - shares, blocks = (int)gridDim.x - shares;
  const int nblk = blocks < U ? blocks : U;                        // blocks that have work
  if (blk >= nblk) return;
  const int v = blk + gi * nblk;
  if (active && v < U) {
    const int64_t gr = grp[v];
    const int sl = slot[v], cnt = (int)(gr >> 32), start = (int)gr;
    if (sl >= 0 && cnt <= split_from) {
      if (cnt > kGroupShort) {
        if (c4 == 0) long_v[atomicAdd(&n_long, 1)] = v;
      } else {
        float4 w, st[kP];
        load_row(sl, w, st);
        D4 s; d4_zero(s);
        add_rows(s, start, start + cnt, 1);
        apply(v, sl, w, st, s);
      }
    }
  }
  __syncthreads();
  const int nl = n_long;
  for (int i = 0; i < nl; ++i) {
    const int id = long_v[i];
    const int64_t gr = grp[id];
    const int sl = slot[id], cnt = (int)(gr >> 32), start = (int)gr;
    float4 w, st[kP];
    if (gi == 0 && active) load_row(sl, w, st);
    const D4 s = block_rows(start, start + cnt);
    if (gi == 0 && active) apply(id, sl, w, st, s);
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------------------------
// Row-wise Adagrad: one accumulator per row (first float of a one-chunk state),
//   acc += mean_j(g_j^2) ; w_j -= lr * g_j / (sqrt(acc) + eps).
// One thread per 16-byte chunk of a row as above; the d4 lanes of a row add their squares with
// shuffles when d4 is a power of two (a row then never straddles a wavefront).  Such rows take the path of the
// element-wise optimizers: the stream passes over the cold groups and leaves its block-edge partials, both are summed
// here (213e3 power-law positions of dim 128, us: stream 29.8 + finish 6.3 + rows 26.5 before, 22.5 + 21.4 this way).
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ float sum_squares(float4 g, int d4) {
  float ss = g.x * g.x + g.y * g.y + g.z * g.z + g.w * g.w;
  for (int d = 1; d < d4; d <<= 1) ss += __shfl_xor(ss, d, kWave);
  return ss;
}

// Widths that are no power of two: one thread per row (the lanes of a row could straddle two wavefronts, and
// the accumulator must be read by all of them before one writes it), every sum from the common matrix.
__global__ __launch_bounds__(256) void k_rowwise_adagrad_any(const float4* __restrict__ common,
                                                              const int* __restrict__ slot,
                                                              const int64_t* __restrict__ unique_ids,
                                                              float4* __restrict__ cw,
                                                              float4* __restrict__ cs, HostRows h,
                                                              int C, int boff, float lr, float eps,
                                                              int d4, const Ctr* ctr) {
  const int64_t stride = (int64_t)gridDim.x * 256;
  const float inv_d = 1.0f / (float)(4 * d4);
  for (int64_t vrow = (int64_t)blockIdx.x * 256 + threadIdx.x; vrow < ctr->U; vrow += stride) {
    const int sl = slot[vrow];
    if (sl < 0) continue;
    float ss = 0.f;
    for (int j = 0; j < d4; ++j) {
      const float4 q = common[vrow * d4 + j];
      ss += q.x * q.x + q.y * q.y + q.z * q.z + q.w * q.w;
    }
    const int64_t row = sl >= C ? sl + boff : sl;
    float4 st = cs[row];
    st.x = st.x + ss * inv_d;
    const float den = sqrtf(st.x) + eps;
    const int64_t id = unique_ids[vrow];
    for (int j = 0; j < d4; ++j) {
      const float4 g = common[vrow * d4 + j];
      float4 w = cw[row * d4 + j];
      w.x = w.x - lr * g.x / den; w.y = w.y - lr * g.y / den;
      w.z = w.z - lr * g.z / den; w.w = w.w - lr * g.w / den;
      cw[row * d4 + j] = w;
      if (sl >= C) h.w[id * h.hs4 + j] = w;
    }
    cs[row] = st;
    if (sl >= C) h.a[id * h.has4] = st;
  }
}

template <bool kOneHot>
__global__ __launch_bounds__(256) void k_rowwise_adagrad_rows(
    const float4* __restrict__ common, const int* __restrict__ slot,
    const int64_t* __restrict__ unique_ids, float4* __restrict__ cw, float4* __restrict__ cs,
    HostRows h, int C, int boff, float lr, float eps, int d4, const Ctr* ctr,
    const int2* __restrict__ cold_pay, const float4* __restrict__ grad,
    const double* __restrict__ bp, const int* __restrict__ bp_vid, int nslots, int nedge) {
  const float inv_d = 1.0f / (float)(4 * d4);
  // chunk c of row `row` (bypass rows: of the Host row `id` as well), its gradient and the row's sum of squares
  auto update = [&](int64_t row, int c, bool bypass, int64_t id, float4 w, float4 st, float4 g, float ss) {
    const float acc = st.x + ss * inv_d;
    const float den = sqrtf(acc) + eps;
    w.x = w.x - lr * g.x / den; w.y = w.y - lr * g.y / den;
    w.z = w.z - lr * g.z / den; w.w = w.w - lr * g.w / den;
    cw[row * d4 + c] = w;
    st.x = acc;
    if (c == 0) cs[row] = st;
    if (bypass) {
      h.w[id * h.hs4 + c] = w;
      if (c == 0) h.a[id * h.has4] = st;
    }
  };
  if ((int)blockIdx.x < nedge) {
    edge_block(bp, bp_vid, nslots, d4, (int)blockIdx.x, [&](int v, int c4, float4 g) {
      const float ss = sum_squares(g, d4);     // the d4 lanes of the row are here together
      const int sl = slot[v];
      if (sl < 0) return;
      const int64_t row = sl >= C ? sl + boff : sl;
      const float4 st = cs[row];
      update(row, c4, sl >= C, sl >= C ? unique_ids[v] : 0, cw[row * d4 + c4], st, g, ss);
    });
    return;
  }
  const int64_t total = (int64_t)ctr->U * d4;
  const int64_t stride = (int64_t)((int)gridDim.x - nedge) * 256;
  // every lane of a wavefront runs the same number of iterations: the shuffles stay convergent.
  // Four rows per thread in flight at each level (slot and cold rows, then gradient, state and weights).
  const int64_t rounds = (total + 4 * stride - 1) / (4 * stride);
  int64_t i0 = (int64_t)((int)blockIdx.x - nedge) * 256 + threadIdx.x;
  for (int64_t it = 0; it < rounds; ++it, i0 += 4 * stride) {
    int vrow[4], c[4], sl[4];
    int2 cp[4];
    float4 g[4], x1[4], st[4], w[4];
    int64_t row[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t i = i0 + u * stride;
      const bool live = i < total;
      vrow[u] = live ? (int)(i / d4) : 0;
      c[u] = live ? (int)(i % d4) : 0;
      sl[u] = live ? slot[vrow[u]] : -1;
      cp[u] = live ? cold_pay[vrow[u]] : make_int2(-1, -1);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      g[u] = x1[u] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (cp[u].x == kEdgeMark) sl[u] = -1;    // updated by the block that chains its partials
      row[u] = sl[u] >= C ? sl[u] + boff : sl[u];
      if (sl[u] < 0) continue;
      st[u] = cs[row[u]]; w[u] = cw[row[u] * d4 + c[u]];
      if (cp[u].x >= 0) {
        g[u] = ld_row<kOneHot>(&grad[(int64_t)cp[u].x * d4 + c[u]]);
        if (cp[u].y >= 0) x1[u] = ld_row<kOneHot>(&grad[(int64_t)cp[u].y * d4 + c[u]]);
      } else {
        g[u] = common[(int64_t)vrow[u] * d4 + c[u]];
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (cp[u].x >= 0 && cp[u].y >= 0) {      // (two terms: the same sum in either order)
        g[u].x = (float)((double)g[u].x + (double)x1[u].x);
        g[u].y = (float)((double)g[u].y + (double)x1[u].y);
        g[u].z = (float)((double)g[u].z + (double)x1[u].z);
        g[u].w = (float)((double)g[u].w + (double)x1[u].w);
      }
      const float ss = sum_squares(g[u], d4);
      if (sl[u] >= 0)
        update(row[u], c[u], sl[u] >= C, sl[u] >= C ? unique_ids[vrow[u]] : 0, w[u], st[u], g[u], ss);
    }
  }
}

template <typename T>
__global__ __launch_bounds__(256) void k_fill(T* p, int64_t n, T v) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) p[i] = v;
}

}  // namespace sfc
