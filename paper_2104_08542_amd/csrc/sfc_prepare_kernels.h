// Kernels of sfc_prepare: Virtual Sparse Id (batch unique with first-appearance order and the
// per-position inverse) and the MixCache manager (resolve against the index in HBM, victim
// selection by batch-granular LRU, slot assignment, index maintenance).
//
// Determinism: every output of sfc_prepare (unique ids, inverse, slots, miss and victim lists,
// cache state) is a function of the input sets and slot numbers only: their orders come from
// prefix scans over positions / virtual ids / slots, and atomics are used only where the result
// is order-free (min, counters, set insert).  The one thing that does follow the arrival order of
// atomics is internal: the order of a group's entries in perm64 (k_rank_resolve ranks the
// positions of an id by the value its counting atomic returns).  It decides the order of an fp64
// sum, nothing else; see the segment-sum kernels for what that means for the results.
#pragma once
#include "sfc_device.h"

namespace sfc {

constexpr int kPosChunk = 2048;   // positions (or slots) per block in the scan passes
constexpr int kVidTile = 256;     // virtual ids per tile in resolve / assign

// ---------------------------------------------------------------------------------------------
// VSI pass 1: insert every position's id into the batch table (open addressing, linear probing,
// in HBM) and keep the smallest position per key; remember the table entry of each position.
//
// What bounds it is atomics and random accesses on the table's lines.  So an entry is one 64-bit word,
// (tag << sh) | smallest position so far (tag = the id, or V for the collapsed out-of-range id; sh = bits of
// a position of this batch): claiming an entry stores its position with the same compare-and-swap,
// and a smaller position is one 64-bit minimum.  (Key and position in two words took two atomics for
// every distinct id and a table twice the size: 53 us instead of 46.5 at 65536 x 39 positions, 159 instead
// of 134 at 8.9e6 in bags, 143 instead of 108 at 1.28e6 uniform ones.)
// Same-address atomics serialise at the memory side (about 10 ns each on this chip), and the
// hottest id of a power-law batch owns a fifth of all positions.  So each block first
// deduplicates its positions in an LDS table (key -> smallest position in the block) and
// only the distinct keys of the block go to HBM, all in flight.  There a plain load
// comes first (the table entry of a key never changes once set, and a stale position can only be too
// large), and an atomic is issued only when the load has not already seen the key / a small enough
// position.
// When all blocks of a large batch start together they all find the table empty, and every block's copy
// of a frequent key goes through the claim / re-read / minimum atomics on one address (thousands in a
// row, about 10 ns each).  So only the first kHeadBlocks blocks go to the table at once; the others that
// are resident from the start sleep a few microseconds first, and then their plain loads find the
// frequent keys in the table with a smaller position than theirs.  (Nothing depends on the sleep being
// long enough.)  us without the sleep / with the head in a launch of its own / this way: 58 / 35 / 29 at
// 16384 x 39 positions, 80 / 47 / 42 at 65536 x 39, 30 / 28 / 20 at 5003 x 39, 95 / 109 / 98 at 1.28e6 uniform ones
// (blocks of 512 positions).
// hslot[p] = HBM table entry of position p.
// first: one bit per position, set for the positions that hold their entry's smallest position in the
// end, all zero before.  Whoever places a position in an entry flips its bit, and whoever replaces one
// flips the bit of the position that was there too; flips commute, so the bits are right whatever the
// order of the blocks.  A block's own flips go out as one atomic per 32 positions.
// ---------------------------------------------------------------------------------------------
// Positions per block: 256, a key per thread, and from 2^22 positions on, where the grid is twenty rounds of resident
// blocks, 512, whose blocks bring fewer copies of an id to the table.  The kernel alone, us, 512 / 256 positions (512 with a
// sleep of five): 7000 13.5 / 9.1, 40e3 12.2 / 9.3, 100e3 14.9 / 12.5, 195e3 18.6 / 13.8, 291e3 20.5 / 15.6, 639e3 26.3 / 24.0, 1.28e6
// uniform ones 98.8 / 87.6, 2.56e6 34.8 / 34.6 and (s = 1.05) 57.6 / 52.4, 5e6 73.6 / 73.9, 8.9e6 116 / 125.  128 positions, a grid of
// twice as many blocks: 40e3 10.0, 291e3 17.8, 2.56e6 37.2.
constexpr int kUniqChunk = 256, kUniqChunkBig = 512;
constexpr int64_t kUniqBigFrom = (int64_t)1 << 22;
constexpr int kHeadBlocks = 64;    // blocks that go to the table at once (128: the same; 256 21.1 against 15.8 us at 291e3)
constexpr int kHeadMin = 512;      // a grid of at most this many blocks does not sleep, and claims without a load first (100e3 positions: 14.4 / 12.0)
constexpr int kResidentBlocks = 2048;        // eight per compute unit
constexpr int kHeadSleep = 3;      // times 2048 clocks, 2.6 us (2 / 3 / 4 / 5: 15.5 / 15.6 / 16.3 / 16.9 us at 291e3, 25.0 / 24.0 / 24.7 / 26.0 at 639e3)

template <typename T>
__device__ __forceinline__ T coherent_load(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The batch table's entries as the insert pass sees them.  Raw: an entry as loaded.  claim: puts (key,
// pos) into an empty entry, returns what was there.  lower: makes pos the entry's position if it is
// smaller, returns the position that was there (kIntMax: none).
struct PackedTab {
  uint64_t* w;
  int sh;
  int64_t V;
  typedef uint64_t Raw;
  static constexpr bool kClaimStoresPos = true;
  __device__ __forceinline__ uint64_t word(int64_t key, int pos) const {
    return ((uint64_t)(key == kNullKey ? V : key) << sh) | (uint32_t)pos;
  }
  __device__ __forceinline__ Raw load(uint32_t h) const { return w[h]; }
  __device__ __forceinline__ Raw coherent(uint32_t h) const { return coherent_load(&w[h]); }
  __device__ __forceinline__ bool empty(Raw r) const { return r == ~0ull; }
  __device__ __forceinline__ bool same(Raw r, int64_t key) const { return r >> sh == word(key, 0) >> sh; }
  __device__ __forceinline__ int pos(Raw r) const { return (int)(r & ((1ull << sh) - 1)); }
  __device__ __forceinline__ Raw claim(uint32_t h, int64_t key, int p) const {
    return atomicCAS((unsigned long long*)&w[h], ~0ull, (unsigned long long)word(key, p));
  }
  __device__ __forceinline__ int lower(uint32_t h, int64_t key, int p) const {
    return pos(atomicMin((unsigned long long*)&w[h], (unsigned long long)word(key, p)));
  }
};
// Where an id and a position do not fit one word together (a Host table of 2^34 rows or more with a
// batch of 2^30 ids): key and position in 16 bytes, the claim takes the key only.
struct WideTab {
  UEntry* e;
  int sh;
  int64_t V;
  struct Raw { int64_t key; int minpos; };
  static constexpr bool kClaimStoresPos = false;
  __device__ __forceinline__ Raw load(uint32_t h) const {
    const int4 q = *reinterpret_cast<const int4*>(&e[h]);
    return Raw{((int64_t)(uint32_t)q.y << 32) | (uint32_t)q.x, q.z};
  }
  __device__ __forceinline__ Raw coherent(uint32_t h) const {
    return Raw{coherent_load(&e[h].key), coherent_load(&e[h].minpos)};
  }
  __device__ __forceinline__ bool empty(Raw r) const { return r.key == kEmpty; }
  __device__ __forceinline__ bool same(Raw r, int64_t key) const { return r.key == key; }
  __device__ __forceinline__ int pos(Raw r) const { return r.minpos; }
  __device__ __forceinline__ Raw claim(uint32_t h, int64_t key, int) const {
    return Raw{(int64_t)atomicCAS((unsigned long long*)&e[h].key, (unsigned long long)kEmpty,
                                  (unsigned long long)key), kIntMax};
  }
  __device__ __forceinline__ int lower(uint32_t h, int64_t, int p) const { return atomicMin(&e[h].minpos, p); }
};

// Rebuild of the hashed cache index: emptied, then every resident id goes back in, by nblk blocks of 256 threads
// each, over the occupied slots [0, f).  The previous step's plan asks for it when too many entries are deleted ones;
// the two halves run between that step's last index update and this step's resolve, as further blocks of the
// insert and the assign pass (rebuild_blocks each, which return at once otherwise), or as kernels of their own
// where those passes are not launched (k_ctr_init, k_index_refill).
// A thread puts its ids back one after the other, so large caches get more blocks.  What a step with a rebuild takes
// longer than one without, us, kernels of their own (2048 blocks each) / 256 blocks inside / 2048 inside: 3e5 slots 45 /
// 26 / 42, 1e6 100 / 82 / 84, 8e6 720 / 820 / 690.
inline int rebuild_blocks(int64_t C) { return C < (1 << 20) ? 256 : C >= (8 << 20) ? 2048 : (int)(C >> 12); }
__device__ __forceinline__ void index_clear(IdxEntry* index, uint32_t hi, int blk, int nblk) {
  IdxEntry e; e.key = kEmpty; e.slot = -1; e.pad = 0;
  for (uint32_t i = blk * 256 + threadIdx.x; i < hi; i += nblk * 256) index[i] = e;
}
__device__ __forceinline__ void index_reinsert(IdxEntry* index, uint32_t hi,
                                               const int64_t* __restrict__ slot_id, int f, int blk, int nblk) {
  for (int s = blk * 256 + threadIdx.x; s < f; s += nblk * 256) {
    const int64_t id = slot_id[s];
    if (id < 0) continue;
    uint32_t h = bucket_of(id, hi);
    for (uint32_t probes = 0; probes < hi; ++probes) {
      if (index[h].key == kEmpty &&
          (int64_t)atomicCAS((unsigned long long*)&index[h].key, (unsigned long long)kEmpty,
                             (unsigned long long)id) == kEmpty) {
        atomicExch(&index[h].slot, s);
        break;
      }
      h = h + 1 == hi ? 0 : h + 1;
    }
  }
}

template <class Tab, int kChunk>
__global__ __launch_bounds__(256) void k_uniq_insert(const int64_t* __restrict__ ids, int n, Tab tab,
                                                      uint32_t hu, int* __restrict__ hslot,
                                                      unsigned* first, int* __restrict__ n_invalid, int blocks,
                                                      const Ctr* prev, IdxEntry* index, uint32_t hi) {
  if ((int)blockIdx.x >= blocks) {            // (only with a hashed index) see index_clear
    if (prev->rebuild) index_clear(index, hi, (int)blockIdx.x - blocks, (int)gridDim.x - blocks);
    return;
  }
  constexpr int kUniqPer = kChunk / 256, kLdsTab = 2 * kChunk, kLdsPer = kLdsTab / 256;
  __shared__ int64_t lkey[kLdsTab];
  __shared__ int lval[kLdsTab];               // smallest position of the key in this block; later its HBM entry
  __shared__ unsigned short lst[kChunk];      // occupied LDS entries, compacted
  __shared__ unsigned flip[kChunk / 32];      // bit per position of the block: placed in an entry by this block
  __shared__ int smem[20];
  for (int i = threadIdx.x; i < kLdsTab; i += 256) { lkey[i] = kEmpty; lval[i] = kIntMax; }
  if (threadIdx.x < kChunk / 32) flip[threadIdx.x] = 0;
  const int64_t V = tab.V;
  const int base = (int)blockIdx.x * kChunk;
  int ls[kUniqPer];
  int64_t idv[kUniqPer];
#pragma unroll
  for (int j = 0; j < kUniqPer; ++j) {      // all loads in flight before the LDS work starts
    const int p = base + j * 256 + (int)threadIdx.x;
    idv[j] = p < n ? ids[p] : 0;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kUniqPer; ++j) {
    const int p = base + j * 256 + (int)threadIdx.x;
    bool invalid = false;
    ls[j] = 0;
    if (p < n) {
      int64_t key = idv[j];
      if (key < 0 || key >= V) { key = kNullKey; invalid = true; }
      uint32_t l = (uint32_t)mix64((uint64_t)key) & (kLdsTab - 1);
      for (int probes = 0; probes < kLdsTab; ++probes) {
        const int64_t k = lkey[l];
        if (k == key) break;
        if (k == kEmpty) {
          const int64_t old = (int64_t)atomicCAS((unsigned long long*)&lkey[l],
                                                 (unsigned long long)kEmpty, (unsigned long long)key);
          if (old == kEmpty || old == key) break;
        }
        l = (l + 1) & (kLdsTab - 1);
      }
      if (lval[l] > p) atomicMin(&lval[l], p);
      ls[j] = (int)l;
    }
    const uint64_t b = __ballot(invalid);
    if (b && lane_id() == 0) atomicAdd(n_invalid, __popcll(b));
  }
  __syncthreads();
  // compact the occupied entries (consecutive entries per thread)
  int nocc;
  {
    unsigned occ = 0;
#pragma unroll
    for (int k = 0; k < kLdsPer; ++k)
      if (lkey[threadIdx.x * kLdsPer + k] != kEmpty) occ |= 1u << k;
    int at = block_excl_scan(__popc(occ), nocc, smem);
#pragma unroll
    for (int k = 0; k < kLdsPer; ++k)
      if (occ & (1u << k)) lst[at++] = (unsigned short)(threadIdx.x * kLdsPer + k);
  }
  __syncthreads();
  if (blocks > kHeadMin && blockIdx.x >= kHeadBlocks && blockIdx.x < kResidentBlocks)
    for (int i = 0; i < kHeadSleep; ++i) __builtin_amdgcn_s_sleep(32);
  // distinct keys of the block -> HBM table, kFly per thread in flight
  constexpr int kFly = kUniqPer;
  const bool all_claim = blocks <= kHeadMin;        // no load first: the table is empty for all of them
  {
    int e[kFly], pm[kFly];
    int64_t key[kFly];
    uint32_t h[kFly];
    typename Tab::Raw r[kFly];
    bool mine[kFly], fresh[kFly];             // fresh: r has just come from the memory side
#pragma unroll
    for (int u = 0; u < kFly; ++u) {
      const int i = (int)threadIdx.x + u * 256;
      e[u] = -1;
      mine[u] = false;
      if (i < nocc) {
        e[u] = lst[i];
        key[u] = lkey[e[u]];
        pm[u] = lval[e[u]];
        h[u] = bucket_of(key[u], hu);
        if (!all_claim) r[u] = tab.load(h[u]);
      }
      fresh[u] = false;
    }
    // first probe: where the plain load saw an empty entry, try to claim it; all in flight
#pragma unroll
    for (int u = 0; u < kFly; ++u)
      if (e[u] >= 0 && (all_claim || tab.empty(r[u]))) {
        r[u] = tab.claim(h[u], key[u], pm[u]);
        mine[u] = tab.empty(r[u]);
        fresh[u] = Tab::kClaimStoresPos;
      }
#pragma unroll
    for (int u = 0; u < kFly; ++u) {
      if (e[u] < 0 || mine[u] || tab.same(r[u], key[u])) continue;
      // the entry belongs to another key: walk on (rare at load factor <= 1/2)
      for (uint32_t probes = 0; probes < hu; ++probes) {
        h[u] = h[u] + 1 == hu ? 0 : h[u] + 1;
        r[u] = tab.coherent(h[u]);
        fresh[u] = true;
        if (tab.same(r[u], key[u])) break;
        if (tab.empty(r[u])) {
          r[u] = tab.claim(h[u], key[u], pm[u]);
          mine[u] = tab.empty(r[u]);
          if (mine[u] || tab.same(r[u], key[u])) break;
        }
      }
    }
    // a plain load may be stale (too large), never too small: ask the memory side before the atomic, where what is
    // known did not come from there just now (a claim that failed)
    bool low[kFly];
#pragma unroll
    for (int u = 0; u < kFly; ++u) {
      low[u] = e[u] >= 0 && (mine[u] ? !Tab::kClaimStoresPos : tab.pos(r[u]) > pm[u]);
      if (low[u] && !mine[u] && !fresh[u]) r[u] = tab.coherent(h[u]);
    }
#pragma unroll
    for (int u = 0; u < kFly; ++u) {
      if (e[u] < 0) continue;
      lval[e[u]] = (int)h[u];
      bool placed = mine[u];
      if (low[u]) {
        placed = false;
        if (mine[u] || tab.pos(r[u]) > pm[u]) {
          const int was = tab.lower(h[u], key[u], pm[u]);
          placed = was > pm[u];
          if (placed && was != kIntMax) atomicXor(&first[was >> 5], 1u << (was & 31));
        }
      }
      const int q = pm[u] - base;
      if (placed) atomicOr(&flip[q >> 5], 1u << (q & 31));
    }
  }
  __syncthreads();
  if (threadIdx.x < kChunk / 32 && flip[threadIdx.x])
    atomicXor(&first[base / 32 + (int)threadIdx.x], flip[threadIdx.x]);
#pragma unroll
  for (int j = 0; j < kUniqPer; ++j) {
    const int p = base + j * 256 + (int)threadIdx.x;
    if (p < n) hslot[p] = lval[ls[j]];
  }
}

// VSI pass 2: how many first appearances each chunk of positions has; a wavefront per chunk.  Up to
// kCountMin positions the next pass adds up the bits itself (at most 64 KB per block, out of L2) and
// this one, 5 us of start-up and drain, is not launched.
constexpr int kCountMin = 1 << 19;
__global__ __launch_bounds__(256) void k_uniq_count(const unsigned* __restrict__ first, int nchunk,
                                                     int* __restrict__ blk_cnt) {
  static_assert(kPosChunk == 32 * kWave, "a word of bits per lane");
  const int chunk = blockIdx.x * 4 + (int)(threadIdx.x >> 6);
  if (chunk >= nchunk) return;
  const int tot = wave_sum(__popc(first[chunk * kWave + lane_id()]));
  if (lane_id() == 0) blk_cnt[chunk] = tot;
}

// Starts the step's counters, once the previous step's prepare has run to its end: they inherit the
// cache-wide fields (watermark, oldest stamp, tombstones, rebuild flag, error) from the previous
// step's and start their own tallies at zero.  Steps in flight on the other streams keep reading
// their own copy.  n_invalid is the insert pass's tally of out-of-range positions, returned to
// zero here.  (An error, once there, stays in every later step's counters; a probe beside this may be flagging one.)
__device__ __forceinline__ void ctr_start(Ctr* cur, const Ctr* prev, const int* n_unique,
                                          int* n_invalid, int t) {
  Ctr c = *prev;
  c.U_prev = c.U;
  c.U = *n_unique;
  if (c.n_bypass) c.last_bypass = t - 1;
  c.M = c.K = c.n_bypass = c.n_hit = 0;
  c.n_invalid = *n_invalid;
  *n_invalid = 0;
  c.f_old = c.f; c.need = 0; c.T = 0; c.r = 0;
  c.t = t; c.bad_offsets = 0;
  static_assert(offsetof(Ctr, err) == 14 * sizeof(int), "the fields around err");
  int* const to = reinterpret_cast<int*>(cur);
  const int* const from = reinterpret_cast<const int*>(&c);
#pragma unroll
  for (int i = 0; i < (int)(sizeof(Ctr) / sizeof(int)); ++i)
    if (i != 14) to[i] = from[i];
  if (c.err) cur->err = c.err;
}

// The counters and the index rebuild as kernels of their own: with a hashed index, for batches prepared by one
// block and empty ones.  They read the flag and the watermark from the previous step's counters, which no kernel
// changes any more (on the very first step prev == cur and both fields are zero before and after).
__global__ __launch_bounds__(256) void k_ctr_init(Ctr* cur, const Ctr* prev, const int* n_unique,
                                                  int* n_invalid, IdxEntry* index, uint32_t hi,
                                                  int t) {
  const bool rebuild = prev->rebuild != 0;
  if (blockIdx.x == 0 && threadIdx.x == 0) ctr_start(cur, prev, n_unique, n_invalid, t);
  if (rebuild) index_clear(index, hi, (int)blockIdx.x, (int)gridDim.x);
}
__global__ __launch_bounds__(256) void k_index_refill(IdxEntry* index, uint32_t hi,
                                                       const int64_t* __restrict__ slot_id,
                                                       const Ctr* ctr) {
  if (ctr->rebuild) index_reinsert(index, hi, slot_id, ctr->f, (int)blockIdx.x, (int)gridDim.x);
}

// VSI pass 3: the first appearances get their virtual ids (rank among all first appearances) and
// the tables keyed by them.  A chunk's first virtual id is the sum of the counts of the chunks
// before it, which every block adds up for itself (a few loads per thread from a list that sits in
// L2: cheaper than a scan kernel between the two passes).  The last chunk leaves the number of
// unique ids in *n_unique.
__global__ __launch_bounds__(256) void k_uniq_assign(const int64_t* __restrict__ ids, int64_t V,
                                                      const int* __restrict__ hslot,
                                                      const unsigned* __restrict__ first, int n,
                                                      const int* __restrict__ blk_cnt,
                                                      int64_t* __restrict__ unique_ids,
                                                      int* __restrict__ uvid,
                                                      int* __restrict__ vid_hslot,
                                                      int* __restrict__ cnt, int* n_unique, int chunks,
                                                      Ctr* ctr, int t, const Ctr* prev, IdxEntry* index, uint32_t hi,
                                                      const int64_t* __restrict__ slot_id) {
  if ((int)blockIdx.x >= chunks) {            // (only with a hashed index) see index_clear
    // the step's number is in its counters before a probe of the resolve can flag an error under it
    if ((int)blockIdx.x == chunks && threadIdx.x == 0) ctr->t = t;
    if (prev->rebuild) index_reinsert(index, hi, slot_id, prev->f, (int)blockIdx.x - chunks, (int)gridDim.x - chunks);
    return;
  }
  __shared__ int smem[20];
  const unsigned flags = reinterpret_cast<const unsigned char*>(first)[blockIdx.x * 256 + threadIdx.x];
  int before = 0;
  if (blk_cnt) {
    for (int i = (int)threadIdx.x; i < (int)blockIdx.x; i += 256) before += blk_cnt[i];
  } else {
    const int4* f4 = reinterpret_cast<const int4*>(first);          // 16 per chunk of positions
    for (int i = (int)threadIdx.x; i < (int)blockIdx.x * (kPosChunk / 128); i += 256) {
      const int4 q = f4[i];
      before += __popc(q.x) + __popc(q.y) + __popc(q.z) + __popc(q.w);
    }
  }
  // the flagged positions' ids and table entries: on their way while the block adds up its counts
  const int base = blockIdx.x * kPosChunk + (int)threadIdx.x * 8;
  int hs[8];
  int64_t id[8];
#pragma unroll
  for (int j = 0; j < 8; ++j)
    if (flags & (1u << j)) { hs[j] = hslot[base + j]; id[j] = ids[base + j]; }
  before = block_sum(before, smem);
  int tot;
  int vid = block_excl_scan(__popc(flags), tot, smem) + before;
  if ((int)blockIdx.x == chunks - 1 && threadIdx.x == 0) *n_unique = before + tot;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    if (flags & (1u << j)) {
      unique_ids[vid] = (id[j] < 0 || id[j] >= V) ? (int64_t)-1 : id[j];
      uvid[hs[j]] = vid;
      vid_hslot[vid] = hs[j];
      cnt[vid] = 0;
      ++vid;
    }
  }
}

// VSI pass 4: virtual id of every position, cnt[v] = number of positions of virtual id v, and the
// place of every position inside its group (rank[p]), so that the grouping pass needs no atomics.
// Virtual ids are handed out in order of first appearance, so the frequent ids of a power-law
// batch are (nearly all) among the lowest ones: those are counted in an LDS histogram per block
// and flushed with one coalesced atomic per bin; the rest go to HBM atomics on distinct words.
// An atomic that counts also ranks: a cold id's returns the position's place in its group, a hot bin's
// LDS atomic its place in the block's share and the flush the start of that share.
// Every block adds its tally of a frequent id to one counter: a thousand atomics in a row on one
// address (about 10 ns each).  The counters of the hot bins are therefore kept in up to kHotRep
// copies, block b using copy b mod nrep (SortGeom); resolve folds the copies into cnt, the miss
// assignment turns them into one group start per copy.
constexpr int kHotRep = 32;

// The shape of the counting and grouping passes by batch size (nothing else of a batch is known to
// the host).  A block's histogram costs its clear and its flush whatever the block counts, and the
// places of a block's positions in a hot group lie side by side, so big batches take many positions
// per block (fewer flushes, fewer 128-byte lines that two XCDs write); small ones are short of blocks
// instead: there a block counts 1024 positions with 1024 threads, which clear and flush eight bins each.
// Counting + grouping us: 195e3 positions 1024x1 and 256x4 (threads x positions per thread) 13.4, 256x16 both
// 33; the same shape for both: 639e3 256x8 28.6, 512x8 29.0, 256x16 38.7; 2.56e6 512x8 57.0, 256x16 63.3, 1024x8
// 61.7; 8.9e6 in bags 1024x8 268, 256x16 310, 512x8 302.
// All bins at every size: with the 2048 lowest only, small batches were no faster (195e3: 256x4 15.2), and
// ids beyond the bins that are frequent all the same, in batches that open with thousands of distinct
// ids, count through one address: 200e3 ids of which 196e3 are 3 ids behind 4000 others 1252 us, 70 with
// 8192 bins; and from 639e3 positions on the counters of the ids just beyond the bins share cache lines
// (2.56e6, 8192 / 4096 / 2048 bins: 57 / 68 / 76 us).
// shift: positions per block = 1 << shift, in both passes.
struct SortGeom { int bins, shift, nrep, blocks; };
inline SortGeom sort_geom(int64_t n) {
  SortGeom g;
  g.bins = kHotBins;
  g.shift = n < ((int64_t)1 << 18) ? 10 : n < ((int64_t)1 << 22) ? 12 : 13;
  g.blocks = (int)((n + (1 << g.shift) - 1) >> g.shift);
  g.nrep = 1;
  while (g.nrep < kHotRep && g.nrep * 16 < g.blocks) g.nrep *= 2;
  return g;
}

// A small batch (k_small_prepare): counted and ranked already, no hot bins.
inline SortGeom small_geom(int64_t n) {
  SortGeom g;
  g.bins = 0; g.shift = 10; g.nrep = 1;
  g.blocks = (int)((n + 1023) >> 10);
  return g;
}

// cnt == nullptr (a batch that is not grouped, see group_now in the host code): the virtual ids alone, kept in rank as well.
// hslot == nullptr (k_count_late): they are there already, in `inverse`.  (At run time: as template arguments these made the counting
// 1.3 us slower at 65536 x 39 positions.)
template <int kPer, int kT>
__device__ __forceinline__ void count_positions(const int* __restrict__ hslot, const int* __restrict__ uvid, int n,
                                                int* __restrict__ inverse, int* cnt, int* cnt_rep, int nrep,
                                                int* __restrict__ rank, unsigned* __restrict__ first, int blk,
                                                int* lh) {
  // the marks of first appearances have been read: all zero again for the next batch
  static_assert(kPer <= 32 && kT * kPer % 32 == 0, "whole words of marks per block");
  if (hslot && (int)threadIdx.x < kT * kPer / 32 && blk * kT * kPer + (int)threadIdx.x * 32 < n)
    first[blk * (kT * kPer / 32) + threadIdx.x] = 0;
  if (cnt)
    for (int i = threadIdx.x; i < kHotBins; i += kT) lh[i] = 0;
  const int base = blk * kT * kPer;
  int hv[kPer], vv[kPer], rr[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {              // kPer loads in flight per level of indirection
    const int p = base + j * kT + (int)threadIdx.x;
    hv[j] = p < n ? (hslot ? hslot[p] : inverse[p]) : -1;
  }
#pragma unroll
  for (int j = 0; j < kPer; ++j) vv[j] = hslot && hv[j] >= 0 ? uvid[hv[j]] : hv[j];
  if (hslot) {
#pragma unroll
    for (int j = 0; j < kPer; ++j)
      if (vv[j] >= 0) inverse[base + j * kT + (int)threadIdx.x] = vv[j];
  }
  if (!cnt) {
#pragma unroll
    for (int j = 0; j < kPer; ++j)
      if (vv[j] >= 0) rank[base + j * kT + (int)threadIdx.x] = vv[j];
    return;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int v = vv[j];
    if (v >= 0) {
      rr[j] = v < kHotBins ? atomicAdd(&lh[v], 1) : atomicAdd(&cnt[v], 1);
    }
  }
  __syncthreads();
  int* mine = cnt_rep + (blk & (nrep - 1)) * kHotBins;
  // the block's share of each non-empty bin: returning atomics, several in flight per thread (each
  // round of them is a round trip to the memory side)
  constexpr int kFlush = kHotBins / kT < 16 ? kHotBins / kT : 16;
  static_assert(kHotBins % (kT * kFlush) == 0, "flush rounds cover the bins exactly");
  for (int b0 = threadIdx.x; b0 < kHotBins; b0 += kT * kFlush) {
    int c[kFlush], r[kFlush];
#pragma unroll
    for (int u = 0; u < kFlush; ++u) c[u] = lh[b0 + u * kT];
#pragma unroll
    for (int u = 0; u < kFlush; ++u) r[u] = c[u] ? atomicAdd(&mine[b0 + u * kT], c[u]) : 0;
#pragma unroll
    for (int u = 0; u < kFlush; ++u) if (c[u]) lh[b0 + u * kT] = r[u];
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int p = base + j * kT + (int)threadIdx.x;
    if (vv[j] >= 0) rank[p] = vv[j] < kHotBins ? lh[vv[j]] + rr[j] : rr[j];
  }
}

// Multi-hot input: bag index of every position.  Also checks the bag structure (first offset 0,
// last offset n, none decreasing); violations are tallied in the step's counters and reported in
// the Host status block.  A malformed structure cannot make any kernel leave its buffers: ranges
// are clamped to [0, n] here and in the forward gather, and a position that no bag covers keeps a
// stale bag number, which the grouping pass clamps to the step's bags.
// A wavefront writes the positions of its 64 bags in order, 64 at a time: the bag of a position is the last
// one that starts at or before it (six steps of a search in LDS).  With a thread per bag every store
// touched a line of its own: 38 us for 852e3 bags of 1 to 20 ids, 17 this way.  A wavefront that has seen a
// violation falls back to a loop per bag.
// starts: a word of LDS per thread, used within the wavefront alone.  kept != nullptr: the check alone, and the offsets
// are kept there; ctr == nullptr: without the check's tally (it has been made).
__device__ __forceinline__ void bags_of_positions(const int64_t* __restrict__ offsets, int n_bags, int n,
                                                  int* __restrict__ pos2bag, int64_t* __restrict__ kept, Ctr* ctr, int blk,
                                                  int* starts_all) {
  const int lane = lane_id(), w = (int)(threadIdx.x >> 6);
  int* const starts = starts_all + w * kWave;
  const int b0 = blk * (int)blockDim.x + w * kWave, b = b0 + lane;
  bool bad = false;
  BagRange r{n, n};                               // lanes beyond the last bag: empty, at the end
  if (b < n_bags) {
    const int64_t lo = offsets[b], hi = offsets[b + 1];
    bad = bag_malformed(lo, hi, b, n_bags, n);
    r = bag_range(lo, hi, n);
    if (kept) {
      kept[b] = lo;
      if (b == n_bags - 1) kept[n_bags] = hi;
    }
  }
  starts[lane] = r.lo;
  const uint64_t m = __ballot(bad);
  if (m && lane == 0 && ctr) {
    atomicAdd(&ctr->bad_offsets, __popcll(m));
    volatile HostStatus* h = ctr->hstat;
    if (h) h->bad_offsets_step = ctr->t;
  }
  if (kept) return;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  if (b0 >= n_bags) return;
  if (m) {
    if (b < n_bags)
      for (int q = r.lo; q < r.hi; ++q) pos2bag[q] = b;
    return;
  }
  // No violation among these bags: their offsets do not decrease, so their clamped ranges tile [first start,
  // last end), also where the offsets lie outside [0, n] (the violation is then another wavefront's).
  const int last = n_bags - b0 < kWave ? n_bags - b0 - 1 : kWave - 1;
  const int begin = starts[0], end = __shfl(r.hi, last, kWave);
  for (int q = begin + lane; q < end; q += kWave) {
    int g = 0;
#pragma unroll
    for (int step = kWave / 2; step > 0; step >>= 1)
      if (g + step <= last && starts[g + step] <= q) g += step;
    pos2bag[q] = b0 + g;
  }
}

// Grouping of positions by virtual id (counting sort): perm64[start of the group + rank] =
// (v << 32) | payload, payload = position (one-hot) or bag index (multi-hot).  The counting pass has
// ranked every position inside its group (a hot bin's copy: inside the copy's share, whose start is in
// cur_rep), so this pass is loads and stores only (65536 x 39 positions: 31 us with a second histogram
// and its returning atomics here, 22 without, and the counting pass is none the slower for ranking).
// rank_slot[p] is read as the rank and overwritten with pos_slot[p] = row of slot[inverse[p]] for the
// forward gather (a bypass slot C + j lives at row C + boff + j: each step in flight has its own
// bypass region).  kRows = false: without that, the rows are there already (k_scatter_late).
// A block takes the same positions as a block of the counting pass: their places in a hot group lie
// side by side, and with half the positions per block two XCDs write into the same 128-byte lines
// (169 against 120 us at 8.9e6 positions in bags).
struct ScatterArgs {
  const int *inverse, *pos2bag; int n; const int64_t* grp; int* cold_pay; const int* cur_rep; int bins, shift, nrep;
  int64_t* perm64; const int* slot; int* rank_slot; int C, boff, n_bags;
};
template <int kScatPer, int kT, bool kRows>
__device__ __forceinline__ void scatter_positions(const int* __restrict__ inverse, const int* __restrict__ pos2bag, int n,
                                                  const int64_t* __restrict__ grp, int* __restrict__ cold_pay,
                                                  const int* __restrict__ cur_rep, int bins, int shift, int nrep,
                                                  int64_t* __restrict__ perm64, const int* __restrict__ slot,
                                                  int* rank_slot, int C, int boff, int n_bags, int blk) {
  const int base = blk * kT * kScatPer + (int)threadIdx.x;
  int vv[kScatPer], rr[kScatPer], sv[kScatPer], pay[kScatPer];
  int64_t gr[kScatPer];
  // two levels of indirection, kScatPer loads in flight at each: position -> vid -> slot / group start
#pragma unroll
  for (int j = 0; j < kScatPer; ++j) {
    const int p = base + j * kT;
    vv[j] = p < n ? inverse[p] : -1;
    rr[j] = p < n ? rank_slot[p] : 0;
    pay[j] = (p < n && pos2bag) ? pos2bag[p] : p;
    // a position that malformed offsets left uncovered carries a stale bag number
    if (pos2bag && (unsigned)pay[j] >= (unsigned)n_bags) pay[j] = 0;
  }
#pragma unroll
  for (int j = 0; j < kScatPer; ++j) {
    const int p = base + j * kT;
    if (vv[j] >= 0) {
      if (kRows) sv[j] = slot[vv[j]];
      gr[j] = vv[j] < bins ? (int64_t)cur_rep[((p >> shift) & (nrep - 1)) * kHotBins + vv[j]] : grp[vv[j]];
    }
  }
#pragma unroll
  for (int j = 0; j < kScatPer; ++j) {
    const int p = base + j * kT;
    if (vv[j] < 0) continue;
    if (kRows) rank_slot[p] = sv[j] >= C ? sv[j] + boff : sv[j];   // pos_slot: row index for the forward gather
    int64_t e = ((int64_t)vv[j] << 32) | (uint32_t)pay[j];
    // a cold group's gradient rows also go where the optimizer kernel finds them without
    // walking the grouping: two words per virtual id, filled in the order of the ranks
    if (vv[j] >= bins && group_cold(gr[j])) {
      cold_pay[2 * vv[j] + rr[j]] = pay[j];
      e |= kColdBit;
    }
    perm64[(int)gr[j] + rr[j]] = e;
  }
}
template <int kScatPer, int kT, bool kRows = true>
__device__ __forceinline__ void scatter_positions(const ScatterArgs& a, int blk) {
  scatter_positions<kScatPer, kT, kRows>(a.inverse, a.pos2bag, a.n, a.grp, a.cold_pay, a.cur_rep, a.bins, a.shift, a.nrep, a.perm64,
                                  a.slot, a.rank_slot, a.C, a.boff, a.n_bags, blk);
}
template <int kScatPer, int kT>
__global__ __launch_bounds__(kT) void k_scatter(const ScatterArgs a) {
  scatter_positions<kScatPer, kT>(a, (int)blockIdx.x);
}

// ---------------------------------------------------------------------------------------------
// The cache index (id -> slot) comes in two kinds.
//   dense: one int per Host row, dmap[id] = slot or -1.  With 288 GB of HBM a map of 4 bytes per
//     Host row (1.6 % of a dim-32 table with its accumulators) is affordable for every table that
//     fits a host, and it needs no probing, no atomics (the ids of a batch are distinct: one writer
//     per word), no tombstones and no rebuild.  The kernels below take it as `dmap`.
//   hashed (dmap == nullptr): open addressing, linear probing, tombstones, rebuilt on the device when
//     deleted entries pass an eighth of the table: for id ranges too large for a dense map, or on
//     request (sfc_config.index_kind).  The helpers that follow are its probe / insert.
// ---------------------------------------------------------------------------------------------
// A probe sequence is walked eight entries (128 bytes) at a time, all eight loads in flight
// together: the longest cluster among the tens of thousands of probes of a step sets the duration
// of the kernel, and a dependent load per entry made that tail tens of microseconds long.
constexpr int kProbeBatch = 8;

__device__ __forceinline__ int64_t idx_key(const int4& raw) {
  return ((int64_t)(uint32_t)raw.y << 32) | (uint32_t)raw.x;
}
__device__ __forceinline__ void idx_load_batch(const IdxEntry* index, uint32_t hi, uint32_t h,
                                               int4 (&raw)[kProbeBatch]) {
#pragma unroll
  for (int j = 0; j < kProbeBatch; ++j) {
    uint32_t hj = h + j;
    if (hj >= hi) hj -= hi;                  // hi >= 64: wraps at most once
    raw[j] = *reinterpret_cast<const int4*>(&index[hj]);
  }
}

__device__ __forceinline__ int index_find(const IdxEntry* __restrict__ index, uint32_t hi,
                                          int64_t id, uint32_t* where, Ctr* ctr) {
  uint32_t h = bucket_of(id, hi);
  for (uint32_t probes = 0; probes < hi; probes += kProbeBatch) {
    int4 raw[kProbeBatch];
    idx_load_batch(index, hi, h, raw);
#pragma unroll
    for (int j = 0; j < kProbeBatch; ++j) {
      const int64_t k = idx_key(raw[j]);
      if (k == id) {
        if (where) { uint32_t hj = h + j; *where = hj >= hi ? hj - hi : hj; }
        return raw[j].z;
      }
      if (k == kEmpty) return -1;
    }
    h += kProbeBatch;
    if (h >= hi) h -= hi;
  }
  flag_err(ctr, 1);
  return -1;
}

// id is known to be absent.  Takes the first empty or deleted entry of its probe sequence.
// Returns true if that was a deleted entry: the caller takes it off the tombstone count.
__device__ __forceinline__ bool index_insert(IdxEntry* index, uint32_t hi, int64_t id, int slot,
                                             Ctr* ctr) {
  uint32_t h = bucket_of(id, hi);
  for (uint32_t probes = 0; probes < hi; probes += kProbeBatch) {
    int4 raw[kProbeBatch];
    idx_load_batch(index, hi, h, raw);
#pragma unroll
    for (int j = 0; j < kProbeBatch; ++j) {
      const int64_t k = idx_key(raw[j]);
      if (k == kEmpty || k == kTomb) {
        uint32_t hj = h + j;
        if (hj >= hi) hj -= hi;
        // an entry seen free may have been taken by another insert since: then walk on
        const int64_t old = (int64_t)atomicCAS((unsigned long long*)&index[hj].key,
                                               (unsigned long long)k, (unsigned long long)id);
        if (old == k) {
          atomicExch(&index[hj].slot, slot);
          return k == kTomb;
        }
      }
    }
    h += kProbeBatch;
    if (h >= hi) h -= hi;
  }
  flag_err(ctr, 2);
  return false;
}

// ---------------------------------------------------------------------------------------------
// Resolve: each unique id against the index.  Hits get their slot and the current stamp.  The
// recency histogram hist[stamp] = #slots with that stamp must stay exact; stamps of hits cluster
// on the last few steps, i.e. on a few words of hist, so each block tallies its hits by age
// (t - old stamp) in LDS and adds its nonzero bins to age_hist, which the plan kernel applies
// to hist and returns to zero.  Only ages beyond the LDS range use an atomic on hist.  Bin 0
// counts the hits.  Also returns the batch-table entries of this step to the empty state, so that
// table never needs a per-step clear.
// ---------------------------------------------------------------------------------------------
constexpr int kAgeBins = 1024;
// One tile per block and iteration, up to 512 blocks: what hides the chain vid -> id -> index entry ->
// stamp is more wavefronts, not more tiles per thread.  (us at 10.6e3 / 40e3 / 132e3 / 200e3 / 837e3 /
// 1.24e6 unique ids: 7.1 / 7.7 / 16 / 17.5 / 48 / 62; four tiles per thread on 256 blocks 16 / 15 / 17 / 25 /
// 60 / 84; one tile on 256 blocks 7.2 / 7.5 / 15 / 21 / 58 / 81, on 1024 6.8 / 7.7 / 16 / 22.5 / 49 / 59.)
constexpr int kResolveThreads = 512 * 256;

template <int kT>
__device__ __forceinline__ void resolve_ids(const int64_t* __restrict__ unique_ids,
                                            const int* __restrict__ vid_hslot, uint64_t* utab, int wide,
                                            const IdxEntry* __restrict__ index, uint32_t hi,
                                            const int* __restrict__ dmap, int* stamp, int* hist, int t,
                                            int* __restrict__ slot_out, int* __restrict__ tile_miss,
                                            int* __restrict__ age_hist, Ctr* ctr, const Ctr* prev,
                                            const int* n_unique, int* n_invalid, int blk, int nblk, int* lds) {
  int* const lage = lds;                       // [kAgeBins]
  int* const wmiss = lds + kAgeBins;           // a word per wavefront
  for (int i = threadIdx.x; i < kAgeBins; i += kT) lage[i] = 0;
  // prev != nullptr: nothing has to happen between the previous step's prepare and this kernel (an index
  // rebuild is done already), so it starts the step's counters itself (k_ctr_init is not launched): the first
  // thread writes them for the kernels that follow, and every block takes the number of unique ids
  // from where the unique passes left it.  Nothing else of the counters is read in this kernel.
  const int U = prev ? *n_unique : ctr->U;
  __syncthreads();
  if (prev && blk == 0 && threadIdx.x == 0) ctr_start(ctr, prev, n_unique, n_invalid, t);
  constexpr int kTiles = kT / kVidTile;        // tiles side by side
  const int sub = (int)threadIdx.x / kVidTile;
  for (int tile0 = blk * kTiles; tile0 * kVidTile < U; tile0 += nblk * kTiles) {
    const int tile = tile0 + sub;
    const int v = tile * kVidTile + (int)threadIdx.x % kVidTile;
    int hs = -1, sl = -1, old = 0;
    int64_t id = -1;
    if (v < U) { hs = vid_hslot[v]; id = unique_ids[v]; }
    if (hs >= 0) {
      if (wide) { UEntry z; z.key = kEmpty; z.minpos = kIntMax; z.pad = 0; reinterpret_cast<UEntry*>(utab)[hs] = z; }
      else utab[hs] = ~0ull;
    }
    if (id >= 0) {
      if (dmap) {
        sl = dmap[id];
      } else {
        const int4 ent = *reinterpret_cast<const int4*>(&index[bucket_of(id, hi)]);
        const int64_t k0 = ((int64_t)(uint32_t)ent.y << 32) | (uint32_t)ent.x;
        if (k0 == id) sl = ent.z;
        else if (k0 != kEmpty) sl = index_find(index, hi, id, nullptr, ctr);   // walk on
      }
    }
    const bool hit = sl >= 0, miss = id >= 0 && sl < 0;
    int age = 0;
    if (v < U) slot_out[v] = hit ? sl : (miss ? kMissMark : -1);
    if (hit) {
      old = stamp[sl];
      stamp[sl] = t;
      age = t - old;
      if (age >= kAgeBins) atomicSub(&hist[old], 1);
    }
    // most hits were last used one step ago: count those per wavefront, the rest one by one
    const uint64_t m1 = __ballot(hit && age == 1), mh = __ballot(hit), mm = __ballot(miss);
    if (lane_id() == 0) {
      if (m1) atomicAdd(&lage[1], __popcll(m1));
      if (mh) atomicAdd(&lage[0], __popcll(mh));
      wmiss[threadIdx.x >> 6] = __popcll(mm);
    }
    if (hit && age > 1 && age < kAgeBins) atomicAdd(&lage[age], 1);
    lds_barrier();
    if (threadIdx.x % kVidTile == 0 && tile * kVidTile < U) {
      const int* const q = wmiss + sub * (kVidTile / kWave);
      tile_miss[tile] = q[0] + q[1] + q[2] + q[3];
    }
    lds_barrier();
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kAgeBins; i += kT)
    if (lage[i]) atomicAdd(&age_hist[i], lage[i]);
}

// Both read what the assign pass has left and neither what the other writes, so they are one launch: the first
// nres blocks resolve, the others count.  us one after the other / in one launch: 1024 x 39 positions 5.3 + 6.6 /
// 5.7, 8192 x 26 with the hashed index 7.5 + 8.5 / 10.1, 16384 x 39 16.3 + 15.6 / 22.1, 65536 x 39 33.3 + 17.6 / 45.8,
// 1.28e6 uniform ones 26.7 + 60.8 / 77.5, 8.9e6 in bags 146 + 48 / 178: what is saved is start-up and drain, the random
// accesses of the two add up.
struct RankArgs {
  const int* hslot; const int* uvid; int n; int* inverse; int* cnt; int* cnt_rep; int nrep; int* rank; unsigned* first;
};
struct ResolveArgs {
  const int64_t* unique_ids; const int* vid_hslot; uint64_t* utab; int wide;
  const IdxEntry* index; uint32_t hi; const int* dmap; int *stamp, *hist; int t;
  int *slot, *tile_miss, *age_hist; Ctr* ctr; const Ctr* prev; const int* n_unique; int* n_invalid;
};
template <int kPer, int kT>
__global__ __launch_bounds__(kT) void k_rank_resolve(const RankArgs a, const ResolveArgs b, int nres) {
  __shared__ int lds[kHotBins];
  static_assert(kHotBins >= kAgeBins + kT / kWave, "the LDS of the counting blocks holds that of the resolving ones");
  if ((int)blockIdx.x < nres)
    resolve_ids<kT>(b.unique_ids, b.vid_hslot, b.utab, b.wide, b.index, b.hi, b.dmap, b.stamp, b.hist, b.t, b.slot,
                    b.tile_miss, b.age_hist, b.ctr, b.prev, b.n_unique, b.n_invalid, (int)blockIdx.x, nres, lds);
  else
    count_positions<kPer, kT>(a.hslot, a.uvid, a.n, a.inverse, a.cnt, a.cnt_rep, a.nrep, a.rank, a.first,
                              (int)blockIdx.x - nres, lds);
}

// ---------------------------------------------------------------------------------------------
// The victims' plan, by one block of 1024 threads: need = M - free; T is the stamp at which the
// running count of evictable slots (stamp < limit, oldest first) passes need; r of the slots stamped T
// go too; K victims in all.
// kAtomic: the kernel also updates the recency histogram with atomics, so every access to it is one.
// ---------------------------------------------------------------------------------------------
struct Plan { int M, need, T, r, K, f_new, n_bypass, oldest; };

__device__ __forceinline__ void hist_add(int* w, int x) {
  const int old = atomicAdd(w, x);
  asm volatile("" :: "v"(old));            // the value has to be back, so the sum has been formed
}

template <bool kAtomic>
__device__ __forceinline__ void plan_decide(Plan& pl, int M, int f, int oldest, int* hist, int t,
                                            int lookahead, int C, int* smem, int* s_found) {
  const int need = M - (C - f);
  const int limit = t - lookahead;       // candidates have stamp < limit
  int T = limit, r = 0, K = 0;
  if (need > 0) {
    // running count of candidates from the oldest stamp upwards
    int cum = 0;           // slots with stamp in [oldest, b)
    bool done = false;
    for (int b = oldest; b < limit && !done; b += 1024) {
      if (threadIdx.x == 0) *s_found = kIntMax;
      __syncthreads();
      const int s = b + (int)threadIdx.x;
      const int x = s < limit ? (kAtomic ? coherent_load(&hist[s]) : hist[s]) : 0;
      int tot;
      const int e = block_excl_scan(x, tot, smem);
      // first stamp whose inclusive count exceeds need
      if (s < limit && cum + e + x > need) atomicMin(s_found, s);
      __syncthreads();
      if (*s_found != kIntMax) {
        T = *s_found;
        if (s == T) smem[18] = cum + e;    // candidates strictly older than T
        __syncthreads();
        r = need - smem[18];
        K = need;
        done = true;
      } else {
        cum += tot;
      }
      __syncthreads();
    }
    if (!done) { T = limit; r = 0; K = cum; }   // everything evictable goes, the rest bypasses
    // the histogram after eviction: stamps below T vanish, r leave stamp T
    for (int s = oldest + (int)threadIdx.x; s < T; s += 1024) {
      if (kAtomic) atomicExch(&hist[s], 0); else hist[s] = 0;
    }
  }
  int f_new = f + (M - K);
  if (f_new > C) f_new = C;
  pl.M = M; pl.need = need; pl.T = T; pl.r = r; pl.K = K;
  pl.f_new = f_new; pl.n_bypass = M - K - (f_new - f);
  pl.oldest = need > 0 && T > oldest ? T : oldest;
}

// The plan into the step's counters.
__device__ __forceinline__ void plan_store(const Plan& pl, Ctr& ctr, int f) {
  ctr.M = pl.M; ctr.K = pl.K; ctr.n_bypass = pl.n_bypass;
  ctr.need = pl.need; ctr.T = pl.T; ctr.r = pl.r;
  ctr.f_old = f; ctr.f = pl.f_new;
  ctr.oldest = pl.oldest;
}

// What the assign pass needs and the plan does not: the positions of every virtual id (the copies of a hot bin, see
// count_positions) and of every tile, by `folds` blocks, and the bags of the positions (multi-hot input), by the
// blocks behind those.  Beside the plan, a chain on one compute unit, they cost nothing (us of plan and bags one after
// the other / this way, 291e3 ids in bags 4.6 + 4.8 / 4.8, 8.9e6 12.8 + 17.0 / 18.8; plan alone, at 1024 x 39 ids,
// 6.2 / 3.5, 65536 x 39 8.8 / 6.2); but a block of the plan's 1024 threads needs a compute unit with sixteen free
// wavefronts, so large pipelined batches give them to the launch of the victims' count: see plan_and_assign.
constexpr int kFoldThreads = 1 << 16;        // of them all, at most
struct FoldArgs { int* cnt; const int* cnt_rep; int bins, nrep; int* tile_cnt; int folds; };
struct BagArgs { const int64_t* offsets; int n_bags, n; int* pos2bag; int64_t* kept; int tally; };

// words: a word of LDS per thread
template <int kT>
__device__ __forceinline__ void fold_or_bags(const FoldArgs& fo, const BagArgs& bags, Ctr* ctr, int blk, int* words) {
  if (blk >= fo.folds) {
    bags_of_positions(bags.offsets, bags.n_bags, bags.n, bags.pos2bag, bags.kept, bags.tally ? ctr : nullptr, blk - fo.folds, words);
    return;
  }
  const int U = ctr->U;
  constexpr int kTiles = kT / kVidTile;
  const int sub = (int)threadIdx.x / kVidTile;
  for (int tile0 = blk * kTiles; tile0 * kVidTile < U; tile0 += fo.folds * kTiles) {
    const int tile = tile0 + sub, v = tile * kVidTile + (int)threadIdx.x % kVidTile;
    int c = 0;
    if (v < U) {
      if (v < fo.bins) {
#pragma unroll 8
        for (int r = 0; r < fo.nrep; ++r) c += fo.cnt_rep[r * kHotBins + v];
        fo.cnt[v] = c;
      } else {
        c = fo.cnt[v];
      }
    }
    c = wave_sum(c);
    if (lane_id() == 0) words[threadIdx.x >> 6] = c;
    lds_barrier();
    if (threadIdx.x % kVidTile == 0 && tile * kVidTile < U) {
      const int* const q = words + sub * (kVidTile / kWave);
      fo.tile_cnt[tile] = q[0] + q[1] + q[2] + q[3];
    }
    lds_barrier();
  }
}

// Plan (the first block): scan the per-tile miss counts, then decide the victims.  It is a chain of a few dependent
// loads and scans on one compute unit.

__global__ __launch_bounds__(1024) void k_plan(int* tile_miss, int* __restrict__ age_hist,
                                               int* __restrict__ tile_reuse, int* hist, int t,
                                               int lookahead, int C, uint32_t hi, int dense, Ctr* ctr,
                                               const FoldArgs fo, const BagArgs bags) {
  static_assert(kAgeBins == 1024, "one thread per age bin");
  __shared__ int smem[20];
  __shared__ int s_found;
  __shared__ int words[1024];
  if (blockIdx.x > 0) {
    fold_or_bags<1024>(fo, bags, ctr, (int)blockIdx.x - 1, words);
    return;
  }
  const int U = ctr->U;
  // every thread reads the counters here; thread 0 overwrites them only after the last barrier
  const int f = ctr->f, oldest = ctr->oldest;
  const int ntiles = (U + kVidTile - 1) / kVidTile;
  const int a = (int)threadIdx.x;
  const int x0 = a < ntiles ? tile_miss[a] : 0;
  const int sum = age_hist[a];
  // deleted index entries that the previous step's miss assignment took back into use
  int reuse = 0;
  if (!dense) {
    const int reuse_tiles = (ctr->U_prev + kVidTile - 1) / kVidTile;
    for (int i = a; i < reuse_tiles; i += 1024) { reuse += tile_reuse[i]; tile_reuse[i] = 0; }
    reuse = block_sum(reuse, smem);
  }
  // hits by age: thread a owns age a.  hist[t] gains the hits, hist[t - a] loses its share.
  if (sum) {
    age_hist[a] = 0;
    if (a == 0) { hist[t] += sum; ctr->n_hit = sum; }
    else hist[t - a] -= sum;
  }
  int carry = 0;
  for (int b = 0; b < ntiles; b += 1024) {
    const int i = b + a;
    const int x = b == 0 ? x0 : i < ntiles ? tile_miss[i] : 0;
    int tot;
    const int e = block_excl_scan(x, tot, smem);
    if (i < ntiles) tile_miss[i] = carry + e;
    carry += tot;
  }
  const int M = carry;
  __syncthreads();                             // the histogram's words are written
  Plan pl;
  plan_decide<false>(pl, M, f, oldest, hist, t, lookahead, C, smem, &s_found);
  __syncthreads();
  if (threadIdx.x == 0) {
    if (pl.need > 0 && pl.r > 0) hist[pl.T] -= pl.r;
    hist[t] += pl.M - pl.n_bypass;
    plan_store(pl, *ctr, f);
    ctr->tomb -= reuse;
    // a rebuild asked for by the previous step has run ahead of this step's resolve
    if (ctr->rebuild) { ctr->rebuild = 0; ctr->tomb = 0; }
    // K deletions are about to add tombstones; ask for a rebuild before the next resolve when a
    // eighth of the index would be deleted entries
    if (!ctr->dense && (unsigned)(ctr->tomb + pl.K) > hi / 8) ctr->rebuild = 1;
  }
}

// ---------------------------------------------------------------------------------------------
// Victim selection over the occupied slots, in slot order (two passes around a scan):
// victim  <=>  stamp < T, or stamp == T and fewer than r earlier slots carry stamp T.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_victim_count(const int* __restrict__ stamp,
                                                       int* __restrict__ tile_lt,
                                                       int* __restrict__ tile_eq, Ctr* ctr, int blocks,
                                                       const FoldArgs fo, const BagArgs bags) {
  __shared__ int smem[256];
  if ((int)blockIdx.x >= blocks) {            // see fold_or_bags
    fold_or_bags<256>(fo, bags, ctr, (int)blockIdx.x - blocks, smem);
    return;
  }
  if (ctr->K == 0) return;
  const int f = ctr->f_old, T = ctr->T;
  for (int tile = blockIdx.x; tile * kPosChunk < f; tile += blocks) {
    const int base = tile * kPosChunk + (int)threadIdx.x * 8;
    int lt = 0, eq = 0;
    if (base + 8 <= f) {
      const int4 a = *reinterpret_cast<const int4*>(stamp + base);
      const int4 b = *reinterpret_cast<const int4*>(stamp + base + 4);
      const int v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
      for (int j = 0; j < 8; ++j) { lt += v[j] < T; eq += v[j] == T; }
    } else {
      for (int j = 0; j < 8; ++j) {
        const int s = base + j;
        if (s < f) { const int st = stamp[s]; lt += st < T; eq += st == T; }
      }
    }
    // both counts in one block reduction: a tile has 2048 slots, so each fits in 16 bits
    const int both = block_sum((lt << 16) | eq, smem);
    if (threadIdx.x == 0) { tile_lt[tile] = both >> 16; tile_eq[tile] = both & 0xffff; }
  }
}

__global__ __launch_bounds__(256) void k_victim_write(const int* __restrict__ stamp,
                                                       const int64_t* __restrict__ slot_id,
                                                       const int* __restrict__ tile_lt,
                                                       const int* __restrict__ tile_eq,
                                                       int* __restrict__ victim_slot,
                                                       int64_t* victim_id, Ctr* ctr,
                                                       int* __restrict__ dmap, IdxEntry* index, uint32_t hi) {
  __shared__ int smem[32];
  if (ctr->K == 0) return;
  const int f = ctr->f_old, T = ctr->T, r = ctr->r, K = ctr->K;
  // victims in the tiles before this block's current one: summed from the per-tile counts, and
  // carried on from tile to tile (each block reads every count at most once)
  int pre_lt = 0, pre_eq = 0, summed = 0;
  for (int tile = blockIdx.x; tile * kPosChunk < f; tile += gridDim.x) {
    const int base = tile * kPosChunk + (int)threadIdx.x * 8;
    unsigned mlt = 0, meq = 0;
    int lt = 0, eq = 0;
    int v[8];
    if (base + 8 <= f) {
      const int4 a = *reinterpret_cast<const int4*>(stamp + base);
      const int4 b = *reinterpret_cast<const int4*>(stamp + base + 4);
      v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = base + j < f ? stamp[base + j] : kIntMax;   // never a victim
    }
    int a = 0, b = 0;
    for (int i = summed + (int)threadIdx.x; i < tile; i += 256) { a += tile_lt[i]; b += tile_eq[i]; }
    summed = tile;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (v[j] < T) { mlt |= 1u << j; ++lt; }
      if (v[j] == T) { meq |= 1u << j; ++eq; }
    }
    // one scan for both counts: a tile has 2048 slots, so each prefix fits in 16 bits
    int tot, both = (lt << 16) | eq, tot_a;
    block_excl_scan2(both, a, tot, tot_a, smem);
    pre_lt += tot_a;
    pre_eq += block_sum(b, smem);
    int lt_before = (both >> 16) + pre_lt;
    int eq_before = (both & 0xffff) + pre_eq;
    // list position of each victim among this thread's eight slots, then the resident ids with all
    // loads in flight (a thread rarely has more than one victim, but a dependent load per victim
    // inside this loop made the pass latency-bound)
    int idx[8];
    int64_t vid8[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const bool is_lt = mlt & (1u << j), is_eq = meq & (1u << j);
      idx[j] = -1;
      if (is_lt || (is_eq && eq_before < r)) {
        idx[j] = lt_before + (eq_before < r ? eq_before : r);
        if (idx[j] >= K) { idx[j] = -1; flag_err(ctr, 4); }     // never while hist mirrors the stamps
      }
      lt_before += is_lt;
      eq_before += is_eq;
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) if (idx[j] >= 0) vid8[j] = slot_id[base + j];
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (idx[j] >= 0) {
        victim_slot[idx[j]] = base + j; victim_id[idx[j]] = vid8[j];
        if (dmap) dmap[vid8[j]] = -1;          // dense index: the victim leaves it here, one store
      }
    if (!dmap) {
      // hashed index: the tile's victims stand side by side in the list; a thread per victim looks its id up and
      // deletes it.  The inserts are in the next kernel and must stay there: with deletions and inserts in one
      // kernel a resident id went missing from the index about once in a hundred steps at the target
      // size (plain stores and memory-side atomics on neighbouring entries of one line from different
      // XCDs); separated, and with every write to the index of a kernel that also uses atomics on it made an
      // atomic itself, it has not been seen again.
      const int k0 = pre_lt + (pre_eq < r ? pre_eq : r);
      const int eq_end = pre_eq + (tot & 0xffff);
      int k1 = pre_lt + (tot >> 16) + (eq_end < r ? eq_end : r);
      if (k1 > K) k1 = K;
      __syncthreads();
      for (int k = k0 + (int)threadIdx.x; k < k1; k += 256) {
        uint32_t where;
        if (index_find(index, hi, victim_id[k], &where, ctr) >= 0)
          atomicExch((unsigned long long*)&index[where].key, (unsigned long long)kTomb);
        else
          flag_err(ctr, 3);
      }
    }
  }
  if (!dmap && blockIdx.x == 0 && threadIdx.x == 0) atomicAdd(&ctr->tomb, ctr->K);
}

// The step's counters, final since the plan, into the Host status block: one 64-bit store by each of the
// first kStatWords lanes of a wavefront (see HostStatus).
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void publish(HostStatus* h, int lane, int t, int U, int n_hit, int M, int K,
                                        int n_bypass, int n_invalid, int bad_offsets) {
  if (!h || lane >= kStatWords) return;
  const int v = lane == kStatU ? U : lane == kStatHit ? n_hit : lane == kStatMiss ? M : lane == kStatEvict ? K
              : lane == kStatBypass ? n_bypass : lane == kStatInvalid ? n_invalid : bad_offsets;
  __hip_atomic_store(&h->word[lane], (uint64_t)(uint32_t)t << 32 | (uint32_t)v, __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_SYSTEM);
}

// ---------------------------------------------------------------------------------------------
// Assignment: the i-th miss in virtual-id order takes the i-th slot of (victims u free) in
// ascending slot order: victims (all below the watermark) first, then never-used slots from the
// watermark up, then transient bypass rows C + j.
// ---------------------------------------------------------------------------------------------
// The groups of the positions: cnt == nullptr where the batch is not grouped (see group_now in the host code).
struct GroupArgs {
  const int* cnt; int* cnt_rep; int* cur_rep; int bins, nrep; const int* tile_cnt; int64_t* grp; int2* cold_pay;
};
// Virtual id v (below U) has nv positions, which start at off: where its group and the copies of a hot bin start.  (The
// arrays as restricted pointers: read through the struct, each copy's count waited for the store of the one before,
// 11.1 us instead of 8.5 for the assign pass at 65536 x 39 ids.)
__device__ __forceinline__ void group_start(int* __restrict__ cnt_rep, int* __restrict__ cur_rep, int bins, int nrep,
                                            int64_t* __restrict__ grp, int2* __restrict__ cold_pay, int v, int nv, int off) {
  grp[v] = ((int64_t)nv << 32) | (uint32_t)off;
  cold_pay[v] = make_int2(-1, -1);              // the grouping pass fills in the cold groups' rows
  if (v < bins) {                               // one group start per copy of a hot bin; copies back to zero
    int at = off;
#pragma unroll 8
    for (int r = 0; r < nrep; ++r) {
      const int c = cnt_rep[r * kHotBins + v];
      cur_rep[r * kHotBins + v] = at;
      at += c;
      cnt_rep[r * kHotBins + v] = 0;
    }
  }
}
__device__ __forceinline__ void group_start(const GroupArgs& g, int v, int nv, int off) {
  group_start(g.cnt_rep, g.cur_rep, g.bins, g.nrep, g.grp, g.cold_pay, v, nv, off);
}

__global__ __launch_bounds__(256) void k_assign_misses(const int64_t* __restrict__ unique_ids, const GroupArgs gr,
                                                        const int* __restrict__ tile_moff,
                                                        const int* __restrict__ victim_slot,
                                                        int* __restrict__ slot_out,
                                                        int* __restrict__ miss_vids,
                                                        int* __restrict__ miss_row,
                                                        int64_t* __restrict__ miss_id, int boff,
                                                        int64_t* __restrict__ slot_id, int* stamp,
                                                        IdxEntry* index, uint32_t hi,
                                                        int* __restrict__ dmap, int t, int C,
                                                        int* __restrict__ tile_reuse, Ctr* ctr) {
  __shared__ int smem[32];
  const int U = ctr->U, K = ctr->K, f = ctr->f_old;
  const int free_slots = C - f;
  if (blockIdx.x == gridDim.x - 1)
    publish(ctr->hstat, (int)threadIdx.x, t, U, ctr->n_hit, ctr->M, K, ctr->n_bypass, ctr->n_invalid, ctr->bad_offsets);
  // positions of the tiles before this block's current one, carried on from tile to tile
  int before = 0, summed = 0;
  for (int tile = blockIdx.x; tile * kVidTile < U; tile += gridDim.x) {
    const int v = tile * kVidTile + (int)threadIdx.x;
    const bool miss = v < U && slot_out[v] == kMissMark;
    const int first_miss = tile_moff[tile];
    int tot, more = 0;
    int i = miss ? 1 : 0, tot_i;
    if (gr.cnt) {
      for (int j = summed + (int)threadIdx.x; j < tile; j += 256) more += gr.tile_cnt[j];
      summed = tile;
      // start of the group of virtual id v in perm64 = exclusive scan of cnt
      const int nv = v < U ? gr.cnt[v] : 0;
      int off = nv;
      block_excl_scan2(off, i, tot, tot_i, smem);
      before += block_sum(more, smem);
      if (v < U) group_start(gr, v, nv, before + off);
    } else {
      i = block_excl_scan(i, tot_i, smem);
    }
    i += first_miss;
    bool reused = false;
    if (miss) {
      miss_vids[i] = v;
      int s;
      if (i < K) s = victim_slot[i];
      else if (i - K < free_slots) s = f + (i - K);
      else s = C + (i - K - free_slots);
      slot_out[v] = s;
      const int64_t id = unique_ids[v];
      miss_row[i] = s >= C ? s + boff : s;      // for the Host copies: cache row and Host row per miss
      miss_id[i] = id;
      if (s < C) {
        slot_id[s] = id;
        stamp[s] = t;
        if (dmap) dmap[id] = s;
        else reused = index_insert(index, hi, id, s, ctr);
      }
    }
    // deleted entries taken back into use: tallied per tile for the next plan pass (thousands of
    // atomics on one counter would serialise at the memory side, about 10 ns each)
    if (!dmap) {
      const int nre = block_sum(reused ? 1 : 0, smem);
      if (threadIdx.x == 0) tile_reuse[tile] = nre;
    }
  }
}

// Row per position of a batch that is not grouped, for the forward gather; 1024 positions per block.
struct RowsArgs { const int *inverse, *slot; int n, C, boff; int* pos_slot; };
__device__ __forceinline__ void rows_of_positions(const RowsArgs& a, int blk) {
  constexpr int kPer = 4;
  const int base = blk * 256 * kPer + (int)threadIdx.x;
  int v[kPer], s[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) v[j] = base + j * 256 < a.n ? a.inverse[base + j * 256] : -1;
#pragma unroll
  for (int j = 0; j < kPer; ++j) s[j] = v[j] >= 0 ? a.slot[v[j]] : -1;
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    if (v[j] >= 0) a.pos_slot[base + j * 256] = s[j] >= a.C ? s[j] + a.boff : s[j];
}
__global__ __launch_bounds__(256) void k_pos_rows(const RowsArgs a) { rows_of_positions(a, (int)blockIdx.x); }

// The grouping of a batch that was prepared without it, when its gradient comes all the same: positions counted and
// ranked, sums and bags, starts of the groups, the grouping pass.  t: the step; where the counters are another step's, a
// graph has been launched that was recorded on this one: nothing to do.
template <int kPer, int kT>
__global__ __launch_bounds__(kT) void k_count_late(const RankArgs a, const Ctr* ctr, int t) {
  __shared__ int lds[kHotBins];
  if (ctr->t != t) return;
  count_positions<kPer, kT>(nullptr, nullptr, a.n, a.inverse, a.cnt, a.cnt_rep, a.nrep, a.rank, nullptr,
                            (int)blockIdx.x, lds);
}
__global__ __launch_bounds__(256) void k_fold_late(Ctr* ctr, const FoldArgs fo, const BagArgs bags, int t) {
  __shared__ int words[256];
  if (ctr->t != t) return;
  fold_or_bags<256>(fo, bags, ctr, (int)blockIdx.x, words);
}
__global__ __launch_bounds__(256) void k_starts_late(const GroupArgs gr, const Ctr* ctr, int t) {
  __shared__ int smem[20];
  if (ctr->t != t) return;
  const int U = ctr->U;
  int before = 0, summed = 0;
  for (int tile = blockIdx.x; tile * kVidTile < U; tile += gridDim.x) {
    const int v = tile * kVidTile + (int)threadIdx.x;
    int tot, more = 0;
    for (int j = summed + (int)threadIdx.x; j < tile; j += 256) more += gr.tile_cnt[j];
    summed = tile;
    const int nv = v < U ? gr.cnt[v] : 0;
    const int off = block_excl_scan(nv, tot, smem);
    before += block_sum(more, smem);
    if (v < U) group_start(gr, v, nv, before + off);
  }
}
template <int kScatPer, int kT>
__global__ __launch_bounds__(kT) void k_scatter_late(const ScatterArgs a, const Ctr* ctr, int t) {
  if (ctr->t == t) scatter_positions<kScatPer, kT, false>(a, (int)blockIdx.x);
}

// ---------------------------------------------------------------------------------------------
// The prepare of a small batch, by ONE block: up to kSmallIds positions fit the LDS of a compute unit
// (their table of distinct ids, counts and slots), and for so few the launches of the passes above were
// all start-up, drain and dependent round trips: what bounds this kernel is the chain ids ->
// table -> rank -> index -> stamp -> lists, walked once with barriers in between instead of kernel
// boundaries, and, from a few thousand positions on, how many scattered accesses one compute unit issues.
// Same outputs, same state.
// So nothing in it waits that need not: the index is read for every position as soon as its id is there, beside
// the table of distinct ids, and the thread that holds an id's first position keeps what it has learned of the
// id (slot, stamp, number) in registers to the end; one scan numbers the distinct ids and the misses; the
// counters are published before the last passes; barriers wait for LDS only.  And what goes to memory goes out in
// order: thread i takes positions i, 1024 + i, ..., virtual ids are numbered by ballots in that order, and the
// grouping is put together in LDS.  us at 1248 / 4992 positions: the kernel from its first to its last instruction
// 14.1 / 23.8 with a thread per run of consecutive positions, the index read per virtual id and the counters
// published last, 5.4 / 14.8 this way (64-bit words in the table of ids 6.3 / 18.7); a pass of 32 x 39 ids looked up
// 19.8 -> 15.2 (13.4 of it host time), of 128 x 39 trained 43.1 -> 34.3.
//
// kWhole (dense index, and either a cache that holds the whole table, so that nothing is ever evicted,
// or one whose stamps a single block can scan: kSmallSlots): everything up to the grouping, one launch.
// Otherwise the unique passes and the resolve only; plan, victims, assignment and grouping follow as
// for any batch (with no hot bins: cnt and the ranks are complete).
// ---------------------------------------------------------------------------------------------
constexpr int kSmallIds = 6144;
constexpr int kSmallPer = kSmallIds / 1024; // positions per thread, at most
constexpr int kSmallBits = 13;              // bits of a position
// entries of the LDS table of distinct ids, for kPer positions per thread: 2.7 to 4 times as many as positions
constexpr int small_tab(int per) { return per <= 2 ? 8192 : 16384; }
constexpr int kSmallSlots = 1 << 16;        // 16 rounds of 16-byte loads over the stamps
constexpr int kSmallBags = 4 * kSmallIds;   // bags may be empty, so there can be more of them than ids

struct SmallArgs {
  const int64_t* ids; int n; int64_t V;
  const int64_t* offsets; int n_bags;       // multi-hot input (else nullptr)
  int64_t* unique_ids; int* inverse; int* slot; int* miss_vids;      // caller's buffers of the step
  const IdxEntry* index; uint32_t hi; int* dmap;
  int* stamp; int64_t* slot_id; int* hist; int t, lookahead, C, boff;
  int *cnt, *tile_miss, *age_hist;                                   // outputs of the short form
  int64_t* grp; int2* cold_pay; int64_t* perm64; int* pos_slot;
  int* victim_slot; int64_t* victim_id; int* miss_row; int64_t* miss_id;
  Ctr* ctr; const Ctr* prev;                // prev: nullptr when k_ctr_init has started the counters
};

// Exclusive prefix of this wavefront's kSmallPer numbers in the order of the positions (all wavefronts' first
// numbers, then all second ones, ...).  x: the numbers, the same in every lane; ent: kSmallPer * 16 words of
// LDS for this call alone.
template <int kPer>
__device__ __forceinline__ void small_prefix(const int (&x)[kPer], int (&pre)[kPer], int& total, int* ent) {
  static_assert(kPer * 16 <= 2 * kWave, "two words per lane");
  const int lane = lane_id(), w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  int mine = 0;
#pragma unroll
  for (int j = 0; j < kPer; ++j) mine = lane == j ? x[j] : mine;
  if (lane < kPer) ent[lane * 16 + w] = mine;
  lds_barrier();
  const int s0 = wave_incl_scan(lane < kPer * 16 ? ent[lane] : 0);
  const int half = __builtin_amdgcn_readlane(s0, kWave - 1);
  const int s1 = half + wave_incl_scan(lane < kPer * 16 - kWave ? ent[kWave + lane] : 0);
  total = __builtin_amdgcn_readlane(s1, kWave - 1);
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int k = j * 16 + w - 1;
    pre[j] = k < 0 ? 0 : k < kWave ? __builtin_amdgcn_readlane(s0, k) : __builtin_amdgcn_readlane(s1, k - kWave);
  }
}
// lanes before this one whose bit is set
__device__ __forceinline__ int bits_before(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0));
}

template <bool kWhole, int kPer>
__global__ __launch_bounds__(1024) void k_small_prepare(const SmallArgs a) {
  constexpr int kIds = kPer * 1024, kTab = small_tab(kPer);
  // Table of distinct ids: 18 bits of the hash and the smallest position with that id in one word, ~0 = empty.
  // (32-bit words, because the claims are what the LDS is busy with.)  Once the virtual ids have been handed
  // out: cache row per virtual id (short form: does it miss) and bag per position.
  __shared__ __align__(16) unsigned tab[kTab];
  __shared__ __align__(16) int64_t lkey[kIds];        // id per position; later the grouping, an entry per position
  __shared__ __align__(16) int cntl[kIds];            // positions per virtual id; later start of the group << 16 | positions
  __shared__ int age[kAgeBins];
  __shared__ int smem[20], ent1[kPer * 16], ent2[kPer * 16];
  __shared__ int s_found, s_bad, s_err, s_inv;
  static_assert(kTab >= 2 * kIds && kIds <= 1 << kSmallBits && kAgeBins == 1024, "sizes of the tables");
  int* const slotl = reinterpret_cast<int*>(tab);
  int* const bagl = slotl + kIds;
  constexpr unsigned kPos = (1u << kSmallBits) - 1;
  const int tid = (int)threadIdx.x, n = a.n, lane = lane_id();
  int64_t key[kPer];
  int e[kPer], sl[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int p = j * 1024 + tid;
    key[j] = p < n ? a.ids[p] : (int64_t)-1;
  }
  {
    const uint4 none = make_uint4(~0u, ~0u, ~0u, ~0u);
#pragma unroll
    for (int i = 0; i < kTab / 4096; ++i) reinterpret_cast<uint4*>(tab)[i * 1024 + tid] = none;
    for (int i = tid; i * 4 < n; i += 1024) reinterpret_cast<int4*>(cntl)[i] = make_int4(0, 0, 0, 0);
    age[tid] = 0;
    if (tid == 0) s_bad = s_err = s_inv = 0;
  }
  // counters of the previous step (on a cache's first step and behind k_ctr_init: of this one, nothing is written
  // there before it has been read)
  const Ctr* const was = a.prev ? a.prev : a.ctr;
  const int f_was = was->f, oldest = was->oldest;
  HostStatus* const hstat = was->hstat;
  if (tid == 0) a.ctr->t = a.t;
  // the dense index by position, on its way while the table is filled (a frequent id's word is one line)
  int n_bad_ids = 0;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int p = j * 1024 + tid;
    if (key[j] < 0 || key[j] >= a.V) { key[j] = kNullKey; n_bad_ids += p < n; }
    lkey[p] = key[j];
    sl[j] = -1;
    if ((kWhole || a.dmap) && key[j] >= 0) sl[j] = a.dmap[key[j]];
  }
  lds_barrier();
  if (n_bad_ids) atomicAdd(&s_inv, n_bad_ids);
  // the distinct ids and their first positions: an entry is claimed together with its position, a smaller one
  // is one minimum; the first probes of a thread's positions go side by side, the few that go on do so one by one
  {
    constexpr int kShift = 32 - __builtin_ctz(kTab);
    auto hash = [](int64_t k) {
      uint32_t h = (uint32_t)k * 0x9e3779b1u + (uint32_t)((uint64_t)k >> 32) * 0x85ebca77u;
      return h ^ h >> 15;
    };
    uint32_t q[kPer], mine[kPer];
    unsigned open = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const uint32_t h = hash(key[j]);
      e[j] = (int)(h >> kShift);
      mine[j] = (h & 0x3ffff) << kSmallBits | (uint32_t)(j * 1024 + tid);
      q[j] = j * 1024 + tid < n ? tab[e[j]] : 0u;
    }
#pragma unroll
    for (int j = 0; j < kPer; ++j)
      if (q[j] == ~0u) q[j] = atomicCAS(&tab[e[j]], ~0u, mine[j]);
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      if (q[j] == ~0u || j * 1024 + tid >= n) continue;            // claimed
      if ((q[j] ^ mine[j]) <= kPos && lkey[q[j] & kPos] == key[j]) {
        if (q[j] > mine[j]) atomicMin(&tab[e[j]], mine[j]);
      } else {
        open |= 1u << j;
      }
    }
    uint32_t l = 0, m = 0;
    int64_t k = 0;
    bool fresh = true;
    while (open) {                            // (at most kTab probes per position: the table is never full)
      const int j = __builtin_ctz(open);
      if (fresh) {
        k = lkey[j * 1024 + tid];
        const uint32_t h = hash(k);
        l = h >> kShift;
        m = (h & 0x3ffff) << kSmallBits | (uint32_t)(j * 1024 + tid);
        fresh = false;
      }
      l = (l + 1) & (kTab - 1);
      uint32_t w = tab[l];
      if (w == ~0u) w = atomicCAS(&tab[l], ~0u, m);
      bool done = w == ~0u;
      if (!done && (w ^ m) <= kPos && lkey[w & kPos] == k) {
        if (w > m) atomicMin(&tab[l], m);
        done = true;
      }
      if (done) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) e[i] = i == j ? (int)l : e[i];
        open &= open - 1;
        fresh = true;
      }
    }
  }
  lds_barrier();
  // first appearances, which of them are resident, and their stamps
  unsigned first = 0, hitm = 0, missm = 0;
  int old[kPer], vid[kPer], mi[kPer], x[kPer], pre[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int p = j * 1024 + tid;
    if (p < n && (int)(tab[e[j]] & kPos) == p) first |= 1u << j;
  }
  if (!kWhole && !a.dmap) {                   // the hashed index: one probe sequence at a time, of the distinct ids only
    for (unsigned m = first; m; m &= m - 1) {
      const int j = __builtin_ctz(m);
      const int64_t k = lkey[j * 1024 + tid];
      const int s = k >= 0 ? index_find(a.index, a.hi, k, nullptr, a.ctr) : -1;
#pragma unroll
      for (int i = 0; i < kPer; ++i) sl[i] = i == j ? s : sl[i];
    }
  }
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const bool is_first = first & (1u << j);
    bool miss = false;
    old[j] = 0;
    if (is_first && key[j] >= 0) {
      if (sl[j] >= 0) { hitm |= 1u << j; old[j] = a.stamp[sl[j]]; }
      else { missm |= 1u << j; miss = true; }
    }
    const uint64_t bf = __ballot(is_first), bm = __ballot(miss);
    x[j] = __popcll(bf) << 16 | __popcll(bm);
    vid[j] = bits_before(bf);
    mi[j] = bits_before(bm);
  }
  int tot;
  small_prefix(x, pre, tot, ent1);
  const int U = tot >> 16, M = tot & 0xffff, n_invalid = s_inv, n_hit = U - M - (n_invalid > 0);
  // virtual ids in order of first appearance, into the table's entries for the other positions (every
  // position has read its entry: the barrier above)
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    vid[j] += pre[j] >> 16;
    mi[j] += pre[j] & 0xffff;
    if (first & (1u << j)) {
      tab[e[j]] = (unsigned)vid[j];
      a.unique_ids[vid[j]] = key[j] == kNullKey ? (int64_t)-1 : key[j];
    }
  }
  lds_barrier();
  int vv[kPer], rr[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const bool in = j * 1024 + tid < n;
    vv[j] = in ? (int)tab[e[j]] : 0;
    rr[j] = 0;
    if (in) {
      a.inverse[j * 1024 + tid] = vv[j];
      rr[j] = atomicAdd(&cntl[vv[j]], 1);
    }
  }
  // hits move to the step's stamp; their old ones by age, as resolve_ids does it
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const bool hit = hitm & (1u << j);
    const int g = a.t - old[j];
    const uint64_t m1 = __ballot(hit && g == 1);
    if (m1 && lane == 0) atomicAdd(&age[1], __popcll(m1));
    if (hit) {
      a.stamp[sl[j]] = a.t;
      if (g >= kAgeBins) hist_add(&a.hist[old[j]], -1);
      else if (g != 1) atomicAdd(&age[g], 1);
    }
  }
  lds_barrier();
  if (!kWhole) {
    // in the form k_plan and its followers take it: slots, counts, ranks, tallies per tile and by age
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      if (j * 1024 + tid < n) a.pos_slot[j * 1024 + tid] = rr[j];
      if (!(first & (1u << j))) continue;
      const bool miss = missm & (1u << j);
      a.slot[vid[j]] = sl[j] >= 0 ? sl[j] : (miss ? kMissMark : -1);
      a.cnt[vid[j]] = cntl[vid[j]];
      slotl[vid[j]] = miss ? 1 : 0;
    }
    lds_barrier();
    a.age_hist[tid] = tid ? age[tid] : n_hit;
    const int w = tid >> 6;
    for (int tile = w; tile * kVidTile < U; tile += 16) {    // a wavefront per tile of kVidTile virtual ids
      int m = 0;
      for (int v = tile * kVidTile + lane; v < U && v < (tile + 1) * kVidTile; v += kWave) m += slotl[v];
      m = wave_sum(m);
      if (lane == 0) a.tile_miss[tile] = m;
    }
    if (tid == 0) {
      Ctr c0 = *was;
      if (a.prev) {
        c0.U_prev = c0.U;
        if (c0.n_bypass) c0.last_bypass = a.t - 1;
        c0.M = c0.K = c0.n_bypass = c0.n_hit = 0;
        c0.f_old = c0.f; c0.need = 0; c0.T = 0; c0.r = 0;
        c0.t = a.t; c0.bad_offsets = 0;
      }
      c0.U = U; c0.n_invalid = n_invalid;
      const int err = a.ctr->err;
      if (err) c0.err = err;                         // a probe above may have flagged one
      *a.ctr = c0;
    }
    return;
  } else {
    if (a.offsets) {
      for (int i = tid; i < n; i += 1024) bagl[i] = 0;
      lds_barrier();
    }
    // the histogram: hits move to stamp t, the rest of the plan as k_plan does it.  Only a search for
    // victims reads it in here, so only then do the sums have to be back.
    const int f = f_was, C = a.C, free_slots = C - f;
    const int moved = tid == 0 ? n_hit : -age[tid];
    if (moved) {
      if (M > free_slots) hist_add(&a.hist[a.t - tid], moved);
      else atomicAdd(&a.hist[a.t - tid], moved);
    }
    Plan pl;
    plan_decide<true>(pl, M, f, oldest, a.hist, a.t, a.lookahead, C, smem, &s_found);
    // bag of every position, checked as bags_of_positions does
    if (a.offsets) {
      int bad = 0;
      for (int b = tid; b < a.n_bags; b += 1024) {
        const int64_t lo = a.offsets[b], hi = a.offsets[b + 1];
        bad += bag_malformed(lo, hi, b, a.n_bags, n);
        const BagRange r = bag_range(lo, hi, n);
        for (int q = r.lo; q < r.hi; ++q) bagl[q] = b;
      }
      if (bad) atomicAdd(&s_bad, bad);
    }
    // victims, in slot order: k_victim_count / k_victim_write by one block
    if (pl.K > 0) {
      int lt_done = 0, eq_done = 0;
      for (int base = 0; base < f; base += 4096) {
        const int s0 = base + tid * 4;
        int v[4];
        if (s0 + 4 <= f) {
          const int4 q = *reinterpret_cast<const int4*>(a.stamp + s0);
          v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) v[j] = s0 + j < f ? a.stamp[s0 + j] : kIntMax;   // never a victim
        }
        int lt = 0, eq = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) { lt += v[j] < pl.T; eq += v[j] == pl.T; }
        int both;
        const int pre2 = block_excl_scan((lt << 16) | eq, both, smem);
        int lt_before = lt_done + (pre2 >> 16), eq_before = eq_done + (pre2 & 0xffff);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const bool is_lt = v[j] < pl.T, is_eq = v[j] == pl.T;
          if (is_lt || (is_eq && eq_before < pl.r)) {
            const int idx = lt_before + (eq_before < pl.r ? eq_before : pl.r);
            if (idx < pl.K) {
              const int64_t vid_out = a.slot_id[s0 + j];
              a.victim_slot[idx] = s0 + j; a.victim_id[idx] = vid_out;
              a.dmap[vid_out] = -1;
            } else {
              s_err = 4;                                     // never while hist mirrors the stamps
              flag_err(a.ctr, 4);
            }
          }
          lt_before += is_lt;
          eq_before += is_eq;
        }
        lt_done += both >> 16; eq_done += both & 0xffff;
      }
    }
    if (pl.K > 0) __syncthreads();                           // the victims are listed (through memory)
    // where the groups start
    int cn[kPer], off[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      cn[j] = first & (1u << j) ? cntl[vid[j]] : 0;
      off[j] = wave_incl_scan(cn[j]);
      x[j] = __builtin_amdgcn_readlane(off[j], kWave - 1);
    }
    small_prefix(x, pre, tot, ent2);                         // (its barrier: the bags are complete)
    // the counters, on their way while the lists are written
    if (tid >= 1024 - kWave) {
      // whoever sees the step's counters also sees that its offsets were malformed: first that, and back
      volatile HostStatus* h = hstat;
      if (s_bad && h) { h->bad_offsets_step = a.t; stores_done(); }
      publish(hstat, lane, a.t, U, n_hit, M, pl.K, pl.n_bypass, n_invalid, s_bad);
    }
    if (tid == 0) {
      if (pl.need > 0 && pl.r > 0) atomicAdd(&a.hist[pl.T], -pl.r);
      if (M != pl.n_bypass) atomicAdd(&a.hist[a.t], M - pl.n_bypass);
      Ctr c0 = *was;
      c0.U_prev = c0.U; c0.U = U; c0.n_hit = n_hit; c0.n_invalid = n_invalid;
      if (c0.n_bypass) c0.last_bypass = a.t - 1;
      c0.t = a.t; c0.bad_offsets = s_bad;
      plan_store(pl, c0, f);
      if (s_err) c0.err = s_err;
      *a.ctr = c0;
    }
    // slots of the misses; groups
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      if (!(first & (1u << j))) continue;
      const int v = vid[j];
      int s = sl[j];
      if (missm & (1u << j)) {
        const int i = mi[j];
        a.miss_vids[i] = v;
        if (i < pl.K) s = a.victim_slot[i];
        else if (i - pl.K < free_slots) s = f + (i - pl.K);
        else s = C + (i - pl.K - free_slots);
        a.miss_row[i] = s >= C ? s + a.boff : s;
        a.miss_id[i] = key[j];
        if (s < C) { a.slot_id[s] = key[j]; a.stamp[s] = a.t; a.dmap[key[j]] = s; }
      }
      off[j] += pre[j] - cn[j];
      a.slot[v] = s;
      slotl[v] = s >= C ? s + a.boff : s;
      cntl[v] = off[j] << 16 | cn[j];
      a.grp[v] = ((int64_t)cn[j] << 32) | (uint32_t)off[j];
    }
    lds_barrier();
    // grouping, put together in LDS; here any group of at most kColdMax positions is a cold one
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const int p = j * 1024 + tid;
      if (p >= n) continue;
      const int v = vv[j], sc = cntl[v];
      a.pos_slot[p] = slotl[v];
      int64_t w = ((int64_t)v << 32) | (uint32_t)(a.offsets ? bagl[p] : p);
      if ((sc & 0xffff) <= kColdMax) w |= kColdBit;
      lkey[(sc >> 16) + rr[j]] = w;
    }
    lds_barrier();
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const int i = j * 1024 + tid;
      if (i < n) a.perm64[i] = lkey[i];
      if (first & (1u << j)) {
        int2 cp = make_int2(-1, -1);
        if (cn[j] <= kColdMax) {
          cp.x = (int)(uint32_t)lkey[off[j]];
          if (cn[j] == kColdMax) cp.y = (int)(uint32_t)lkey[off[j] + 1];
        }
        a.cold_pay[vid[j]] = cp;
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Test aid (sfc_verify): recount of the manager state after a complete prepare.
//   bad[0]  occupied slots (below the watermark) whose id the index does not map to that slot
//   bad[1]  live index entries that do not point at a slot holding their id
//   bad[2]  words of the recency histogram that differ from the recount of the slots' stamps
//   bad[3]  live index entries (the host compares them with the number of occupied slots)
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ void tally(unsigned long long* word, int mine) {
  const int w = wave_sum(mine);
  if (w && lane_id() == 0) atomicAdd(word, (unsigned long long)w);
}

__global__ __launch_bounds__(256) void k_verify_slots(const int64_t* __restrict__ slot_id,
                                                       const int* __restrict__ stamp,
                                                       const IdxEntry* __restrict__ index,
                                                       uint32_t hi, const int* __restrict__ dmap,
                                                       int* recount, int hist_len,
                                                       unsigned long long* bad, Ctr* ctr) {
  const int f = ctr->f;
  const int rounds = (f + (int)gridDim.x * 256 - 1) / ((int)gridDim.x * 256);
  int s = blockIdx.x * 256 + (int)threadIdx.x;
  for (int it = 0; it < rounds; ++it, s += gridDim.x * 256) {   // every lane stays for the wave sums
    int lost = 0, off = 0;
    if (s < f) {
      const int64_t id = slot_id[s];
      if (id < 0 || (dmap ? dmap[id] : index_find(index, hi, id, nullptr, ctr)) != s) lost = 1;
      const int st = stamp[s];
      if (st >= 0 && st < hist_len) atomicAdd(&recount[st], 1); else off = 1;
    }
    tally(&bad[0], lost);
    tally(&bad[2], off);
  }
}

__global__ __launch_bounds__(256) void k_verify_entries(const IdxEntry* __restrict__ index,
                                                         uint32_t hi,
                                                         const int64_t* __restrict__ slot_id, int C,
                                                         unsigned long long* bad) {
  const uint32_t stride = gridDim.x * 256;
  const uint32_t rounds = (hi + stride - 1) / stride;
  uint32_t i = blockIdx.x * 256 + threadIdx.x;
  int live = 0, stray = 0;
  for (uint32_t it = 0; it < rounds; ++it, i += stride) {
    if (i < hi) {
      const int4 raw = *reinterpret_cast<const int4*>(&index[i]);
      const int64_t key = idx_key(raw);
      if (key >= 0) {
        ++live;
        if (raw.z < 0 || raw.z >= C || slot_id[raw.z] != key) ++stray;
      }
    }
  }
  tally(&bad[3], live);
  tally(&bad[1], stray);
}

// the same for the dense index: every entry >= 0 is live and must point at a slot holding its id
__global__ __launch_bounds__(256) void k_verify_dense(const int* __restrict__ dmap, int64_t V,
                                                       const int64_t* __restrict__ slot_id, int C,
                                                       unsigned long long* bad) {
  const int64_t stride = (int64_t)gridDim.x * 256;
  const int64_t rounds = (V + stride - 1) / stride;
  int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  int live = 0, stray = 0;
  for (int64_t it = 0; it < rounds; ++it, i += stride) {
    if (i < V) {
      const int s = dmap[i];
      if (s >= 0) {
        ++live;
        if (s >= C || slot_id[s] != i) ++stray;
      }
    }
  }
  tally(&bad[3], live);
  tally(&bad[1], stray);
}

__global__ __launch_bounds__(256) void k_verify_hist(const int* __restrict__ hist,
                                                      const int* __restrict__ recount, int hist_len,
                                                      unsigned long long* bad) {
  const int stride = (int)gridDim.x * 256;
  const int rounds = (hist_len + stride - 1) / stride;
  int i = blockIdx.x * 256 + (int)threadIdx.x, off = 0;
  for (int it = 0; it < rounds; ++it, i += stride)
    if (i < hist_len && hist[i] != recount[i]) ++off;
  tally(&bad[2], off);
}

}  // namespace sfc
