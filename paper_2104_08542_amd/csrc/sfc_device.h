// Device-side building blocks shared by the kernels of the sparse-embedding step:
// hashing, wavefront/block scans and reductions for 64-wide wavefronts, 16-byte row chunks.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace sfc {

constexpr int kWave = 64;
constexpr int64_t kEmpty = -1;      // never-used entry of a hash table
constexpr int64_t kNullKey = -2;    // batch-unique table: the collapsed out-of-range id
constexpr int64_t kTomb = -2;       // cache index: deleted entry (ids in the index are >= 0)
constexpr int kMissMark = -2;       // d_slot value between resolve and assignment
constexpr int kIntMax = 0x7fffffff;

// Grouped positions (perm64): one 64-bit entry per position, (virtual id << 32) | gradient row,
// groups in virtual-id order.  Virtual ids stay below 2^30, so bit 62 is free: it marks the
// entries of a *cold* group, one of at most kColdMax positions whose virtual id lies outside the
// range the counting pass treats in LDS.  Nine rows in ten of a power-law batch are such rows.
// Their gradients are summed by the optimizer kernel itself, straight from the gradient rows;
// the segment-sum stream passes over them, and their rows of the common-gradient matrix are
// neither written nor read.
constexpr int kHotBins = 8192;      // lowest virtual ids, at most: counted through LDS histograms
constexpr int kColdMax = 2;
constexpr int64_t kColdBit = (int64_t)1 << 62;
// cold_pay[v] holds the (at most two) gradient rows of a cold group, (-1, -1) for any other group.
// A third value of its first word marks a group that the segment-sum stream left as block-edge
// partials: the optimizer kernel chains those itself and updates the row there.
constexpr int kEdgeMark = -2;
__device__ __forceinline__ int entry_vid(int64_t e) { return (int)(e >> 32) & 0x3fffffff; }
__device__ __forceinline__ bool entry_cold(int64_t e) { return (e & kColdBit) != 0; }
// per virtual id: (positions << 32) | start of its group in perm64
__device__ __forceinline__ bool group_cold(int64_t grp) { return (int)(grp >> 32) <= kColdMax; }

// Positions [lo, hi) of a bag by its two offsets, whatever these hold: each clamped to [0, n] in 64 bits
// before it becomes a 32-bit position (an offset below -2^31 narrowed as it is can look like any position).
// Empty where lo >= hi.
struct BagRange { int lo, hi; };
__host__ __device__ __forceinline__ int clamp_offset(int64_t x, int n) { return x < 0 ? 0 : (x > n ? n : (int)x); }
__host__ __device__ __forceinline__ BagRange bag_range(int64_t lo, int64_t hi, int n) {
  return BagRange{clamp_offset(lo, n), clamp_offset(hi, n)};
}
// Is bag b of n_bags malformed: decreasing, or the first one not at 0, or the last one not ending at n?
__host__ __device__ __forceinline__ bool bag_malformed(int64_t lo, int64_t hi, int b, int n_bags, int n) {
  return hi < lo || (b == 0 && lo != 0) || (b == n_bags - 1 && hi != n);
}

// Status block in pinned, device-mapped Host memory: kernels write it, the host reads it without
// waiting for any stream (sfc_check, sfc_peek_stats and the first lines of every step call).
// A published counter and the step it belongs to share a 64-bit word, step above, and are stored as one: the
// host has a step's counters when all words carry the same step, and the writer has nothing to order or to
// wait for.  (A sequence word around plain counters took two waits for the host link, 5 us at the end of
// the one-block prepare.)
enum { kStatU, kStatHit, kStatMiss, kStatEvict, kStatBypass, kStatInvalid, kStatBadOffsets, kStatWords };
struct HostStatus {
  int err;               // first device-side consistency check that fired (0 = none); never cleared
  int err_step;          // step of that check
  int bad_offsets_step;  // most recent step whose bag offsets were malformed (0 = none)
  int pad;
  uint64_t word[kStatWords];   // step << 32 | counter; step 0 = none yet
};

// Device counters of one cache.  Written by kernels only; the host reads a copy in get_stats.
struct Ctr {
  int U;          // unique ids of the batch
  int M;          // misses
  int K;          // victims
  int n_bypass;
  int n_hit;
  int n_invalid;
  int f;          // slots [0, f) are occupied, [f, C) have never been used
  int f_old;      // f before this step's inserts
  int need;       // misses that found no free slot
  int T;          // stamp threshold: stamp < T is evicted, stamp == T partly
  int r;          // how many slots with stamp == T are evicted (lowest slots first)
  int oldest;     // no occupied slot has a stamp below this
  int tomb;       // deleted entries in the cache index
  int rebuild;    // set when the index must be rebuilt before the next resolve
  int err;        // nonzero: a probe loop ran off its bound
  int last_bypass;    // the latest step before this one that had bypass rows (0: none)
  int U_prev;     // unique ids of the previous step (its per-tile tallies are still to be read)
  int dense;      // the id -> slot index is a dense map (no hashed entries, no tombstones, no rebuild)
  int t;          // number of the step these counters belong to
  int bad_offsets;    // violations found in the step's bag offsets (multi-hot input)
  HostStatus* hstat;  // device view of the cache's status block
};

// A device-side consistency check fired: remembered in the step's counters (every later step
// inherits it) and in the Host status block (plain stores over the link: if several checks fire
// together any one of their codes is kept, which is all the host needs to know).
__device__ __forceinline__ void flag_err(Ctr* ctr, int code) {
  ctr->err = code;
  volatile HostStatus* h = ctr->hstat;
  if (h) { h->err_step = ctr->t; h->err = code; }
}

// Entry of the per-step batch table where an id and a position do not fit 64 bits together (WideTab):
// key and the smallest position that carries it, one 16-byte access for both.
struct __attribute__((aligned(16))) UEntry {
  int64_t key;    // id, kEmpty or kNullKey
  int32_t minpos; // kIntMax when unset
  int32_t pad;
};

struct __attribute__((aligned(16))) IdxEntry {
  int64_t key;    // id, kEmpty or kTomb
  int32_t slot;
  int32_t pad;
};

// murmur3 64-bit finaliser
__device__ __forceinline__ uint64_t mix64(uint64_t x) {
  x ^= x >> 33; x *= 0xff51afd7ed558ccdULL;
  x ^= x >> 33; x *= 0xc4ceb9fe1a85ec53ULL;
  x ^= x >> 33;
  return x;
}
// bucket in [0, n) without a power-of-two table: high half of a 32x32 product
__device__ __forceinline__ uint32_t bucket_of(int64_t key, uint32_t n) {
  return (uint32_t)(((mix64((uint64_t)key) >> 32) * (uint64_t)n) >> 32);
}

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & (kWave - 1)); }

// Sums across the wavefront in registers (DPP): lanes 1, 2, 4, 8 to the left within a row of 16, then the last
// lane of a row into the rows behind it.  Six dependent additions; six shuffles through the LDS crossbar took
// several times as long, and most of the prepare's kernels are a few such scans long.
template <int kCtrl, int kRowMask>
__device__ __forceinline__ int dpp_add(int x) {
  return x + __builtin_amdgcn_update_dpp(0, x, kCtrl, kRowMask, 0xf, false);
}
// inclusive scan over each row of 16 lanes
__device__ __forceinline__ int row_incl_scan(int x) {
  x = dpp_add<0x111, 0xf>(x);      // row_shr:1
  x = dpp_add<0x112, 0xf>(x);      // row_shr:2
  x = dpp_add<0x114, 0xf>(x);      // row_shr:4
  return dpp_add<0x118, 0xf>(x);   // row_shr:8
}
__device__ __forceinline__ int wave_incl_scan(int x) {
  x = row_incl_scan(x);
  x = dpp_add<0x142, 0xa>(x);      // row_bcast:15 into rows 1 and 3
  return dpp_add<0x143, 0xc>(x);   // row_bcast:31 into rows 2 and 3
}
// (every lane of the wavefront has to be active in these three)
__device__ __forceinline__ int wave_sum(int x) { return __builtin_amdgcn_readlane(wave_incl_scan(x), kWave - 1); }

// A barrier for what the block shares in LDS alone: accesses to memory stay in flight across it (__syncthreads
// waits for them, a microsecond or more each time).  What goes through memory from one thread of the block to
// another needs __syncthreads.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Exclusive scan of one int per thread over the block (blockDim.x multiple of 64, <= 1024).
// smem: at least 16 ints, which nothing else may touch between this call and the next barrier.
// total = sum over the block.
__device__ __forceinline__ int block_excl_scan_once(int x, int& total, int* smem) {
  const int lane = lane_id(), nw = (int)(blockDim.x >> 6);
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int inc = wave_incl_scan(x);
  if (lane == kWave - 1) smem[w] = inc;
  __syncthreads();
  const int sums = row_incl_scan(lane < nw ? smem[lane] : 0);     // at most 16 wavefronts: one row
  total = __builtin_amdgcn_readlane(sums, nw - 1);
  const int before = w > 0 ? __builtin_amdgcn_readlane(sums, w - 1) : 0;
  return before + inc - x;
}
// Safe to call repeatedly with the same smem.
__device__ __forceinline__ int block_excl_scan(int x, int& total, int* smem) {
  const int res = block_excl_scan_once(x, total, smem);
  __syncthreads();
  return res;
}

// Two such scans (of two sums) at the barriers of one.  smem: at least 32 ints.
__device__ __forceinline__ void block_excl_scan2(int& x, int& y, int& total_x, int& total_y, int* smem) {
  const int lane = lane_id(), nw = (int)(blockDim.x >> 6);
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int ix = wave_incl_scan(x), iy = wave_incl_scan(y);
  if (lane == kWave - 1) { smem[w] = ix; smem[16 + w] = iy; }
  __syncthreads();
  const int sx = row_incl_scan(lane < nw ? smem[lane] : 0), sy = row_incl_scan(lane < nw ? smem[16 + lane] : 0);
  total_x = __builtin_amdgcn_readlane(sx, nw - 1);
  total_y = __builtin_amdgcn_readlane(sy, nw - 1);
  x = (w > 0 ? __builtin_amdgcn_readlane(sx, w - 1) : 0) + ix - x;
  y = (w > 0 ? __builtin_amdgcn_readlane(sy, w - 1) : 0) + iy - y;
  __syncthreads();
}

__device__ __forceinline__ int block_sum(int x, int* smem) {
  const int lane = lane_id(), w = (int)(threadIdx.x >> 6), nw = (int)(blockDim.x >> 6);
  x = wave_sum(x);
  if (lane == 0) smem[w] = x;
  __syncthreads();
  int s = 0;
  for (int i = 0; i < nw; ++i) s += smem[i];
  __syncthreads();
  return s;
}

}  // namespace sfc
