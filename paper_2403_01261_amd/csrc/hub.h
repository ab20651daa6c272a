// What the hub kernels of whole-number and of float weights share: the hash
// partitions of a hub's labels, the arguments and a block-wide scan.
#pragma once

#include "device_common.h"
#include "gsl_internal.h"

namespace gsl {

namespace {

constexpr int kHubBlock = 256;
constexpr int kHubK = kHubChunk / kHubBlock;  // row entries per lane
constexpr int kTabLog2 = 12;                  // 4096 LDS slots (2 per chunk entry)
constexpr int kTabSlots = 1 << kTabLog2;
constexpr int kMaxParts = kHubMaxParts;
constexpr int kPartSize = 2048;               // expected distinct labels per partition
constexpr int kMergeBlock = 256;
constexpr int kMergeAhead = 4;                // staged records each lane of a merge has on the way
constexpr int kHubFoldRounds = 1;  // label fold rounds per wave before the inserts (as in the tiers)
// Claims before a merge pass gives up and the partition is split into
// sub-passes: at most kHubMergeCapMax, so that a free slot always remains
// (up to kMergeBlock threads may pass the check at once); a smaller cap can
// be set at run time to exercise the sub-pass path on small graphs.
static_assert(kHubMergeCapMax + kMergeBlock < kTabSlots, "a free slot must always remain");
constexpr int kChunkGroup = 512;                        // chunks whose slices one merge step indexes

static_assert(kHubChunk % kHubBlock == 0, "chunk must split evenly over the block");
static_assert(2 * kHubChunk <= kTabSlots, "insert table must hold every chunk entry");

__device__ __forceinline__ int hub_parts(int64_t d) {
  int64_t p = (d + kPartSize - 1) / kPartSize;
  return (int)(p < 1 ? 1 : (p > kMaxParts ? kMaxParts : p));
}

// Label mixers independent of the Fibonacci slot hash (murmur3 finalizer).
__device__ __forceinline__ uint32_t mix32(uint32_t h) {
  h ^= h >> 16;
  h *= 0x85ebca6bu;
  h ^= h >> 13;
  h *= 0xc2b2ae35u;
  h ^= h >> 16;
  return h;
}
__device__ __forceinline__ int part_of(uint32_t label, int P) {
  return (int)(((uint64_t)mix32(label) * (uint64_t)P) >> 32);
}
__device__ __forceinline__ uint32_t sub_of(uint32_t label) { return mix32(label ^ 0x9e3779b9u); }

struct HubArgs {
  const int32_t *hubs;           // hub vertex ids (NULL: hub k is vertex k)
  HubLayout L;                   // [H+1] prefix arrays
  unsigned long long *staging;   // chunk c of the batch at (c - chunk_start[k0]) * kHubChunk
  int32_t *hist;                 // partition bounds, relative to hist_start[k0]
  unsigned long long *best;      // [H] packed argmax keys
  unsigned long long *rowsum;    // [H] summed row weights
  int64_t k0, k1;                // hubs of this batch
  int merge_cap;                 // claims before a merge pass splits (1 .. kHubMergeCapMax)
};

// Exclusive scan of a[0..n) (n <= kMaxParts) in LDS by the whole block;
// a[n] receives the total.  `part` needs blockDim.x / 64 entries.  The threads'
// sums are scanned within each wavefront first: two barriers in all (with a scan
// of them in LDS, two barriers per doubling, float weights on R-MAT scale 20
// took 8.20 ms a call instead of 7.86, scale 26 224.4 instead of 223.9).
template <int BLOCK>
__device__ void block_exclusive_scan(int *a, int n, int *part) {
  const int per = (n + BLOCK - 1) / BLOCK;
  const int lo = threadIdx.x * per, hi = lo + per < n ? lo + per : n;
  const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
  int s = 0;
  for (int i = lo; i < hi; ++i) s += a[i];
  int incl = s;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int y = __shfl_up(incl, o, kWave);
    incl += lane >= o ? y : 0;
  }
  if (lane == kWave - 1) part[wid] = incl;
  __syncthreads();
  int run = incl - s;
#pragma unroll
  for (int w = 0; w < BLOCK / kWave; ++w) run += w < wid ? part[w] : 0;
  for (int i = lo; i < hi; ++i) {
    const int c = a[i];
    a[i] = run;
    run += c;
  }
  if (threadIdx.x == BLOCK - 1) a[n] = run;
  __syncthreads();
}

}  // namespace

}  // namespace gsl
