// Degree-ordered renumbering of the graph.
//
// The plan's list orders the vertices hubs first and isolated vertices last;
// new id p stands for old vertex list[p].  A renumbered copy of the CSR lets
// every tier kernel walk a contiguous id range (coalesced offsets, rows and
// flags) and packs the labels of the highest-degree vertices -- the targets of
// most label gathers -- into a few megabytes that stay in L2.  Labels keep
// their original-id values, so the smallest-label tie-break and the output are
// unchanged; only storage positions move.
//
// Graphs of short rows whose neighbours lie far apart in the caller's ids are
// renumbered too, for another reason: every label gather of such a graph
// misses L2 (see launch_cluster_order).
#include "device_common.h"
#include "gsl_internal.h"

namespace gsl {

namespace {

constexpr int kScanBlock = 1024;

__global__ void reorder_invert(const int32_t *__restrict__ list, int64_t first, int64_t end,
                               int32_t *__restrict__ old2new) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t p = first + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < end; p += stride)
    old2new[list[p]] = (int32_t)p;
}

// off2[p + 1] = degree of list[p] for the np non-isolated rows; off2[0] = 0.
// Also the initial labels of all n vertices (an isolated vertex keeps its
// own, even where an entry of a graph that is not symmetric names it).
// Positions [row0, row0 + nrows) that cluster_place described in `rows` come
// from there, their list entries included.
__global__ void reorder_degrees(const int64_t *__restrict__ off, int32_t *list, int64_t np, int64_t n,
                                const ClusterRow *__restrict__ rows, int64_t row0, int64_t nrows,
                                int64_t *__restrict__ off2, int32_t *__restrict__ lab) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += stride) {
    int32_t v;
    if (p >= row0 && p < row0 + nrows) {
      const ClusterRow r = rows[p - row0];
      v = r.v;
      list[p] = v;
      off2[p + 1] = r.d;
    } else {
      v = list[p];
      if (p < np) off2[p + 1] = off[v + 1] - off[v];
    }
    lab[p] = v;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) off2[0] = 0;
}

// In-place inclusive scan of a[0..n): per-block scan, block totals to sums.
template <class T>
__global__ __launch_bounds__(kScanBlock) void scan_local(T *a, int64_t n, int64_t *sums) {
  __shared__ int64_t part[kScanBlock];
  const int64_t i = (int64_t)blockIdx.x * kScanBlock + threadIdx.x;
  part[threadIdx.x] = i < n ? a[i] : 0;
  __syncthreads();
  for (int o = 1; o < kScanBlock; o <<= 1) {
    const int64_t y = threadIdx.x >= o ? part[threadIdx.x - o] : 0;
    __syncthreads();
    part[threadIdx.x] += y;
    __syncthreads();
  }
  if (i < n) a[i] = (T)part[threadIdx.x];
  if (threadIdx.x == kScanBlock - 1) sums[blockIdx.x] = part[kScanBlock - 1];
}

// Exclusive scan of sums[0..nb) in one block.
__global__ __launch_bounds__(kScanBlock) void scan_sums(int64_t *sums, int64_t nb) {
  __shared__ int64_t part[kScanBlock];
  const int64_t per = (nb + kScanBlock - 1) / kScanBlock;
  const int64_t lo = threadIdx.x * per, hi = lo + per < nb ? lo + per : nb;
  int64_t s = 0;
  for (int64_t b = lo; b < hi; ++b) s += sums[b];
  part[threadIdx.x] = s;
  __syncthreads();
  for (int o = 1; o < kScanBlock; o <<= 1) {
    const int64_t y = threadIdx.x >= o ? part[threadIdx.x - o] : 0;
    __syncthreads();
    part[threadIdx.x] += y;
    __syncthreads();
  }
  int64_t run = threadIdx.x > 0 ? part[threadIdx.x - 1] : 0;
  for (int64_t b = lo; b < hi; ++b) {
    const int64_t c = sums[b];
    sums[b] = run;
    run += c;
  }
}

template <class T>
__global__ __launch_bounds__(kScanBlock) void scan_add(T *a, int64_t n, const int64_t *sums) {
  const int64_t i = (int64_t)blockIdx.x * kScanBlock + threadIdx.x;
  if (i < n) a[i] += (T)sums[blockIdx.x];
}

template <class T>
void scan_inclusive(T *a, int64_t n, int64_t *sums, hipStream_t s) {
  const int64_t nb = (n + kScanBlock - 1) / kScanBlock;
  scan_local<T><<<(unsigned)nb, kScanBlock, 0, s>>>(a, n, sums);
  scan_sums<<<1, kScanBlock, 0, s>>>(sums, nb);
  scan_add<T><<<(unsigned)nb, kScanBlock, 0, s>>>(a, n, sums);
}

// ---- cluster order of the short rows (launch_cluster_order) ----

// Two entries of each of up to kSpreadSamples vertices spread over
// the graph (not the ends of the row: sorted rows have their farthest there).
constexpr int64_t kSpreadSamples = 1 << 16;
__global__ __launch_bounds__(256) void sample_spread(const int64_t *__restrict__ off, const int32_t *__restrict__ cols,
                                                     int64_t n, int64_t samples, unsigned long long *out) {
  __shared__ unsigned long long red[256 / kWave];
  unsigned long long seen = 0, far = 0, near = 0;
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < samples) {
    const int64_t v = (int64_t)((unsigned long long)k * (unsigned long long)n / (unsigned long long)samples);
    const int64_t b = off[v], e = off[v + 1];
    if (e > b) {
      const int64_t p = cols[b + (e - b) / 4], q = cols[b + (e - b) * 3 / 4];
      const int64_t x = p > v ? p - v : v - p, y = q > v ? q - v : v - q;
      seen = 2;
      far = (x > kSpreadFar) + (y > kSpreadFar);
      near = (x <= kSpreadNear) + (y <= kSpreadNear);
    }
  }
  seen = block_sum(seen, red);
  far = block_sum(far, red);
  near = block_sum(near, red);
  if (threadIdx.x == 0 && seen) {
    atomicAdd(&out[0], seen);
    atomicAdd(&out[1], far);
    atomicAdd(&out[2], near);
  }
}

// first[v] = smallest neighbour of v (v itself without one), count cleared.
__global__ __launch_bounds__(256) void cluster_first(const int64_t *__restrict__ off,
                                                     const int32_t *__restrict__ cols, int64_t n, int64_t longest,
                                                     int32_t *__restrict__ first, int32_t *__restrict__ count) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) {
    const int64_t b = off[v], e = off[v + 1];
    int32_t m = 0x7fffffff;
    if (e - b <= longest)
      for (int64_t p = b; p < e; ++p) {
        const int32_t j = cols[p];
        m = j != (int32_t)v && j < m ? j : m;
      }
    first[v] = m == 0x7fffffff ? (int32_t)v : m;
    count[v] = 0;
  }
}

// The cluster of v -- the smaller of its smallest neighbour and that one's.
__device__ __forceinline__ int32_t cluster_of(const int64_t *__restrict__ off, int64_t longest,
                                              const int32_t *__restrict__ first, int64_t v) {
  const int64_t d = off[v + 1] - off[v];
  if (d <= 0 || d > longest) return -1;
  const int32_t m = first[v], mm = first[m];
  return mm < m ? mm : m;
}

// The clusters and every vertex's rank in its own (any order will do): where all
// rows are short, and so are the clusters, with an atomic per vertex.
__global__ __launch_bounds__(256) void cluster_rank(const int64_t *__restrict__ off, int64_t n, int64_t longest,
                                                    const int32_t *__restrict__ first, int32_t *__restrict__ cluster,
                                                    int32_t *__restrict__ rank, int32_t *count) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) {
    const int32_t c = cluster_of(off, longest, first, v);
    cluster[v] = c;
    if (c >= 0) rank[v] = atomicAdd(&count[c], 1);
  }
}

// The same where a long row may lend its vertex's id to all that it names: the
// vertices of a workgroup that share a cluster are counted in an LDS table
// first, one atomic on the cluster's counter for all of them (stars of 3 M and 20
// M vertices: 37.6 and 252 ms a call with an atomic each, 3.5 and 24.8 here, 4.4
// and 29.8 in the caller's order; 24 M road vertices would take 14.87 ms instead
// of 14.57).
constexpr int kRankBlock = 1024;
constexpr int kRankTableLog2 = 11, kRankTable = 1 << kRankTableLog2;
static_assert(kRankTable >= 2 * kRankBlock, "two slots per vertex of the block");
__global__ __launch_bounds__(kRankBlock) void cluster_rank_hubs(const int64_t *__restrict__ off, int64_t n, int64_t longest,
                                                                const int32_t *__restrict__ first,
                                                                int32_t *__restrict__ cluster,
                                                                int32_t *__restrict__ rank, int32_t *count) {
  __shared__ uint32_t key[kRankTable];
  __shared__ int32_t num[kRankTable];  // vertices of the slot's cluster, then their first rank
  for (int64_t v0 = (int64_t)blockIdx.x * kRankBlock; v0 < n; v0 += (int64_t)gridDim.x * kRankBlock) {
    for (int q = threadIdx.x; q < kRankTable; q += kRankBlock) {
      key[q] = kNoLabel;
      num[q] = 0;
    }
    const int64_t v = v0 + threadIdx.x;
    int32_t c = -1;
    if (v < n) cluster[v] = c = cluster_of(off, longest, first, v);
    __syncthreads();
    uint32_t h = 0;
    int32_t at = 0;
    if (c >= 0) {
      h = slot_hash((uint32_t)c, kRankTableLog2);
      for (;;) {  // at most kRankBlock clusters: a free slot remains
        const uint32_t prev = atomicCAS(&key[h], kNoLabel, (uint32_t)c);
        if (prev == kNoLabel || prev == (uint32_t)c) break;
        h = (h + 1) & (kRankTable - 1);
      }
      at = atomicAdd(&num[h], 1);
    }
    __syncthreads();
    for (int q = threadIdx.x; q < kRankTable; q += kRankBlock)
      if (key[q] != kNoLabel) num[q] = atomicAdd(&count[key[q]], num[q]);
    __syncthreads();
    if (c >= 0) rank[v] = num[h] + at;
    __syncthreads();  // the table is cleared next
  }
}

// The short rows at their positions (one 16-byte record each: the list, the
// degrees and the copy then read them in order instead of gathering offsets by
// vertex) and the inverse of the list; end[c] is the end of cluster c.
__global__ __launch_bounds__(256) void cluster_place(const int64_t *__restrict__ off, const int32_t *__restrict__ cluster,
                                                     const int32_t *__restrict__ rank,
                                                     const int32_t *__restrict__ end, int64_t n, int64_t start,
                                                     ClusterRow *__restrict__ rows, int32_t *__restrict__ old2new) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) {
    const int32_t c = cluster[v];
    if (c < 0) continue;
    const int64_t q = end[c] - 1 - rank[v], b = off[v];
    rows[q] = ClusterRow{b, (int32_t)v, (int32_t)(off[v + 1] - b)};
    old2new[v] = (int32_t)(start + q);
  }
}

struct CopyArgs {
  const int64_t *off;
  const int32_t *cols;
  const uint32_t *w;
  bool f32;  // w holds floats: as bits they order like their values, but for a negative zero
  const int32_t *list;
  const int32_t *old2new;
  const int64_t *off2;
  int32_t *cols2;
  uint32_t *w2;
  const ClusterRow *rows;  // the launch's rows, or NULL: through list and off
  // First sweep, folded into the copy: while the labels are still the vertex
  // ids, a row without duplicate entries holds every label once, so its winner
  // is the heaviest entry (smallest id on ties) -- no table, no label gather.
  unsigned long long *first_key;   // per new row: packed argmax key (0: none)
  unsigned long long *hub_rowsum;  // per hub: summed row weight
  unsigned long long *flags;       // bit 0: a row is not strictly increasing
                                   // bit 1: a row's weight sum reaches 2^32
};

// Rows [first, first + count) of the new numbering, G lanes per row (G <= 64
// or the whole block), each lane owning at most K entries of the row (the
// tier bound is G * K) with all its loads issued before any use.
template <int G, int BLOCK, int K>
__global__ __launch_bounds__(BLOCK) void reorder_rows(CopyArgs c, int64_t first, int64_t count) {
  constexpr int GPB = BLOCK / G;
  __shared__ unsigned long long red[BLOCK / kWave], red2[BLOCK / kWave];
  const int g = threadIdx.x / G, lane = threadIdx.x % G;
  int unsorted = 0, ovf = 0;
  for (int64_t base = (int64_t)blockIdx.x * GPB; base < count; base += (int64_t)gridDim.x * GPB) {
    const int64_t idx = base + g;
    unsigned long long best = 0, rowsum = 0;
    int64_t p = -1, b = 0, e = 0, b2 = 0;
    int32_t v = -1;
    if (idx < count) {
      p = first + idx;
      b2 = c.off2[p];
      if (c.rows) {
        const ClusterRow r = c.rows[idx];
        v = r.v;
        b = r.b;
        e = b + r.d;
      } else {
        v = c.list[p];
        b = c.off[v];
        e = c.off[v + 1];
      }
    }
    int32_t j[K], jn[K];
    uint32_t w[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int64_t q = b + lane + (int64_t)k * G;
      const bool in = q < e;
      j[k] = in ? c.cols[q] : -1;
      jn[k] = in && q + 1 < e ? c.cols[q + 1] : 0x7fffffff;
      w[k] = in ? (c.w ? c.w[q] : 1u) : 0u;
    }
    // every old->new lookup is issued before the first store (a store could
    // alias a later lookup's address as far as the compiler knows, which
    // would keep one random gather in flight per lane)
    int32_t nj[K];
#pragma unroll
    for (int k = 0; k < K; ++k) nj[k] = j[k] >= 0 ? c.old2new[j[k]] : 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (j[k] < 0) continue;
      const int64_t q = b + lane + (int64_t)k * G;
      c.cols2[b2 + (q - b)] = nj[k];
      if (c.w) c.w2[b2 + (q - b)] = w[k];
      unsorted |= jn[k] <= j[k];
      rowsum += w[k];
      if (j[k] != v) {
        const unsigned long long key = argmax_key((uint32_t)j[k], c.f32 && w[k] == 0x80000000u ? 0u : w[k]);
        best = key > best ? key : best;
      }
    }
    if constexpr (G <= 64) {
      best = group_max<G>(best);
      rowsum = group_sum<G>(rowsum);
    } else {
      best = group_max<kWave>(best);
      rowsum = wave_sum(rowsum);
      if (threadIdx.x % kWave == 0) {
        red[threadIdx.x / kWave] = best;
        red2[threadIdx.x / kWave] = rowsum;
      }
      __syncthreads();
      best = 0;
      rowsum = 0;
      for (int ww = 0; ww < BLOCK / kWave; ++ww) {
        best = red[ww] > best ? red[ww] : best;
        rowsum += red2[ww];
      }
      __syncthreads();
    }
    if (p >= 0 && lane == 0) {
      c.first_key[p] = best;
      ovf |= rowsum >> 32 ? 1 : 0;
    }
  }
  const int any_unsorted = __syncthreads_or(unsorted);
  const int any_ovf = __syncthreads_or(ovf);
  if (threadIdx.x == 0 && (any_unsorted || any_ovf))
    atomicOr(c.flags, (unsigned long long)(any_unsorted ? 1 : 0) | (any_ovf ? 2 : 0));
}

// Hub rows in chunks of kHubChunk entries, one block per chunk; chunk_start
// and chunk_owner are the hub layout (hubs = new ids 0..H-1).  Each lane
// loads its kChunk / 256 entries, then issues all their old->new lookups,
// then stores.  The first-sweep key and weight sum of a hub are combined
// across its chunks.
constexpr int kChunk = kHubChunk;
constexpr int kChunkPerLane = kChunk / 256;
__global__ __launch_bounds__(256) void reorder_hub_rows(CopyArgs c, const int64_t *chunk_start,
                                                        const int32_t *chunk_owner) {
  __shared__ unsigned long long red[256 / kWave], red2[256 / kWave];
  const int64_t ch = blockIdx.x;
  const int64_t p = chunk_owner[ch];
  const int32_t v = c.list[p];
  const int64_t rb = c.off[v], re = c.off[v + 1], b2 = c.off2[p];
  const int64_t b = rb + (ch - chunk_start[p]) * kChunk;
  const int64_t e = b + kChunk < re ? b + kChunk : re;
  unsigned long long best = 0, rowsum = 0;
  int unsorted = 0;
  int32_t j[kChunkPerLane], jn[kChunkPerLane], nj[kChunkPerLane];
  uint32_t w[kChunkPerLane];
#pragma unroll
  for (int k = 0; k < kChunkPerLane; ++k) {
    const int64_t q = b + threadIdx.x + (int64_t)k * 256;
    const bool in = q < e;
    j[k] = in ? c.cols[q] : -1;
    jn[k] = in && q + 1 < re ? c.cols[q + 1] : 0x7fffffff;
    w[k] = in ? (c.w ? c.w[q] : 1u) : 0u;
  }
#pragma unroll
  for (int k = 0; k < kChunkPerLane; ++k) nj[k] = j[k] >= 0 ? c.old2new[j[k]] : 0;
#pragma unroll
  for (int k = 0; k < kChunkPerLane; ++k) {
    if (j[k] < 0) continue;
    const int64_t q = b + threadIdx.x + (int64_t)k * 256;
    c.cols2[b2 + (q - rb)] = nj[k];
    if (c.w) c.w2[b2 + (q - rb)] = w[k];
    unsorted |= jn[k] <= j[k];
    rowsum += w[k];
    if (j[k] != v) {
      const unsigned long long key = argmax_key((uint32_t)j[k], c.f32 && w[k] == 0x80000000u ? 0u : w[k]);
      best = key > best ? key : best;
    }
  }
  best = group_max<kWave>(best);
  rowsum = wave_sum(rowsum);
  if (threadIdx.x % kWave == 0) {
    red[threadIdx.x / kWave] = best;
    red2[threadIdx.x / kWave] = rowsum;
  }
  const int any_unsorted = __syncthreads_or(unsorted);
  if (threadIdx.x == 0) {
    for (int w = 1; w < 256 / kWave; ++w) {
      red[0] = red[w] > red[0] ? red[w] : red[0];
      red2[0] += red2[w];
    }
    if (red[0]) __hip_atomic_fetch_max(&c.first_key[p], red[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (red2[0]) __hip_atomic_fetch_add(&c.hub_rowsum[p], red2[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (any_unsorted) atomicOr(c.flags, 1ull);
  }
}

// Applies the folded first sweep (if `apply` and no row failed the strict
// increase test): lab[p] becomes the winner of row p, changes are counted into
// *dn.  Hub weight sums are always checked (bit 1 of flags) and reset.
__global__ __launch_bounds__(256) void first_apply(const unsigned long long *__restrict__ first_key,
                                                   const int32_t *__restrict__ orig, int64_t np,
                                                   unsigned long long *hub_rowsum, int64_t H,
                                                   unsigned long long *flags, int32_t *lab,
                                                   unsigned long long *dn, int apply) {
  __shared__ unsigned long long red[256 / kWave];
  const bool skip = !apply || (*flags & 1ull) != 0;  // uniform
  unsigned long long changes = 0;
  int ovf = 0;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < np; p += stride) {
    if (p < H) {
      ovf |= hub_rowsum[p] >> 32 ? 1 : 0;
      hub_rowsum[p] = 0;
    }
    if (skip) continue;
    const unsigned long long key = first_key[p];
    if (key) {
      const uint32_t cstar = key_label(key);
      if ((int32_t)cstar != orig[p]) {
        lab[p] = (int32_t)cstar;
        changes += 1;
      }
    }
  }
  const unsigned long long t = block_sum(changes, red);
  const int any_ovf = __syncthreads_or(ovf);
  if (threadIdx.x == 0) {
    if (t) atomicAdd(dn, t);
    if (any_ovf) atomicOr(flags, 2ull);
  }
}

// Output in old ids: out[list[p]] = val[p] for p < np, out[list[p]] = list[p]
// for the isolated vertices p >= np.
__global__ void reorder_scatter(const int32_t *__restrict__ list, const int32_t *__restrict__ val,
                                int64_t np, int64_t n, int32_t *__restrict__ out) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += stride) {
    const int32_t v = list[p];
    out[v] = p < np ? val[p] : v;
  }
}

int grid_of(int64_t items, int per_block, int cap) {
  int64_t g = (items + per_block - 1) / per_block;
  if (g < 1) g = 1;
  return (int)(g > cap ? cap : g);
}

}  // namespace

// Renumbered CSR (off2, cols2, w2) of the np non-isolated vertices and their
// initial labels lab[p] = list[p].  scan_tmp needs plan_blocks(np) + 1 entries.
hipError_t launch_reorder(const int64_t *off, const int32_t *cols, const uint32_t *w, int64_t n,
                          int32_t *list, const int64_t *tier_count_h, const int64_t *tier_start_h,
                          const int64_t *hub_chunk_start, const int32_t *hub_chunk_owner, int64_t hub_chunks,
                          int32_t *old2new, int64_t *off2, int32_t *cols2, uint32_t *w2, int32_t *lab,
                          int64_t *scan_tmp, unsigned long long *first_key,
                          unsigned long long *hub_rowsum, unsigned long long *flags,
                          unsigned long long *dn0, int apply_first, const TierConfig &cfg, int64_t max_degree,
                          const ClusterRow *rows, bool f32, hipStream_t s) {
  const int64_t np = n - tier_count_h[0];
  constexpr int kCap = 256 * 32;
  if (!rows) reorder_invert<<<grid_of(n, 256, kCap), 256, 0, s>>>(list, 0, n, old2new);
  reorder_degrees<<<grid_of(n, 256, kCap), 256, 0, s>>>(off, list, np, n, rows, tier_start_h[1], rows ? tier_count_h[1] : 0,
                                                        off2, lab);
  if (np > 0) scan_inclusive(off2 + 1, np, scan_tmp, s);
  CopyArgs c{off, cols, w, f32, list, old2new, off2, cols2, w2, nullptr, first_key, hub_rowsum, flags};
  const int64_t H = tier_count_h[kNumTiers - 1];
  if (H > 0) launch_fill_u64(reinterpret_cast<uint64_t *>(first_key), 0, H, s);
  for (int t = 1; t < kNumTiers; ++t) {
    const int64_t cnt = tier_count_h[t], first = tier_start_h[t];
    if (cnt <= 0) continue;
    // the copy kernel takes rows up to G * K entries: the smallest that
    // covers the tier's degree bound (and the graph's longest row)
    const int64_t d = cfg.bound[t] < max_degree ? cfg.bound[t] : max_degree;
    c.rows = t == 1 ? rows : nullptr;
    if (t == kNumTiers - 1) {
      if (hub_chunks > 0)
        reorder_hub_rows<<<(unsigned)hub_chunks, 256, 0, s>>>(c, hub_chunk_start, hub_chunk_owner);
    } else if (d <= 8) {
      reorder_rows<1, 256, 8><<<grid_of(cnt, 256, kCap), 256, 0, s>>>(c, first, cnt);
    } else if (d <= 16) {
      reorder_rows<8, 256, 2><<<grid_of(cnt, 32, kCap), 256, 0, s>>>(c, first, cnt);
    } else if (d <= 32) {
      reorder_rows<16, 256, 2><<<grid_of(cnt, 16, kCap), 256, 0, s>>>(c, first, cnt);
    } else if (d <= 64) {
      reorder_rows<32, 256, 2><<<grid_of(cnt, 8, kCap), 256, 0, s>>>(c, first, cnt);
    } else if (d <= 128) {
      reorder_rows<64, 256, 2><<<grid_of(cnt, 4, kCap), 256, 0, s>>>(c, first, cnt);
    } else if (d <= 512) {
      reorder_rows<64, 256, 8><<<grid_of(cnt, 4, kCap), 256, 0, s>>>(c, first, cnt);
    } else if (d <= 2048) {
      reorder_rows<256, 256, 8><<<grid_of(cnt, 1, kCap), 256, 0, s>>>(c, first, cnt);
    } else {
      reorder_rows<1024, 1024, 8><<<grid_of(cnt, 1, kCap), 1024, 0, s>>>(c, first, cnt);
    }
  }
  if (np > 0)
    first_apply<<<grid_of(np, 256, 1024), 256, 0, s>>>(first_key, list, np, hub_rowsum, H, flags, lab, dn0,
                                                       apply_first);
  return hipGetLastError();
}

hipError_t launch_spread(const int64_t *off, const int32_t *cols, int64_t n, uint64_t *out, hipStream_t s) {
  const int64_t samples = n < kSpreadSamples ? n : kSpreadSamples;
  if (samples <= 0) return hipSuccess;
  sample_spread<<<grid_of(samples, 256, 1 << 20), 256, 0, s>>>(off, cols, n, samples,
                                                               reinterpret_cast<unsigned long long *>(out));
  return hipGetLastError();
}

hipError_t launch_cluster_order(const int64_t *off, const int32_t *cols, int64_t n, const int64_t *tier_count_h,
                                const int64_t *tier_start_h, int64_t longest, int64_t max_degree, int32_t *first,
                                int32_t *cluster, int32_t *rank, int32_t *count, int64_t *scan_tmp,
                                const int32_t *list, ClusterRow *rows, int32_t *old2new, hipStream_t s) {
  constexpr int kCap = 256 * 32;
  const int g = grid_of(n, 256, kCap);
  cluster_first<<<g, 256, 0, s>>>(off, cols, n, longest, first, count);
  if (max_degree > longest)
    cluster_rank_hubs<<<grid_of(n, kRankBlock, kCap), kRankBlock, 0, s>>>(off, n, longest, first, cluster, rank, count);
  else
    cluster_rank<<<g, 256, 0, s>>>(off, n, longest, first, cluster, rank, count);
  scan_inclusive(count, n, scan_tmp, s);
  cluster_place<<<g, 256, 0, s>>>(off, cluster, rank, count, n, tier_start_h[1], rows, old2new);
  // the other tiers keep their order: the list's ranges before and after tier 1
  const int64_t before = tier_start_h[1], after = tier_start_h[1] + tier_count_h[1];
  if (before > 0) reorder_invert<<<grid_of(before, 256, kCap), 256, 0, s>>>(list, 0, before, old2new);
  if (after < n) reorder_invert<<<grid_of(n - after, 256, kCap), 256, 0, s>>>(list, after, n, old2new);
  return hipGetLastError();
}

hipError_t launch_reorder_scatter(const int32_t *list, const int32_t *val, int64_t np, int64_t n,
                                  int32_t *out, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  reorder_scatter<<<grid_of(n, 256, 256 * 32), 256, 0, s>>>(list, val, np, n, out);
  return hipGetLastError();
}

}  // namespace gsl
