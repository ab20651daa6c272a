// Sweeps with fp32 weights summed in fp64 -- the paper's precision
// (Sec. 5.1.2: float weights, double accumulators).  The label rule is Eq. 2
// as in sweep.hip: per processed vertex the label of largest summed weight
// among its row entries (j != i), smallest label on ties; a row without such
// entries keeps its label.
//
// Same tiers, loop state, pruning and change records as the integer path;
// only the accumulation differs.  Tables keep labels and fp64 sums in two
// LDS arrays (12 bytes per slot).  The thread tier sums in CSR entry order,
// like the oracle; LDS and hub tables add with atomics, so a sum may differ
// from the entry-order sum in its last bits when weights span more than 2^29
// in magnitude -- only exact ties can then resolve differently.  Hubs (rows
// longer than the last tier) are summed chunk by chunk and merged by hash
// partition, as with whole-number weights.
#include "hub.h"

namespace gsl {

namespace {

constexpr uint32_t kEmptyKey = 0xFFFFFFFFu;

// (sum, label) pairs: larger sum first, then smaller label; label kNoLabel
// (with sum -1) is "no candidate".
__device__ __forceinline__ bool better(double w, uint32_t l, double bw, uint32_t bl) {
  if (l == kNoLabel) return false;
  return bl == kNoLabel || w > bw || (w == bw && l < bl);
}

template <int W>
__device__ __forceinline__ void shfl_best(double &w, uint32_t &l) {
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) {
    const double ow = __shfl_xor(w, o, W);
    const uint32_t ol = (uint32_t)__shfl_xor((int)l, o, W);
    if (better(ow, ol, w, l)) {
      w = ow;
      l = ol;
    }
  }
}

__device__ __forceinline__ float wf(const SweepArgs &a, int64_t p) {
  return a.w ? reinterpret_cast<const float *>(a.w)[p] : 1.0f;
}

__device__ __forceinline__ void change(const SweepArgs &a, int32_t v, uint32_t cstar, LocalCounts &lc) {
  if (a.inplace)
    __hip_atomic_store(const_cast<int32_t *>(a.C) + v, (int32_t)cstar, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  else
    a.Cn[v] = (int32_t)cstar;
  a.chg[v] = 1;
  lc.dn += 1;
}

__device__ __forceinline__ void flush(const SweepArgs &a, const LocalCounts &lc, unsigned long long *red) {
  const unsigned long long dn = block_sum(lc.dn, red);
  const unsigned long long pr = block_sum(lc.processed, red);
  const unsigned long long ed = block_sum(lc.edges, red);
  const unsigned long long mk = block_sum(lc.marked, red);
  if (threadIdx.x == 0) {
    unsigned long long *r = a.part + (size_t)blockIdx.x * kCountFields;
    r[0] = dn;
    r[1] = pr;
    r[2] = ed;
    r[3] = mk;
    r[4] = 0;  // fp64 sums do not overflow
  }
}

// Adds w to `label` in an LDS table (keys / sums, 2^log2s slots).  Returns the
// slot if this call claimed it, else -1.
__device__ __forceinline__ int lds_insert_f64(uint32_t *keys, double *sums, int log2s, uint32_t label,
                                              double w) {
  const uint32_t mask = (1u << log2s) - 1u;
  uint32_t h = slot_hash(label, log2s);
  for (;;) {
    const uint32_t prev = atomicCAS(&keys[h], kEmptyKey, label);
    if (prev == kEmptyKey || prev == label) {
      atomicAdd(&sums[h], w);
      return prev == kEmptyKey ? (int)h : -1;
    }
    h = (h + 1u) & mask;
  }
}

// Folds the label of the wavefront's first entry: the weights of its other
// entries with that label are added to it and those entries dropped (every lane
// works on the same table).  On power-law graphs most entries of a long row
// carry a few labels after the first sweeps, and each would be an atomic on
// one LDS address.
template <int K>
__device__ __forceinline__ void wave_fold_f64(uint32_t (&lab)[K], double (&wt)[K]) {
  const int lane = threadIdx.x % kWave;
  int kk = -1, leader = 0;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const unsigned long long b = __ballot(lab[k] != kNoLabel);
    if (kk < 0 && b) {
      kk = k;
      leader = __ffsll((long long)b) - 1;
    }
  }
  if (kk < 0) return;  // uniform
  uint32_t mine = kNoLabel;
#pragma unroll
  for (int k = 0; k < K; ++k) mine = k == kk ? lab[k] : mine;
  const uint32_t L = (uint32_t)__shfl((int)mine, leader);
  int count = 0;
  double sum = 0.0;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    count += __popcll(__ballot(lab[k] == L));
    sum += lab[k] == L ? wt[k] : 0.0;
  }
  if (count < 2) return;  // uniform
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) sum += __shfl_xor(sum, o, kWave);
#pragma unroll
  for (int k = 0; k < K; ++k)
    if (lab[k] == L) {
      if (lane == leader && k == kk)
        wt[k] = sum;
      else
        lab[k] = kNoLabel;
    }
}

// Tier 1: a thread per vertex, row in registers, sums in entry order.
template <int D>
__global__ __launch_bounds__(256) void sweepf_thread(SweepArgs a, const int32_t *__restrict__ list, int64_t first,
                                                     int64_t count) {
  __shared__ unsigned long long red[256 / kWave];
  SweepView sv;
  if (!sweep_view(a, sv)) return;
  LocalCounts lc;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < count; idx += stride) {
    const int32_t v = list ? list[first + idx] : (int32_t)(first + idx);
    if (!sweep_takes(a, sv, v)) continue;
    const int64_t b = a.off[v];
    const int d = (int)(a.off[v + 1] - b);
    int32_t col[D];
    uint32_t lab[D];
    double w[D];
#pragma unroll
    for (int k = 0; k < D; ++k) col[k] = k < d ? a.cols[b + k] : v;
#pragma unroll
    for (int k = 0; k < D; ++k) {
      lab[k] = col[k] != v ? (uint32_t)a.C[col[k]] : kNoLabel;
      w[k] = k < d ? (double)wf(a, b + k) : 0.0;
    }
    double bw = -1.0;
    uint32_t bl = kNoLabel;
#pragma unroll
    for (int k = 0; k < D; ++k) {
      if (lab[k] == kNoLabel) continue;
      double s = 0.0;
#pragma unroll
      for (int m = 0; m < D; ++m) s += lab[m] == lab[k] ? w[m] : 0.0;
      if (better(s, lab[k], bw, bl)) {
        bw = s;
        bl = lab[k];
      }
    }
    lc.processed += 1;
    lc.edges += (unsigned long long)d;
    if (bl != kNoLabel && bl != (uint32_t)a.C[v]) {
      change(a, v, bl, lc);
      if (sv.mark)
#pragma unroll
        for (int k = 0; k < D; ++k)
          if (k < d) {
            if (!sv.nact[col[k]]) sv.nact[col[k]] = 1;
            lc.marked += 1;
          }
    }
  }
  flush(a, lc, red);
}

// Tiers 2-7: a group of G lanes per vertex (a wave slice, or the block), K
// entries per lane, LDS keys / sums of 2^LOG2S slots per group.
template <int G, int LOG2S, int BLOCK, int K>
__global__ __launch_bounds__(BLOCK) void sweepf_lds(SweepArgs a, const int32_t *__restrict__ list, int64_t first,
                                                    int64_t count) {
  static_assert(G <= 64 || G == BLOCK, "group is a wave slice or the block");
  constexpr int GPB = BLOCK / G;
  constexpr int S = 1 << LOG2S;
  constexpr int NW = BLOCK / kWave;
  __shared__ uint32_t keys[GPB * S];
  __shared__ double sums[GPB * S];
  __shared__ double rw[NW];
  __shared__ uint32_t rl[NW];
  __shared__ unsigned long long red[NW];
  SweepView sv;
  if (!sweep_view(a, sv)) return;
  for (int s = threadIdx.x; s < GPB * S; s += BLOCK) {
    keys[s] = kEmptyKey;
    sums[s] = 0.0;
  }
  __syncthreads();
  const int g = threadIdx.x / G, lane = threadIdx.x % G;
  uint32_t *Tk = keys + g * S;
  double *Ts = sums + g * S;
  LocalCounts lc;
  for (int64_t base = (int64_t)blockIdx.x * GPB; base < count; base += (int64_t)gridDim.x * GPB) {
    const int64_t idx = base + g;
    int32_t v = -1;
    if (idx < count) {
      v = list ? list[first + idx] : (int32_t)(first + idx);
      if (!sweep_takes(a, sv, v)) v = -1;
    }
    int64_t b = 0, e = 0;
    int log2s = 1;
    if (v >= 0) {
      b = a.off[v];
      e = a.off[v + 1];
      log2s = table_log2(e - b, 1, LOG2S);
    }
    int32_t j[K];
    uint32_t lab[K];
    double wt[K];
    int slot[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int64_t p = b + lane + (int64_t)k * G;
      const bool in = p < e;
      j[k] = in ? a.cols[p] : -1;
      wt[k] = in ? (double)wf(a, p) : 0.0;
    }
#pragma unroll
    for (int k = 0; k < K; ++k) lab[k] = (j[k] >= 0 && j[k] != v) ? (uint32_t)a.C[j[k]] : kNoLabel;
    if constexpr (G >= kWave) wave_fold_f64<K>(lab, wt);  // one vertex per wave
#pragma unroll
    for (int k = 0; k < K; ++k) slot[k] = lab[k] != kNoLabel ? lds_insert_f64(Tk, Ts, log2s, lab[k], wt[k]) : -1;
    group_sync<G>();
    double bw = -1.0;
    uint32_t bl = kNoLabel;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (slot[k] < 0) continue;
      const double s = Ts[slot[k]];
      if (better(s, Tk[slot[k]], bw, bl)) {
        bw = s;
        bl = Tk[slot[k]];
      }
      Tk[slot[k]] = kEmptyKey;
      Ts[slot[k]] = 0.0;
    }
    if constexpr (G <= 64) {
      shfl_best<G>(bw, bl);
    } else {
      shfl_best<kWave>(bw, bl);
      if (threadIdx.x % kWave == 0) {
        rw[threadIdx.x / kWave] = bw;
        rl[threadIdx.x / kWave] = bl;
      }
      __syncthreads();
      bw = -1.0;
      bl = kNoLabel;
#pragma unroll
      for (int w = 0; w < NW; ++w)
        if (better(rw[w], rl[w], bw, bl)) {
          bw = rw[w];
          bl = rl[w];
        }
    }
    if (v >= 0) {
      if (lane == 0) {
        lc.processed += 1;
        lc.edges += (unsigned long long)(e - b);
      }
      if (bl != kNoLabel && bl != (uint32_t)a.C[v]) {
        if (lane == 0) change(a, v, bl, lc);
        if (sv.mark)
#pragma unroll
          for (int k = 0; k < K; ++k)
            if (j[k] >= 0) {
              if (!sv.nact[j[k]]) sv.nact[j[k]] = 1;
              lc.marked += 1;
            }
      }
    }
    group_sync<G>();
  }
  flush(a, lc, red);
}

// Hubs, as in hub.hip: a workgroup per chunk sums the chunk's labels in LDS and
// stages the distinct (label, sum) pairs by hash partition, a workgroup per
// partition (or group of them) merges what the hub's chunks staged there, and a
// wavefront per hub picks the winner of its partitions.  A global table per hub
// instead (one compare-and-swap and one fp64 add per pair, and a scan of all
// its slots by one workgroup) took 0.48 + 0.33 ms per sweep of R-MAT scale 20,
// edge factor 16 (33 M entries), against 0.09 + 0.29 + 0.02 ms here.
// Labels are staged in `labels` and sums in `sums`, both indexed like
// HubArgs::staging; won_* hold a winner per partition of the batch.
struct HubF {
  uint32_t *labels;
  double *sums;
  uint32_t *won_label;
  double *won_sum;
};
constexpr int kHubBlockF = 512;
constexpr int kHubKF = kHubChunk / kHubBlockF;
// A merge workgroup's 12-byte slots leave room for two of them per compute
// unit, so they are wide, and each lane has kMergeAhead records on the way.
constexpr int kMergeBlockF = 512;
constexpr int kMergeCapF = kTabSlots - kMergeBlockF - 1;  // a free slot always remains

// Partitions that one merge workgroup takes (see hub_merge).
__device__ __forceinline__ int hubf_group(const HubArgs &h, unsigned long long records, int P) {
  const unsigned long long fit = (unsigned long long)h.merge_cap * 3 / 4 * (unsigned long long)P;
  return records <= (unsigned long long)h.merge_cap ? P
         : (int)(fit / records < 1 ? 1 : (fit / records > (unsigned long long)P ? P : fit / records));
}

// Dynamic LDS: the partition histogram, (largest P of the batch + 1) ints.
__global__ __launch_bounds__(kHubBlockF) void hubf_insert(SweepArgs a, HubArgs h, HubF f) {
  __shared__ uint32_t keys[kTabSlots];
  __shared__ double sums[kTabSlots];
  extern __shared__ int hist[];
  __shared__ int scan_part[kHubBlockF / kWave];
  SweepView sv;
  if (!sweep_view(a, sv)) return;
  const int64_t c = h.L.chunk_start[h.k0] + blockIdx.x;
  const int64_t k = h.L.chunk_owner[c];
  const int32_t v = h.hubs ? h.hubs[k] : (int32_t)k;
  if (!sweep_takes(a, sv, v)) return;  // uniform over the block
  const int64_t rb = a.off[v], re = a.off[v + 1];
  const int P = hub_parts(re - rb);
  const int64_t cl = c - h.L.chunk_start[k];
  const int64_t b = rb + cl * kHubChunk;
  const int64_t e = b + kHubChunk < re ? b + kHubChunk : re;
  int32_t j[kHubKF];
  uint32_t lab[kHubKF];
  double wt[kHubKF];
#pragma unroll
  for (int q = 0; q < kHubKF; ++q) {
    const int64_t p = b + threadIdx.x + (int64_t)q * kHubBlockF;
    const bool in = p < e;
    j[q] = in ? a.cols[p] : -1;
    wt[q] = in ? (double)wf(a, p) : 0.0;
  }
#pragma unroll
  for (int q = 0; q < kHubKF; ++q) lab[q] = (j[q] >= 0 && j[q] != v) ? (uint32_t)a.C[j[q]] : kNoLabel;
  for (int s = threadIdx.x; s < kTabSlots; s += kHubBlockF) {
    keys[s] = kEmptyKey;
    sums[s] = 0.0;
  }
  for (int i = threadIdx.x; i <= P; i += kHubBlockF) hist[i] = 0;
  wave_fold_f64<kHubKF>(lab, wt);
  __syncthreads();  // table and histogram initialised
  int slot[kHubKF];
#pragma unroll
  for (int q = 0; q < kHubKF; ++q) slot[q] = lab[q] != kNoLabel ? lds_insert_f64(keys, sums, kTabLog2, lab[q], wt[q]) : -1;
  __syncthreads();
  int pp[kHubKF], rank[kHubKF];
#pragma unroll
  for (int q = 0; q < kHubKF; ++q) {
    pp[q] = 0;
    rank[q] = 0;
    if (slot[q] >= 0) {
      pp[q] = part_of(lab[q], P);
      rank[q] = atomicAdd(&hist[pp[q]], 1);
    }
  }
  __syncthreads();
  block_exclusive_scan<kHubBlockF>(hist, P, scan_part);
  const int64_t stage = (c - h.L.chunk_start[h.k0]) * kHubChunk;
#pragma unroll
  for (int q = 0; q < kHubKF; ++q)
    if (slot[q] >= 0) {
      f.labels[stage + hist[pp[q]] + rank[q]] = lab[q];
      f.sums[stage + hist[pp[q]] + rank[q]] = sums[slot[q]];
    }
  int32_t *gh = h.hist + (h.L.hist_start[k] - h.L.hist_start[h.k0]) + cl * (P + 1);
  for (int i = threadIdx.x; i <= P; i += kHubBlockF) gh[i] = hist[i];
  if (threadIdx.x == 0 && hist[P])
    __hip_atomic_fetch_add(&h.L.records[k], (unsigned long long)hist[P], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ __launch_bounds__(kMergeBlockF) void hubf_merge(SweepArgs a, HubArgs h, HubF f) {
  __shared__ uint32_t keys[kTabSlots];
  __shared__ double sums[kTabSlots];
  __shared__ int pre[kChunkGroup + 1], slice[kChunkGroup];
  __shared__ int scan_part[kMergeBlockF / kWave];
  __shared__ int claimed, overflow;
  __shared__ double rw[kMergeBlockF / kWave];
  __shared__ uint32_t rl[kMergeBlockF / kWave];
  SweepView sv;
  if (!sweep_view(a, sv)) return;
  const int64_t gp = h.L.part_start[h.k0] + blockIdx.x;
  const int64_t k = h.L.part_owner[gp];
  const int p = (int)(gp - h.L.part_start[k]);
  const int32_t v = h.hubs ? h.hubs[k] : (int32_t)k;
  const int P = hub_parts(a.off[v + 1] - a.off[v]);
  const int g = hubf_group(h, h.L.records[k], P);
  if ((int64_t)p * g >= P) return;  // uniform
  if (!sweep_takes(a, sv, v)) return;
  const int64_t c0 = h.L.chunk_start[k], nc = h.L.chunk_start[k + 1] - c0;
  const int32_t *gh = h.hist + (h.L.hist_start[k] - h.L.hist_start[h.k0]);
  const int64_t stage = (c0 - h.L.chunk_start[h.k0]) * kHubChunk;
  const int p_lo = p * g, p_hi = p_lo + g < P ? p_lo + g : P;  // partitions merged here
  double bw = -1.0;
  uint32_t bl = kNoLabel;
  for (uint32_t R = 1;; R <<= 1) {
    bool ok = true;
    bw = -1.0;
    bl = kNoLabel;
    for (uint32_t r = 0; r < R && ok; ++r) {
      for (int s = threadIdx.x; s < kTabSlots; s += kMergeBlockF) {
        keys[s] = kEmptyKey;
        sums[s] = 0.0;
      }
      if (threadIdx.x == 0) {
        claimed = 0;
        overflow = 0;
      }
      __syncthreads();
      for (int64_t g0 = 0; g0 < nc; g0 += kChunkGroup) {
        const int gn = (int)(nc - g0 < kChunkGroup ? nc - g0 : kChunkGroup);
        for (int i = threadIdx.x; i < gn; i += kMergeBlockF) {
          const int32_t *hc = gh + (g0 + i) * (P + 1);
          slice[i] = hc[p_lo];
          pre[i] = hc[p_hi] - slice[i];
        }
        __syncthreads();
        block_exclusive_scan<kMergeBlockF>(pre, gn, scan_part);
        const int total = pre[gn];
        for (int t0 = 0; t0 < total; t0 += kMergeAhead * kMergeBlockF) {
          uint32_t lab[kMergeAhead];
          double wt[kMergeAhead];
          int64_t at[kMergeAhead];
#pragma unroll
          for (int u = 0; u < kMergeAhead; ++u) {
            const int t = t0 + u * kMergeBlockF + threadIdx.x;
            int lo = 0, hi = gn;  // chunk i with pre[i] <= t < pre[i + 1]
            while (hi - lo > 1) {
              const int mid = (lo + hi) / 2;
              if (pre[mid] <= t)
                lo = mid;
              else
                hi = mid;
            }
            at[u] = t < total ? stage + (g0 + lo) * kHubChunk + slice[lo] + (t - pre[lo]) : -1;
          }
#pragma unroll
          for (int u = 0; u < kMergeAhead; ++u) {
            lab[u] = at[u] >= 0 ? f.labels[at[u]] : kNoLabel;
            wt[u] = at[u] >= 0 ? f.sums[at[u]] : 0.0;
          }
#pragma unroll
          for (int u = 0; u < kMergeAhead; ++u)
            if (R > 1 && lab[u] != kNoLabel && (sub_of(lab[u]) & (R - 1)) != r) lab[u] = kNoLabel;
          wave_fold_f64<kMergeAhead>(lab, wt);
#pragma unroll
          for (int u = 0; u < kMergeAhead; ++u) {
            if (lab[u] == kNoLabel) continue;
            if (__hip_atomic_load(&overflow, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) continue;
            if (__hip_atomic_load(&claimed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) >= h.merge_cap) {
              overflow = 1;
              continue;
            }
            if (lds_insert_f64(keys, sums, kTabLog2, lab[u], wt[u]) >= 0) atomicAdd(&claimed, 1);
          }
        }
        __syncthreads();
      }
      if (overflow) {
        ok = false;  // uniform: read after the barrier
      } else {
        for (int s = threadIdx.x; s < kTabSlots; s += kMergeBlockF)
          if (better(sums[s], keys[s], bw, bl)) {  // an empty key is no candidate
            bw = sums[s];
            bl = keys[s];
          }
      }
      __syncthreads();
    }
    if (ok) break;
  }
  shfl_best<kWave>(bw, bl);
  if (threadIdx.x % kWave == 0) {
    rw[threadIdx.x / kWave] = bw;
    rl[threadIdx.x / kWave] = bl;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kMergeBlockF / kWave; ++w)
      if (better(rw[w], rl[w], bw, bl)) {
        bw = rw[w];
        bl = rl[w];
      }
    f.won_sum[blockIdx.x] = bw;
    f.won_label[blockIdx.x] = bl;
  }
}

// A wavefront per hub: the winner of its merged groups and the decision.
__global__ __launch_bounds__(256) void hubf_decide(SweepArgs a, HubArgs h, HubF f) {
  __shared__ unsigned long long red[256 / kWave];
  SweepView sv;
  if (!sweep_view(a, sv)) return;
  LocalCounts lc;
  const int lane = threadIdx.x % kWave;
  const int64_t k = h.k0 + (int64_t)blockIdx.x * (256 / kWave) + threadIdx.x / kWave;
  const int32_t v = k < h.k1 ? (h.hubs ? h.hubs[k] : (int32_t)k) : -1;
  if (v >= 0 && sweep_takes(a, sv, v)) {  // uniform over the wavefront
    const int64_t d = a.off[v + 1] - a.off[v];
    const int P = hub_parts(d), g = hubf_group(h, h.L.records[k], P);
    const int64_t first = h.L.part_start[k] - h.L.part_start[h.k0];
    double bw = -1.0;
    uint32_t bl = kNoLabel;
    for (int p = lane; (int64_t)p * g < P; p += kWave)
      if (better(f.won_sum[first + p], f.won_label[first + p], bw, bl)) {
        bw = f.won_sum[first + p];
        bl = f.won_label[first + p];
      }
    shfl_best<kWave>(bw, bl);
    if (lane == 0) {
      h.L.records[k] = 0;
      lc.processed = 1;
      lc.edges = (unsigned long long)d;
      if (bl != kNoLabel && bl != (uint32_t)a.C[v]) {
        change(a, v, bl, lc);
        if (sv.mark) lc.marked = lc.edges;  // hub_mark flags the whole row
      }
    }
  }
  const unsigned long long dn = block_sum(lc.dn, red);
  const unsigned long long pr = block_sum(lc.processed, red);
  const unsigned long long ed = block_sum(lc.edges, red);
  const unsigned long long mk = block_sum(lc.marked, red);
  if (threadIdx.x == 0) {
    if (mk) atomicAdd(a.tier + 3, mk);
    if (dn) {
      atomicAdd(a.dn + sv.it, dn);
      atomicAdd(a.tier + 2, dn);
    }
    if (pr) {
      atomicAdd(a.processed + sv.it, pr);
      atomicAdd(a.tier + 0, pr);
    }
    if (ed) {
      atomicAdd(a.edges + sv.it, ed);
      atomicAdd(a.tier + 1, ed);
    }
  }
}

__global__ void check_f32(const float *__restrict__ w, int64_t nnz, unsigned long long *bad) {
  int b = 0;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < nnz; e += stride)
    b |= (w[e] >= 0.0f && w[e] <= 3.4e38f) ? 0 : 1;
  if (__ballot(b) && threadIdx.x % kWave == 0) atomicOr(bad, 1ull);
}

int grid_f(int64_t items, int per_block) {
  int64_t g = (items + per_block - 1) / per_block;
  if (g < 1) g = 1;
  return (int)(g > kMaxTierGrid ? kMaxTierGrid : g);
}

}  // namespace

// Tiers 1-7 with the default bounds (8/16/32/64/128/512/2048).
hipError_t launch_sweep_tier_f32(int tier, const SweepArgs &a, const int32_t *list, int64_t first, int64_t count,
                                 int *grid_out, hipStream_t s) {
  *grid_out = 0;
  if (count <= 0) return hipSuccess;
  int grid = 0;
  switch (tier) {
    case 1:
      grid = grid_f(count, 256);
      sweepf_thread<8><<<grid, 256, 0, s>>>(a, list, first, count);
      break;
    case 2:
      grid = grid_f(count, 256 / 8);
      sweepf_lds<8, 5, 256, 2><<<grid, 256, 0, s>>>(a, list, first, count);
      break;
    case 3:
      grid = grid_f(count, 256 / 16);
      sweepf_lds<16, 6, 256, 2><<<grid, 256, 0, s>>>(a, list, first, count);
      break;
    case 4:
      grid = grid_f(count, 256 / 32);
      sweepf_lds<32, 7, 256, 2><<<grid, 256, 0, s>>>(a, list, first, count);
      break;
    case 5:
      grid = grid_f(count, 256 / 64);
      sweepf_lds<64, 8, 256, 2><<<grid, 256, 0, s>>>(a, list, first, count);
      break;
    case 6:
      grid = grid_f(count, 256 / 64);
      sweepf_lds<64, 10, 256, 8><<<grid, 256, 0, s>>>(a, list, first, count);
      break;
    case 7:
      grid = grid_f(count, 1);
      sweepf_lds<256, 12, 256, 8><<<grid, 256, 0, s>>>(a, list, first, count);
      break;
    default:
      return hipErrorInvalidValue;
  }
  *grid_out = grid;
  return hipGetLastError();
}

hipError_t launch_hub_f32(const SweepArgs &a, const int32_t *hubs, HubLayout L, const int64_t *chunk_start_h,
                          const int64_t *part_start_h, unsigned long long *staging, int32_t *hist, uint32_t *labels,
                          double *won, int64_t k0, int64_t k1, int max_parts, int merge_cap, int stage, hipStream_t s) {
  if (k1 <= k0) return hipSuccess;
  if (merge_cap < 1 || merge_cap > kHubMergeCapMax) return hipErrorInvalidValue;
  const int64_t chunks = chunk_start_h[k1] - chunk_start_h[k0], parts = part_start_h[k1] - part_start_h[k0];
  HubArgs h{hubs, L, nullptr, hist, nullptr, nullptr, k0, k1, merge_cap < kMergeCapF ? merge_cap : kMergeCapF};
  HubF f{labels, reinterpret_cast<double *>(staging), labels + chunks * kHubChunk, won};
  if (stage == 0) {
    hubf_insert<<<(unsigned)chunks, kHubBlockF, (size_t)(max_parts + 1) * sizeof(int), s>>>(a, h, f);
    return hipGetLastError();
  }
  hubf_merge<<<(unsigned)parts, kMergeBlockF, 0, s>>>(a, h, f);
  hubf_decide<<<(unsigned)((k1 - k0 + 3) / 4), 256, 0, s>>>(a, h, f);
  return launch_hub_mark(a, hubs, L, chunk_start_h, k0, k1, s);
}

hipError_t launch_check_f32(const float *w, int64_t nnz, unsigned long long *bad, hipStream_t s) {
  if (nnz <= 0) return hipSuccess;
  check_f32<<<grid_f(nnz, 256 * 4), 256, 0, s>>>(w, nnz, bad);
  return hipGetLastError();
}

}  // namespace gsl
