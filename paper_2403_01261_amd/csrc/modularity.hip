// Modularity of a labelling (Eq. 1, second form) with exact integer sums.
//
//   2m      = sum of w over all CSR entries
//   I       = sum of w over entries (i, j) with C_i == C_j      (= sum_c sigma_c)
//   Sigma_c = sum of w over entries (i, j) with C_i == c
//   S2      = sum_c Sigma_c^2                                    (128-bit)
//   Q       = I / 2m - S2 / (2m)^2, each operation IEEE double, round to nearest
//
// Integer sums are order independent, so Q does not depend on the schedule.
#include "device_common.h"
#include "gsl_internal.h"

namespace gsl {

namespace {

constexpr int kModBlock = 256;
constexpr int kShortRow = 32;
constexpr int kFinishBlock = 1024;

// Strength and intra-community weight of the entries [b, e) that start at this
// lane and lie `step` apart, kModAhead of them on the way at once: a long row is
// a chain of column and label loads otherwise.
constexpr int kModAhead = 8;
__device__ __forceinline__ void mod_entries(const int32_t *__restrict__ cols, const uint32_t *__restrict__ w,
                                            const int32_t *__restrict__ C, int64_t b, int64_t e, int64_t step, int32_t c,
                                            unsigned long long &k, unsigned long long &in) {
  for (int64_t p0 = b; p0 < e; p0 += kModAhead * step) {
    int32_t j[kModAhead];
    uint32_t we[kModAhead];
#pragma unroll
    for (int u = 0; u < kModAhead; ++u) {
      const int64_t p = p0 + u * step;
      j[u] = p < e ? cols[p] : -1;
      we[u] = p < e ? (w ? w[p] : 1u) : 0u;
    }
    bool same[kModAhead];
#pragma unroll
    for (int u = 0; u < kModAhead; ++u) same[u] = j[u] >= 0 && C[j[u]] == c;
#pragma unroll
    for (int u = 0; u < kModAhead; ++u) {
      k += we[u];
      in += same[u] ? we[u] : 0u;
    }
  }
}

// Per vertex: K_i and the intra-community weight.  Rows up to kShortRow are
// scanned by their own thread; longer rows are collected by ballot and scanned
// by the whole wavefront, those above kHugeRow by the workgroup.
constexpr int kHugeRow = 4096;
constexpr int kModTableLog2 = 9, kModTable = 1 << kModTableLog2;
static_assert(kModTable >= 2 * kModBlock, "two slots per vertex of the block");
__global__ __launch_bounds__(kModBlock) void mod_rows(const int64_t *__restrict__ off,
                                                      const int32_t *__restrict__ cols,
                                                      const uint32_t *__restrict__ w, int64_t n,
                                                      const int32_t *__restrict__ C,
                                                      unsigned long long *sigma_tot, Counters *ctr) {
  __shared__ unsigned long long red[kModBlock / kWave];
  __shared__ int64_t huge[kModBlock];
  __shared__ int huge_n;
  const int lane = threadIdx.x % kWave;
  unsigned long long my_two_m = 0, my_intra = 0;
  // Strengths of the communities of a block's vertices meet in an LDS table
  // first: where many vertices share a community an atomic on its sum for each
  // of them serialises (R-MAT scale 20, 33 M weighted entries, took 8.5 ms for
  // both quality measures, planted with 1 M vertices in 100 blocks 5.1 ms; 0.93
  // and 0.75 ms now).
  __shared__ uint32_t key[kModTable];
  __shared__ unsigned long long sum[kModTable];
  for (int q = threadIdx.x; q < kModTable; q += kModBlock) {
    key[q] = kNoLabel;
    sum[q] = 0;
  }
  auto strength = [&](int32_t c, unsigned long long k) {
    if (!k) return;
    uint32_t h = slot_hash((uint32_t)c, kModTableLog2);
    for (;;) {  // at most kModBlock communities: a free slot remains
      const uint32_t prev = atomicCAS(&key[h], kNoLabel, (uint32_t)c);
      if (prev == kNoLabel || prev == (uint32_t)c) break;
      h = (h + 1) & (kModTable - 1);
    }
    atomicAdd(&sum[h], k);
  };
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t base = (int64_t)blockIdx.x * blockDim.x; base < n; base += stride) {
    if (threadIdx.x == 0) huge_n = 0;
    __syncthreads();
    const int64_t v = base + threadIdx.x;
    int64_t b = 0, e = 0;
    int32_t c = 0;
    if (v < n) {
      b = off[v];
      e = off[v + 1];
      c = C[v];
    }
    const bool longrow = v < n && e - b > kShortRow;
    if (v < n && !longrow) {
      unsigned long long k = 0, in = 0;
      for (int64_t p = b; p < e; ++p) {
        const unsigned long long we = w ? w[p] : 1u;
        k += we;
        if (C[cols[p]] == c) in += we;
      }
      my_two_m += k;
      my_intra += in;
      strength(c, k);
    }
    if (longrow && e - b > kHugeRow) huge[atomicAdd(&huge_n, 1)] = v;
    unsigned long long pending = __ballot(longrow && e - b <= kHugeRow);
    while (pending) {
      const int src = __ffsll((long long)pending) - 1;
      pending &= pending - 1;
      const int64_t vb = __shfl(b, src, kWave), ve = __shfl(e, src, kWave);
      const int32_t vc = __shfl(c, src, kWave);
      unsigned long long k = 0, in = 0;
      if (ve - vb <= kWave) {  // one entry a lane: nothing to have on the way
        const int64_t p = vb + lane;
        const int32_t j = p < ve ? cols[p] : -1;
        const uint32_t we = p < ve ? (w ? w[p] : 1u) : 0u;
        k = we;
        in = j >= 0 && C[j] == vc ? we : 0u;
      } else {
        mod_entries(cols, w, C, vb + lane, ve, kWave, vc, k, in);
      }
      k = wave_sum(k);
      in = wave_sum(in);
      if (lane == 0) {
        my_two_m += k;
        my_intra += in;
        strength(vc, k);
      }
    }
    __syncthreads();
    const int rows = huge_n;
    for (int r = 0; r < rows; ++r) {
      const int64_t u = huge[r];
      const int32_t uc = C[u];
      unsigned long long k = 0, in = 0;
      mod_entries(cols, w, C, off[u] + threadIdx.x, off[u + 1], kModBlock, uc, k, in);
      k = wave_sum(k);
      in = wave_sum(in);
      if (lane == 0) {
        my_two_m += k;
        my_intra += in;
        strength(uc, k);
      }
    }
    __syncthreads();
    for (int q = threadIdx.x; q < kModTable; q += kModBlock)
      if (key[q] != kNoLabel) {
        atomicAdd(&sigma_tot[key[q]], sum[q]);
        key[q] = kNoLabel;
        sum[q] = 0;
      }
    // the next round starts with a barrier
  }
  const unsigned long long t2 = block_sum(my_two_m, red);
  const unsigned long long ti = block_sum(my_intra, red);
  if (threadIdx.x == 0) {
    if (t2) atomicAdd(reinterpret_cast<unsigned long long *>(&ctr->two_m), t2);
    if (ti) atomicAdd(reinterpret_cast<unsigned long long *>(&ctr->intra), ti);
  }
}

struct U128 {
  unsigned long long lo, hi;
};

__device__ __forceinline__ U128 add128(U128 a, U128 b) {
  U128 r;
  r.lo = a.lo + b.lo;
  r.hi = a.hi + b.hi + (r.lo < a.lo ? 1ull : 0ull);
  return r;
}

__device__ __forceinline__ U128 shfl_xor128(U128 x, int o) {
  U128 r;
  r.lo = __shfl_xor(x.lo, o, kWave);
  r.hi = __shfl_xor(x.hi, o, kWave);
  return r;
}

// Per-block partial of sum_c Sigma_c^2 (128-bit) -> partials[2 * block].
__global__ __launch_bounds__(kModBlock) void mod_squares(const unsigned long long *__restrict__ sig,
                                                         int64_t n,
                                                         unsigned long long *__restrict__ partials) {
  __shared__ U128 red[kModBlock / kWave];
  U128 acc = {0, 0};
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < n; c += stride) {
    const unsigned long long s = sig[c];
    U128 sq = {s * s, __umul64hi(s, s)};
    acc = add128(acc, sq);
  }
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) acc = add128(acc, shfl_xor128(acc, o));
  if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    U128 t = {0, 0};
    for (int k = 0; k < kModBlock / kWave; ++k) t = add128(t, red[k]);
    partials[2 * blockIdx.x] = t.lo;
    partials[2 * blockIdx.x + 1] = t.hi;
  }
}

// Correctly rounded (to nearest even) conversion of a 128-bit unsigned integer.
__device__ __forceinline__ double u128_to_double(unsigned long long hi, unsigned long long lo) {
  if (hi == 0) return (double)lo;
  const int s = __clzll((long long)hi);
  unsigned long long top = s ? (hi << s) | (lo >> (64 - s)) : hi;
  const unsigned long long rest = s ? lo << s : lo;
  top |= rest ? 1ull : 0ull;  // sticky bit: below the rounding position
  return ldexp((double)top, 64 - s);
}

// One block: the total of the partials (a single thread adding up to 4,096 of
// them took 482 us, a fifth of what a caller of both quality measures on 6 M
// road vertices waits for; 7 us with a block).
__global__ __launch_bounds__(kFinishBlock) void mod_finish(const unsigned long long *__restrict__ partials, int nparts,
                                                           Counters *ctr) {
  __shared__ U128 red[kFinishBlock / kWave];
  U128 t = {0, 0};
  for (int k = threadIdx.x; k < nparts; k += kFinishBlock) t = add128(t, U128{partials[2 * k], partials[2 * k + 1]});
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) t = add128(t, shfl_xor128(t, o));
  if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = t;
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (int w = 1; w < kFinishBlock / kWave; ++w) t = add128(t, red[w]);
  ctr->s2_lo = t.lo;
  ctr->s2_hi = t.hi;
  const unsigned long long two_m = ctr->two_m, I = ctr->intra;
  if (two_m == 0) {
    ctr->q = 0.0;
    return;
  }
  const double M = (double)two_m;
  const double a = __ddiv_rn((double)I, M);
  const double b = __ddiv_rn(u128_to_double(t.hi, t.lo), __dmul_rn(M, M));
  ctr->q = __dsub_rn(a, b);
}

}  // namespace

hipError_t launch_modularity(const int64_t *off, const int32_t *cols, const uint32_t *w, int64_t n,
                             const int32_t *labels, unsigned long long *sigma_tot,
                             unsigned long long *partials, int partial_blocks, Counters *ctr,
                             hipStream_t s) {
  if (n <= 0) return hipSuccess;
  int64_t g = (n + kModBlock - 1) / kModBlock;
  if (g > 256 * 16) g = 256 * 16;
  mod_rows<<<(unsigned)g, kModBlock, 0, s>>>(off, cols, w, n, labels, sigma_tot, ctr);
  int64_t g2 = (n + kModBlock - 1) / kModBlock;
  if (g2 > partial_blocks) g2 = partial_blocks;
  mod_squares<<<(unsigned)g2, kModBlock, 0, s>>>(sigma_tot, n, partials);
  mod_finish<<<1, kFinishBlock, 0, s>>>(partials, (int)g2, ctr);
  return hipGetLastError();
}

}  // namespace gsl
