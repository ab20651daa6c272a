// Small graphs: the whole call -- every sweep of Alg. 3 and the split of
// Alg. 2 -- in one launch.
//
// A graph of a few hundred to a few hundred thousand vertices spends its time
// on launches, not on its rows: a sweep is about seven kernels, most of them
// shorter than the gap to the next one.  Here a fixed set of workgroups stays
// on the device for the whole call; every vertex belongs to one of them, and
// the workgroups meet once per sweep.
//
//  - Two lanes share a vertex, 16 row entries each (longer rows 4 lanes, a
//    wavefront or the workgroup): a row is sorted by label across its lanes
//    (lanes_best), so the chain of dependent steps is short.  While every
//    workgroup has one window of vertices only, their rows stay in registers
//    from sweep to sweep.
//  - Labels are double buffered (sweep t reads lab[t & 1] and writes the label
//    of every vertex, changed or not, to the other array), so one meeting per
//    sweep replaces the sweep / copy / decide launches.
//  - A meeting is a slot per workgroup: its count of changed labels and the
//    meeting's number in one word, a plain store without contention (two words
//    in turn, meeting.h).  Up to kDirect workgroups read every slot and each
//    draws the same conclusion; more of them (and batches, whose graphs stop
//    one by one) leave that to workgroup 0, which publishes it in the release
//    word.  The rules are those of sweep_end and graph_end.
//  - Up to kSmallOne vertices run in one workgroup with labels, flags and the
//    split's forest in LDS; its meetings are barriers.
//  - The split needs three more meetings: link, flatten, hook, write out.
//
// Measured (MI355X, whole calls, general path -> here): planted graphs of 200
// vertices 596 -> 83 us (16 sweeps), 10,000 vertices 626 -> 146 us, 28,901
// vertices (no allocation) 653 -> 185 us, 131,072 weighted vertices 855 -> 667
// us.  All device functions are inlined and no member of the arguments is
// indexed by a variable: a call by reference or such an index moves the
// arguments to scratch memory, where every use reads them (some 35 us a call).  A
// sweep of the 10,000 vertices takes 3.9 us of work (1.6 us gather and sort, the
// rest flags, counts and barriers) and 3 us of meeting; the launches of such a
// sweep took about 25 us.  What bounds it is latency: the label gathers after a
// meeting miss both caches.
//
// The workgroups wait for each other, so all of them must be resident at
// once: the host launches at most kSmallGrid and keeps the sum over concurrent
// calls below what the device holds.  Other kernels end by themselves, and
// every wait ends after `spin_limit` ticks of the realtime clock: a workgroup
// that waits longer reports it in the result, marks the release word and
// leaves, as does every other one that sees the mark, and the host runs the
// call on the general path.
//
// A session's step is such a launch too, from the labels, flags and counts that
// the step before left (`init` clear), with the split of the graphs that stop.
//
// Results are those of the general path: the labels of a sweep depend on the
// labels of the one before only, and the same vertices are processed.
#include "device_common.h"
#include "gsl_internal.h"
#include "meeting.h"
#include "rows.h"

namespace gsl {

namespace {

constexpr int kBlock = 256;
constexpr int kOneBlock = 512;
constexpr int kDirect = 256;              // workgroups that read each other's slots directly
constexpr int kRegs = 16;                 // row entries a lane holds
constexpr int kLanes = 2;                 // lanes of a vertex: rows up to 32 entries
constexpr int kRowMain = kRegs * kLanes;
constexpr int kGroup = 4;                 // lanes of a longer row, up to
constexpr int kRowGroup = kGroup * kRegs;
constexpr int kRowWave = 512;             // up to here: half a wavefront
constexpr int kWaveLanes = kRowWave / kRegs;
// longer rows (up to kSmallMaxDegree): the workgroup, an LDS table
constexpr int kTable = 4096;
static_assert(2 * kSmallMaxDegree <= kTable, "the workgroup's table holds two slots per entry");
static_assert(kOneBlock / kLanes == kSmallOne, "one window per graph in one workgroup");
static_assert(kBlock / kLanes == kSmallWindow, "a window has two lanes per vertex");
static_assert(kBlock / kWaveLanes == kSmallPerPass, "half a wavefront per row of up to kRowWave entries");

// Payload of a slot: changed vertices in the low bits, events above.
constexpr uint32_t kDnMask = (1u << 28) - 1;
constexpr uint32_t kOverflow = 1u << 28, kDecline = 1u << 29, kAbort = 1u << 30;
// Release word's payload.
constexpr uint32_t kDone = 1, kDense = 2, kMark = 4, kError = 8;

template <int BLOCK>
struct Shared {
  static constexpr int V = BLOCK / kLanes;  // vertices of a window
  static constexpr int NW = BLOCK / kWave;
  static constexpr int ONE = BLOCK == kOneBlock ? kSmallOne : 1;
  unsigned long long tab[kTable];
  uint16_t q[3][V];          // vertices of the window with longer rows
  int qn[3];
  int64_t rb[V], re[V];      // row bounds of the window's vertices
  uint32_t own[V];           // and their labels
  uint8_t chg[V];            // vertices of the window that changed label
  // this sweep's processed rows, their entries, changed and marked: rows of
  // kLanes lanes, of kGroup lanes, longer ones
  unsigned int cnt[3][4];
  unsigned int events;
  int32_t gone;              // batches: the graph whose changes are summed here until the workgroup
  unsigned int gsum;         // comes to another or the sweep ends
  unsigned int tstat[kNumTiers][kSmallTierFields];
  unsigned long long red[NW], red2[NW];
  unsigned int acc[kMeetingCopies][2];  // a meeting's sums (meeting_copy): changed vertices, events
  unsigned long long active;
  uint32_t word;
  // workgroup 0: changes of every sweep, whether it marked, and (one workgroup) its rows
  uint32_t dn_of[kSmallMaxSweeps], processed_of[kSmallMaxSweeps], edges_of[kSmallMaxSweeps];
  uint8_t marked[kSmallMaxSweeps];
  // one workgroup: the graph's labels, flags and forest
  int32_t lab[2][ONE], parent[ONE], root[ONE], rep[ONE];
  uint8_t act[2][ONE];
};

__device__ __forceinline__ unsigned long long word_of(const SmallArgs &a, uint32_t meeting, uint32_t payload) {
  return meeting_word(a.epoch, meeting, payload);
}

__device__ __forceinline__ bool spun_out(const SmallArgs &a, long long t0) {
  return wall_clock64() - t0 > a.spin_limit;
}

// Reports a wait that ran out and has the others leave.
__device__ __forceinline__ void give_up(const SmallArgs &a, uint32_t m) {
  __hip_atomic_store(&a.result->aborted, a.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __hip_atomic_store(a.release, word_of(a, m, kAbort), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ bool given_up(const SmallArgs &a) {
  const unsigned long long r = __hip_atomic_load(a.release, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return (r >> 40) == a.epoch && ((uint32_t)r & kAbort);
}

// The slots of every workgroup at meeting m, read by all threads of this one:
// their sums are added to the meeting's s.acc.
template <int BLOCK>
__device__ __forceinline__ void small_collect(const SmallArgs &a, Shared<BLOCK> &s, uint32_t m) {
  const long long t0 = wall_clock64();
  uint32_t sum = 0, ev = 0;
  const unsigned long long *slots = a.slots + meeting_copy(m) * kSmallGrid;
  for (unsigned int b = threadIdx.x; b < gridDim.x; b += BLOCK) {
    for (int spins = 0;; ++spins) {
      const unsigned long long x = __hip_atomic_load(slots + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (meeting_posted(x, a.epoch, m)) {
        sum += (uint32_t)x & kDnMask;
        ev |= (uint32_t)x & ~kDnMask;
        break;
      }
      if ((spins & 15) == 15) {
        if (given_up(a)) {
          ev |= kAbort;
          break;
        }
        if (spun_out(a, t0)) {
          give_up(a, m);
          ev |= kAbort;
          break;
        }
      }
      __builtin_amdgcn_s_sleep(1);
    }
  }
  sum = wave_sum_u32(sum);
  unsigned int *acc = s.acc[meeting_copy(m)];
  if (threadIdx.x % kWave == 0 && sum) atomicAdd(&acc[0], sum);
  if (ev) atomicOr(&acc[1], ev);
}

// This workgroup's part of meeting m: what it wrote becomes visible, then its
// slot says so.  With `all` (uniform over the grid) every workgroup returns
// with the sums in s.acc; else workgroup 0 does, and calls small_release with
// the payload that the others return.  Returns kAbort: leave.
template <int BLOCK>
__device__ __forceinline__ uint32_t small_arrive(const SmallArgs &a, Shared<BLOCK> &s, uint32_t m, uint32_t payload, bool all) {
  // no barrier before the sums are written: their last readers were at meeting
  // m - 2, and everyone has been through m - 1's barriers since
  unsigned int *acc = s.acc[meeting_copy(m)];
  if constexpr (BLOCK == kOneBlock) {
    __syncthreads();
    if (threadIdx.x == 0) {
      acc[0] = payload & kDnMask;
      acc[1] = payload & ~kDnMask;
    }
    __syncthreads();
    return 0;
  }
  if (threadIdx.x == 0) acc[0] = acc[1] = 0;
  __syncthreads();
  if (threadIdx.x == 0) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __hip_atomic_store(a.slots + meeting_copy(m) * kSmallGrid + blockIdx.x, word_of(a, m, payload), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  }
  if (all || blockIdx.x == 0) {
    small_collect(a, s, m);
    __syncthreads();
    if (threadIdx.x == 0) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    __syncthreads();
    return acc[1] & kAbort;
  }
  if (threadIdx.x == 0) {
    const long long t0 = wall_clock64();
    uint32_t got = kAbort;
    for (;;) {
      const unsigned long long x = __hip_atomic_load(a.release, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (meeting_posted(x, a.epoch, m)) {
        got = (uint32_t)x;
        break;
      }
      if ((x >> 40) == a.epoch && ((uint32_t)x & kAbort)) break;
      if (spun_out(a, t0)) {
        give_up(a, m);
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    s.word = got;
  }
  __syncthreads();
  const uint32_t got = s.word;
  __syncthreads();  // s.word is written again at the next meeting
  return got;
}

__device__ __forceinline__ void small_release(const SmallArgs &a, uint32_t m, uint32_t payload) {
  if (threadIdx.x == 0) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __hip_atomic_store(a.release, word_of(a, m, payload), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// A meeting without a decision.  Returns false when the kernel must leave.
template <int BLOCK>
__device__ __forceinline__ bool small_meet(const SmallArgs &a, Shared<BLOCK> &s, uint32_t m) {
  if constexpr (BLOCK == kOneBlock) {
    __syncthreads();
    return true;
  }
  const bool all = gridDim.x <= kDirect;
  const uint32_t r = small_arrive(a, s, m, 0, all);
  if (!all && blockIdx.x == 0) small_release(a, m, r & kAbort);
  return !(r & kAbort);
}

// ---- rows ----

template <int BLOCK>
struct Sweep {
  const int32_t *C;    // labels read (NULL: every vertex its own id)
  int32_t *Cn;         // labels written
  uint8_t *act, *nact;
  int par;             // parity of the sweep (one workgroup: its arrays in LDS)
  bool dense, mark;
};

// Label of vertex j in this sweep.
template <int BLOCK>
__device__ __forceinline__ uint32_t label_of(const Shared<BLOCK> &s, const Sweep<BLOCK> &m, uint32_t j) {
  if constexpr (BLOCK == kOneBlock)
    return (uint32_t)s.lab[m.par][j];
  else
    return *reinterpret_cast<const uint32_t *>(reinterpret_cast<const char *>(m.C) + (j << 2));
}

template <int BLOCK>
__device__ __forceinline__ void set_label(Shared<BLOCK> &s, const Sweep<BLOCK> &m, int32_t v, uint32_t c) {
  if constexpr (BLOCK == kOneBlock)
    s.lab[m.par ^ 1][v] = (int32_t)c;
  else
    m.Cn[v] = (int32_t)c;
}

template <int BLOCK>
__device__ __forceinline__ uint8_t *flag_of(Shared<BLOCK> &s, const Sweep<BLOCK> &m, int32_t j, bool next) {
  if constexpr (BLOCK == kOneBlock)
    return &s.act[m.par ^ (next ? 1 : 0)][j];
  else
    return (next ? m.nact : m.act) + j;
}

// The entries of a row that one lane holds, the row's own vertex past its end.
template <bool W, bool V4>
__device__ __forceinline__ void load_slice(const SmallArgs &a, int32_t v, int64_t b, int d, int lane, uint32_t (&col)[kRegs],
                                           uint32_t (&w)[kRegs]) {
  const int at = lane * kRegs;
  const int dl = d - at < 0 ? 0 : (d - at > kRegs ? kRegs : d - at);
  load_row<kRegs, V4>(reinterpret_cast<const uint32_t *>(a.cols), b + at, dl, (uint32_t)v, col);
  if constexpr (W) load_row<kRegs, V4>(a.w, b + at, dl, 0u, w);
}

// Packed argmax key of a row of d entries (0: no candidate) from the slices of
// its L lanes.
template <int L, bool W, int BLOCK>
__device__ __forceinline__ unsigned long long row_best(const Shared<BLOCK> &s, const Sweep<BLOCK> &m, int32_t v, int d,
                                                       const uint32_t (&col)[kRegs], const uint32_t (&w0)[kRegs],
                                                       unsigned long long &rowsum) {
  int longest = 1;
#pragma unroll
  for (int h = 1; h < L; h <<= 1) longest = __ballot(d > h * kRegs) ? 2 * h * kRegs : longest;
  uint32_t lab[kRegs], w[kRegs];
  if (BLOCK == kOneBlock || m.C) {
#pragma unroll
    for (int k = 0; k < kRegs; ++k) lab[k] = col[k] != (uint32_t)v ? label_of(s, m, col[k]) : kNoLabel;
  } else {
#pragma unroll
    for (int k = 0; k < kRegs; ++k) lab[k] = col[k] != (uint32_t)v ? col[k] : kNoLabel;
  }
  rowsum = (unsigned long long)d;
  if constexpr (W) {
    rowsum = 0;
#pragma unroll
    for (int k = 0; k < kRegs; ++k) {
      w[k] = w0[k];
      rowsum += w0[k];
    }
    rowsum = group_sum<L>(rowsum);
  }
  return lanes_best<L, kRegs, W>(lab, w, longest);
}

// The same for a row of up to kSmallMaxDegree entries shared by the workgroup,
// summed in an LDS table that is empty before and after.
template <int BLOCK, bool W>
__device__ __forceinline__ unsigned long long row_best_block(const SmallArgs &a, Shared<BLOCK> &s, const Sweep<BLOCK> &m,
                                                             int32_t v, int64_t b, int64_t e, unsigned long long &rowsum) {
  constexpr int K = kSmallMaxDegree / BLOCK;
  const int log2s = table_log2(e - b, 1, 12);
  uint32_t lab[K], wt[K];
  int slot[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int64_t p = b + threadIdx.x + (int64_t)k * BLOCK;
    const bool in = p < e;
    lab[k] = in ? (uint32_t)a.cols[p] : (uint32_t)v;
    wt[k] = in ? (W ? a.w[p] : 1u) : 0u;
  }
#pragma unroll
  for (int k = 0; k < K; ++k)
    lab[k] = lab[k] != (uint32_t)v ? (BLOCK == kOneBlock || m.C ? label_of(s, m, lab[k]) : lab[k]) : kNoLabel;
  rowsum = 0;
#pragma unroll
  for (int k = 0; k < K; ++k) rowsum += wt[k];
#pragma unroll
  for (int k = 0; k < K; ++k) slot[k] = lab[k] != kNoLabel ? lds_insert(s.tab, log2s, lab[k], wt[k]) : -1;
  __syncthreads();
  unsigned long long best = 0;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    if (slot[k] >= 0) {
      const unsigned long long x = s.tab[slot[k]];
      const unsigned long long key = argmax_key((uint32_t)(x >> 32), (uint32_t)x);
      best = key > best ? key : best;
      s.tab[slot[k]] = kEmptySlot;
    }
  }
  best = group_max<kWave>(best);
  rowsum = wave_sum(rowsum);
  if (threadIdx.x % kWave == 0) {
    s.red[threadIdx.x / kWave] = best;
    s.red2[threadIdx.x / kWave] = rowsum;
  }
  __syncthreads();
  best = 0;
  rowsum = 0;
#pragma unroll
  for (int w = 0; w < Shared<BLOCK>::NW; ++w) {
    best = s.red[w] > best ? s.red[w] : best;
    rowsum += s.red2[w];
  }
  __syncthreads();
  return best;
}

// Flags the entries of a changed vertex's row that a lane holds for the next
// sweep: every flag is read before the first is set.
template <int BLOCK>
__device__ __forceinline__ void mark_slice(Shared<BLOCK> &s, const Sweep<BLOCK> &m, int32_t v, const uint32_t (&col)[kRegs],
                                           bool self) {
  uint8_t f[kRegs];
#pragma unroll
  for (int k = 0; k < kRegs; ++k) f[k] = col[k] != (uint32_t)v ? *flag_of(s, m, (int32_t)col[k], true) : 1;
#pragma unroll
  for (int k = 0; k < kRegs; ++k)
    if (!f[k]) *flag_of(s, m, (int32_t)col[k], true) = 1;
  if (self) *flag_of(s, m, v, true) = 1;  // an entry of its own row
}

// The decision for a processed row, by every lane that shares it (lane 0
// writes): the new label.  Returns whether it changed.
template <int BLOCK>
__device__ __forceinline__ bool row_decide(Shared<BLOCK> &s, const Sweep<BLOCK> &m, int t, int32_t v, uint32_t own,
                                           unsigned long long best, unsigned long long rowsum, int lane) {
  // a row whose weights sum to 2^32 or more keeps its label: the call fails
  const bool over = rowsum >> 32;
  const uint32_t next = best && !over ? key_label(best) : own;
  if (lane == 0) {
    if (over) atomicOr(&s.events, kOverflow);
    set_label(s, m, v, next);
    if (next != own) s.chg[t] = 1;
  }
  return next != own;
}

// Counts of a wavefront's rows (`on`: the lane leads one, of d entries), all
// lanes active.
template <int BLOCK>
__device__ __forceinline__ void wave_count(Shared<BLOCK> &s, const Sweep<BLOCK> &m, int cls, bool on, unsigned int d, bool ch) {
  const unsigned long long rows = __ballot(on), changed = __ballot(on && ch);
  if (!rows) return;
  const uint32_t edges = wave_sum_u32(on ? d : 0u);
  const uint32_t marks = changed && m.mark ? wave_sum_u32(on && ch ? d : 0u) : 0u;
  if (threadIdx.x % kWave == 0) {
    atomicAdd(&s.cnt[cls][0], (unsigned int)__popcll(rows));
    atomicAdd(&s.cnt[cls][1], edges);
    if (changed) atomicAdd(&s.cnt[cls][2], (unsigned int)__popcll(changed));
    if (marks) atomicAdd(&s.cnt[cls][3], marks);
  }
}

// Counts of one longer row (one thread).
template <int BLOCK>
__device__ __forceinline__ void row_count(const SmallArgs &a, Shared<BLOCK> &s, const Sweep<BLOCK> &m, unsigned int d, bool ch) {
  const int t = tier_of(d, a.tiers);
  atomicAdd(&s.cnt[2][0], 1u);
  atomicAdd(&s.cnt[2][1], d);
  atomicAdd(&s.tstat[t][0], 1u);
  atomicAdd(&s.tstat[t][1], d);
  if (ch) {
    atomicAdd(&s.cnt[2][2], 1u);
    atomicAdd(&s.tstat[t][2], 1u);
    if (m.mark) atomicAdd(&s.tstat[t][3], d);
  }
}

// What a lane keeps of its vertex.
struct Row {
  int64_t b, e;
  int32_t v;          // -1: none
  bool self;          // the lane's slice names the vertex itself
  uint32_t col[kRegs], w[kRegs];
};

template <bool W, bool V4>
__device__ __forceinline__ void row_slice(const SmallArgs &a, Row &r, bool wanted) {
  const int sub = threadIdx.x % kLanes;
  const int d = wanted && r.e - r.b <= kRowMain ? (int)(r.e - r.b) : 0;
  load_slice<W, V4>(a, r.v, r.b, d, sub, r.col, r.w);
  const int dl = d - sub * kRegs;
  r.self = false;
#pragma unroll
  for (int k = 0; k < kRegs; ++k) r.self = r.self || (k < dl && r.col[k] == (uint32_t)r.v);
}

__device__ __forceinline__ void row_bounds(const SmallArgs &a, Row &r, int64_t v) {
  r.v = v < a.n ? (int32_t)v : -1;
  r.b = r.e = 0;
  if (r.v >= 0) {
    r.b = a.off[v];
    r.e = a.off[v + 1];
  }
}

// A longer row taken by L lanes (L <= 64).
template <int L, int BLOCK, bool W, bool V4>
__device__ __forceinline__ void long_row(const SmallArgs &a, Shared<BLOCK> &s, const Sweep<BLOCK> &m, int64_t base, int r,
                                         bool on) {
  const int lane = threadIdx.x % L;
  const int32_t u = (int32_t)(base + r);
  const int64_t ub = s.rb[r];
  const int d = on ? (int)(s.re[r] - ub) : 0;
  uint32_t col[kRegs], w[kRegs];
  load_slice<W, V4>(a, u, ub, d, lane, col, w);
  unsigned long long rowsum = 0;
  const unsigned long long best = row_best<L, W, BLOCK>(s, m, u, d, col, w, rowsum);
  bool ch = false;
  if (on) ch = row_decide(s, m, r, u, s.own[r], best, rowsum, lane);
  if (ch && m.mark) {
    bool self = false;
#pragma unroll
    for (int k = 0; k < kRegs; ++k) self = self || (lane * kRegs + k < d && col[k] == (uint32_t)u);
    mark_slice(s, m, u, col, self);
  }
  if constexpr (L == kGroup)
    wave_count(s, m, 1, on && lane == 0, (unsigned int)d, ch);
  else if (on && lane == 0)
    row_count(a, s, m, (unsigned int)d, ch);
}

// Thread 0: the summed changes of graph s.gone to its counter.
template <int BLOCK>
__device__ __forceinline__ void small_graph_changes(const SmallArgs &a, Shared<BLOCK> &s) {
  if (s.gsum)
    __hip_atomic_fetch_add(reinterpret_cast<unsigned long long *>(a.gdn) + s.gone, (unsigned long long)s.gsum,
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  s.gsum = 0;
}

// One window of BLOCK / kLanes consecutive vertices in one sweep; rows that
// need more lanes are packed and follow.  `r` holds the window's rows
// (`resident`) or just their bounds.
template <int BLOCK, bool W, bool V4>
__device__ __forceinline__ void small_window(const SmallArgs &a, Shared<BLOCK> &s, const Sweep<BLOCK> &m, int64_t base,
                                             bool first, Row &r, bool resident) {
  const int t = threadIdx.x / kLanes;
  const int lane = threadIdx.x % kWave;
  const bool in = r.v >= 0, lead = threadIdx.x % kLanes == 0;
  const int64_t d = r.e - r.b;
  uint32_t own = (uint32_t)r.v;
  bool on = in;
  if (in) {
    if (BLOCK == kOneBlock || m.C) own = label_of(s, m, (uint32_t)r.v);
    if (!m.dense) on = *flag_of(s, m, r.v, false) != 0;
    if (a.gdone && a.gdone[a.gid[r.v]]) on = false;
  }
  bool take = on && d > 0;
  if (threadIdx.x < 3) s.qn[threadIdx.x] = 0;
  if (BLOCK != kOneBlock && a.gdn && threadIdx.x == 0) {  // a batch is never one workgroup of its own
    const int32_t g = a.gid[base];
    if (g != s.gone) {
      small_graph_changes(a, s);
      s.gone = g;
    }
  }
  if (lead) s.chg[t] = 0;
  __syncthreads();
  if (first && a.init) {
    // degree statistics of the call, and rows this kernel does not take
    const int tier = tier_of(d, a.tiers);
    for (int k = 0; k < kNumTiers; ++k) {
      const unsigned long long c = __ballot(in && lead && tier == k);
      if (!c) continue;
      const uint32_t de = wave_sum_u32(in && lead && tier == k && d > 0 ? (uint32_t)d : 0u);
      if (lane == 0) {
        atomicAdd(&s.tstat[k][4], (unsigned int)__popcll(c));
        atomicAdd(&s.tstat[k][5], de);
      }
    }
    const unsigned long long longest = group_max<kWave>(in && d > 0 ? (unsigned long long)d : 0ull);
    if (lane == 0) atomicMax(&s.tstat[0][0], (unsigned int)(longest < 0x7fffffff ? longest : 0x7fffffff));
    if (take && d > kSmallMaxDegree) {
      if (lead) atomicOr(&s.events, kDecline);
      take = false;
    }
  }
  const bool mine = take && d <= kRowMain;
  if (!resident) row_slice<W, V4>(a, r, mine);
  if (take && !mine && lead) {
    const int c = d <= kRowGroup ? 0 : d <= kRowWave ? 1 : 2;
    s.q[c][atomicAdd(&s.qn[c], 1)] = (uint16_t)t;
    s.rb[t] = r.b;
    s.re[t] = r.e;
    s.own[t] = own;
  }
  // the flag is consumed (its next user marks it after the next meeting)
  if (!m.dense && in && lead && on) *flag_of(s, m, r.v, false) = 0;
  const unsigned long long am = __ballot(mine);
  bool changed = false;
  if (am) {
    unsigned long long rowsum = 0;
    const unsigned long long best = row_best<kLanes, W, BLOCK>(s, m, r.v, mine ? (int)d : 0, r.col, r.w, rowsum);
    if (mine) changed = row_decide(s, m, t, r.v, own, best, rowsum, (int)threadIdx.x % kLanes);
    if (changed && m.mark) mark_slice(s, m, r.v, r.col, r.self);
    wave_count(s, m, 0, mine && lead, (unsigned int)d, changed);
  }
  if (in && !take && lead) set_label(s, m, r.v, own);  // every label is written
  __syncthreads();
  const int n0 = s.qn[0], n1 = s.qn[1], n2 = s.qn[2];
  // long rows that the sample missed because they lie together: twice the line in
  // this window alone, as rows spread evenly vary around their mean
  if (first && a.init && n1 + n2 &&
      small_rows_cost(W, 0, 64u * (uint32_t)n1, 64u * (uint32_t)n2, BLOCK / kWaveLanes) >
          2 * small_rows_line(BLOCK == kOneBlock ? 1 : small_windows(a.n, (int)gridDim.x))) {
    if (threadIdx.x == 0) atomicOr(&s.events, kDecline);
    return;
  }
  if (n0 + n1 + n2) {
    for (int i0 = 0; i0 < n0; i0 += BLOCK / kGroup) {
      const int i = i0 + (int)threadIdx.x / kGroup;
      if (!__ballot(i < n0)) break;
      long_row<kGroup, BLOCK, W, V4>(a, s, m, base, i < n0 ? s.q[0][i] : s.q[0][0], i < n0);
    }
    for (int i0 = 0; i0 < n1; i0 += BLOCK / kWaveLanes) {
      const int i = i0 + (int)threadIdx.x / kWaveLanes;
      if (!__ballot(i < n1)) break;
      long_row<kWaveLanes, BLOCK, W, V4>(a, s, m, base, i < n1 ? s.q[1][i] : s.q[1][0], i < n1);
    }
    for (int i = 0; i < n2; ++i) {
      const int q = s.q[2][i];
      const int32_t u = (int32_t)(base + q);
      const int64_t ub = s.rb[q], ue = s.re[q];
      unsigned long long rowsum = 0;
      const unsigned long long best = row_best_block<BLOCK, W>(a, s, m, u, ub, ue, rowsum);
      const bool ch = row_decide(s, m, q, u, s.own[q], best, rowsum, (int)threadIdx.x);
      if (ch && m.mark)
        for (int64_t p = ub + threadIdx.x; p < ue; p += BLOCK) {
          uint8_t *f = flag_of(s, m, a.cols[p], true);
          if (!*f) *f = 1;
        }
      if (threadIdx.x == 0) row_count(a, s, m, (unsigned int)(ue - ub), ch);
    }
    __syncthreads();
  }
  if (BLOCK != kOneBlock && a.gdn) {
    // changes per graph of a batch, by runs of vertices of a graph: those of the
    // window's first graph meet in LDS, one atomic for all of the sweep's (with
    // one per run a batch of four graphs, 260,000 vertices in all that keep
    // changing, took 2,160 us a call)
    const bool c = lead && s.chg[t];
    unsigned long long pending = __ballot(c);
    const int32_t g = c ? a.gid[r.v] : -1;
    while (pending) {
      const int32_t lg = __shfl(g, __ffsll((long long)pending) - 1);
      const unsigned long long same = __ballot(c && g == lg);
      if (lane == 0) {
        if (lg == s.gone)
          atomicAdd(&s.gsum, (unsigned int)__popcll(same));
        else
          __hip_atomic_fetch_add(reinterpret_cast<unsigned long long *>(a.gdn) + lg, (unsigned long long)__popcll(same),
                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      pending &= ~same;
    }
  }
}

// Whether a fixed sample of the rows already says that the call is for the
// general path: a row above kSmallMaxDegree, rows that cost more than the launches
// saved (small_rows_cost), or most entries in rows that the layout rule counts.  A
// sweep takes 60 us (2^16 vertices of an R-MAT graph) to 120 us (2^18), which
// the general path would repeat.  Every wavefront of the grid reads the same rows
// and answers alike, without a meeting or a barrier.
// 512 rows say enough where none has more than 64 entries or there are very many
// of them; else up to kSampleRounds times as many are read, 1 us each time, until
// the answer is clear.  Where the share is near a half either way will do, and a
// call turned away loses 400 us and up: the line is nine sixteenths (an R-MAT graph
// of 4,096 vertices, half of its entries in such rows, runs in 166 us here and 632
// on the general path; it was 651 when the exact share, known after the first
// sweep, turned it away).  (R-MAT of 2^16 vertices, 400,000 weighted edges, in turn
// on three graphs: 1,884 us a call when the first sweep found out, 1,800 here and
// on the general path alone.)  The rows are spread by a multiplicative hash: no
// period of the ids meets it.
constexpr int kSampleRows = 8;  // rows per lane and round
constexpr int kSampleRounds = 8;

template <int BLOCK, bool W>
__device__ __forceinline__ bool small_sampled_out(const SmallArgs &a) {
  const int windows = BLOCK == kOneBlock ? 1 : small_windows(a.n, (int)gridDim.x);
  const uint32_t line = small_rows_line(windows);
  const uint32_t V = BLOCK == kOneBlock ? (uint32_t)a.n : (uint32_t)kSmallWindow;
  uint32_t sum = 0, heavy = 0, cost = 0, c1 = 0, c2 = 0, c3 = 0;
#pragma unroll 1
  for (uint32_t round = 1; round <= kSampleRounds; ++round) {
    int64_t d[kSampleRows];
#pragma unroll
    for (int k = 0; k < kSampleRows; ++k) {
      const uint32_t h = (uint32_t)(threadIdx.x % kWave + ((round - 1) * kSampleRows + k) * kWave + 1) * 2654435761u;
      const int64_t v = (int64_t)(((uint64_t)h * (uint64_t)a.n) >> 32);  // < n
      d[k] = a.off[v + 1] - a.off[v];
    }
    uint32_t rs = 0, rh = 0, rc = 0;  // entries, those of rows above 64; the three kinds of those rows, 10 bits each
    bool over = false;
#pragma unroll
    for (int k = 0; k < kSampleRows; ++k) {
      over = over || d[k] > kSmallMaxDegree;
      const uint32_t c = d[k] > 0 && d[k] <= kSmallMaxDegree ? (uint32_t)d[k] : 0u;
      rs += c;
      rh += c > 64 ? c : 0u;
      rc += c > kRowWave ? 1u << 20 : c > 128 ? 1u << 10 : c > 64 ? 1u : 0u;
    }
    if (__ballot(over)) return true;
    sum += wave_sum_u32(rs);
    heavy += wave_sum_u32(rh);
    if (!heavy) return false;
    rc = wave_sum_u32(rc);
    c1 += rc & 1023u;
    c2 += rc >> 10 & 1023u;
    c3 += rc >> 20;
    // of a window of V rows, in 64ths
    const uint32_t rows = 64u * kSampleRows * round;
    cost = (uint32_t)windows * small_rows_cost(W, 64u * V * c1 / rows, 64u * V * c2 / rows, 64u * V * c3 / rows, BLOCK / kWaveLanes);
    // the more rows, the closer to the lines an answer may lie
    if (cost * round > line * (round + 1) || (a.layout_auto && (round < 4 ? 4 * heavy > 3 * sum : 8 * heavy > 5 * sum))) return true;
    if (cost * (round + 1) < line * round && (!a.layout_auto || (round < 4 ? 4 * heavy < sum : 8 * heavy < 3 * sum))) return false;
    if (rows >= 4 * (uint32_t)a.n) break;
  }
  return cost > line || (a.layout_auto && 16 * heavy > 9 * sum);
}

// After a sweep (every slot in at meeting m): per-graph stops of a batch (workgroup 0) and
// the next sweep's mode, the rules of graph_end and sweep_end.
template <int BLOCK>
__device__ __forceinline__ void small_decide(const SmallArgs &a, Shared<BLOCK> &s, uint32_t m, SweepCtrl &c) {
  const unsigned int *acc = s.acc[meeting_copy(m)];
  if (a.gdn) {
    unsigned long long active = 0;
    // the loads of four graphs on the way at once: a round trip each made the
    // decisions of 4,096 graphs a good part of a sweep
    constexpr int K = 4;
    for (int64_t g0 = threadIdx.x; g0 < a.graphs; g0 += K * BLOCK) {
      bool run[K];
      long long d[K], most[K];
      int32_t it[K];
#pragma unroll
      for (int k = 0; k < K; ++k) run[k] = g0 + k * BLOCK < a.graphs && !a.gdone[g0 + k * BLOCK];
#pragma unroll
      for (int k = 0; k < K; ++k)
        if (run[k]) {
          d[k] = (long long)__hip_atomic_load(a.gdn + g0 + k * BLOCK, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          most[k] = a.glimit[g0 + k * BLOCK];
          it[k] = a.giters[g0 + k * BLOCK] + 1;
        }
#pragma unroll
      for (int k = 0; k < K; ++k)
        if (run[k]) {
          const int64_t g = g0 + k * BLOCK;
          a.giters[g] = it[k];
          if (d[k] <= most[k] || it[k] >= c.graph_max_iters)
            a.gdone[g] = 1;
          else
            active += 1;
          __hip_atomic_store(a.gdn + g, (int64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    active = block_sum(active, s.red);
    if (threadIdx.x == 0) s.active = active;
    __syncthreads();
  }
  const long long d = (long long)acc[0];
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    s.dn_of[c.it - a.ctrl.it] = (uint32_t)d;
    s.marked[c.it - a.ctrl.it] = (uint8_t)c.mark;
  }
  const int marked = c.mark;
  c.it += 1;
  if (acc[1] & kOverflow) {
    c.error = 1;
    c.done = 1;
    return;
  }
  bool stop = c.it >= c.max_iters;
  stop = stop || (a.gdn ? s.active == 0 : d <= c.limit);
  c.done = stop ? 1 : 0;
  c.dense = (c.prune && marked) ? 0 : 1;
  c.mark = (c.prune && d * 8 <= c.n) ? 1 : 0;
}

// ---- split (the union-find of split.hip, over this kernel's windows) ----
// The forest: global memory, or LDS when one workgroup holds the graph.
template <int BLOCK>
struct Forest {
  static constexpr bool kLds = BLOCK == kOneBlock;
  int32_t *p;
  __device__ __forceinline__ int32_t load(int32_t x) const {
    return __hip_atomic_load(p + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  __device__ __forceinline__ int32_t fresh(int32_t x) const {
    if constexpr (kLds) return load(x);
    return __hip_atomic_load(p + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ bool hook(int32_t x, int32_t &expected, int32_t y) const {
    if constexpr (kLds)
      return __hip_atomic_compare_exchange_strong(p + x, &expected, y, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_WORKGROUP);
    return __hip_atomic_compare_exchange_strong(p + x, &expected, y, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ int32_t root(int32_t x) const {
    for (;;) {
      const int32_t q = load(x);
      if (q == x) return x;
      const int32_t g = load(q);
      if (g != q) __hip_atomic_store(p + x, g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      x = g;
    }
  }
  __device__ __forceinline__ void unite(int32_t x, int32_t y) const {
    x = root(x);
    y = root(y);
    for (;;) {
      if (x == y) return;
      if (x < y) {
        const int32_t t = x;
        x = y;
        y = t;
      }
      int32_t expected = fresh(x);
      if (expected == x && hook(x, expected, y)) return;
      x = root(expected);
      y = root(y);
    }
  }
};

// The split takes vertex v: in a session, if its graph has just stopped (or
// stopped before and waits to be collected).
__device__ __forceinline__ bool splits(const SmallArgs &a, int64_t v) {
  if (!a.session) return true;
  const int32_t g = a.gid[v];
  return g != a.graphs - 1 && a.gdone[g];
}

constexpr int kLinkScanS = 16;  // entries scanned for the two that are linked

// First pass: the first two intra-community entries among a row's first 16,
// one by each of the vertex's lanes.
template <int BLOCK>
__device__ __forceinline__ void split_link(const SmallArgs &a, Shared<BLOCK> &s, const Forest<BLOCK> &f, const int32_t *L,
                                           int64_t base) {
  const int64_t v = base + threadIdx.x / kLanes;
  if (v >= a.n || !splits(a, v)) return;
  const int64_t b = a.off[v], e = a.off[v + 1];
  const int32_t cu = BLOCK == kOneBlock ? s.root[v] : L[v];
  uint32_t u[kLinkScanS];
#pragma unroll
  for (int k = 0; k < kLinkScanS; ++k) u[k] = b + k < e ? (uint32_t)a.cols[b + k] : (uint32_t)v;
  unsigned int hits = 0;
#pragma unroll
  for (int k = 0; k < kLinkScanS; ++k)
    hits |= u[k] != (uint32_t)v && (BLOCK == kOneBlock ? s.root[u[k]] : L[u[k]]) == cu ? 1u << k : 0u;
  if (threadIdx.x % kLanes) hits &= hits - 1;
  int32_t to = -1;
#pragma unroll
  for (int k = kLinkScanS - 1; k >= 0; --k) to = (hits >> k) & 1 ? (int32_t)u[k] : to;
  if (to >= 0) f.unite((int32_t)v, to);
}

// Second pass, rows outside their community's representative component: every
// entry that was in the community but in another component is united.  A
// vertex's lanes take its entries 16 at a time; long rows (`lane`, `lanes`) by
// more of them.
template <int BLOCK>
__device__ __forceinline__ void split_hook(const SmallArgs &a, Shared<BLOCK> &s, const Forest<BLOCK> &f, int32_t v,
                                           unsigned long long x, int64_t b, int64_t e, int lane, int lanes) {
  constexpr int K = 8;
  for (int64_t p = b + lane; p < e; p += (int64_t)K * lanes) {
    uint32_t u[K];
    unsigned long long y[K];
#pragma unroll
    for (int k = 0; k < K; ++k) u[k] = p + (int64_t)k * lanes < e ? (uint32_t)a.cols[p + (int64_t)k * lanes] : (uint32_t)v;
#pragma unroll
    for (int k = 0; k < K; ++k) y[k] = a.cp[u[k]];
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (u[k] != (uint32_t)v && (uint32_t)(y[k] >> 32) == (uint32_t)(x >> 32) && (uint32_t)y[k] != (uint32_t)x)
        f.unite(v, (int32_t)u[k]);
  }
}

template <int BLOCK>
__device__ __forceinline__ void split_hooks(const SmallArgs &a, Shared<BLOCK> &s, const Forest<BLOCK> &f, int64_t base) {
  const int64_t v = base + threadIdx.x / kLanes;
  const int lane = threadIdx.x % kWave;
  unsigned long long x = 0;
  int64_t b = 0, e = 0;
  if (v < a.n && splits(a, v)) {
    x = a.cp[v];
    const int32_t rep = BLOCK == kOneBlock ? s.rep[x >> 32] : a.rep[x >> 32];
    if (rep != (int32_t)(uint32_t)x) {
      b = a.off[v];
      e = a.off[v + 1];
    }
  }
  if (e - b <= kRowGroup) split_hook(a, s, f, (int32_t)v, x, b, e, (int)threadIdx.x % kLanes, kLanes);
  unsigned long long pending = __ballot(e - b > kRowGroup && threadIdx.x % kLanes == 0);
  while (pending) {
    const int src = __ffsll((long long)pending) - 1;
    pending &= pending - 1;
    split_hook(a, s, f, __shfl((int32_t)v, src), (unsigned long long)__shfl((long long)x, src), (int64_t)__shfl((long long)b, src),
               (int64_t)__shfl((long long)e, src), lane, kWave);
  }
}

// Totals of the statistics over the workgroups, a wavefront of the grid per
// count (one workgroup: its own counts).
template <int BLOCK>
__device__ __forceinline__ void small_totals(const SmallArgs &a, Shared<BLOCK> &s, int sweeps) {
  constexpr int F = kNumTiers * kSmallTierFields;
  if constexpr (BLOCK == kOneBlock) {
    for (int f = threadIdx.x; f < F; f += BLOCK)
      a.result->tier[f / kSmallTierFields][f % kSmallTierFields] = (&s.tstat[0][0])[f];
    for (int k = threadIdx.x; k < sweeps; k += BLOCK) {
      a.result->processed[k] = s.processed_of[k];
      a.result->edges[k] = s.edges_of[k];
    }
    return;
  }
  const int lane = threadIdx.x % kWave;
  for (int f = (int)(threadIdx.x / kWave * gridDim.x + blockIdx.x); f < F + sweeps; f += Shared<BLOCK>::NW * gridDim.x) {
    unsigned long long x = 0, y = 0;
    if (f < F) {
      for (unsigned int b = lane; b < gridDim.x; b += kWave) {
        const unsigned int r = a.tier_rec[(size_t)b * F + f];
        x = f == 0 ? (r > x ? r : x) : x + r;
      }
      x = f == 0 ? group_max<kWave>(x) : wave_sum(x);
      if (lane == 0) a.result->tier[f / kSmallTierFields][f % kSmallTierFields] = (int64_t)x;
    } else {
      const int k = f - F;
      for (unsigned int b = lane; b < gridDim.x; b += kWave) {
        const unsigned long long r = a.rec[(size_t)k * kSmallGrid + b];
        x += r >> 32;
        y += (uint32_t)r;
      }
      x = wave_sum(x);
      y = wave_sum(y);
      if (lane == 0) {
        a.result->processed[k] = (int64_t)x;
        a.result->edges[k] = (int64_t)y;
      }
    }
  }
}

template <int BLOCK, bool W, bool V4>
__global__ __launch_bounds__(BLOCK, W || BLOCK == kOneBlock ? 2 : 4) void small_lpa(SmallArgs a) {
  constexpr bool kOne = BLOCK == kOneBlock;
  constexpr int V = Shared<BLOCK>::V, F = kNumTiers * kSmallTierFields;
  __shared__ Shared<BLOCK> s;
  const int64_t nnz = a.off[a.n];
  // uniform over the grid: every workgroup reads the same words
  if (a.off[0] != 0 || nnz < 0 || (nnz > 0 && !a.cols) || nnz > a.max_nnz) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      a.result->status = a.off[0] != 0 ? kSmallBadStart : nnz < 0 ? kSmallBadEnd : nnz > a.max_nnz ? kSmallDeclined : kSmallNoCols;
      a.result->first_offset = a.off[0];
      a.result->nnz = nnz;
    }
    return;
  }
  if (a.init && a.ctrl.max_iters > 0 && small_sampled_out<BLOCK, W>(a)) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      // the host looks for this word while the launch runs
      __hip_atomic_store(&a.result->declined, a.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      a.result->status = kSmallDeclined;
    }
    return;
  }
  const int64_t base0 = (int64_t)blockIdx.x * V, step = (int64_t)gridDim.x * V;
  const bool resident = step >= a.n;
  const bool all = gridDim.x <= kDirect && !a.gdn;
  Row r;
  row_bounds(a, r, base0 + threadIdx.x / kLanes);
  if (resident) row_slice<W, V4>(a, r, true);
  for (int i = threadIdx.x; i < kTable; i += BLOCK) s.tab[i] = kEmptySlot;
  for (int i = threadIdx.x; i < F; i += BLOCK) (&s.tstat[0][0])[i] = 0;
  if (threadIdx.x == 0) {
    s.events = s.gsum = 0;
    s.gone = -1;
  }
  if (threadIdx.x < 12) s.cnt[threadIdx.x / 4][threadIdx.x % 4] = 0;
  SweepCtrl c = a.ctrl;
  const int it0 = c.it;
  // the call's own state (one workgroup: into LDS)
  const int32_t *labels_in = it0 & 1 ? a.lab1 : a.lab0;
  if constexpr (kOne) {
    for (int v = threadIdx.x; v < a.n; v += BLOCK) {
      s.lab[it0 & 1][v] = a.init ? v : labels_in[v];
      s.act[0][v] = a.init ? 0 : a.act0[v];
      s.act[1][v] = a.init ? 0 : a.act1[v];
      s.parent[v] = v;
    }
  } else {
    for (int64_t v = (int64_t)blockIdx.x * BLOCK + threadIdx.x; v < a.n; v += (int64_t)gridDim.x * BLOCK) {
      if (a.init) a.act0[v] = a.act1[v] = 0;
      a.parent[v] = (int32_t)v;
    }
  }
  __syncthreads();
  uint32_t m = 0;  // meetings held
  int it = it0;
  while (c.max_iters > it0) {
    Sweep<BLOCK> md;
    md.C = a.init && it == it0 ? nullptr : it & 1 ? a.lab1 : a.lab0;
    md.Cn = it & 1 ? a.lab0 : a.lab1;
    md.act = it & 1 ? a.act1 : a.act0;
    md.nact = it & 1 ? a.act0 : a.act1;
    md.par = it & 1;
    md.dense = c.dense != 0;
    md.mark = c.mark != 0;
    for (int64_t base = base0; base < a.n; base += step) {
      if (!resident) row_bounds(a, r, base + threadIdx.x / kLanes);
      small_window<BLOCK, W, V4>(a, s, md, base, it == it0, r, resident);
      __syncthreads();  // the next window clears the queues and change flags
    }
    if (!kOne && a.gdn && threadIdx.x == 0) small_graph_changes(a, s);
    const uint32_t payload = ((s.cnt[0][2] + s.cnt[1][2] + s.cnt[2][2]) & kDnMask) | s.events;
    if (threadIdx.x == 0) {
      const uint32_t processed = s.cnt[0][0] + s.cnt[1][0] + s.cnt[2][0], edges = s.cnt[0][1] + s.cnt[1][1] + s.cnt[2][1];
      if constexpr (kOne) {
        s.processed_of[it - it0] = processed;
        s.edges_of[it - it0] = edges;
      } else {
        a.rec[(size_t)(it - it0) * kSmallGrid + blockIdx.x] = ((unsigned long long)processed << 32) | edges;
      }
    }
    // the classes of kLanes and kGroup lanes are the tier table's first two tiers
    if (threadIdx.x < 8) s.tstat[1 + threadIdx.x / 4][threadIdx.x % 4] += s.cnt[threadIdx.x / 4][threadIdx.x % 4];
    __syncthreads();
    if (threadIdx.x < 12) s.cnt[threadIdx.x / 4][threadIdx.x % 4] = 0;
    const uint32_t got = small_arrive(a, s, m, payload, all);
    uint32_t leave = got & (kAbort | kDecline);
    if (kOne || all || blockIdx.x == 0) {
      if (!leave) {
        if (s.acc[meeting_copy(m)][1] & kDecline)
          leave = kDecline;
        else
          small_decide(a, s, m, c);
      }
      if (!kOne && !all) {
        __syncthreads();
        small_release(a, m, leave | (c.done ? kDone : 0) | (c.dense ? kDense : 0) | (c.mark ? kMark : 0) |
                                (c.error ? kError : 0));
      }
    } else {
      c.done = (got & kDone) != 0;
      c.dense = (got & kDense) != 0;
      c.mark = (got & kMark) != 0;
      c.error = (got & kError) != 0;
    }
    ++m;
    ++it;
    if (leave) {
      if (blockIdx.x == 0 && threadIdx.x == 0) a.result->status = leave & kAbort ? kSmallAborted : kSmallDeclined;
      return;
    }
    if (c.done) break;
  }
  // this workgroup's counts of the whole call, summed after the next meeting
  if (!kOne && a.stats)
    for (int i = threadIdx.x; i < F; i += BLOCK) a.tier_rec[(size_t)blockIdx.x * F + i] = (&s.tstat[0][0])[i];
  const int32_t *L = it & 1 ? a.lab1 : a.lab0;
  const int64_t v0 = (int64_t)blockIdx.x * BLOCK + threadIdx.x, stride = (int64_t)gridDim.x * BLOCK;
  Forest<BLOCK> f;
  if constexpr (kOne) {
    f.p = s.parent;
    // the labels move to s.root, which names them until the flattening
    __syncthreads();
    for (int v = threadIdx.x; v < a.n; v += BLOCK) s.root[v] = s.lab[it & 1][v];
    __syncthreads();
  } else {
    f.p = a.parent;
  }
  bool ok = true;
  if (a.split && !c.error) {
    for (int64_t base = base0; base < a.n; base += step) split_link(a, s, f, L, base);
    ok = small_meet(a, s, m++);
    if (ok && a.stats) small_totals(a, s, it - it0);
    if (ok) {
      for (int64_t v = v0; v < a.n; v += stride) {
        if (!splits(a, v)) continue;
        const int32_t q = f.root((int32_t)v), l = kOne ? s.root[v] : L[v];
        f.p[v] = q;
        a.cp[v] = ((unsigned long long)(uint32_t)l << 32) | (uint32_t)q;
        if constexpr (kOne)
          s.rep[l] = q;
        else
          a.rep[l] = q;
      }
      ok = small_meet(a, s, m++);
    }
    if (ok) {
      for (int64_t base = base0; base < a.n; base += step) split_hooks(a, s, f, base);
      ok = small_meet(a, s, m++);
    }
    if (ok)
      for (int64_t v = v0; v < a.n; v += stride)
        if (splits(a, v)) a.out[v] = f.root((int32_t)v);
  } else {
    for (int64_t v = v0; v < a.n; v += stride) {
      if constexpr (kOne)
        a.out[v] = s.root[v];
      else if (a.out != L)
        a.out[v] = L[v];
    }
    if (a.stats) {
      ok = small_meet(a, s, m++);
      if (ok) small_totals(a, s, it - it0);
    }
  }
  if (blockIdx.x != 0) return;
  if (a.session)
    for (int64_t g = threadIdx.x; g < a.graphs; g += BLOCK) {
      a.gdone_host[g] = a.gdone[g];
      a.giters_host[g] = a.giters[g];
    }
  for (int q = threadIdx.x; a.stats && q < it - it0; q += BLOCK) {
    a.result->changed[q] = s.dn_of[q];
    a.result->marked[q] = s.marked[q];
  }
  if (threadIdx.x == 0) {
    a.result->ctrl = c;
    a.result->nnz = nnz;
    a.result->status = ok ? kSmallOk : kSmallAborted;
  }
}

}  // namespace

namespace {

template <int BLOCK>
void launch_rows(const SmallArgs &a, int grid, hipStream_t s) {
  const bool v4 = ((uintptr_t)a.cols & 15) == 0 && ((uintptr_t)a.w & 15) == 0;
  if (a.w) {
    if (v4)
      small_lpa<BLOCK, true, true><<<grid, BLOCK, 0, s>>>(a);
    else
      small_lpa<BLOCK, true, false><<<grid, BLOCK, 0, s>>>(a);
  } else {
    if (v4)
      small_lpa<BLOCK, false, true><<<grid, BLOCK, 0, s>>>(a);
    else
      small_lpa<BLOCK, false, false><<<grid, BLOCK, 0, s>>>(a);
  }
}

}  // namespace

hipError_t launch_small(const SmallArgs &a, int grid, hipStream_t s) {
  if (grid < 1 || grid > kSmallGrid) return hipErrorInvalidValue;
  if (a.n <= kSmallOne && !a.gdn)
    launch_rows<kOneBlock>(a, 1, s);
  else
    launch_rows<kBlock>(a, grid, s);
  return hipGetLastError();
}

}  // namespace gsl
