// Rows held in registers: 16-byte row loads and label gathers of one thread,
// and rows sorted across the lanes of a wavefront slice.
#pragma once

#include <utility>

#include "device_common.h"

namespace gsl {

namespace {

template <bool O32>
__device__ __forceinline__ uint32_t gather_label(const int32_t *__restrict__ C, int32_t c) {
  if constexpr (O32)
    return *reinterpret_cast<const uint32_t *>(reinterpret_cast<const char *>(C) + ((uint32_t)c << 2));
  else
    return (uint32_t)C[c];
}

// Row entries [b, b + d) of a 4-byte array into r[0..D), `fill` beyond d.
// V4: 16-byte loads of the aligned words that cover the row -- at most
// D / 4 + 1 loads instead of D, vector memory instructions being what the
// thread-per-vertex sweep waits on -- then shifted into place in registers.
// Only words that hold an entry of the row are loaded (none where d is 0: a lane
// past its row's end, whose b may lie past the array's), and an aligned 16-byte
// word lies within one page (the page of that entry), so no load reaches
// unmapped memory.  V4 needs a 16-byte aligned array.  Register indices are
// template constants (index sequences rather than loops), so the words stay
// in registers.
template <int... Q>
__device__ __forceinline__ void load_words(const uint4 *__restrict__ p, int lim, uint32_t fill, uint32_t *t,
                                           std::integer_sequence<int, Q...>) {
  ((t[4 * Q] = fill, t[4 * Q + 1] = fill, t[4 * Q + 2] = fill, t[4 * Q + 3] = fill), ...);
  ([&] {
    if (4 * Q < lim) {
      const uint4 v = p[Q];
      t[4 * Q] = v.x;
      t[4 * Q + 1] = v.y;
      t[4 * Q + 2] = v.z;
      t[4 * Q + 3] = v.w;
    }
  }(), ...);
}

// Word K + sh of t (sh in 0..3).  The empty asm hands the selects plain
// register values: a select between two array elements would otherwise
// become a load through a selected address, which keeps the array in
// scratch memory.
template <int K>
__device__ __forceinline__ uint32_t shifted_word(const uint32_t *t, int sh, int d, uint32_t fill) {
  uint32_t c0 = t[K], c1 = t[K + 1], c2 = t[K + 2], c3 = t[K + 3];
  asm("" : "+v"(c0), "+v"(c1), "+v"(c2), "+v"(c3));
  const uint32_t lo = (sh & 1) ? c1 : c0, hi = (sh & 1) ? c3 : c2;
  return K < d ? ((sh & 2) ? hi : lo) : fill;
}

template <int... K>
__device__ __forceinline__ void shift_words(const uint32_t *t, int sh, int d, uint32_t fill, uint32_t *r,
                                            std::integer_sequence<int, K...>) {
  ((r[K] = shifted_word<K>(t, sh, d, fill)), ...);
}

template <int D, bool V4>
__device__ __forceinline__ void load_row(const uint32_t *__restrict__ x, int64_t b, int d, uint32_t fill,
                                         uint32_t (&r)[D]) {
  if constexpr (!V4) {
#pragma unroll
    for (int k = 0; k < D; ++k) r[k] = k < d ? x[b + k] : fill;
  } else {
    constexpr int Q = D / 4 + 1;
    const int64_t b4 = b & ~int64_t(3);
    const int sh = (int)(b - b4);
    uint32_t t[4 * Q];
    load_words(reinterpret_cast<const uint4 *>(x + b4), d > 0 ? sh + d : 0, fill, t, std::make_integer_sequence<int, Q>{});
    shift_words(t, sh, d, fill, r, std::make_integer_sequence<int, D>{});
  }
}

// Value of x in lane (this lane ^ X): a DPP move where one reaches (quad
// permutations, mirrors of 8 and 16 lanes), else an LDS-crossbar swizzle or
// permute.
template <int X>
__device__ __forceinline__ uint32_t lane_xor(uint32_t x) {
  if constexpr (X == 1)
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, true);
  else if constexpr (X == 2)
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xF, 0xF, true);
  else if constexpr (X == 3)
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x1B, 0xF, 0xF, true);
  else if constexpr (X == 7)
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xF, 0xF, true);
  else if constexpr (X == 15)
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x140, 0xF, 0xF, true);
  else if constexpr (X < 32)
    return (uint32_t)__builtin_amdgcn_ds_swizzle((int)x, (X << 10) | 0x1F);
  else
    return (uint32_t)__shfl_xor((int)x, X, kWave);
}

// One compare-exchange across lanes: register r against register RR of lane ^ X;
// the lanes of the upper half (`upper`) keep the larger.
template <int R, bool W, int X, bool MIRROR>
__device__ __forceinline__ void lanes_exchange(uint32_t (&l)[R], uint32_t (&w)[R], bool upper) {
  uint32_t ol[R], ow[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    ol[r] = lane_xor<X>(l[MIRROR ? R - 1 - r : r]);
    if constexpr (W) ow[r] = lane_xor<X>(w[MIRROR ? R - 1 - r : r]);
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if constexpr (W) {
      const bool take = upper ? ol[r] > l[r] : ol[r] < l[r];
      l[r] = take ? ol[r] : l[r];
      w[r] = take ? ow[r] : w[r];
    } else {
      const uint32_t lo = l[r] < ol[r] ? l[r] : ol[r], hi = l[r] < ol[r] ? ol[r] : l[r];
      l[r] = upper ? hi : lo;
    }
  }
}

template <int R, bool W, int X>
__device__ __forceinline__ void lanes_half_clean(uint32_t (&l)[R], uint32_t (&w)[R], int lane) {
  if constexpr (X >= 1) {
    lanes_exchange<R, W, X, false>(l, w, (lane & X) != 0);
    lanes_half_clean<R, W, X / 2>(l, w, lane);
  }
}

// Bitonic sequence of R registers into ascending order.
template <int R, bool W>
__device__ __forceinline__ void clean_registers(uint32_t (&l)[R], uint32_t (&w)[R]) {
#pragma unroll
  for (int k = R / 2; k >= 1; k >>= 1)
#pragma unroll
    for (int x = 0; x < R; ++x) {
      if (x & k) continue;
      const int y = x + k;
      const uint32_t lx = l[x], ly = l[y];
      if constexpr (W) {
        const bool sw = lx > ly;
        const uint32_t wx = w[x];
        w[x] = sw ? w[y] : wx;
        w[y] = sw ? wx : w[y];
      }
      l[x] = lx < ly ? lx : ly;
      l[y] = lx < ly ? ly : lx;
    }
}

// Merges the sorted slices of H lanes into sorted slices of 2H lanes, for H =
// 1, 2, .. below L, while a row of the wavefront is longer than H slices
// (`longest` entries, uniform; a slice past a row's end holds no-label values,
// which are last already).
template <int L, int R, bool W, int H>
__device__ __forceinline__ void lanes_merge(uint32_t (&l)[R], uint32_t (&w)[R], int lane, int longest) {
  if constexpr (H < L) {
    if (longest <= H * R) return;
    lanes_exchange<R, W, 2 * H - 1, true>(l, w, (lane & H) != 0);
    lanes_half_clean<R, W, H / 2>(l, w, lane);
    clean_registers<R, W>(l, w);
    lanes_merge<L, R, W, 2 * H>(l, w, lane, longest);
  }
}

// Largest argmax key of a row whose L * R labels (no-label values last) are in
// the registers of L lanes, R consecutive entries each; every lane returns
// it.  Each lane sorts its slice, the slices are merged across the lanes, and
// one pass over the sorted runs sums their weights; a run that began in
// another lane gets the sum it has reached there.  Partial sums never exceed
// a run's total, so the largest key seen is the winner's.
template <int L, int R, bool W>
__device__ __forceinline__ unsigned long long lanes_best(uint32_t (&lab)[R], uint32_t (&w)[R], int longest) {
  const int lane = threadIdx.x % L;
  sort_by_label<R, W>(lab, w);
  lanes_merge<L, R, W, 1>(lab, w, lane, longest);
  // labels ascend, so a strictly larger sum is the only reason to change the
  // lane's best; its first label stands where every sum is zero
  uint32_t s = 0, head = 0, bs = 0, bl = lab[0];
  bool in_head = true;
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const uint32_t wk = W ? w[k] : 1u;
    const bool same = k > 0 && lab[k] == lab[k - 1];
    if (k > 0) in_head = in_head && same;
    s = same ? s + wk : wk;
    head = in_head ? s : head;
    const bool more = s > bs && lab[k] != kNoLabel;
    bs = more ? s : bs;
    bl = more ? lab[k] : bl;
  }
  unsigned long long best = bl != kNoLabel ? argmax_key(bl, bs) : 0ull;
  if constexpr (L > 1) {
    // sum of the run that ends the lane, carried over lanes of one label
    uint32_t tail = s;
    const uint32_t before = (uint32_t)__shfl_up((int)lab[R - 1], 1, L);
    const bool joins = lane > 0 && before == lab[0];
    if constexpr (L > 2) {
      bool open = joins && lab[0] == lab[R - 1];  // the run of the lane before goes on through this one
#pragma unroll
      for (int o = 1; o < L; o <<= 1) {
        const uint32_t t = (uint32_t)__shfl_up((int)tail, o, L);
        const int q = __shfl_up((int)open, o, L);
        if (open) tail += t;
        open = open && lane >= o && q;
      }
    }
    const uint32_t carry = (uint32_t)__shfl_up((int)tail, 1, L);
    if (joins && lab[0] != kNoLabel) {
      const unsigned long long key = argmax_key(lab[0], head + carry);
      best = key > best ? key : best;
    }
    best = group_max<L>(best);
  }
  return best;
}

}  // namespace

}  // namespace gsl
