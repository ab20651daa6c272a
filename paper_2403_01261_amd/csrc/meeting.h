// How many workgroups a small-graph launch has and the words through which they
// meet (small.hip): plain arithmetic, for the device and for a host compiler.
#pragma once

#include <cstdint>

namespace gsl {

// Most workgroups of a launch, all resident at once: two per CU, with weights
// one.  Registers and LDS are given out in one piece, so what a CU has room for
// is what fits however the workgroups there lie, other streams' kernels having
// come and gone between them: beside one of 128 registers (or of 256) a second
// of 128 always fits, a third need not, nor a second of 256.  Four and two per
// CU, which fit an idle device exactly, leave one of two concurrent launches
// waiting for its limit now and then (a server with two slots at 2,000 and 5,000
// requests a second: 17 and 24 waits of 3,000 and 870 calls ran out, p99 8 and 10
// ms; none here, p99 3.0 and 4.5).  kSmallGrid of them where a device has 256 CUs
// or more; a partitioned one has fewer.
constexpr int kSmallGrid = 512;
constexpr int64_t kSmallOne = 256;     // graphs up to here run in one workgroup, in LDS
constexpr int64_t kSmallWindow = 128;  // vertices that a workgroup of a larger launch takes at a time
constexpr uint32_t kSmallPerPass = 8;  // rows of 65 - 512 entries that it takes at a time
constexpr int small_most(int cus) { return 2 * cus < kSmallGrid ? 2 * cus : kSmallGrid; }

// Workgroups of a launch on n vertices, and how many of small_most each counts
// for: with weights two, for its registers.
constexpr int small_share(bool weighted) { return weighted ? 2 : 1; }
constexpr int small_grid(int64_t n, bool weighted, bool batch, int cus) {
  if (n <= kSmallOne && !batch) return 1;
  const int64_t g = (n + kSmallWindow - 1) / kSmallWindow, most = small_most(cus) / small_share(weighted);
  return (int)(g < most ? g : most);
}

// Workgroups of small-graph launches that a device may hold at once: all of
// small_most for a call alone, a quarter of them beside another call of the
// library, where the rest takes the general path.  Either fits (of 24,000 calls
// of that server no wait ran out): the line decides who waits for whom.  At
// 2,000, 5,000 and 20,000 requests a second p50 is 0.75, 1.63 and 6.0 ms and p99
// 3.0, 4.5 and 26 ms with a quarter, 0.63, 1.38 and 7.7 and 2.6, 5.6 and 28 with
// all of them.
constexpr int small_room(int cus, bool alone) { return alone ? small_most(cus) : small_most(cus) / 4; }

// Windows that a workgroup takes in every sweep.
constexpr int small_windows(int64_t n, int grid) {
  return ((int)((n + kSmallWindow - 1) / kSmallWindow) + grid - 1) / grid;
}

// What a window's rows of more than 64 entries cost in one sweep, in half
// microseconds: those of up to 512 go through the workgroup `per` at a time, the
// longer ones one by one.  e1, e2 and e3 are 64ths of rows of 65 - 128, 129 - 512
// and more entries.  small_rows_line is what the launches saved by the one kernel
// leave for that, by windows: where the rows cost more the general path, whose
// kernels spread them over the whole device, is the faster one.  Both are fitted
// to 236 graphs of 256 to 250,000 vertices with a hundredth to all of their rows
// of 80 to 1,500 entries: 80 of them ran slower in one launch than on the general
// path (8,000 vertices of 1,700 neighbours: 1,758 us instead of 540, with weights
// 3,818 instead of 750), 2 of those that the rule leaves there (0.97 and 0.98
// times as fast); 4,000 vertices, 30 % with 120 neighbours, run in 267 us instead
// of 623.
constexpr uint32_t small_rows_cost(bool weighted, uint32_t e1, uint32_t e2, uint32_t e3, uint32_t per) {
  const uint32_t r = e1 + e2, u1 = weighted ? 10 : 3, u2 = weighted ? 20 : 5, u3 = 10;
  const uint32_t passes = r >= 64 ? (r + 64 * per - 1) / (64 * per) * 64 : r;
  return (r ? passes * ((u1 * e1 + u2 * e2) / r) : 0) / 64 + u3 * e3 / 64;
}
constexpr uint32_t small_rows_line(int windows) { return windows < 6 ? 88u - 12u * (uint32_t)windows : 16u; }

// A workgroup posts meeting m in its own word and waits until every other has
// posted m.  It may post m + 1 while another still looks for its m, so each
// has two words, taken in turn: m + 2, which overwrites m, comes after all have
// posted m + 1 and so have read m.  The sums that a workgroup keeps of a
// meeting's words in LDS have two copies for the same reason: thread 0 clears
// those of m + 1 while a slower wavefront still reads those of m.
constexpr uint32_t kMeetingCopies = 2;
constexpr uint32_t meeting_copy(uint32_t meeting) { return meeting % kMeetingCopies; }

// A word: the launch's number (24 bits), the meeting's (8) and a payload.
constexpr unsigned long long meeting_word(uint32_t epoch, uint32_t meeting, uint32_t payload) {
  return ((unsigned long long)epoch << 40) | ((unsigned long long)meeting << 32) | payload;
}
constexpr bool meeting_posted(unsigned long long word, uint32_t epoch, uint32_t meeting) {
  return (word >> 32) == (meeting_word(epoch, meeting, 0) >> 32);
}

}  // namespace gsl
