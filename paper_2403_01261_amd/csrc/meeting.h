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
// CU, which fit an idle device exactly, left one of two concurrent launches
// waiting for its limit (a server with two slots: p50 805 ms at 2,000 requests
// a second).  kSmallGrid of them where a device has 256 CUs or more; a
// partitioned one has fewer.
constexpr int kSmallGrid = 512;
constexpr int64_t kSmallOne = 256;     // graphs up to here run in one workgroup, in LDS
constexpr int64_t kSmallWindow = 128;  // vertices that a workgroup of a larger launch takes at a time
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
// small_most for a call alone.  Beside another call of the library a launch is
// taken up to half a workgroup per CU only: each launch deals its workgroups out
// over the XCDs from the first one on, so two that just fit the device may not
// fit an XCD, and a workgroup of another call that needs much LDS holds up those
// queued behind it.
constexpr int small_room(int cus, bool alone) { return alone ? small_most(cus) : small_most(cus) / 4; }

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
