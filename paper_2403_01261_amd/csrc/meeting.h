// The words through which the workgroups of a small-graph launch meet
// (small.hip): plain arithmetic, for the device and for a host compiler.
#pragma once

#include <cstdint>

namespace gsl {

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
