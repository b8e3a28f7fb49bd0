// Which words of a payload's arrays the receive side reads: plain arithmetic, for the host too.
#ifndef DGC_PROBE_H_
#define DGC_PROBE_H_

#include <stdint.h>

namespace dgc {

// First round of a search in a list of up to 2^31 - 1 values: 1 << shift probes (32 at least), evenly spaced over a list of m values.  The last probe's position stays below
// m + 2^shift, and every product below in 32 bits without a sign, because a probe beyond the last is told by its
// number, not by where it would lie: in a list of 2^30 values and more, 63 steps of a round of 32 are 2^31.
struct FirstRound {
  uint32_t m, step, probes;
  constexpr FirstRound(int length, int shift)
      : m((uint32_t)length), step((m + (1u << shift) - 1u) >> shift), probes(1u << shift) {}
  constexpr bool asks(uint32_t probe) const { return probe < probes && probe * step < m; }
  constexpr int at(uint32_t probe) const { return asks(probe) ? (int)(probe * step) : 0; }
  // the answer lies in [lo, hi] if `below` probes, a prefix of those that ask, are less than what is looked for
  constexpr int lo(int below) const { return below > 0 ? (int)((uint32_t)(below - 1) * step + 1u) : 0; }
  constexpr int hi(int below) const { return below > 0 ? (int)((uint32_t)below * step < m ? (uint32_t)below * step : m) : 0; }
};

// log2 of the probes that the range merge's first round makes in a list of m values, whatever other list is searched
// beside it: enough to leave brackets of 32, for which one more round of 32 is the last, in up to 4224 values; in
// longer lists, which take three rounds anyway, the fewest.
constexpr int first_round_shift(int m) { return m > 128 * 33 ? 5 : m > 64 * 33 ? 7 : 6; }

// Four consecutive slots of which some lie outside [head, end), the slots that hold a part's pairs.  Those behind
// `end` may not exist: a payload need not go on behind its last pair.  Those before `head` do, as far back as the
// payload's first slot (`pos` is the place of `slot` in the payload).  So one load of four that ends at `end` gets all
// that are wanted, and only at the start of a payload it takes one load each.
struct EdgeFour {
  bool any;    // some are wanted
  int back;    // the load starts this many slots before `slot` (0 to 3)
  bool whole;  // ... and not before the payload
  constexpr EdgeFour(int slot, int head, int end, int pos)
      : any(slot < end && head - slot < 4), back(any && end - slot < 4 ? 4 - (end - slot) : 0), whole(any && pos >= back) {}
  static constexpr bool wanted(int slot, int head, int end) { return slot >= head && slot < end; }
};

}  // namespace dgc
#endif  // DGC_PROBE_H_
