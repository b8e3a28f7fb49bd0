// Caller of the arithmetic of a part's first and last loads (csrc/dgc_probe.h) on the host: a payload of `extent` pairs,
// a part whose pairs are [first, first + length), slots counted from the line below its first pair.  Every slot that is
// read has to be a slot of the payload that is not behind the part's last pair, and every pair has to arrive in its place.
#include "dgc_probe.h"

#include <cstdio>

int main() {
  long checked = 0;
  for (int head = 0; head < 32; ++head) {
    for (int first = 0; first < 40; ++first) {
      for (int length = 1; length < 300; length += length < 40 ? 1 : 29) {
        const int end = head + length, pos0 = first - head;  // slot s is pair pos0 + s of the payload, which ends at the part's
        for (int slot = 0; slot < end + 12; slot += 4) {
          const dgc::EdgeFour four(slot, head, end, pos0 + slot);
          for (int k = 0; k < 4; ++k) {
            const bool wanted = dgc::EdgeFour::wanted(slot + k, head, end);
            if (wanted != (slot + k >= head && slot + k < end)) return std::printf("wanted\n"), 1;
            if (wanted && !four.any) return std::printf("head %d end %d slot %d: pair %d lost\n", head, end, slot, k), 1;
            if (four.whole) {
              const int read = slot - four.back + k;
              if (read >= end || pos0 + read < 0) return std::printf("head %d first %d end %d slot %d reads %d\n", head, first, end, slot, read), 1;
              if (wanted && k + four.back > 3) return std::printf("head %d end %d slot %d: pair %d not loaded\n", head, end, slot, k), 1;
            }
            ++checked;
          }
          if (four.whole && !four.any) return std::printf("loads nothing wanted\n"), 1;
        }
      }
    }
  }
  std::printf("ok %ld\n", checked);
  return 0;
}
