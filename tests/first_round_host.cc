// Caller of the first round's arithmetic (csrc/dgc_probe.h) on the host: every probe of all 128 lanes' numbers in the
// list, and the bracket it leaves around the answer.  The list is its own positions, so that no memory is needed.
#include "dgc_probe.h"

#include <algorithm>
#include <cstdio>
#include <vector>

int main() {
  std::vector<int> lengths;
  for (int m = 0; m <= 4300; ++m) lengths.push_back(m);
  const int around[] = {1 << 16, 1 << 24, (1 << 30) - 64, 1073741824, 1090785344, 1090785345, 1431655766, 2147483647 - 200};
  for (int a : around)
    for (int d = -70; d <= 130; ++d) lengths.push_back(a + d);
  for (int d = 0; d <= 70; ++d) lengths.push_back(2147483647 - d);
  long checked = 0;
  for (int m : lengths) {
    const dgc::FirstRound own(m, dgc::first_round_shift(m));
    if (m <= 4224 && own.step > 33) return std::printf("m %d: brackets of %u\n", m, own.step - 1), 1;
    if (m > 4224 && own.probes != 32) return std::printf("m %d: %u probes\n", m, own.probes), 1;
    for (int shift = 5; shift <= 7; ++shift) {
      const dgc::FirstRound r(m, shift);
      std::vector<int> asked;
      for (uint32_t p = 0; p < 128; ++p) {
        const int at = r.at(p);
        if (at < 0 || (m > 0 && at >= m) || (m == 0 && at != 0)) return std::printf("m %d shift %d probe %u at %d\n", m, shift, p, at), 1;
        if (r.asks(p)) {
          if (p >= 1u << shift) return std::printf("m %d shift %d probe %u asks\n", m, shift, p), 1;
          if (!asked.empty() && at <= asked.back()) return std::printf("m %d shift %d probe %u does not ascend\n", m, shift, p), 1;
          asked.push_back(at);
        }
      }
      std::vector<int> answers = {0, m / 3, m / 2, m - (m > 0), m};
      for (int a : asked)
        for (int d = -1; d <= 2; ++d)
          if ((long)a + d >= 0 && (long)a + d <= m) answers.push_back(a + d);
      for (int x : answers) {  // the first position not below x is x itself
        const int below = (int)(std::lower_bound(asked.begin(), asked.end(), x) - asked.begin());
        const int lo = r.lo(below), hi = r.hi(below);
        if (!(0 <= lo && lo <= x && x <= hi && hi <= m)) return std::printf("m %d shift %d answer %d in [%d, %d]\n", m, shift, x, lo, hi), 1;
        if ((unsigned)(hi - lo) >= std::max(1u, r.step)) return std::printf("m %d shift %d bracket [%d, %d]\n", m, shift, lo, hi), 1;
        ++checked;
      }
    }
  }
  std::printf("ok %ld\n", checked);
  return 0;
}
