// Where the band of an exact selection lies in its sample, and whether its floor may be the threshold of the streaming
// pass: plain arithmetic, for the host too.
#ifndef DGC_BAND_H_
#define DGC_BAND_H_

#include <math.h>
#include <stdint.h>

#ifdef __HIPCC__
#define DGC_BOTH __host__ __device__
#else
#define DGC_BOTH
#endif

namespace dgc {

struct BandRanks {
  double mid, spread;  // sampled keys above the exact threshold: expected, and the standard deviation if each is drawn by itself
  DGC_BOTH BandRanks(double share, double sample) : mid(share * sample), spread(sqrt(mid * (1.0 - share))) {}

  // The floor in the pass lies five standard deviations and 16 keys below the wanted rank, if the sample can be relied on.
  DGC_BOTH double floor_in_pass() const { return ceil(mid) + 16.0 + ceil(5.0 * spread); }
  // Neighbours are no independent draws: keys that come c to a block have a standard deviation sqrt(c) times as large.
  // `keys` of the sample do not lie below the floor, and the sum over its blocks of the squares of their numbers is
  // `squares`: c is about squares / keys, and up to two the floor is still more than five of them away.
  DGC_BOTH static bool clustered(uint32_t keys, uint32_t squares) { return squares > 2u * keys + 16u; }
  // With many equal to the floor, those above it may be fewer than are wanted: half the distance is asked for.  (Above a
  // floor of zero is everything that could be wanted.)
  DGC_BOTH bool tied(uint32_t above, uint32_t floor_key) const {
    return floor_key != 0u && (double)above < mid + 0.5 * (floor_in_pass() - mid);
  }

  // How far the band reaches to either side of the wanted rank where its keys are collected: seven standard deviations and
  // 32 keys.
  DGC_BOTH double reach() const { return 32.0 + ceil(7.0 * spread); }
};

}  // namespace dgc
#endif  // DGC_BAND_H_
