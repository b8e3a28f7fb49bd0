// Device code shared by the kernels: wavefront scans and searches.
#ifndef DGC_DEVICE_H_
#define DGC_DEVICE_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dgc {

// Inclusive prefix sum over the 64 lanes of a wavefront; every lane must be active.  Data-parallel
// primitives move the operand between lanes inside the vector unit (shifts by 1, 2, 4, 8 inside a row of
// 16 lanes, then the last lane of a row to the rows behind it), six dependent additions in all, where
// __shfl_up goes through the LDS unit six times.
__device__ __forceinline__ uint32_t wave_inclusive_sum(uint32_t x) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);  // row_shr:1
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);  // row_shr:2
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);  // row_shr:4
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);  // row_shr:8
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);  // row_bcast:15 to rows 1 and 3
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);  // row_bcast:31 to rows 2 and 3
  return x;
}

// The last lane's value of an inclusive sum: the sum over the wavefront, the same in every lane.
__device__ __forceinline__ uint32_t wave_last(uint32_t x) { return (uint32_t)__builtin_amdgcn_readlane((int)x, 63); }

__device__ __forceinline__ uint32_t wave_sum(uint32_t x) { return wave_last(wave_inclusive_sum(x)); }

// The largest of the wavefront's values, the same in every lane.
__device__ __forceinline__ uint32_t wave_max(uint32_t x) {
  auto larger = [](uint32_t a, int b) { return a > (uint32_t)b ? a : (uint32_t)b; };
  x = larger(x, __builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false));
  x = larger(x, __builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false));
  x = larger(x, __builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false));
  x = larger(x, __builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false));
  x = larger(x, __builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false));
  x = larger(x, __builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false));
  return wave_last(x);
}

// Where to look first for x in an ascending list of m values that lie in [from, to): the place it has if they
// are spread evenly, and the standard deviation of that place if they are spread at random.  Only the number
// of probes depends on it.
struct Guess {
  int place, sigma;
  __device__ __forceinline__ Guess(int m, int32_t x, int32_t from, int32_t to) {
    float f = (float)(x - from) / (float)(to - from);
    f = f < 0.0f ? 0.0f : f > 1.0f ? 1.0f : f;
    const float at = f * (float)m;
    place = at < (float)m ? (int)at : m;
    sigma = (int)sqrtf((float)m * f * (1.0f - f));
  }
};

// One round of PROBES probes around a guess, by as many neighbouring lanes (this one is number `sub`, the
// group's votes start at bit `shift` of a ballot): the probe of this lane, and after the vote the bracket
// [lo, hi] that the answer lies in.  The probes cover four standard deviations to either side.
template <int PROBES>
struct GuessRound {
  int start, step, last;  // probe i is at clamp(start + i * step, 0, last)
  __device__ __forceinline__ GuessRound(const Guess& g, int m) {
    step = g.sigma / (PROBES / 8) + 1;
    start = g.place - PROBES / 2 * step;
    last = m - 1;
  }
  __device__ __forceinline__ int at(int i) const {
    const int64_t p = (int64_t)start + (int64_t)i * step;
    return p < 0 ? 0 : p > last ? last : (int)p;
  }
  __device__ __forceinline__ void narrow(int below, int& lo, int& hi) const {  // `below` probes are less than x: a prefix
    if (below < PROBES) hi = at(below);
    if (below > 0) lo = at(below - 1) + 1;
    if (lo > hi) lo = hi;
  }
};
constexpr int kGuessFrom = 1024;  // shorter lists take two rounds of 32 probes anyhow

// Positions [lo, hi) of the list L[0, m) whose values lie in [xa, xb), for a list in which
// "value < xa" and "value < xb" are monotone; every lane of the wavefront takes part and
// gets the same answer.  GUESS: the values lie in [from, to), about evenly.
template <bool GUESS>
__device__ __forceinline__ void wave_equal_range(const int32_t* __restrict__ L, int m, int32_t xa, int32_t xb,
                                                 int32_t from, int32_t to, int lane, int& out_lo, int& out_hi) {
  const int half = lane >> 5;  // 0: lower bound of xa, 1: lower bound of xb
  const int sub = lane & 31;
  const int32_t x = half ? xb : xa;
  int lo = 0, hi = m;  // the answer of this lane's half lies in [lo, hi]
  if (GUESS && m > kGuessFrom) {
    const GuessRound<32> r(Guess(m, x, from, to), m);
    const unsigned long long votes = __ballot(L[r.at(sub)] < x);
    r.narrow(__popc((uint32_t)(votes >> (32 * half))), lo, hi);
  }
  while (__ballot(hi > lo)) {
    const int span = hi - lo;
    const int step = (span + 31) >> 5;
    const int pos = lo + sub * step;
    const bool less = span > 0 && pos < hi && L[pos] < x;
    const unsigned long long votes = __ballot(less);
    const int c = __popc((uint32_t)(votes >> (32 * half)));  // probes below x form a prefix
    if (span > 0) {
      if (c == 0) {
        hi = lo;
      } else {
        const int next = lo + c * step;
        lo = lo + (c - 1) * step + 1;
        hi = next < hi ? next : hi;
      }
    }
  }
  out_lo = __shfl(lo, 0);
  out_hi = __shfl(lo, 32);
}

}  // namespace dgc
#endif  // DGC_DEVICE_H_
