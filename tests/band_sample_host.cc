// How often the floor of an exact selection misses, and how often it may go into the streaming pass: the sample of
// select_kernel (1024 draws of 32 neighbours, held by 16 wavefronts of 64 threads) drawn from tensors of different
// structure, and the decision of csrc/dgc_band.h on it.
#include "dgc_band.h"

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <random>
#include <vector>

namespace {

std::mt19937_64 gen(5);
double uniform() { return (double)(gen() >> 11) * 0x1p-53; }

struct Tensor {  // values above 1 where `large`, below it elsewhere
  long n;
  double share_large;
  std::function<bool(long)> large;
};

// runs of `run` neighbours placed anew, `count` of them
Tensor runs(long n, long run, long count) {
  std::vector<long> start(count);
  for (long& s : start) s = (long)(uniform() * (double)(n / run)) * run;
  std::sort(start.begin(), start.end());
  return {n, (double)(std::unique(start.begin(), start.end()) - start.begin()) * (double)run / (double)n, [start, run](long e) {
            auto it = std::upper_bound(start.begin(), start.end(), e);
            return it != start.begin() && e < it[-1] + run;
          }};
}

}  // namespace

// band_sample_host <density> <run> <count> <n> <draws>: prints the shares of draws that went into the pass, that missed there,
// and that missed where the band was collected
int main(int argc, char** argv) {
  if (argc != 6) return 2;
  const double density = std::atof(argv[1]);
  const long run = std::atol(argv[2]), count = std::atol(argv[3]), n = std::atol(argv[4]);
  const int draws = std::atoi(argv[5]);
  constexpr int kBlocks = 1024, kBlock = 32;
  int passed = 0, missed_there = 0, missed_collected = 0;
  std::vector<float> key(kBlocks * kBlock), sorted;
  for (int d = 0; d < draws; ++d) {
    const Tensor t = count > 0 ? runs(n, run, count) : Tensor{n, 0.0, [](long) { return false; }};
    // uniform values in [1, 2) where large and [0, 1) elsewhere: the exact threshold of the wanted share
    const float exact = (float)(density <= t.share_large ? 2.0 - density / t.share_large : 1.0 - (density - t.share_large) / (1.0 - t.share_large));
    for (int b = 0; b < kBlocks; ++b) {
      const long first = (long)(uniform() * (double)(n / kBlock)) * kBlock;
      for (int e = 0; e < kBlock; ++e) key[b * kBlock + e] = (float)(uniform() + (t.large(first + e) ? 1.0 : 0.0));
    }
    const dgc::BandRanks at(density, (double)key.size());
    sorted = key;
    const int rank = (int)at.floor_in_pass();
    std::nth_element(sorted.begin(), sorted.begin() + rank, sorted.end(), std::greater<float>());
    const float floor = sorted[rank];
    uint32_t bits, above = 0, keys = 0, squares = 0;
    std::memcpy(&bits, &floor, 4);
    for (int b = 0; b < kBlocks; ++b) {
      uint32_t c = 0;
      for (int e = 0; e < kBlock; ++e) {
        c += key[b * kBlock + e] >= floor;
        above += key[b * kBlock + e] > floor;
      }
      keys += c;
      squares += c * c;
    }
    if (!dgc::BandRanks::clustered(keys, squares) && !at.tied(above, bits)) {
      ++passed;
      missed_there += floor > exact;
      continue;
    }
    // the floor of the collected band: the smallest of the wavefronts' t-th largest thread maxima
    const int t_th = (int)(std::ceil(at.mid) + at.reach()) / 16 + 1;
    float lowest = 3.0f;
    for (int wave = 0; wave < 16; ++wave) {
      std::vector<float> top(64, 0.0f);
      for (int lane = 0; lane < 64; ++lane)
        for (int i = 0; i < 8; ++i) {
          const int quad = wave * 64 + lane + i * 1024;
          for (int c = 0; c < 4; ++c) top[lane] = std::max(top[lane], key[quad * 4 + c]);
        }
      std::nth_element(top.begin(), top.begin() + (t_th - 1), top.end(), std::greater<float>());
      lowest = std::min(lowest, top[t_th - 1]);
    }
    missed_collected += lowest > exact;
  }
  std::printf("%.5f %.5f %.5f\n", (double)passed / draws, (double)missed_there / draws, (double)missed_collected / draws);
  return 0;
}
