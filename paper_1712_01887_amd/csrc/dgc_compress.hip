// HIP kernels of the DGC hot path for gfx950 (wave64, CDNA4).
//
// The path is memory-bound: one streaming pass reads g, u, v and writes u, v
// (20 bytes per element); everything else touches a sample or the sparse
// payload only.  No kernel here is a contraction, so no MFMA is used.
//
// Arithmetic contract (shared with nothing, stated for the reader): binary32,
// one rounding per operation, in this order
//     gs = g * scale;  t = m * u;  u' = t + gs;  v' = v + u'          (vanilla)
//     gs = g * scale;  s = u + gs; u' = m * s;   w = v + u'; v' = w + gs  (Nesterov)
// The file must be compiled with -ffp-contract=off so that no pair of these is
// fused; the threshold pass and the streaming pass evaluate v' with the same
// inline function, which makes the sampled threshold an exact member of the
// values the streaming pass later compares against it.

#include "dgc_device.h"
#include "dgc_internal.h"

namespace dgc {
namespace {

// ---------------------------------------------------------------------------
// Momentum correction (paper: equation 7; Algorithm 3 / Algorithm 4 update lines)
// ---------------------------------------------------------------------------
__device__ __forceinline__ void momentum_update(float g, float u, float v, float m, float scale,
                                                bool nesterov, float& u1, float& v1) {
  const float gs = g * scale;
  if (!nesterov) {
    const float t = m * u;
    u1 = t + gs;
    v1 = v + u1;
  } else {
    const float s = u + gs;
    u1 = m * s;
    const float w = v + u1;
    v1 = w + gs;
  }
}

// Zero fill of small pieces of the workspace (a kernel rather than a memset: the calls of
// the library may be captured into a HIP graph).
__global__ __launch_bounds__(256) void clear_words_kernel(uint32_t* __restrict__ p, size_t words) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < words; i += (size_t)gridDim.x * 256) p[i] = 0u;
}

// ---------------------------------------------------------------------------
// Clipping norm (paper: Section 3.2 "Local Gradient Clipping"; Appendix C eq. 12)
// ---------------------------------------------------------------------------
// Every workgroup accumulates squares in binary64 over a grid-stride range and stores
// one partial sum; nothing else.  The partials are added up, in a fixed order, by the
// kernel that runs next (every workgroup of the threshold selection does it for itself),
// so that the result does not depend on scheduling and no workgroup has to wait for
// another: a version in which the last workgroup to arrive finished the sum needed two
// chained device-scope atomics per workgroup and ran 6 us longer (52 against 46 us on
// 66 M elements).  (Small sets have no launch for it: see select_kernel.)
__global__ __launch_bounds__(kNormThreads) void norm_kernel(const float* __restrict__ g, int64_t n,
                                                            double* __restrict__ partials) {
  __shared__ double red[kNormThreads / 64];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int64_t nvec = n >> 2;
  const float4* __restrict__ g4 = reinterpret_cast<const float4*>(g);
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
  const int64_t stride = (int64_t)gridDim.x * kNormThreads;
  int64_t i = (int64_t)blockIdx.x * kNormThreads + tid;
  // four independent 16-byte loads in flight per thread; ordinary (cached) loads, because
  // the streaming pass reads g again right after this kernel
  for (; i + 3 * stride < nvec; i += 4 * stride) {
    const float4 x0 = g4[i];
    const float4 x1 = g4[i + stride];
    const float4 x2 = g4[i + 2 * stride];
    const float4 x3 = g4[i + 3 * stride];
    a0 += (double)x0.x * (double)x0.x;
    a1 += (double)x0.y * (double)x0.y;
    a2 += (double)x0.z * (double)x0.z;
    a3 += (double)x0.w * (double)x0.w;
    a0 += (double)x1.x * (double)x1.x;
    a1 += (double)x1.y * (double)x1.y;
    a2 += (double)x1.z * (double)x1.z;
    a3 += (double)x1.w * (double)x1.w;
    a0 += (double)x2.x * (double)x2.x;
    a1 += (double)x2.y * (double)x2.y;
    a2 += (double)x2.z * (double)x2.z;
    a3 += (double)x2.w * (double)x2.w;
    a0 += (double)x3.x * (double)x3.x;
    a1 += (double)x3.y * (double)x3.y;
    a2 += (double)x3.z * (double)x3.z;
    a3 += (double)x3.w * (double)x3.w;
  }
  for (; i < nvec; i += stride) {
    const float4 x = g4[i];
    a0 += (double)x.x * (double)x.x;
    a1 += (double)x.y * (double)x.y;
    a2 += (double)x.z * (double)x.z;
    a3 += (double)x.w * (double)x.w;
  }
  if (blockIdx.x == 0 && tid < (int)(n & 3)) {
    const double x = (double)g[(nvec << 2) + tid];
    a0 += x * x;
  }
  double acc = (a0 + a1) + (a2 + a3);
  for (int d = 32; d >= 1; d >>= 1) acc += __shfl_down(acc, d);
  if (lane == 0) red[wave] = acc;
  __syncthreads();
  if (tid == 0) {
    double s = 0.0;
    for (int w = 0; w < kNormThreads / 64; ++w) s += red[w];
    partials[blockIdx.x] = s;
  }
}

// ---------------------------------------------------------------------------
// Sampled threshold (paper: Section 5 -- top-k on a sample estimates the
// threshold of the whole tensor; Algorithm 3 "thr <- s% of |V[j]|")
// ---------------------------------------------------------------------------
// 32-bit xorshift-multiply finaliser; a bijection on 32-bit words.
__device__ __forceinline__ uint32_t mix32(uint32_t x) {
  x ^= x >> 16;
  x *= 0x7FEB352Du;
  x ^= x >> 15;
  x *= 0x846CA68Bu;
  x ^= x >> 16;
  return x;
}

struct Candidates {
  const float* g;
  const float* u;
  const float* v;
  int64_t offset;
  uint32_t key;      // folded (seed, iteration, tensor)
  uint32_t nblocks;
  int32_t block_shift;
  int32_t exact;
  float m, scale;
  bool nesterov;

  // Position (relative to the tensor) of candidate p.
  __device__ __forceinline__ int64_t position(int32_t p) const {
    if (exact) return p;
    const uint32_t draw = (uint32_t)p >> block_shift;
    const uint32_t r = mix32(key ^ (draw * 0x9E3779B1u));
    const uint32_t blk = __umulhi(r, nblocks);
    return ((int64_t)blk << block_shift) + (p & ((1 << block_shift) - 1));
  }
};

// One workgroup per tensor finds the candidate key of a given descending rank
// exactly.  Keys are the bit patterns of |v'| (order-isomorphic to the
// magnitudes).  Histograms of 2048 bins narrow the interval that holds the key down; as soon as the bin that holds the
// rank has few enough members they are gathered and ranked directly, mostly after the first.  Low ranks are ranked
// from a list of the largest keys without any.
//
// Up to kSelectRegKeys * kSelectThreads candidates live in registers (each
// thread gathers its own once and keeps them); a larger candidate set (exact
// selection on a big tensor) is re-evaluated from g, u, v in every pass.
struct SelectShared {
  alignas(16) double red[kSelectThreads / 64];
  unsigned long long missing[kSelectThreads / 64];
  float scale;
  uint32_t hist[kSelectBins];
  uint32_t wave_tot[kSelectThreads / 64];
  alignas(16) uint32_t surv[kSelectThreads];
  uint32_t sel[3];
  uint32_t surv_n, result;
};

// After a histogram pass: the bin that holds descending rank `rank`, how many
// candidates lie above it, and how many it holds; and the number of all of them, not above which the rank is for the others
// to mean anything.  Every thread returns the same.
// `sel` is three words of LDS, `wave_tot` one word per wavefront.
template <int THREADS>
__device__ __forceinline__ void find_bin(const uint32_t* hist, uint32_t* wave_tot, uint32_t* sel, int tid,
                                         uint32_t rank, uint32_t& bin, uint32_t& above_out,
                                         uint32_t& members, uint32_t& total) {
  constexpr int PER = kSelectBins / THREADS;  // consecutive bins owned by a thread
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint32_t h[PER];
  uint32_t local = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    h[i] = hist[PER * tid + i];
    local += h[i];
  }
  const uint32_t incl = wave_inclusive_sum(local);
  if (lane == 63) wave_tot[wave] = incl;
  __syncthreads();
  uint32_t run = wave_last(incl) - incl;  // candidates above this thread's bins: in its wavefront, and in those behind
  total = 0;
#pragma unroll
  for (int w = 0; w < THREADS / 64; ++w) {  // (all asked for together)
    const uint32_t t = wave_tot[w];
    run += w > wave ? t : 0u;
    total += t;
  }
#pragma unroll
  for (int i = PER - 1; i >= 0; --i) {
    if (run <= rank && rank < run + h[i]) {
      sel[0] = PER * tid + i;
      sel[1] = run;
      sel[2] = h[i];
    }
    run += h[i];
  }
  __syncthreads();
  bin = sel[0];
  above_out = sel[1];
  members = sel[2];
}

// The `m` <= kSelectThreads keys in sh.surv, which is zero behind them up to a multiple of four: the one of
// descending rank `rank`.  Up to 256 keys, the usual case, have four neighbouring threads each, up to 512 two, which compare
// it with a share of the keys, four to an LDS read, and add up through the vector unit; more have one.
__device__ __forceinline__ uint32_t rank_directly(SelectShared& sh, int tid, uint32_t m, uint32_t rank) {
  const uint4* __restrict__ four = reinterpret_cast<const uint4*>(sh.surv);
  const uint32_t shift = 4 * m <= (uint32_t)kSelectThreads ? 2u : 2 * m <= (uint32_t)kSelectThreads ? 1u : 0u;  // uniform
  const uint32_t own = (uint32_t)tid >> shift, step = 1u << shift;
  if (own < m) {
    const uint32_t x = sh.surv[own];
    uint32_t greater = 0, equal = 0;  // (a zero behind the keys can only add to the last rank's ties)
    for (uint32_t i = (uint32_t)tid & (step - 1u); 4 * i < m; i += step) {
      const uint4 y = four[i];
      greater += (y.x > x) + (y.y > x) + (y.z > x) + (y.w > x);
      equal += (y.x == x) + (y.y == x) + (y.z == x) + (y.w == x);
    }
    if (shift > 0) {
      uint32_t both = greater | (equal << 16);
      both += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)both, 0xB1, 0xf, 0xf, false);  // the neighbour's
      const uint32_t other = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)both, 0x4E, 0xf, 0xf, false);  // the other pair's
      both += shift > 1 ? other : 0u;
      greater = both & 0xFFFFu;
      equal = both >> 16;
    }
    if (greater <= rank && rank < greater + equal) sh.result = x;  // ties write the same value
  }
  __syncthreads();
  return sh.result;
}

constexpr uint32_t kNoKey = 0xFFFFFFFFu;  // real keys have the sign bit clear
constexpr uint32_t kInfinity = 0x7F800000u;  // the keys of NaNs lie above: they are ranked, and not sent
__device__ __forceinline__ bool sent(uint32_t key, uint32_t thr) { return key > thr && key <= kInfinity; }

// Key of descending rank `rank` among the keys a workgroup holds in registers (NKEYS per thread, the first `live` of which may be
// in use), ignoring empty slots; the caller guarantees that there are more than `rank`.  Every thread returns the same.
// Histograms of 2048 bins over the interval that holds the key, until the bin has few enough members to rank directly.
// `guess`, if not zero: the key probably lies in the eight octaves from there on.  The first histogram then has 256 bins to an
// octave, where one over all keys has eight and leaves several hundred members in the bin, for another round, and
// collisions of the lanes' additions on the way (selection at 25 % and 1.6 % on 122 M elements 21.3 -> 17.8 and 21.4 -> 17.4 us, at
// 6.25 % on 25.6 M 17.0 -> 15.1, on 2 M 11.1 -> 8.0).  A guess that is wrong costs that round.
template <int NKEYS>
__device__ __forceinline__ uint32_t select_in_registers(SelectShared& sh, const uint32_t (&key)[NKEYS], int live,
                                                        uint32_t guess, uint32_t rank, int tid) {
  constexpr uint32_t kLastBin = (uint32_t)kSelectBins - 1u;
  uint32_t lo = guess, width = guess != 0u ? kNoKey - guess : 0x80000000u;  // the key is one of [lo, lo + width)
  int shift = guess != 0u ? 15 : 20;  // what lies beyond the bins counts in the last one
#pragma unroll 1
  for (bool first = guess != 0u;; first = false) {
    for (int i = tid; i < kSelectBins; i += kSelectThreads) sh.hist[i] = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NKEYS; ++i) {
      if (i % 4 == 0 && i >= live) break;  // uniform
      const uint32_t from = key[i] - lo;   // (an empty slot's is beyond every width)
      if (from < width) {
        const uint32_t bin = from >> shift;
        atomicAdd(&sh.hist[bin < kLastBin ? bin : kLastBin], 1u);
      }
    }
    __syncthreads();
    uint32_t bin, above, members, total;
    find_bin<kSelectThreads>(sh.hist, sh.wave_tot, sh.sel, tid, rank, bin, above, members, total);
    if (first && rank >= total) {  // it lies below what was guessed
      rank -= total;
      lo = 0u;
      width = guess;
    } else {
      rank -= above;
      const uint32_t rest = width - (bin << shift);  // (the interval's end may lie inside its last bin)
      lo += bin << shift;
      width = (first && bin == kLastBin) || rest < 1u << shift ? rest : 1u << shift;
      if (width == 1u) return lo;
      if (members <= (uint32_t)kSelectDirect) {
        if (tid == 0) sh.surv_n = 0;
        if (tid < 4) sh.surv[(members & ~3u) + tid] = 0;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NKEYS; ++i) {
          if (i % 4 == 0 && i >= live) break;  // uniform
          if (key[i] - lo < width) sh.surv[atomicAdd(&sh.surv_n, 1u)] = key[i];
        }
        __syncthreads();
        return rank_directly(sh, tid, members, rank);
      }
    }
    shift = width > (uint32_t)kSelectBins ? 21 - __clz((int)(width - 1u)) : 0;  // 11 bits stay
  }
}

// The smallest of what the first `full_waves` wavefronts name as the t-th largest of their threads' largest keys: a key that
// t * full_waves keys at least do not lie below.  `top` gets this thread's largest key (-1: it has none).
__device__ __forceinline__ uint32_t floor_of_waves(SelectShared& sh, const uint32_t (&key)[kSelectRegKeys], int live,
                                                   uint32_t full_waves, uint32_t t, int tid, int32_t& top) {
  constexpr int kWaves = kSelectThreads / 64;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  top = -1;  // (an empty slot counts as -1)
#pragma unroll
  for (int i = 0; i < kSelectRegKeys; ++i) {
    if (i % 4 == 0 && i >= live) break;  // uniform
    top = (int32_t)key[i] > top ? (int32_t)key[i] : top;
  }
  uint32_t rest = top > 0 ? (uint32_t)top : 0u;
  uint32_t tth = 0;
  for (uint32_t round = 0; round < t; ++round) {
    tth = wave_max(rest);
    const unsigned long long holding = __ballot(rest == tth);
    if (lane == __ffsll((long long)holding) - 1) rest = 0;  // one holder of the maximum steps down
  }
  if (lane == 0) sh.wave_tot[wave] = (uint32_t)wave < full_waves ? tth : 0x7FFFFFFFu;
  __syncthreads();
  uint32_t floor_key = sh.wave_tot[0];
#pragma unroll
  for (int w = 1; w < kWaves; ++w) floor_key = sh.wave_tot[w] < floor_key ? sh.wave_tot[w] : floor_key;
  return full_waves == 0 ? 0u : floor_key;
}

// Key of descending rank `rank` among the `count` keys a workgroup holds in registers (kNoKey marks an empty
// slot); threads 0 .. holders - 1 have at least one, none has one behind its first `live`.  Every thread returns the same.
__device__ __forceinline__ uint32_t rank_registers(SelectShared& sh, const uint32_t (&key)[kSelectRegKeys], int32_t count,
                                                   int32_t holders, int live, uint32_t rank, int tid) {
  // Gradients of one tensor share a few exponents, so a histogram over the leading key
  // bits of all candidates piles tens of thousands of LDS atomics on a handful of bins,
  // and every histogram pass costs half a dozen barriers of 1024 threads (ranking 32 Ki
  // keys that way took 20 us, against 3 us this way).  At the paper's densities the
  // rank r is a few dozen, and a floor below which no key matters is cheap to get: if
  // every one of the (up to 16) wavefronts whose threads all hold keys names the t-th largest of
  // its threads' largest keys, with t times the wavefronts more than r, then the smallest of the
  // answers has more than r keys at or above it.  What lies at or above that floor (a few times r
  // keys; everything, if there are fewer than 64 holders) is listed in LDS
  // and ranked by direct counting.  Anything that does not fit this pattern takes the
  // histogram passes.
  constexpr int kWaves = kSelectThreads / 64;
  const uint32_t full_waves = (uint32_t)holders >= (uint32_t)kSelectThreads ? (uint32_t)kWaves : (uint32_t)holders >> 6;
  const uint32_t t_rounds = full_waves > 0 ? rank / full_waves + 1 : 0;  // full_waves * t_rounds > rank
  // (Of a key or two per thread, the list is several hundred long from a rank of 80 or so on: 20000 tensors of
  // 1500 elements, rank 120, 739 us this way and 553 by histograms, rank 94 618 and 571, rank 45 472 and 535.)
  if (t_rounds <= (uint32_t)kSelectFloorRounds && (count > 2 * kSelectThreads || rank < 80u)) {
    int32_t top;
    if (tid == 0) sh.surv_n = 0;
    sh.surv[tid] = 0;
    const uint32_t floor_key = floor_of_waves(sh, key, live, full_waves, t_rounds, tid, top);
    // One addition to the list's length per wavefront.  Most threads that have a key to list have one, their largest.
    uint32_t mine = 0;
#pragma unroll
    for (int i = 0; i < kSelectRegKeys; ++i) {
      if (i % 4 == 0 && i >= live) break;  // uniform
      mine += (int32_t)key[i] >= (int32_t)floor_key ? 1u : 0u;
    }
    const uint32_t upto = wave_inclusive_sum(mine);
    uint32_t pos = 0;
    if ((tid & 63) == 63 && upto > 0u) pos = atomicAdd(&sh.surv_n, upto);
    pos = wave_last(pos) + upto - mine;
    if (mine == 1u && pos < (uint32_t)kSelectThreads) sh.surv[pos] = (uint32_t)top;
    if (__ballot(mine > 1u) != 0) {
#pragma unroll
      for (int i = 0; i < kSelectRegKeys; ++i) {
        if (i % 4 == 0 && i >= live) break;  // uniform
        if (mine > 1u && (int32_t)key[i] >= (int32_t)floor_key) {
          if (pos < (uint32_t)kSelectThreads) sh.surv[pos] = key[i];
          ++pos;
        }
      }
    }
    __syncthreads();
    const uint32_t listed = sh.surv_n;
    if (listed <= (uint32_t)kSelectThreads) return rank_directly(sh, tid, listed, rank);
    __syncthreads();
  }
  // The smallest of the wavefronts' largest keys is among the largest few in a thousand, however large a few others are: the
  // key is looked for from seven octaves below on.
  int32_t top;
  const uint32_t anchor = floor_of_waves(sh, key, live, full_waves, 1u, tid, top);
  constexpr uint32_t kSevenOctaves = 7u << 23;
  return select_in_registers<kSelectRegKeys>(sh, key, live, anchor > kSevenOctaves ? anchor - kSevenOctaves : 0u, rank, tid);
}

// How many keys of a band's sample lie above `floor_key`, how many do not lie below it, and the sum over the sampled
// blocks of the squares of the latter's numbers.  Eight neighbouring threads hold the 32 keys of a block, four to a
// thread, and eight blocks (see the gather).
__device__ __forceinline__ void keys_by_block(SelectShared& sh, const uint32_t (&key)[kSelectRegKeys], uint32_t floor_key,
                                              int tid, uint32_t& above, uint32_t& keys, uint32_t& squares) {
  static_assert(kBandBlockShift == 5 && kSelectRegKeys == 32 && kBandSample == kSelectRegKeys * kSelectThreads, "every thread is full");
  uint32_t four[2] = {0u, 0u};  // of the thread's eight blocks, a byte each
  uint32_t strict = 0;
#pragma unroll
  for (int i = 0; i < kSelectRegKeys; ++i) {
    four[i >> 4] += key[i] >= floor_key ? 1u << (8 * ((i >> 2) & 3)) : 0u;
    strict += key[i] > floor_key ? 1u : 0u;
  }
  uint32_t own = 0;  // a wavefront's 64 blocks: up to 2048 keys, squares up to 65536
#pragma unroll
  for (int h = 0; h < 2; ++h) {  // over the eight lanes: up to 32 in a byte
    uint32_t x = four[h];
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xf, 0xf, false);   // the neighbour's
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xf, 0xf, false);   // the other pair's of the quad
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xf, 0xf, false);  // the other quad's of the half row
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const uint32_t n = (x >> (8 * b)) & 0xFFu;
      own += (n << 20) + n * n;
    }
  }
  own = wave_sum((tid & 7) == 0 ? own : 0u);
  strict = wave_sum(strict);
  if ((tid & 63) == 0) {
    sh.wave_tot[tid >> 6] = own;
    sh.surv[tid >> 6] = strict;
  }
  __syncthreads();
  above = keys = squares = 0;
#pragma unroll
  for (int w = 0; w < kSelectThreads / 64; ++w) {
    keys += sh.wave_tot[w] >> 20;
    squares += sh.wave_tot[w] & 0xFFFFFu;
    above += sh.surv[w];
  }
  __syncthreads();
}

// The same among `count` candidates that are evaluated from g, u, v anew in every pass.
__device__ __forceinline__ uint32_t rank_reevaluated(SelectShared& sh, const Candidates& c, int32_t count, uint32_t rank,
                                                     int tid) {
  uint32_t prefix = 0;
  int consumed = 0;
#pragma unroll 1
  for (int pass = 0; pass < 3; ++pass) {
    const int bits = pass == 2 ? 9 : 11;
    const int shift = 31 - consumed - bits;
    const uint32_t digit_mask = (1u << bits) - 1u;
    for (int i = tid; i < kSelectBins; i += kSelectThreads) sh.hist[i] = 0;
    __syncthreads();
    for (int32_t p0 = tid; p0 < count; p0 += kSelectInFlight * kSelectThreads) {
      float gg[kSelectInFlight], uu[kSelectInFlight], vv[kSelectInFlight];
#pragma unroll
      for (int q = 0; q < kSelectInFlight; ++q) {
        const int32_t p = p0 + q * kSelectThreads;
        gg[q] = uu[q] = vv[q] = 0.0f;
        if (p < count) {
          const int64_t e = c.offset + c.position(p);
          gg[q] = c.g[e];
          uu[q] = c.u[e];
          vv[q] = c.v[e];
        }
      }
#pragma unroll
      for (int q = 0; q < kSelectInFlight; ++q) {
        const int32_t p = p0 + q * kSelectThreads;
        if (p < count) {
          float u1, v1;
          momentum_update(gg[q], uu[q], vv[q], c.m, c.scale, c.nesterov, u1, v1);
          const uint32_t k = __float_as_uint(v1) & 0x7FFFFFFFu;
          if (pass == 0 || (k >> (shift + bits)) == prefix)
            atomicAdd(&sh.hist[(k >> shift) & digit_mask], 1u);
        }
      }
    }
    __syncthreads();
    uint32_t bin, above, members, all;
    find_bin<kSelectThreads>(sh.hist, sh.wave_tot, sh.sel, tid, rank, bin, above, members, all);
    prefix = (prefix << bits) | bin;
    rank -= above;
    consumed += bits;
  }
  return prefix;
}

// The threshold of tensor j into the tables.  Tiles that lie wholly inside the tensor get it into the
// per-tile table, which is all the streaming pass looks at on its fast path.
__device__ __forceinline__ void write_threshold(const SelectArgs& a, int j, const TensorPlan& plan, float thr, int tid) {
  const int64_t tile_first = (plan.offset + kWaveTile - 1) / kWaveTile;
  const int64_t tile_end = (plan.offset + plan.n) / kWaveTile;
  if (tid == 0) {
    a.thr[j] = thr;
    if (a.out_thr) a.out_thr[j] = thr;
  }
  for (int64_t t = tile_first + tid; t < tile_end; t += kSelectThreads) a.tile_thr[t] = thr;
}

__device__ __forceinline__ Candidates candidates_of(const SelectArgs& a, int j, const TensorPlan& plan, float scale,
                                                    bool nesterov) {
  Candidates c;
  c.g = a.g;
  c.u = a.u;
  c.v = a.v;
  c.offset = plan.offset;
  c.nblocks = plan.nblocks;
  c.block_shift = a.block_shift;
  c.exact = plan.exact;
  c.m = a.momentum;
  c.scale = scale;
  c.nesterov = nesterov;
  uint32_t h = mix32(a.seed_lo ^ 0x9E3779B9u);
  h = mix32(h ^ a.seed_hi);
  h = mix32(h ^ a.iter_lo);
  h = mix32(h ^ a.iter_hi);
  c.key = mix32(h ^ (uint32_t)j);
  return c;
}

// For a tensor with a band, after select_kernel.
__device__ __forceinline__ bool floor_went_into_pass(const FloorArgs& f, const DeviceState* state, int j) {
  const int64_t crowded = state->crowded;
  const int32_t collected = f.collected[j];  // (asked for in any case: no chain of loads)
  return f.in_pass != 0 && collected == 0 && (crowded == 0 || f.elements - crowded > kBandMixedElements);
}

__device__ __forceinline__ BandState* band_state(const SelectArgs& a, const TensorPlan& plan) {
  return reinterpret_cast<BandState*>(reinterpret_cast<char*>(a.bands) + (size_t)plan.nblocks * kBandStride);
}
__device__ __forceinline__ int64_t band_list_begin(int64_t offset) { return 3 * (offset >> kBandListShift); }

// Sum of squares of share `c` of `shares` of g by a workgroup of select_kernel's size; every thread returns it.
__device__ __forceinline__ double norm_share(const float* __restrict__ g, int64_t n, int c, int shares, SelectShared& sh, int tid) {
  constexpr int kInFlight = 4;
  const int64_t nvec = n >> 2;
  const float4* __restrict__ g4 = reinterpret_cast<const float4*>(g);
  const int64_t stride = (int64_t)shares * kSelectThreads;
  double a[4] = {0.0, 0.0, 0.0, 0.0};
  for (int64_t i = (int64_t)c * kSelectThreads + tid; i < nvec; i += kInFlight * stride) {
    float4 x[kInFlight];
#pragma unroll
    for (int q = 0; q < kInFlight; ++q) {
      const int64_t at = i + q * stride;
      x[q] = at < nvec ? g4[at] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
#pragma unroll
    for (int q = 0; q < kInFlight; ++q) {
      a[0] += (double)x[q].x * (double)x[q].x;
      a[1] += (double)x[q].y * (double)x[q].y;
      a[2] += (double)x[q].z * (double)x[q].z;
      a[3] += (double)x[q].w * (double)x[q].w;
    }
  }
  if (c == 0 && tid < (int)(n & 3)) {
    const double x = (double)g[(nvec << 2) + tid];
    a[0] += x * x;
  }
  const double s = wave_sum_down((a[0] + a[1]) + (a[2] + a[3]));
  __syncthreads();  // (`red` may be in use)
  if ((tid & 63) == 0) sh.red[tid >> 6] = s;
  __syncthreads();
  double total = 0.0;
#pragma unroll
  for (int w = 0; w < kSelectThreads / 64; ++w) total += sh.red[w];
  return total;
}

// A share's place holds zero until its sum is there, which is stored with the sign turned: a sum of nothing is -0.
__device__ __forceinline__ unsigned long long share_word(double sum) { return (unsigned long long)__double_as_longlong(-sum); }

// Clipping scale (paper: Appendix C equation 12).  With clipping on, the norm kernel has left its partial
// sums, of which `part` is this thread's (thread t has partial t, or zero); every workgroup adds them in the
// same fixed order (lanes, then wavefronts, in order), so all of them get the same bits, and the first one
// also files the result for the streaming pass and for the diagnostics.
// FUSED: other workgroups of this launch form the partial sums.  A workgroup looks for them for a while (they are there by
// the time the candidates are, in a set that this is done for); what is missing then, because those workgroups
// have found no place on the device, say, it forms itself.  So nothing here waits without an end, whatever else runs.
static_assert(kNormMaxBlocks <= kSelectThreads, "a partial sum per thread");
template <bool FUSED>
__device__ __forceinline__ float settle_scale(const SelectArgs& a, SelectShared& sh, double part, int j, int tid) {
  if (!a.scale_from_state) {
    if (tid == 0 && j == 0) {  // no clipping: start a clean record
      a.state->norm = __longlong_as_double(0x7FF8000000000000ll);
      a.state->scale = a.scale_const;
      a.state->flags = 0;
    }
    return a.scale_const;
  }
  if (FUSED) {
    unsigned long long word = ~0ull;
    if (tid < a.num_partials) {
      word = 0;
      const int looks = looks_for(a.looks, tid);
      for (int look = 0; look < looks; ++look) {
        word = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(a.partials) + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (word != 0) break;
        __builtin_amdgcn_s_sleep(1);
      }
      part = -__longlong_as_double((long long)word);
    }
    const unsigned long long lacking = __ballot(word == 0);
    if ((tid & 63) == 0) sh.missing[tid >> 6] = lacking;
  }
  const double s = wave_sum_down(part);
  if ((tid & 63) == 0) sh.red[tid >> 6] = s;
  __syncthreads();
  if (FUSED) {
    unsigned long long any = 0;
#pragma unroll
    for (int w = 0; w < kSelectThreads / 64; ++w) any |= sh.missing[w];
    if (__builtin_amdgcn_readfirstlane((int)(any != 0)) != 0) {  // the same in every wavefront
      for (int c = 0; c < a.num_partials; ++c) {
        if ((sh.missing[c >> 6] >> (c & 63)) & 1u) {
          const double sum = norm_share(a.g, a.n, c, a.num_partials, sh, tid);
          if (tid == c) part = sum;
        }
      }
      const double again = wave_sum_down(part);
      __syncthreads();
      if ((tid & 63) == 0) sh.red[tid >> 6] = again;
      __syncthreads();
    }
  }
  if (tid == 0) {
    double total = 0.0;
#pragma unroll
    for (int w = 0; w < kSelectThreads / 64; ++w) total += sh.red[w];
    const double norm = sqrt(total);
    float sc = 1.0f;
    if (norm > a.thr_local) sc = (float)(a.thr_local / norm);
    if (a.scale_override == a.scale_override) sc = a.scale_override;
    sh.scale = sc;
    if (j == 0) {
      uint32_t flags = 0;
      if (!(norm <= 1.79769313486231570e308)) flags |= DGC_DIAG_NONFINITE;  // NaN or infinity
      a.state->norm = norm;
      a.state->scale = sc;
      a.state->flags = flags;
    }
  }
  __syncthreads();
  return sh.scale;
}

// Bound by latency: the gather of the candidates, then the ranking, in one workgroup per tensor.  16.9 us on eleven tensors of
// 66 M elements, 12.8 on 161 of 25.6 M (13.7 with chains as they were before the next sentence).  Inside the workgroup,
// 1 M elements, from its start:
// 8.0 -> 6.6 us with the list's length asked for once per wavefront and not per key, four threads to a listed key, no
// walk over empty slots, and the scale's sum over the lanes inside the vector unit; the step of that set 27.5 ->
// 26.3, of 23 tensors of 0.27 M elements in all 33.9 -> 31.9.
// FUSED: the norm's partial sums are formed by the first workgroups of the launch, while the others gather (rule and
// figures at kNormInSelectElements; steps with clipping: 23 tensors of 0.27 M elements 31.7 -> 30.1 us, 1 M 26.0 -> 24.4).
// MODE: whether some tensors are ranked by way of a band (TensorPlan.exact == 2), and whether its floor may go into the pass.
enum SelectMode : int { kSelectNoBands = 0, kSelectLists = 1, kSelectInPass = 2 };

template <bool NESTEROV, int MODE, bool FUSED>
__global__ __launch_bounds__(kSelectThreads) void select_kernel(SelectArgs a) {
  __shared__ SelectShared sh;
  const int tid = threadIdx.x;
  if (FUSED && (int)blockIdx.x < a.num_partials) {  // the first workgroups form the partial sums of the norm
    const double sum = norm_share(a.g, a.n, blockIdx.x, a.num_partials, sh, tid);
    if (tid == 0)
      __hip_atomic_store(reinterpret_cast<unsigned long long*>(a.partials) + blockIdx.x, share_word(sum), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return;
  }
  const int j = FUSED ? (int)blockIdx.x - a.num_partials : (int)blockIdx.x;
  const TensorPlan plan = a.plans[j];
  // Asked for before the candidates and used after their first loads are on their way, so that the scale's
  // chain of steps (sum over the lanes, over the wavefronts, square root) runs while those are outstanding.
  const double part = !FUSED && a.scale_from_state && tid < a.num_partials ? a.partials[tid] : 0.0;

  if (plan.rank >= plan.count) {  // the strict comparison then passes everything
    settle_scale<FUSED>(a, sh, part, j, tid);
    write_threshold(a, j, plan, -1.0f, tid);
    return;
  }

  Candidates c = candidates_of(a, j, plan, a.scale_const, NESTEROV);
  if (MODE != kSelectNoBands && plan.exact == 2) {  // a sample for the band of an exact selection
    c.exact = 0;
    c.block_shift = kBandBlockShift;
    c.nblocks = (uint32_t)(plan.n >> kBandBlockShift);
  }

  const int32_t count = (MODE != kSelectNoBands && plan.exact == 2) ? kBandSample : plan.count;
  const uint32_t rank = (uint32_t)plan.rank;
  uint32_t thr_bits = 0;

  if (count <= kSelectRegKeys * kSelectThreads) {
    // ---- candidates in registers ------------------------------------------------
    uint32_t key[kSelectRegKeys];
#pragma unroll
    for (int i = 0; i < kSelectRegKeys; ++i) key[i] = kNoKey;
    const bool quads_of_blocks = !c.exact && c.block_shift >= 2;
    const int32_t holders = quads_of_blocks ? count >> 2 : count;  // threads with at least one candidate
    // candidates of a thread that has most
    const int live = quads_of_blocks ? 4 * (((count >> 2) + kSelectThreads - 1) / kSelectThreads) : (count + kSelectThreads - 1) / kSelectThreads;
    // The gather is written without branches around the loads and without conditional stores into
    // key[]: a candidate beyond the count reads candidate 0 instead and its key is replaced by the
    // empty mark afterwards.  (With `if (p < count)` around them the compiler copied the whole
    // register array at every such branch: some 400 moves per thread in a kernel that spends as
    // much time issuing instructions as waiting for memory, 16 wavefronts sharing four SIMDs.)
    if (quads_of_blocks) {
      // Sampled blocks of at least four elements: a thread takes four consecutive elements of a
      // drawn block at a time (one 16-byte load per array; a block starts at a multiple of its size
      // from the tensor's start, which need not be 16-byte aligned: dword-aligned vector loads), so
      // that the draw's position is worked out once per four candidates.  Which thread holds which
      // candidate does not matter: the rank is taken over all of them.
      typedef float vec4u __attribute__((ext_vector_type(4), aligned(4)));
      constexpr int kQuads = kSelectRegKeys / 4;       // per thread
      constexpr int kQuadsInFlight = 4;
      const int32_t quads = count >> 2;                // blocks are whole multiples of four elements
      const int qshift = c.block_shift - 2;            // log2(quads per block)
#pragma unroll
      for (int r = 0; r < kQuads / kQuadsInFlight; ++r) {
        if (r == 0 || r * kQuadsInFlight * kSelectThreads < quads) {  // uniform
          vec4u gg[kQuadsInFlight], uu[kQuadsInFlight], vv[kQuadsInFlight];
#pragma unroll
          for (int q = 0; q < kQuadsInFlight; ++q) {
            const int32_t qd = tid + (r * kQuadsInFlight + q) * kSelectThreads;
            const int32_t qq = qd < quads ? qd : 0;
            const int64_t e = c.offset + c.position((qq >> qshift) << c.block_shift) + ((qq & ((1 << qshift) - 1)) << 2);
            gg[q] = *reinterpret_cast<const vec4u*>(c.g + e);
            uu[q] = *reinterpret_cast<const vec4u*>(c.u + e);
            vv[q] = *reinterpret_cast<const vec4u*>(c.v + e);
          }
          if (r == 0) c.scale = settle_scale<FUSED>(a, sh, part, j, tid);
#pragma unroll
          for (int q = 0; q < kQuadsInFlight; ++q) {
            const bool ok = tid + (r * kQuadsInFlight + q) * kSelectThreads < quads;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              float u1, v1;
              momentum_update(gg[q][k], uu[q][k], vv[q][k], c.m, c.scale, NESTEROV, u1, v1);
              key[4 * (r * kQuadsInFlight + q) + k] = ok ? (__float_as_uint(v1) & 0x7FFFFFFFu) : kNoKey;
            }
          }
        }
      }
    } else {
      // one candidate per load: kSelectInFlight of them are loaded before any is used
#pragma unroll
      for (int r = 0; r < kSelectRegKeys / kSelectInFlight; ++r) {
        if (r == 0 || r * kSelectInFlight * kSelectThreads < count) {  // uniform
          float gg[kSelectInFlight], uu[kSelectInFlight], vv[kSelectInFlight];
#pragma unroll
          for (int q = 0; q < kSelectInFlight; ++q) {
            const int32_t p = tid + (r * kSelectInFlight + q) * kSelectThreads;
            const int64_t e = c.offset + c.position(p < count ? p : 0);
            gg[q] = c.g[e];
            uu[q] = c.u[e];
            vv[q] = c.v[e];
          }
          if (r == 0) c.scale = settle_scale<FUSED>(a, sh, part, j, tid);
#pragma unroll
          for (int q = 0; q < kSelectInFlight; ++q) {
            const bool ok = tid + (r * kSelectInFlight + q) * kSelectThreads < count;
            float u1, v1;
            momentum_update(gg[q], uu[q], vv[q], c.m, c.scale, NESTEROV, u1, v1);
            key[r * kSelectInFlight + q] = ok ? (__float_as_uint(v1) & 0x7FFFFFFFu) : kNoKey;
          }
        }
      }
    }
    if (MODE != kSelectNoBands && plan.exact == 2) {
      // A band that holds the wanted rank almost surely.  Nothing depends on it but the time: a band that misses is
      // noticed.  In the pass it is a floor alone, and only for values that the sample can be relied on for; the
      // others are collected.
      const BandRanks at((double)plan.rank / (double)plan.n, (double)kBandSample);
      if (MODE == kSelectInPass) {
        const uint32_t floor_key = rank_registers(sh, key, count, holders, live, (uint32_t)at.floor_in_pass(), tid);
        bool reliable = true, in_clusters = false;
        if (a.band_list) {  // (a set without lists has no tensor so long that a miss would cost more than looking)
          uint32_t above, keys, squares;
          keys_by_block(sh, key, floor_key, tid, above, keys, squares);
          in_clusters = at.clustered(keys, squares);
          reliable = !in_clusters && !at.tied(above, floor_key);
        }
        if (tid == 0) {
          a.floor.collected[j] = reliable ? 0 : 1;
          if (!reliable) atomicAdd(&a.state->crowded, (uint32_t)plan.n);
        }
        // What exceeds the floor passes, and refine_kernel ranks it ...
        write_threshold(a, j, plan, __uint_as_float(floor_key < kInfinity ? floor_key : kInfinity), tid);
        // ... or the band is collected, and rank_band_kernel writes the threshold.  Ties at the floor are counted then.
        // Clusters need a floor further down: they fill eight lanes each and so spare some wavefront, whose own floor is the
        // smallest; the list gets two or three times the keys that the rank below asks for, and which they are does
        // not matter.  No ceiling: at the densities of the pass it would lie above everything.
        if (a.band_list) {
          uint32_t band_floor = floor_key;
          int32_t top;
          if (in_clusters) band_floor = floor_of_waves(sh, key, live, kSelectThreads / 64, (uint32_t)(ceil(at.mid) + at.reach()) / (kSelectThreads / 64) + 1u, tid, top);
          if (tid == 0) *band_state(a, plan) = BandState{band_floor, 0x80000000u, 0u, 0u, 0u};
        }
        return;
      }
      const double reach = at.reach();
      const double low = ceil(at.mid) + reach, high = floor(at.mid) - reach;
      const uint32_t floor_key = low < (double)count ? rank_registers(sh, key, count, holders, live, (uint32_t)low, tid) : 0xFFFFFFFFu;
      uint32_t ceil_key = high >= 0.0 ? rank_registers(sh, key, count, holders, live, (uint32_t)high, tid) : 0x80000000u;
      if (ceil_key == floor_key) ++ceil_key;
      if (tid == 0) *band_state(a, plan) = BandState{floor_key, ceil_key, 0u, 0u, 0u};
      return;
    }
    thr_bits = rank_registers(sh, key, count, holders, live, rank, tid);
  } else {
    c.scale = settle_scale<FUSED>(a, sh, part, j, tid);
    thr_bits = rank_reevaluated(sh, c, count, rank, tid);
  }
  write_threshold(a, j, plan, __uint_as_float(thr_bits), tid);
}

// ---------------------------------------------------------------------------
// Exact threshold of a tensor too large for a workgroup's registers
// (paper: Algorithm 3 "thr <- s% of |V[j]|" taken literally)
// ---------------------------------------------------------------------------
// Two kernels after select_kernel, which has named the band (see kBandSample).  A workgroup of the
// collecting pass reads kBandElements elements of g, u, v (12 bytes each, once: HBM bounds it), counts
// the keys above the band and those equal to its floor, and appends those inside it to the tensor's
// list, one returning atomic per workgroup.  A wavefront collects its keys in a segment of LDS of its
// own, placed by votes.
template <bool NESTEROV>
__global__ __launch_bounds__(kBandThreads) void collect_band_kernel(SelectArgs a, const EmitBlock* __restrict__ blocks) {
  constexpr int kWaves = kBandThreads / 64;
  constexpr int kRounds = kBandElements / (4 * kBandThreads);
  constexpr int kRoundsInFlight = 4;
  constexpr int kSegment = kBandElements / kWaves;
  typedef float quad __attribute__((ext_vector_type(4)));
  __shared__ uint32_t list[kBandElements];
  __shared__ uint32_t counts[3][kWaves];
  __shared__ uint32_t base_sh;
  if (a.floor.in_pass && a.state->crowded == 0) return;  // every floor went into the pass
  const EmitBlock blk = blocks[blockIdx.x / kBandsPerPart];
  const TensorPlan plan = a.plans[blk.tensor];
  const bool into_pass = floor_went_into_pass(a.floor, a.state, blk.tensor);
  if (plan.exact != 2 || into_pass) return;
  const int64_t base = (int64_t)blk.first_tile * kWaveTile + (int64_t)(blockIdx.x % kBandsPerPart) * kBandElements;
  if (base >= blk.hi || base + kBandElements <= blk.lo) return;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const float scale = a.scale_from_state ? a.state->scale : a.scale_const;
  BandState* st = band_state(a, plan);
  const uint32_t floor_key = st->floor_key, ceil_key = st->ceil_key;
  uint32_t above = 0, ties = 0, listed = 0;  // of the wavefront
#pragma unroll 1
  for (int r0 = 0; r0 < kRounds; r0 += kRoundsInFlight) {
    quad x[kRoundsInFlight], y[kRoundsInFlight], z[kRoundsInFlight];
    bool in[kRoundsInFlight];  // all four elements belong to the tensor
#pragma unroll
    for (int r = 0; r < kRoundsInFlight; ++r) {
      const int64_t e = base + (r0 + r) * (4 * kBandThreads) + tid * 4;
      in[r] = e >= blk.lo && e + 4 <= blk.hi;
      if (in[r]) {
        x[r] = __builtin_nontemporal_load(reinterpret_cast<const quad*>(a.g + e));
        y[r] = __builtin_nontemporal_load(reinterpret_cast<const quad*>(a.u + e));
        z[r] = __builtin_nontemporal_load(reinterpret_cast<const quad*>(a.v + e));
      } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const bool one = e + c >= blk.lo && e + c < blk.hi;
          x[r][c] = one ? a.g[e + c] : 0.0f;
          y[r][c] = one ? a.u[e + c] : 0.0f;
          z[r][c] = one ? a.v[e + c] : 0.0f;
        }
      }
    }
#pragma unroll
    for (int r = 0; r < kRoundsInFlight; ++r) {
      const int64_t e = base + (r0 + r) * (4 * kBandThreads) + tid * 4;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        float u1, v1;
        momentum_update(x[r][c], y[r][c], z[r][c], a.momentum, scale, NESTEROV, u1, v1);
        const uint32_t key = __float_as_uint(v1) & 0x7FFFFFFFu;
        const bool mine = in[r] || (e + c >= blk.lo && e + c < blk.hi);
        above += (uint32_t)__popcll(__ballot(mine && key >= ceil_key));
        ties += (uint32_t)__popcll(__ballot(mine && key == floor_key));
        // (a floor of all ones lies below every key)
        const bool inside = mine && (int32_t)key > (int32_t)floor_key && key < ceil_key;
        const unsigned long long votes = __ballot(inside);
        if (inside)
          list[wave * kSegment + listed +
               __builtin_amdgcn_mbcnt_hi((uint32_t)(votes >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)votes, 0u))] = key;
        listed += (uint32_t)__popcll(votes);
      }
    }
  }
  if (lane == 0) {
    counts[0][wave] = above;
    counts[1][wave] = ties;
    counts[2][wave] = listed;
  }
  __syncthreads();
  uint32_t before = 0, total = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    if (w < wave) before += counts[2][w];
    total += counts[2][w];
  }
  if (tid == 0) {
    uint32_t all_above = 0, all_ties = 0;
    for (int w = 0; w < kWaves; ++w) {
      all_above += counts[0][w];
      all_ties += counts[1][w];
    }
    if (all_above) atomicAdd(&st->above, all_above);
    if (all_ties) atomicAdd(&st->ties, all_ties);
    base_sh = total ? atomicAdd(&st->listed, total) : 0u;
  }
  __syncthreads();
  const int64_t begin = band_list_begin(blk.lo);
  const int64_t cap = band_list_begin(blk.hi) - begin;
  const int64_t at = (int64_t)base_sh + before;
  uint32_t* __restrict__ out = a.band_list + begin;
  for (uint32_t i = lane; i < listed; i += 64)
    if (at + i < cap) out[at + i] = list[wave * kSegment + i];  // (a list that does not fit is not used)
}

// One workgroup per tensor: the key of the wanted rank, from the band's list by histograms of 2048 bins
// over the interval that holds it, the last few hundred ranked directly.
template <bool NESTEROV>
__global__ __launch_bounds__(kSelectThreads) void rank_band_kernel(SelectArgs a) {
  typedef uint32_t vec4u __attribute__((ext_vector_type(4), aligned(4)));
  constexpr int kLoads = 4;
  __shared__ SelectShared sh;
  const int tid = threadIdx.x;
  const int j = blockIdx.x;
  if (a.floor.in_pass && a.state->crowded == 0) return;  // every floor went into the pass
  const TensorPlan plan = a.plans[j];
  const bool into_pass = floor_went_into_pass(a.floor, a.state, j);
  if (plan.exact != 2 || into_pass) return;
  const BandState st = *band_state(a, plan);
  const int64_t begin = band_list_begin(plan.offset);
  const int64_t cap = band_list_begin(plan.offset + plan.n) - begin;
  const uint32_t k = (uint32_t)plan.rank;
  const uint32_t m = st.listed;
  uint32_t thr_bits = 0;
  if (k >= st.above && k - st.above < m && (int64_t)m <= cap) {
    const uint32_t* __restrict__ list = a.band_list + begin;
    uint32_t rank = k - st.above;
    uint32_t lo = st.floor_key + 1u, width = st.ceil_key - lo;  // the keys lie in [lo, lo + width)
    const uint32_t quads = m >> 2;
    auto walk = [&](auto f) {  // f(key) for every key of the list
      for (uint32_t q0 = tid; q0 < quads; q0 += kLoads * kSelectThreads) {
        vec4u x[kLoads];
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
          const uint32_t q = q0 + i * kSelectThreads;
          x[i] = *reinterpret_cast<const vec4u*>(list + 4 * (int64_t)(q < quads ? q : 0u));
        }
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
          if (q0 + i * kSelectThreads < quads) {
#pragma unroll
            for (int c = 0; c < 4; ++c) f(x[i][c]);
          }
        }
      }
      if (tid < (int)(m & 3u)) f(list[4 * (int64_t)quads + tid]);
    };
#pragma unroll 1
    for (;;) {
      const int shift = width > (uint32_t)kSelectBins ? 21 - __clz((int)(width - 1u)) : 0;  // 11 bits stay
      for (int i = tid; i < kSelectBins; i += kSelectThreads) sh.hist[i] = 0;
      if (tid == 0) sh.surv_n = 0;
      __syncthreads();
      walk([&](uint32_t key) {
        if (key - lo < width) atomicAdd(&sh.hist[(key - lo) >> shift], 1u);
      });
      __syncthreads();
      uint32_t bin, over, members, all;
      find_bin<kSelectThreads>(sh.hist, sh.wave_tot, sh.sel, tid, rank, bin, over, members, all);
      rank -= over;
      lo += bin << shift;
      width = 1u << shift;
      if (shift == 0) {
        thr_bits = lo;
        break;
      }
      if (members <= (uint32_t)kSelectDirect) {
        if (tid < 4) sh.surv[(members & ~3u) + tid] = 0;
        __syncthreads();
        walk([&](uint32_t key) {
          if (key - lo < width) sh.surv[atomicAdd(&sh.surv_n, 1u)] = key;
        });
        __syncthreads();
        thr_bits = rank_directly(sh, tid, members, rank);
        break;
      }
    }
  } else if (k >= st.above + m && k - (st.above + m) < st.ties) {
    thr_bits = st.floor_key;
  } else {  // the band missed, or its list did not fit
    const float scale = a.scale_from_state ? a.state->scale : a.scale_const;
    const Candidates c = candidates_of(a, j, plan, scale, NESTEROV);
    thr_bits = rank_reevaluated(sh, c, plan.count, k, tid);
  }
  write_threshold(a, j, plan, __uint_as_float(thr_bits), tid);
}

// ---------------------------------------------------------------------------
// Streaming pass: momentum correction + mask
// (paper: Algorithm 3, the U and V update lines and the Mask line)
// ---------------------------------------------------------------------------
// A wavefront owns kWaveTile consecutive elements, read as kStreamUnroll rounds
// of one 16-byte vector per lane.  g, u and v are touched exactly once per
// iteration, so they are loaded and stored with the non-temporal hint.  The
// pass writes the pre-mask u', v' and one bit per element (|v'| > thr) and
// nothing else: no atomics, no scattered stores, nothing that depends on how
// many elements pass.  The emit pass below turns the bits into the payload and
// applies the mask to u and v.
//
// Mask layout: lane l of the wavefront that owns tile t stores a 16-bit word at
// mask[t * 64 + l]; bit q = r * 4 + c of it belongs to element
// t * kWaveTile + r * 256 + l * 4 + c.
//
// Tiles that lie inside one tensor (all but a few hundred) compare against one
// threshold.  Tiles that straddle tensors, and the ragged last tile, look up each
// element's tensor.
typedef float vec4 __attribute__((ext_vector_type(4)));

static_assert(kStreamUnroll >= 1 && kStreamUnroll <= 4, "mask words hold at most 16 bits per lane");

__device__ __forceinline__ int64_t tile_element(int64_t tile, int lane, int q) {
  return tile * kWaveTile + (q >> 2) * 256 + lane * 4 + (q & 3);
}

// Mask bits of a lane's sixteen elements (its v' in z) in a tile that is not wholly inside one tensor.
// `j0` is the tensor of the tile's first element.  The starts of the tensors after it are
// fetched 64 at a time, one per lane (those inside the tile form a prefix of the lanes because
// the offsets ascend) and handed round with readlane: one round of loads per 64 tensors, however many
// tensors share the tile.  The tile's thresholds are laid out in LDS, one per element (`thr_at`, one word
// per element of the tile), segment by segment, and every lane reads those of its elements: a tile of a
// handful of tiny tensors took 16 dependent reads per segment when the lanes' values lay there instead.
__device__ __forceinline__ uint32_t mixed_tile_mask(const StreamArgs& a, int64_t base, int lane, int32_t j0,
                                                    const vec4 (&z)[kStreamUnroll], float* thr_at) {
  const int32_t tile_end = base + kWaveTile <= a.n ? kWaveTile : (int32_t)(a.n - base);
  int32_t seg_lo = 0;            // the segment being closed starts here (relative to the tile)
  float seg_thr = a.thr[j0];     // ... and belongs to a tensor with this threshold
  auto fill = [&](int32_t from, int32_t to, float t) {
#pragma unroll 1
    for (int32_t p = from + lane; p < to; p += 64) thr_at[p] = t;
  };
  for (int32_t jb = j0 + 1; jb < a.num_tensors; jb += 64) {
    const int32_t jj = jb + lane;
    int32_t rel = kWaveTile;  // start of tensor jj relative to the tile, kWaveTile = not inside it
    float t = 0.0f;
    if (jj < a.num_tensors) {
      const int64_t o = a.offsets[jj];
      if (o < base + tile_end) {
        rel = o > base ? (int32_t)(o - base) : 0;
        t = a.thr[jj];
      }
    }
    const int cnt = __popcll(__ballot(rel < kWaveTile));
    for (int i = 0; i < cnt; ++i) {
      const int32_t seg_hi = __builtin_amdgcn_readlane(rel, i);
      fill(seg_lo, seg_hi, seg_thr);
      seg_lo = seg_hi;
      seg_thr = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int32_t)__float_as_uint(t), i));
    }
    if (cnt < 64) break;
  }
  fill(seg_lo, tile_end, seg_thr);
  fill(tile_end, kWaveTile, __builtin_inff());  // beyond the set: nothing passes
  wave_lds_fence();
  uint32_t cand = 0;
#pragma unroll
  for (int r = 0; r < kStreamUnroll; ++r) {
    const float4 t = *reinterpret_cast<const float4*>(thr_at + r * 256 + lane * 4);
    const float tc[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (fabsf(z[r][c]) > tc[c]) cand |= 1u << (4 * r + c);
  }
  return cand;
}

// Mask bits of the lane's NaNs that belong to tensors with a floor.  (Rare: `j0` is the tensor of the tile's first
// element, those behind it are walked over.)
__device__ __forceinline__ uint32_t band_nans(const StreamArgs& a, int64_t base, int lane, int32_t j0, const vec4 (&z)[kStreamUnroll]) {
  uint32_t found = 0;
#pragma unroll
  for (int q = 0; q < 4 * kStreamUnroll; ++q) {
    const float v = z[q >> 2][q & 3];
    const int64_t e = base + (q >> 2) * 256 + lane * 4 + (q & 3);
    if (v == v || e >= a.n) continue;
    int32_t j = j0;
    while (a.offsets[j + 1] <= e) ++j;
    if (a.plans[j].exact == 2 && floor_went_into_pass(a.floor, a.state, j)) found |= 1u << q;
  }
  return found;
}

// NESTEROV and SCALED are compile-time so that the sixteen updates of a lane are straight
// code: SCALED = false is the case scale == 1 exactly (no clipping), where g * 1.0f == g
// bit for bit and the multiplication is left out.  The kernel is memory-bound but a
// wave64 instruction occupies its SIMD for four cycles, so instructions saved per tile
// show in the run time.
//
// Every tile, whatever it holds, asks for its data first and all at once, then learns from
// ONE table word (a scalar load that depends on nothing) whether it lies wholly inside one
// tensor, in which case the word is its threshold, or not (NaN), in which case it fetches
// the tensor starts and thresholds it needs in one more round of loads.  A tile that took
// several dependent rounds, as a first version did, held up the end of the whole launch
// whenever it was dispatched late: 5 us of 88 on the 161-tensor set.
//
// STAGED (densities of the warm-up epochs, paper: Section 4): with a quarter of the elements
// selected, an emit pass that comes back for them reads every sector of v and rewrites
// every sector of u and v a second time.  Here a tile that lies wholly inside one tensor
// applies the mask to u and v before it stores them, and parks the selected v' (and u',
// which a full payload region needs to put back) in the tile's 1024 slots of a staging
// array, in index order: the emit pass then copies from there and touches u and v only
// where a region overflows.  An element's position among the tile's selected ones is
// rows before it + bits of its row in lower lanes (from the votes) + lower bits of its
// nibble.  Tiles shared between tensors are left to the emit pass as before.
//
// SLOTTED (densities up to 0.5 %, i.e. the 99.9 % sparsity the method runs at after its
// warm-up): a tile holds one or two selected elements, seldom more than a handful.  A tile
// that lies wholly inside one tensor and selects at most kSlotsPerTile elements parks their
// index, v' and u' (which a full payload region needs to put back) in a record that takes the
// place of the tile's mask words, in index order, and stores u and v masked: the emit pass copies
// from the record and neither decodes a mask word nor reads or rewrites u and v for such a tile.  Tiles with more selected elements, and tiles shared between tensors, are
// left to the emit pass as in the plain case (u', v' unmasked, mask bits set).
//
// BAND (exact selection at those densities): the threshold is a floor under the exact one, and refine_kernel settles
// which of the elements that pass are sent.  NaNs, which rank above everything, have to pass with them (those of
// tensors whose threshold comes from a band: the comparison lets none pass).
enum StreamMode : int { kStreamPlain = 0, kStreamStaged = 1, kStreamSlotted = 2, kStreamBand = 3 };



template <bool NESTEROV, bool SCALED, int MODE>
__global__ __launch_bounds__(kStreamThreads) void stream_kernel(StreamArgs a) {
  constexpr bool STAGED = MODE == kStreamStaged;
  constexpr bool SLOTTED = MODE == kStreamSlotted || MODE == kStreamBand;
  __shared__ alignas(16) float mixed_thr[kStreamWaves][kWaveTile];  // for tiles shared between tensors only
  constexpr int U = kStreamUnroll;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // uniform: table reads go scalar
  const int64_t tile = (int64_t)blockIdx.x * kStreamWaves + wave;
  const int64_t base = tile * kWaveTile;
  if (base >= a.n) return;
  const float scale = SCALED ? (a.scale_from_state ? a.state->scale : a.scale_const) : 1.0f;
  const bool full = base + kWaveTile <= a.n;
  const vec4* __restrict__ g4 = reinterpret_cast<const vec4*>(a.g + base) + lane;
  vec4* __restrict__ u4 = reinterpret_cast<vec4*>(a.u + base) + lane;
  vec4* __restrict__ v4 = reinterpret_cast<vec4*>(a.v + base) + lane;
  vec4 x[U], y[U], z[U];
  if (full) {
#pragma unroll
    for (int r = 0; r < U; ++r) {
      x[r] = __builtin_nontemporal_load(g4 + r * 64);
      y[r] = __builtin_nontemporal_load(u4 + r * 64);
      z[r] = __builtin_nontemporal_load(v4 + r * 64);
    }
  } else {  // the ragged last tile: element by element, zero beyond the end
#pragma unroll
    for (int r = 0; r < U; ++r) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int64_t e = base + r * 256 + lane * 4 + c;
        const bool in = e < a.n;
        x[r][c] = in ? a.g[e] : 0.0f;
        y[r][c] = in ? a.u[e] : 0.0f;
        z[r][c] = in ? a.v[e] : 0.0f;
      }
    }
  }
  const float thr = a.tile_thr[tile];
  const int32_t j0 = (int32_t)(a.tile_info[tile] & ~kTileMixed);

  const float m = a.momentum;
#pragma unroll
  for (int r = 0; r < U; ++r) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const float gs = SCALED ? x[r][c] * scale : x[r][c];
      float u1, v1;
      if (!NESTEROV) {
        const float t = m * y[r][c];
        u1 = t + gs;
        v1 = z[r][c] + u1;
      } else {
        const float s = y[r][c] + gs;
        u1 = m * s;
        const float w = z[r][c] + u1;
        v1 = w + gs;
      }
      y[r][c] = u1;
      z[r][c] = v1;
    }
  }
  uint32_t nans = 0;
  if (MODE == kStreamBand) {
    float sum = 0.0f;  // a NaN if any of the elements is one (or there are infinities of both signs)
#pragma unroll
    for (int q = 0; q < 4 * U; ++q) sum += z[q >> 2][q & 3];
    if (__ballot(sum != sum) != 0) nans = band_nans(a, base, lane, j0, z);
  }
  if (STAGED && thr == thr) {  // wholly inside one tensor (and so a whole tile)
    uint32_t cand = 0;
#pragma unroll
    for (int q = 0; q < 4 * U; ++q)
      if (fabsf(z[q >> 2][q & 3]) > thr) cand |= 1u << q;
    float* __restrict__ stage_v = a.stage_v + base;
    float* __restrict__ stage_u = a.stage_u ? a.stage_u + base : nullptr;
    const bool clear_u = a.factor_masking != 0;
    int row_base = 0;
#pragma unroll
    for (int r = 0; r < U; ++r) {
      const uint32_t nib = (cand >> (4 * r)) & 0xFu;
      int lower = 0, row = 0;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const unsigned long long vote = __ballot((nib >> c) & 1u);
        lower += (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(vote >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)vote, 0u));
        row += __popcll(vote);
      }
      int pos = row_base + lower;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if ((nib >> c) & 1u) {
          stage_v[pos] = z[r][c];
          if (stage_u) stage_u[pos] = y[r][c];
          z[r][c] = 0.0f;
          if (clear_u) y[r][c] = 0.0f;
          ++pos;
        }
      }
      row_base += row;
    }
#pragma unroll
    for (int r = 0; r < U; ++r) {
      __builtin_nontemporal_store(y[r], u4 + r * 64);
      __builtin_nontemporal_store(z[r], v4 + r * 64);
    }
    a.mask[tile * 64 + lane] = (uint16_t)cand;
    if (lane == 0) a.tile_count[tile] = (uint32_t)row_base;
    return;
  }
  if (SLOTTED && thr == thr) {  // wholly inside one tensor (and so a whole tile)
    uint32_t cand = nans;
#pragma unroll
    for (int q = 0; q < 4 * U; ++q)
      if (fabsf(z[q >> 2][q & 3]) > thr) cand |= 1u << q;
    // A row (one 16-byte vector per lane) without a selected element, which is most rows, goes out
    // at once: how long a wavefront holds on to its data after the loads have come back is what
    // the pass's throughput hangs on, and the bookkeeping below is long enough to show.
    unsigned long long row_holders[U];
#pragma unroll
    for (int r = 0; r < U; ++r) {
      row_holders[r] = __ballot(((cand >> (4 * r)) & 0xFu) != 0);
      if (row_holders[r] == 0) {
        __builtin_nontemporal_store(y[r], u4 + r * 64);
        __builtin_nontemporal_store(z[r], v4 + r * 64);
      }
    }
    const int total = (int)wave_sum((uint32_t)__popc(cand));
    if (total > 0 && total <= kSlotsPerTile) {  // uniform
      // The few selected elements are taken row by row, one at a time, everything about them in
      // scalar registers (which lane, which of its four elements): the values are read from that
      // lane, and the tile's record is put together across lanes 0 .. 31 (index of element p in
      // lane p, its v' in lane 8 + p, its u' in lane 16 + p) and stored whole, as one 128-byte
      // line.  (Scattered 4-byte stores from inside this pass cost 26 us on a 122 M-element set:
      // every one is a partial write of a line; a record array of its own with a line for every
      // tile that has a record, a stream of stores with holes in it, 7 us.)
      const bool clear_u = a.factor_masking != 0;
      int record = 0;
      int pos = 0;
#pragma unroll
      for (int r = 0; r < U; ++r) {
        unsigned long long holders = row_holders[r];
        if (holders == 0) continue;
        const uint32_t nib = (cand >> (4 * r)) & 0xFu;
        do {
          const int l = __ffsll((long long)holders) - 1;
          holders &= holders - 1;
          uint32_t w = (uint32_t)__builtin_amdgcn_readlane((int)nib, l);
          do {
            const int c = __ffs(w) - 1;  // uniform: the component is picked in every lane, then read from lane l
            w &= w - 1;
            const float zc = c == 0 ? z[r][0] : c == 1 ? z[r][1] : c == 2 ? z[r][2] : z[r][3];
            const float yc = c == 0 ? y[r][0] : c == 1 ? y[r][1] : c == 2 ? y[r][2] : y[r][3];
            const int zv = __builtin_amdgcn_readlane(__float_as_int(zc), l);
            const int yv = __builtin_amdgcn_readlane(__float_as_int(yc), l);
            const int e = (int32_t)(base + r * 256 + l * 4 + c);
            if (lane == pos) record = e;
            if (lane == kSlotsPerTile + pos) record = zv;
            if (lane == 2 * kSlotsPerTile + pos) record = yv;
            ++pos;
          } while (w);
        } while (holders);
        // the mask applied to this row of u and v
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const bool sel = (nib >> c) & 1u;
          z[r][c] = sel ? 0.0f : z[r][c];
          if (clear_u) y[r][c] = sel ? 0.0f : y[r][c];
        }
      }
      // the record takes the place of the tile's mask words (both are one 128-byte line per tile;
      // the count says which of the two the line holds)
      if (lane < kSlotRecord) reinterpret_cast<int32_t*>(a.mask)[tile * kSlotRecord + lane] = record;
    } else {  // (an empty tile's line is written too: a stream of stores with holes in it runs slower)
      a.mask[tile * 64 + lane] = (uint16_t)cand;
    }
#pragma unroll
    for (int r = 0; r < U; ++r) {
      if (row_holders[r] != 0) {
        __builtin_nontemporal_store(y[r], u4 + r * 64);
        __builtin_nontemporal_store(z[r], v4 + r * 64);
      }
    }
    // (the flag: this line holds mask words although the tile lies inside one tensor -- a count that
    // the re-threshold pass lowers to kSlotsPerTile or less must not make the line pass for a record)
    if (lane == 0) a.tile_count[tile] = (uint32_t)total | (total > kSlotsPerTile ? kTileCountHasMask : 0u);
    return;
  }
  // u' and v' go out first: once stored, u' need not be kept while the mask is worked out
  if (full) {
#pragma unroll
    for (int r = 0; r < U; ++r) {
      __builtin_nontemporal_store(y[r], u4 + r * 64);
      __builtin_nontemporal_store(z[r], v4 + r * 64);
    }
  } else {
#pragma unroll
    for (int r = 0; r < U; ++r) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int64_t e = base + r * 256 + lane * 4 + c;
        if (e < a.n) {
          a.u[e] = y[r][c];
          a.v[e] = z[r][c];
        }
      }
    }
  }
  uint32_t cand = 0;
  if (thr == thr) {  // the whole tile belongs to one tensor
#pragma unroll
    for (int q = 0; q < 4 * U; ++q)
      if (fabsf(z[q >> 2][q & 3]) > thr) cand |= 1u << q;
  } else {
    cand = mixed_tile_mask(a, base, lane, j0, z, mixed_thr[wave]) | nans;
  }
  a.mask[tile * 64 + lane] = (uint16_t)cand;
  // bits set in the tile, for the index-ordered emit pass (measured: no cost here)
  const int bits = (int)wave_sum((uint32_t)__popc(cand));
  if (lane == 0) a.tile_count[tile] = (uint32_t)bits;
}

// Yardstick for the streaming pass: the same traffic (three arrays read, two written,
// non-temporal, one wave tile per wavefront) with next to no arithmetic, no table and no
// mask.  What this kernel reaches on a box is the ceiling the streaming pass can be held
// against besides the nominal HBM peak.  Whole tiles only.
__global__ __launch_bounds__(64) void ceiling_kernel(const float* __restrict__ a, float* __restrict__ b,
                                                     float* __restrict__ c, int64_t tiles) {
  constexpr int U = kStreamUnroll;
  const int lane = threadIdx.x;
  const int64_t tile = blockIdx.x;  // one wavefront per workgroup: the residency is set in wavefronts
  if (tile >= tiles) return;
  const vec4* a4 = reinterpret_cast<const vec4*>(a + tile * kWaveTile) + lane;
  vec4* b4 = reinterpret_cast<vec4*>(b + tile * kWaveTile) + lane;
  vec4* c4 = reinterpret_cast<vec4*>(c + tile * kWaveTile) + lane;
  vec4 x[U], y[U], z[U];
#pragma unroll
  for (int r = 0; r < U; ++r) {
    x[r] = __builtin_nontemporal_load(a4 + r * 64);
    y[r] = __builtin_nontemporal_load(b4 + r * 64);
    z[r] = __builtin_nontemporal_load(c4 + r * 64);
  }
#pragma unroll
  for (int r = 0; r < U; ++r) {
    y[r] = y[r] + x[r];
    z[r] = z[r] + y[r];
    __builtin_nontemporal_store(y[r], b4 + r * 64);
    __builtin_nontemporal_store(z[r], c4 + r * 64);
  }
}

// This thread's share of the sum of tile_count[b .. e) (the counts proper: the flag of the slotted
// pass is masked off): the counts are fetched four to a load
// (the last workgroup of a 4.7 M-element tensor adds up 4600 of them: with one count per load
// that was three rounds of loads in a row, 6 us of the emit pass on a 122 M-element set).
template <int THREADS>
__device__ __forceinline__ int tile_counts_partial(const uint32_t* __restrict__ tc, int64_t b64, int64_t e64, int tid) {
  const int32_t b = (int32_t)b64, e = (int32_t)e64;  // tiles: below 2^21
  int sum = 0;
  if (b >= e) return 0;
  int32_t b4 = (b + 3) & ~3;  // first multiple of four at or above b
  if (b4 > e) b4 = e;
  int32_t e4 = e & ~3;
  if (e4 < b4) e4 = b4;
  // at most three counts before the aligned body and three behind it
  if (tid < b4 - b) sum += (int)(tc[b + tid] & kTileCountMask);
  if (tid < e - e4) sum += (int)(tc[e4 + tid] & kTileCountMask);
  const uint4* __restrict__ tc4 = reinterpret_cast<const uint4*>(tc);  // the table starts on a 256-byte boundary
  const int32_t q0 = b4 >> 2, q1 = e4 >> 2;
  int32_t q = q0 + tid;
  for (; q + 3 * THREADS < q1; q += 4 * THREADS) {  // four loads in flight per thread
    uint4 c[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) c[k] = tc4[q + k * THREADS];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      sum += (int)((c[k].x & kTileCountMask) + (c[k].y & kTileCountMask) + (c[k].z & kTileCountMask) + (c[k].w & kTileCountMask));
  }
  for (; q < q1; q += THREADS) {
    const uint4 c = tc4[q];
    sum += (int)((c.x & kTileCountMask) + (c.y & kTileCountMask) + (c.z & kTileCountMask) + (c.w & kTileCountMask));
  }
  return sum;
}

// ---------------------------------------------------------------------------
// Re-threshold on over-selection
// (paper: Section 5 -- the exact threshold among the elements that passed, for a
//  tensor that let too many pass)
// ---------------------------------------------------------------------------
// Runs between the streaming and the emit pass, one workgroup per tensor.  The workgroup adds up
// the mask-bit counts the streaming pass has left for the tensor's tiles; only if the total
// exceeds refine_limit does it go on: it finds the magnitude of descending rank k among |v'| of
// the selected elements exactly, and a last walk clears the mask bits, and lowers the counts of the records, of
// elements that do not exceed it.  What the emit pass then extracts is the exact top k of the
// tensor.  (A first version ran over the emit work list: every workgroup recounted its part's
// mask words and took a ticket on the tensor's counter, the last to arrive went on; 17 us on the
// 161-tensor set and 34 us on the 122 M-element set for what the per-tile counts already say.)
// EXACT SELECTION at densities up to kBandInPassDensity comes here, too: select_kernel has named a floor that lies below
// the exact threshold almost surely, the pass took what exceeds it, and every such tensor is ranked here.  The streaming
// pass is then the only one over g, u, v: 161 tensors of 25.6 M elements, 0.1 %, call 175 -> 139 us where bands were
// collected by another pass.  (Tensors whose sample does not bear the floor out still are: with large values in rows of
// every second large tensor, placed anew every third call, the median of the calls is 195 us and the worst 220, where bands
// alone take 187 and 1467; with such rows in one tensor of fifty 158, against 178.)
// After a slotted pass over a tensor of up to 4096 tiles the keys of the records stay in registers, from the one read of the
// lines to the lowered counts; what mask words say, and the elements of larger tensors or of other passes, up to
// kRefineList of them, is listed in LDS.  One histogram and a direct ranking settle the threshold; the over-selection of a big
// tensor goes to the payload region, which is free until the emit
// pass, and through three histogram passes.  Bound by latency, a chain of dependent steps in the dozen
// workgroups that go on: 11 us on the 161-tensor set (14.4 with the records' elements listed in LDS and read again for the
// counts, two look-ups of every line, and a prefix over the bins through LDS; 23 with the list always in the payload region),
// and with exact selection there, where every large tensor goes on, 14.5 (21.5).  The lists
// (and 16 wavefronts of more than 64 registers) leave one workgroup per compute unit; 20000 tensors, most of which
// only add up their counts, take 133 us as they did without the lists.
struct RefineShared {
  SelectShared s;
  uint32_t list[kRefineList];
  uint32_t keys[kRefineList];
  alignas(16) int red[kRefineThreads / 64];
  uint32_t listed;
};
static_assert(kRefineThreads == kSelectThreads, "the ranking is shared with select_kernel");

// This thread's filtered mask word `wi` (0-based within the tensor's tiles) of tensor [lo, hi).
__device__ __forceinline__ uint32_t tensor_mask_word(const uint16_t* mask, int64_t t0, int64_t wi, int64_t lo,
                                                     int64_t hi, int64_t& tile, int& lane) {
  constexpr int kBits = kStreamUnroll * 4;
  tile = t0 + (wi >> 6);
  lane = (int)(wi & 63);
  uint32_t w = mask[tile * 64 + lane];
  if (w && (tile * kWaveTile < lo || (tile + 1) * kWaveTile > hi)) {
    uint32_t keep = 0;
    for (int q = 0; q < kBits; ++q) {
      const int64_t e = tile_element(tile, lane, q);
      if (e >= lo && e < hi) keep |= 1u << q;
    }
    w &= keep;
  }
  return w;
}

__global__ __launch_bounds__(kRefineThreads) void refine_kernel(RefineArgs a) {
  constexpr int kWaves = kRefineThreads / 64;
  __shared__ RefineShared sh;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int j = blockIdx.x;
  const TensorPlan plan = a.plans[j];
  const int64_t region = a.out_offsets[j];  // asked for early: needed late
  const int64_t cap = a.out_offsets[j + 1] - region;
  const int64_t lo = plan.offset;
  const int64_t hi = plan.offset + plan.n;
  const int64_t t0 = lo / kWaveTile;
  const int64_t t1 = (hi - 1) / kWaveTile;
  // Exact selection: the pass took whatever exceeds a floor, NaNs too, and the threshold is settled here in any case.
  const bool into_pass = floor_went_into_pass(a.floor, a.state, j);
  const bool banded = plan.exact == 2 && into_pass;
  if (!banded && !a.on_excess) return;

  // How many elements of the tensor passed: the counts the streaming pass has left for the tiles
  // that lie wholly inside the tensor, and the tensor's share of a first or last tile that it
  // shares with a neighbour (or that is the ragged end of the set), recounted from the mask words.
  const bool shared0 = t0 * kWaveTile < lo || (t0 == t1 && (t1 + 1) * kWaveTile > hi);
  const bool shared1 = t1 != t0 && (t1 + 1) * kWaveTile > hi;
  // After a slotted pass over up to kRefineHeld / 2 tiles per thread the counts stay in registers, and the keys of the records
  // will, which are asked for before the counts are there where they are wanted in any case.  Two neighbouring threads share a
  // tile, half a record's keys each: a line is looked up once for both.
  constexpr int kHalf = kSlotsPerTile / 2;
  const int half = tid & 1;
  auto tile_of = [&](int k) { return t0 + ((k * kRefineThreads + tid) >> 1); };
  const int groups = (int)((2 * (t1 - t0) + 1) / kRefineThreads) + 1;  // of items to a thread that are in use
  const bool held = a.slotted && groups <= kRefineHeld;
  uint32_t held_count[kRefineHeld];     // elements in a record
  bool held_words[kRefineHeld];         // the tile has mask words, and the thread looks after them
  int4 held_keys[kRefineHeld];
  auto load_keys = [&](int k) {
    const int64_t tile = tile_of(k);
    held_keys[k] = reinterpret_cast<const int4*>(a.mask)[(tile <= t1 ? tile : t1) * (kSlotRecord / 4) + kSlotsPerTile / 4 + half];
  };
  int cnt = 0;
  if (held) {
    uint32_t c[kRefineHeld];
#pragma unroll
    for (int k = 0; k < kRefineHeld; ++k) {
      c[k] = 0;
      held_keys[k] = make_int4(0, 0, 0, 0);
      if (k >= groups) continue;  // uniform
      const int64_t tile = tile_of(k);
      c[k] = a.tile_count[tile <= t1 ? tile : t1];
    }
    if (banded) {
#pragma unroll
      for (int k = 0; k < kRefineHeld; ++k)
        if (k < groups) load_keys(k);  // uniform
    }
#pragma unroll
    for (int k = 0; k < kRefineHeld; ++k) {
      const int64_t tile = tile_of(k);
      const bool whole = tile <= t1 && tile * kWaveTile >= lo && (tile + 1) * kWaveTile <= hi;
      held_words[k] = half == 0 && tile <= t1 && (!whole || c[k] > (uint32_t)kSlotsPerTile);
      held_count[k] = whole && c[k] <= (uint32_t)kSlotsPerTile ? c[k] : 0u;
      if (whole && half == 0) cnt += (int)(c[k] & kTileCountMask);
    }
  } else {
    cnt = tile_counts_partial<kRefineThreads>(a.tile_count, shared0 ? t0 + 1 : t0, shared1 ? t1 : t1 + 1, tid);
  }
  {
    int64_t tile;
    int l;
    if (shared0 && wave == 0) cnt += __popc(tensor_mask_word(a.mask, t0, lane, lo, hi, tile, l));
    if (shared1 && wave == 1) cnt += __popc(tensor_mask_word(a.mask, t0, (t1 - t0) * 64 + lane, lo, hi, tile, l));
  }
  cnt = (int)wave_sum((uint32_t)cnt);
  if (lane == 0) sh.red[wave] = cnt;
  if (tid == 0) sh.listed = 0;
  __syncthreads();
  int total = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) total += sh.red[w];
  if (!banded && (uint32_t)total <= (uint32_t)plan.refine_limit) return;

  // ---- exact threshold among the selected elements of tensor j (rare) ---------------
  // After a slotted streaming pass a tile that lies wholly inside the tensor and selected 1 to
  // kSlotsPerTile elements holds a record in place of its mask words (indices, v', u'), and u and
  // v are masked there already; every other tile has mask words and u', v' as they were.
  const int64_t words = (t1 - t0 + 1) * 64;
  const int64_t passed = total;
  uint32_t prefix = 0;
  uint32_t rank = (uint32_t)plan.k;
  int consumed = 0;
  uint32_t* mask32 = reinterpret_cast<uint32_t*>(a.mask);
  const int32_t* records = reinterpret_cast<const int32_t*>(a.mask);
  auto is_record = [&](int64_t tile) {
    if (!a.slotted || tile * kWaveTile < lo || (tile + 1) * kWaveTile > hi) return false;
    const uint32_t c = a.tile_count[tile];  // (with the flag: mask words, whatever the count)
    return c >= 1u && c <= (uint32_t)kSlotsPerTile;
  };
  constexpr uint32_t kFromRecord = 0x80000000u;  // list entry: the element sits in a record (indices are below 2^31)
  const float floor = a.thr[j];  // every selected element exceeds it
  // Takes the mask bit of element e away, and one from the count of its tile; by whole wavefronts.  Neighbours in a
  // list mostly lie in one tile, and additions to words of one line are carried out one by one: one per tile and
  // wavefront (3.8 M elements whose largest values fill 20 rows of 650, all above the floor: call 167 -> 105 us).
  auto drop_bit = [&](bool drop, uint32_t e) {
    const uint32_t tile = e / kWaveTile, r = e % kWaveTile;
    if (drop) {
      const int64_t h = (int64_t)tile * 64 + ((r & 255u) >> 2);  // the lane's 16-bit word
      const uint32_t b = (r >> 8) * 4u + (r & 3u);
      atomicAnd(&mask32[h >> 1], ~((1u << b) << (16 * (int)(h & 1))));
    }
    for (unsigned long long left = __ballot(drop); left;) {
      const int leader = __ffsll((long long)left) - 1;
      const uint32_t its = (uint32_t)__shfl((int)tile, leader);
      const unsigned long long same = __ballot(drop && tile == its);
      if (lane == leader) atomicSub(&a.tile_count[its], (uint32_t)__popcll(same));
      left &= ~same;
    }
  };

  bool missed = banded && passed <= (int64_t)rank && floor > 0.0f;
  if (missed) {
    // Values that occur many times (rounded or ternary gradients): the floor is itself the threshold if enough
    // elements equal it, and what has passed is what is sent.  As much of the tensor is looked at as that takes
    // (A set without lists, see select_kernel; in others such tensors do not come here.)
    constexpr int kPer = 32;
    const uint32_t floor_key = __float_as_uint(floor);
    const uint32_t enough = rank - (uint32_t)passed + 1u;
#pragma unroll 1
    for (int64_t first = lo; missed && first < hi; first += kPer * kRefineThreads) {
      uint32_t key[kPer];
#pragma unroll
      for (int q = 0; q < kPer; ++q) {
        const int64_t e = first + q * kRefineThreads + tid;
        key[q] = __float_as_uint(a.v_out[e < hi ? e : hi - 1]) & 0x7FFFFFFFu;
        if (e >= hi) key[q] = kNoKey;
      }
      uint32_t same = 0;
#pragma unroll
      for (int q = 0; q < kPer; ++q) same += key[q] == floor_key ? 1u : 0u;
      same = wave_sum(same);
      if (lane == 0 && same) atomicAdd(&sh.listed, same);
      __syncthreads();
      missed = sh.listed < enough;
      __syncthreads();
    }
    if (!missed) {
      prefix = floor_key;
      if (tid == 0) sh.listed = 0;
      __syncthreads();
    }
  }
  if (missed) {
    // The floor lies above the threshold (the sample missed): everything goes back to u and v, the whole tensor is
    // ranked as it stands there, and its tiles get mask words.  One workgroup over the tensor four times, 1.9 ms for
    // 3 M elements; this
    // takes single values that are large where the sample looks, or the chance of one in a million.
    for (int64_t tile = t0 + tid; tile <= t1; tile += kRefineThreads) {
      if (!is_record(tile)) continue;
      const int c = (int)a.tile_count[tile];
      for (int q = 0; q < c; ++q) {
        const int32_t* r = records + tile * kSlotRecord + q;
        a.v_out[r[0]] = __int_as_float(r[kSlotsPerTile]);
        if (a.factor_masking) a.u_out[r[0]] = __int_as_float(r[2 * kSlotsPerTile]);
      }
    }
    __syncthreads();
    auto key_at = [&](int64_t e) { return __float_as_uint(a.v_out[e]) & 0x7FFFFFFFu; };
#pragma unroll 1
    for (int pass = 0; pass < 3; ++pass) {
      const int bits = pass == 2 ? 9 : 11;
      const int shift = 31 - consumed - bits;
      const uint32_t digit_mask = (1u << bits) - 1u;
      for (int i = tid; i < kSelectBins; i += kRefineThreads) sh.s.hist[i] = 0;
      __syncthreads();
      constexpr int kPer = 16;  // loads on their way
#pragma unroll 1
      for (int64_t first = lo; first < hi; first += kPer * kRefineThreads) {
        uint32_t key[kPer];
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
          const int64_t e = first + q * kRefineThreads + tid;
          key[q] = key_at(e < hi ? e : hi - 1);
          if (e >= hi) key[q] = kNoKey;
        }
#pragma unroll
        for (int q = 0; q < kPer; ++q)
          if (key[q] != kNoKey && (pass == 0 || (key[q] >> (shift + bits)) == prefix)) atomicAdd(&sh.s.hist[(key[q] >> shift) & digit_mask], 1u);
      }
      __syncthreads();
      uint32_t bin, above, members, all;
      find_bin<kRefineThreads>(sh.s.hist, sh.s.wave_tot, sh.s.sel, tid, rank, bin, above, members, all);
      prefix = (prefix << bits) | bin;
      rank -= above;
      consumed += bits;
    }
    for (int64_t tile = t0 + wave; tile <= t1; tile += kWaves) {
      uint32_t own = 0, word = 0;  // the lane's elements that belong to the tensor, and those that are sent
      uint32_t key[4 * kStreamUnroll];
#pragma unroll
      for (int q = 0; q < 4 * kStreamUnroll; ++q) {
        const int64_t e = tile_element(tile, lane, q);
        key[q] = key_at(e < lo ? lo : e < hi ? e : hi - 1);
        if (e >= lo && e < hi) own |= 1u << q;
      }
#pragma unroll
      for (int q = 0; q < 4 * kStreamUnroll; ++q)
        if (sent(key[q], prefix)) word |= (own >> q & 1u) << q;
      if (tile * kWaveTile >= lo && (tile + 1) * kWaveTile <= hi) {
        a.mask[tile * 64 + lane] = (uint16_t)word;
        const uint32_t c = wave_sum((uint32_t)__popc(word));
        if (lane == 0) a.tile_count[tile] = c ? c | kTileCountHasMask : 0u;
      } else {  // shared with a neighbour, whose bits stay (counts of such tiles are formed from the words)
        const int64_t h = tile * 64 + lane;
        const int sh16 = 16 * (int)(h & 1);
        atomicAnd(&mask32[h >> 1], ~(own << sh16));
        atomicOr(&mask32[h >> 1], word << sh16);
      }
    }
    if (tid == 0) {
      const float thr = __uint_as_float(prefix);
      a.thr[j] = thr;
      if (a.out_thr) a.out_thr[j] = thr;
    }
    return;
  }

  auto list_words = [&](int64_t tile, int l, uint32_t w) {  // a lane's mask word, this tensor's bits only
    int pos = (int)atomicAdd(&sh.listed, (uint32_t)__popc(w));
    while (w) {
      const int q = __ffs(w) - 1;
      w &= w - 1;
      sh.list[pos++] = (uint32_t)tile_element(tile, l, q);
    }
  };
  // One histogram over the four octaves above the sampled threshold, where the wanted rank nearly always
  // is (the last bin takes everything beyond), and direct ranking of its bin; if that does not fit, the
  // passes over the key's bits.  `sh.s.hist` and `sh.s.surv_n` are zero.
  // `in_use(q)`, uniform: some thread may have a key in slot q.
  auto settle = [&](const auto& key, auto in_use) {
    constexpr int kKeys = sizeof(key) / sizeof(uint32_t);
    constexpr int kShift = 14;
    const uint32_t low = floor >= 0.0f ? __float_as_uint(floor) : 0u;  // -1: everything was let through
#pragma unroll
    for (int q = 0; q < kKeys; ++q) {
      if (!in_use(q)) continue;
      const uint32_t b = (key[q] - low) >> kShift;
      if (key[q] != kNoKey) atomicAdd(&sh.s.hist[b < (uint32_t)kSelectBins ? b : (uint32_t)kSelectBins - 1u], 1u);
    }
    __syncthreads();
    uint32_t bin, above, members, all;
    find_bin<kRefineThreads>(sh.s.hist, sh.s.wave_tot, sh.s.sel, tid, rank, bin, above, members, all);
    if (members <= (uint32_t)kSelectDirect) {
      if (tid < 4) sh.s.surv[(members & ~3u) + tid] = 0;
      __syncthreads();
      const uint32_t first = low + (bin << kShift);  // the bin's keys: this one, and `span` behind it
      const uint32_t span = bin < (uint32_t)kSelectBins - 1u ? (1u << kShift) - 1u : kNoKey - 1u - first;
#pragma unroll
      for (int q = 0; q < kKeys; ++q)
        if (in_use(q) && key[q] - first <= span) sh.s.surv[atomicAdd(&sh.s.surv_n, 1u)] = key[q];
      __syncthreads();
      return rank_directly(sh.s, tid, members, rank - above);
    }
    __syncthreads();
    return select_in_registers<kKeys>(sh.s, key, kKeys, 0u, rank, tid);
  };
  auto clear_bins = [&]() {
    for (int b = tid; b < kSelectBins; b += kRefineThreads) sh.s.hist[b] = 0;
    if (tid == 0) sh.s.surv_n = 0;
  };

  if (held && passed <= kRefineList) {
    // The keys of the records in registers, where they stay until the tiles' counts are lowered; what mask words say, which
    // is little as a rule, is listed.
    constexpr int kRecordKeys = kRefineHeld * kHalf;
    constexpr int kWordKeys = 4;
    clear_bins();
#pragma unroll
    for (int k = 0; k < kRefineHeld; ++k) {
      if (k >= groups) continue;  // uniform
      if (!banded) load_keys(k);
      for (unsigned long long m = __ballot(held_words[k]); m; m &= m - 1) {
        const int64_t wi = (((int64_t)k * kRefineThreads + wave * 64 + (__ffsll((long long)m) - 1)) >> 1) * 64 + lane;
        int64_t tile;
        int l;
        const uint32_t w = tensor_mask_word(a.mask, t0, wi, lo, hi, tile, l);
        if (w) list_words(tile, l, w);
      }
    }
    __syncthreads();
    const uint32_t listed = sh.listed;
    if (listed <= (uint32_t)(kWordKeys * kRefineThreads)) {
      uint32_t key[kRecordKeys + kWordKeys];
      uint32_t from[kWordKeys];
#pragma unroll
      for (int q = 0; q < kWordKeys; ++q) {
        const uint32_t p = (uint32_t)(tid + q * kRefineThreads);
        from[q] = p < listed ? sh.list[p] : 0u;
        key[kRecordKeys + q] = kNoKey;
        if (p < listed) key[kRecordKeys + q] = __float_as_uint(a.v[from[q]]) & 0x7FFFFFFFu;
      }
#pragma unroll
      for (int k = 0; k < kRefineHeld; ++k) {
        const int32_t x[kHalf] = {held_keys[k].x, held_keys[k].y, held_keys[k].z, held_keys[k].w};
#pragma unroll
        for (int q = 0; q < kHalf; ++q)
          key[k * kHalf + q] = (uint32_t)(half * kHalf + q) < held_count[k] ? (uint32_t)x[q] & 0x7FFFFFFFu : kNoKey;
      }
      auto in_use = [&](int q) {
        return q < kRecordKeys ? q / kHalf < groups : (q - kRecordKeys) * kRefineThreads < (int)listed;
      };
      if (passed > (int64_t)rank) prefix = settle(key, in_use);  // (else: see below)
#pragma unroll
      for (int q = 0; q < kWordKeys; ++q) {
        const bool drop = (uint32_t)(tid + q * kRefineThreads) < listed && !sent(key[kRecordKeys + q], prefix);
        if (q * kRefineThreads < (int)listed) drop_bit(drop, from[q]);  // uniform
      }
#pragma unroll
      for (int k = 0; k < kRefineHeld; ++k) {
        if (k >= groups) break;  // uniform
        uint32_t kept = 0;
#pragma unroll
        for (int q = 0; q < kHalf; ++q) kept += sent(key[k * kHalf + q], prefix) ? 1u : 0u;
        kept += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)kept, 0xB1, 0xf, 0xf, false);  // the neighbour's
        if (half == 0 && kept != held_count[k]) a.tile_count[tile_of(k)] = kept | (held_count[k] << kTileCountHeldShift);
      }
      if (tid == 0) {
        const float thr = __uint_as_float(prefix);
        a.thr[j] = thr;
        if (a.out_thr) a.out_thr[j] = thr;
      }
      return;
    }
    __syncthreads();  // (the list's length is read before it is formed anew)
  }

  if (passed <= kRefineList) {
    // From the records: one thread per tile, the counts of four tiles and then their records in flight
    // together; from the mask words of the other tiles: by the wavefront whose lanes met them.
    if (tid == 0) sh.listed = 0;
    __syncthreads();
    if (a.slotted) {
      constexpr int kTilesInFlight = 4;
#pragma unroll 1
      for (int64_t first = t0; first <= t1; first += kTilesInFlight * kRefineThreads) {
        uint32_t c[kTilesInFlight];
        bool words_here[kTilesInFlight];
#pragma unroll
        for (int k = 0; k < kTilesInFlight; ++k) {
          const int64_t tile = first + k * kRefineThreads + tid;
          c[k] = tile <= t1 ? a.tile_count[tile] : 0u;
        }
        int4 e[kTilesInFlight][2], x[kTilesInFlight][2];
#pragma unroll
        for (int k = 0; k < kTilesInFlight; ++k) {
          const int64_t tile = first + k * kRefineThreads + tid;
          const bool whole = tile * kWaveTile >= lo && (tile + 1) * kWaveTile <= hi;
          words_here[k] = tile <= t1 && (!whole || c[k] > (uint32_t)kSlotsPerTile);
          if (words_here[k]) c[k] = 0u;
          const int4* __restrict__ r = reinterpret_cast<const int4*>(records + tile * kSlotRecord);
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            e[k][h] = x[k][h] = make_int4(0, 0, 0, 0);
            if (c[k] > 4u * h) {
              e[k][h] = r[h];
              x[k][h] = r[kSlotsPerTile / 4 + h];
            }
          }
        }
        // one addition to the list's length per wavefront: those of its lanes would be carried out one by one
        uint32_t at[kTilesInFlight], all = 0;
#pragma unroll
        for (int k = 0; k < kTilesInFlight; ++k) {
          at[k] = all;
          all += c[k];
        }
        const uint32_t upto = wave_inclusive_sum(all);
        uint32_t from = 0;
        if (lane == 63 && upto > 0u) from = atomicAdd(&sh.listed, upto);
        from = wave_last(from) + upto - all;
#pragma unroll
        for (int k = 0; k < kTilesInFlight; ++k) {
          if (c[k] == 0u) continue;
          const uint32_t pos = from + at[k];
          const int32_t ee[8] = {e[k][0].x, e[k][0].y, e[k][0].z, e[k][0].w, e[k][1].x, e[k][1].y, e[k][1].z, e[k][1].w};
          const int32_t xx[8] = {x[k][0].x, x[k][0].y, x[k][0].z, x[k][0].w, x[k][1].x, x[k][1].y, x[k][1].z, x[k][1].w};
#pragma unroll
          for (uint32_t q = 0; q < (uint32_t)kSlotsPerTile; ++q) {
            if (q < c[k]) {
              sh.list[pos + q] = (uint32_t)ee[q] | kFromRecord;
              sh.keys[pos + q] = (uint32_t)xx[q] & 0x7FFFFFFFu;
            }
          }
        }
#pragma unroll
        for (int k = 0; k < kTilesInFlight; ++k) {
          for (unsigned long long m = __ballot(words_here[k]); m; m &= m - 1) {
            const int64_t wi = (first - t0 + k * kRefineThreads + wave * 64 + (__ffsll((long long)m) - 1)) * 64 + lane;
            int64_t tile;
            int l;
            const uint32_t w = tensor_mask_word(a.mask, t0, wi, lo, hi, tile, l);
            if (w) list_words(tile, l, w);
          }
        }
      }
    } else {
      // eight words (16 bytes) per load, four loads in flight per thread
      const uint4* mask128 = reinterpret_cast<const uint4*>(a.mask + t0 * 64);
      const int64_t chunks = words >> 3;
      for (int64_t c0 = tid; c0 < chunks; c0 += 4 * kRefineThreads) {
        uint4 m[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int64_t c = c0 + k * kRefineThreads;
          m[k] = c < chunks ? mask128[c] : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int64_t c = c0 + k * kRefineThreads;
          if ((m[k].x | m[k].y | m[k].z | m[k].w) == 0) continue;
          const uint32_t pair[4] = {m[k].x, m[k].y, m[k].z, m[k].w};
#pragma unroll
          for (int h = 0; h < 8; ++h) {
            uint32_t w = (pair[h >> 1] >> (16 * (h & 1))) & 0xFFFFu;
            if (!w) continue;
            const int64_t wi = c * 8 + h;
            const int64_t tile = t0 + (wi >> 6);
            const int l = (int)(wi & 63);
            if (tile * kWaveTile < lo || (tile + 1) * kWaveTile > hi) {  // tile shared with a neighbour
              uint32_t keep = 0;
              for (int q = 0; q < kStreamUnroll * 4; ++q) {
                const int64_t e = tile_element(tile, l, q);
                if (e >= lo && e < hi) keep |= 1u << q;
              }
              w &= keep;
              if (!w) continue;
            }
            list_words(tile, l, w);
          }
        }
      }
    }
    clear_bins();
    __syncthreads();
    const int count = (int)passed;
    uint32_t key[kRefinePer];
#pragma unroll
    for (int q = 0; q < kRefinePer; ++q) {
      const int p = tid + q * kRefineThreads;
      key[q] = kNoKey;
      if (p < count) {
        const uint32_t e = sh.list[p];
        key[q] = (e & kFromRecord) ? sh.keys[p] : (__float_as_uint(a.v[e]) & 0x7FFFFFFFu);
      }
    }
    if (passed > (int64_t)rank) prefix = settle(key, [](int) { return true; });
    // (else the floor is the threshold: settled above, or zero, with fewer elements than wanted anything else)
    // Clear the mask bit of every selected element that does not exceed the new threshold.
    // A 16-bit mask word of a tile shared with a neighbour tensor also holds that tensor's
    // bits, and its re-threshold may run at the same time: atomic AND on the 32-bit word.
    // (Elements in records are dropped tile by tile below.)
#pragma unroll
    for (int q = 0; q < kRefinePer; ++q) {
      const int p = tid + q * kRefineThreads;
      const bool drop = p < count && !sent(key[q], prefix) && !(sh.list[p] & kFromRecord);
      drop_bit(drop, drop ? sh.list[p] : 0u);
    }
  } else if (passed <= cap) {
    // The tensor's payload region is free until the emit pass: list the selected elements
    // there, then their keys, so that everything after one walk over the tiles is coalesced.
    uint32_t* list = reinterpret_cast<uint32_t*>(a.out_idx + region);
    uint32_t* keys = reinterpret_cast<uint32_t*>(a.out_val + region);
    if (tid == 0) sh.listed = 0;
    __syncthreads();
    // records: one thread per tile (keys come with them)
    if (a.slotted) {
      for (int64_t tile = t0 + tid; tile <= t1; tile += kRefineThreads) {
        if (!is_record(tile)) continue;
        const int c = (int)a.tile_count[tile];
        int pos = (int)atomicAdd(&sh.listed, (uint32_t)c);
        for (int q = 0; q < c; ++q) {
          list[pos] = (uint32_t)records[tile * kSlotRecord + q] | kFromRecord;
          keys[pos] = (uint32_t)records[tile * kSlotRecord + kSlotsPerTile + q] & 0x7FFFFFFFu;
          ++pos;
        }
      }
    }
    // mask words: eight (16 bytes) per load, four loads in flight per thread
    const uint4* mask128 = reinterpret_cast<const uint4*>(a.mask + t0 * 64);
    const int64_t chunks = words >> 3;
    for (int64_t c0 = tid; c0 < chunks; c0 += 4 * kRefineThreads) {
      uint4 m[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int64_t c = c0 + k * kRefineThreads;
        m[k] = c < chunks ? mask128[c] : make_uint4(0, 0, 0, 0);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int64_t c = c0 + k * kRefineThreads;
        if ((m[k].x | m[k].y | m[k].z | m[k].w) == 0) continue;
        if (c < chunks && is_record(t0 + (c >> 3))) continue;  // that line is a record, taken above
        const uint32_t pair[4] = {m[k].x, m[k].y, m[k].z, m[k].w};
#pragma unroll
        for (int h = 0; h < 8; ++h) {
          uint32_t w = (pair[h >> 1] >> (16 * (h & 1))) & 0xFFFFu;
          if (!w) continue;
          const int64_t wi = c * 8 + h;
          const int64_t tile = t0 + (wi >> 6);
          const int l = (int)(wi & 63);
          if (tile * kWaveTile < lo || (tile + 1) * kWaveTile > hi) {  // tile shared with a neighbour
            uint32_t keep = 0;
            for (int q = 0; q < kStreamUnroll * 4; ++q) {
              const int64_t e = tile_element(tile, l, q);
              if (e >= lo && e < hi) keep |= 1u << q;
            }
            w &= keep;
            if (!w) continue;
          }
          int pos = (int)atomicAdd(&sh.listed, (uint32_t)__popc(w));
          while (w) {
            const int q = __ffs(w) - 1;
            w &= w - 1;
            list[pos++] = (uint32_t)tile_element(tile, l, q);
          }
        }
      }
    }
    __syncthreads();
    const int count = (int)passed;
    for (int p0 = tid; p0 < count; p0 += 4 * kRefineThreads) {
      uint32_t e[4];
      float x[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int p = p0 + q * kRefineThreads;
        e[q] = p < count ? list[p] : kFromRecord;
        x[q] = (e[q] & kFromRecord) ? 0.0f : a.v[e[q]];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int p = p0 + q * kRefineThreads;
        if (p < count && !(e[q] & kFromRecord)) keys[p] = __float_as_uint(x[q]) & 0x7FFFFFFFu;
      }
    }
    __syncthreads();
#pragma unroll 1
    for (int pass = 0; pass < 3; ++pass) {
      const int bits = pass == 2 ? 9 : 11;
      const int shift = 31 - consumed - bits;
      const uint32_t digit_mask = (1u << bits) - 1u;
      for (int i = tid; i < kSelectBins; i += kRefineThreads) sh.s.hist[i] = 0;
      __syncthreads();
      for (int p = tid; p < count; p += kRefineThreads) {
        const uint32_t key = keys[p];
        if (pass == 0 || (key >> (shift + bits)) == prefix) atomicAdd(&sh.s.hist[(key >> shift) & digit_mask], 1u);
      }
      __syncthreads();
      uint32_t bin, above, members, all;
      find_bin<kRefineThreads>(sh.s.hist, sh.s.wave_tot, sh.s.sel, tid, rank, bin, above, members, all);
      prefix = (prefix << bits) | bin;
      rank -= above;
      consumed += bits;
    }
    // mask bits as above
    for (int p0 = 0; p0 < count; p0 += kRefineThreads) {
      const int p = p0 + tid;
      const bool drop = p < count && !sent(keys[p], prefix) && !(list[p] & kFromRecord);
      drop_bit(drop, drop ? list[p] : 0u);
    }
  } else {
    // More passed than the payload region holds (the caller's capacity is below the
    // over-selection): walk the tiles in every pass and read v' element by element.
#pragma unroll 1
    for (int pass = 0; pass < 3; ++pass) {
      const int bits = pass == 2 ? 9 : 11;
      const int shift = 31 - consumed - bits;
      const uint32_t digit_mask = (1u << bits) - 1u;
      for (int i = tid; i < kSelectBins; i += kRefineThreads) sh.s.hist[i] = 0;
      __syncthreads();
      if (a.slotted) {
        for (int64_t tile = t0 + tid; tile <= t1; tile += kRefineThreads) {
          if (!is_record(tile)) continue;
          const int c = (int)a.tile_count[tile];
          for (int q = 0; q < c; ++q) {
            const uint32_t key = (uint32_t)records[tile * kSlotRecord + kSlotsPerTile + q] & 0x7FFFFFFFu;
            if (pass == 0 || (key >> (shift + bits)) == prefix) atomicAdd(&sh.s.hist[(key >> shift) & digit_mask], 1u);
          }
        }
      }
      for (int64_t wi = tid; wi < words; wi += kRefineThreads) {
        if (is_record(t0 + (wi >> 6))) continue;
        int64_t tile;
        int l;
        uint32_t w = tensor_mask_word(a.mask, t0, wi, lo, hi, tile, l);
        while (w) {
          const int q = __ffs(w) - 1;
          w &= w - 1;
          const uint32_t key = __float_as_uint(a.v[tile_element(tile, l, q)]) & 0x7FFFFFFFu;
          if (pass == 0 || (key >> (shift + bits)) == prefix)
            atomicAdd(&sh.s.hist[(key >> shift) & digit_mask], 1u);
        }
      }
      __syncthreads();
      uint32_t bin, above, members, all;
      find_bin<kRefineThreads>(sh.s.hist, sh.s.wave_tot, sh.s.sel, tid, rank, bin, above, members, all);
      prefix = (prefix << bits) | bin;
      rank -= above;
      consumed += bits;
    }
    for (int64_t wi = tid; wi < words; wi += kRefineThreads) {
      if (is_record(t0 + (wi >> 6))) continue;
      int64_t tile;
      int l;
      uint32_t w = tensor_mask_word(a.mask, t0, wi, lo, hi, tile, l);
      uint32_t drop = 0;
      while (w) {
        const int q = __ffs(w) - 1;
        w &= w - 1;
        const uint32_t key = __float_as_uint(a.v[tile_element(tile, l, q)]) & 0x7FFFFFFFu;
        if (!sent(key, prefix)) drop |= 1u << q;
      }
      if (drop) {
        const int64_t h = tile * 64 + l;  // index of the 16-bit word
        atomicAnd(&mask32[h >> 1], ~(drop << (16 * (int)(h & 1))));
        atomicSub(&a.tile_count[tile], (uint32_t)__popc(drop));
      }
    }
  }
  // Records: a tile's count becomes the elements that exceed the new threshold, with the number that the record holds
  // beside it, and the emit pass tells them apart and puts the others back.  (Put back from here, 2400 elements of one
  // tensor took 16 us: one compute unit stores to half a scattered word per ns.)  One thread per tile: a record belongs
  // to this tensor alone.
  if (a.slotted) {
    __syncthreads();  // every walk over records and counts above is over
    constexpr int kTilesInFlight = 4;
#pragma unroll 1
    for (int64_t first = t0; first <= t1; first += kTilesInFlight * kRefineThreads) {
      uint32_t c[kTilesInFlight];
      int4 x[kTilesInFlight][2];
#pragma unroll
      for (int k = 0; k < kTilesInFlight; ++k) {
        // the counts of the tiles and their lines (a record only if the count says so) are asked for together
        const int64_t tile = first + k * kRefineThreads + tid;
        const bool whole = tile <= t1 && tile * kWaveTile >= lo && (tile + 1) * kWaveTile <= hi;
        const int64_t from = tile <= t1 ? tile : t0;
        const int4* line = reinterpret_cast<const int4*>(records + from * kSlotRecord + kSlotsPerTile);
        const uint32_t count = a.tile_count[from];
        x[k][0] = line[0];
        x[k][1] = line[1];
        c[k] = whole && count <= (uint32_t)kSlotsPerTile ? count : 0u;
      }
#pragma unroll
      for (int k = 0; k < kTilesInFlight; ++k) {
        const int32_t xx[8] = {x[k][0].x, x[k][0].y, x[k][0].z, x[k][0].w, x[k][1].x, x[k][1].y, x[k][1].z, x[k][1].w};
        uint32_t kept = 0;
#pragma unroll
        for (int q = 0; q < kSlotsPerTile; ++q)
          if ((uint32_t)q < c[k] && sent((uint32_t)xx[q] & 0x7FFFFFFFu, prefix)) ++kept;
        if (kept != c[k]) a.tile_count[first + k * kRefineThreads + tid] = kept | (c[k] << kTileCountHeldShift);
      }
    }
  }
  if (tid == 0) {
    const float thr = __uint_as_float(prefix);
    a.thr[j] = thr;
    if (a.out_thr) a.out_thr[j] = thr;
  }
}

// ---------------------------------------------------------------------------
// Emit pass: sparse extract + residual + momentum factor masking
// (paper: Algorithm 3, the three lines after Mask; Section 3.3)
// ---------------------------------------------------------------------------
// One workgroup per entry of a host-built list of (tensor, first tile): it owns up
// to kEmitTiles consecutive tiles of that tensor, counts the mask bits that fall
// inside the tensor, obtains that many slots of the tensor's payload region, then
// for every set bit moves v' into the payload and clears v and u.  An element that
// finds the region full is left untouched (it stays in u, v) and the overflow flag
// is set.
//
// The streaming pass has left the number of mask bits of every tile; a workgroup starts
// after the sum over the tensor's tiles before its own, so the workgroups' parts follow
// each other in index order and the region is the same on every run.  Inside its part, too, a
// workgroup places its elements in index order: the whole region ascends, and a full region keeps
// the lowest indices, whether or not DGC_FLAG_SORTED_OUTPUT asks for it.
// (A first version reserved slots with one atomic per workgroup in order of arrival; the
// receive side can find a range of elements in a region by search only if the parts are
// in order.)

// The places of the norm's shares for the next call (see share_word): nothing behind the selection reads them.
template <int THREADS>
__device__ __forceinline__ void clear_shares(const EmitArgs& a, int tid) {
  for (int c = tid; c < a.shares; c += THREADS) a.norm_shares[c] = 0;
}

// This lane's mask word of tile t with the bits outside tensor [lo, hi) removed.
__device__ __forceinline__ uint32_t tensor_tile_word(const uint16_t* __restrict__ mask, int64_t t, int lane,
                                                     int64_t lo, int64_t hi) {
  constexpr int kBits = kStreamUnroll * 4;
  uint32_t w = mask[t * 64 + lane];
  // (the test must not depend on w: the loads of several tiles are to be in flight together)
  if (t * kWaveTile < lo || (t + 1) * kWaveTile > hi) {  // tile shared with a neighbour tensor
    uint32_t keep = 0;
    for (int q = 0; q < kBits; ++q) {
      const int64_t e = tile_element(t, lane, q);
      if (e >= lo && e < hi) keep |= 1u << q;
    }
    w &= keep;
  }
  return w;
}

// From mask words, in index order: everything but a slotted streaming pass.  A thread owns 128 consecutive elements
// of the part, half a row of a tile: it puts their bits together from the mask words (64 bytes), one scan over the
// workgroup says where in the part they go, and the thread lists them in LDS by a walk over its bits.  Then slots
// are dealt to threads, so that every thread has as many elements to move however they are spread.
// STAGED (densities of the warm-up epochs with the staging workspace): the selected values of a tile that lies
// wholly inside one tensor wait in the tile's slots of the staging array, in index order, and u and v are masked
// already: values are copied from there, four slots to a thread, u and v touched only where the region is full (the
// element is put back: v' and, under factor masking, u') and in tiles shared between tensors, which the streaming
// pass leaves alone.
// Otherwise every element's v' is read where it is, and v and u are cleared there (neighbouring lanes take
// neighbouring slots: they meet in the same sectors).
//
// Staged, 122 M elements: 42 -> 17.5 us at 1.6 %, where positions worked out tile by tile in every lane's four
// rows were bound by instructions; 113 -> 108 at 25 % (pairs stored with the non-temporal hint, which leaves the
// last-level cache to what follows: the streaming pass of the next call 402 -> 392 us, the merge 430 -> 422; 115
// without it), of which the walk and the dealing take 42 and the stores, 245 MB, the rest.  From a plain pass,
// 25.6 M elements, 6.25 %: 65 -> 60.5 us (scattered reads of v and clears of v and u, a sector each), 23 tensors of
// 0.27 M elements, 1 %: 6.9 -> 5.0.  Also measured at 25 %: four slots to a lane 146 us (a wavefront nearly always
// has a four that straddles two tiles and takes the long way), a thread's first element found by bisection over the
// owners and halving of its 128 bits instead of the list 118, and 56 at 1.6 %.
template <bool STAGED>
struct EmitOrderedShared {
  static constexpr int kWindow = STAGED ? 9216 : 4096;  // elements listed at a time
  uint16_t list[kWindow];                               // offsets from the part's first tile
  int start[kEmitThreads];                              // elements of the part before those of every thread
  int wave_tot[kEmitThreads / 64];
  int pre_tot[kEmitThreads / 64];
};

template <bool STAGED>
__global__ __launch_bounds__(kEmitThreads) void emit_ordered_kernel(EmitArgs a) {
  constexpr int kWaves = kEmitThreads / 64;
  constexpr int kPerTile = kEmitThreads / kEmitTiles;  // threads of a tile
  constexpr int kOwn = kWaveTile / kPerTile;           // elements of a thread
  static_assert(kOwn == 128 && kStreamUnroll == 4, "half a row of a tile: 32 mask words, a nibble of each");
  static_assert(kEmitElements <= 65536, "16-bit offsets");
  __shared__ EmitOrderedShared<STAGED> sh;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const EmitBlock blk = a.blocks[blockIdx.x];
  const int j = blk.tensor;
  const int64_t region = a.out_offsets[j];  // asked for early: needed late
  const int64_t cap = a.out_offsets[j + 1] - region;
  const int64_t lo = blk.lo;
  const int64_t hi = blk.hi;
  const int64_t t0 = lo / kWaveTile;
  const int64_t t1 = (hi - 1) / kWaveTile;
  const int64_t first = blk.first_tile;

  // Everything the workgroup needs before it can place its elements is asked for at once: the mask words of its own
  // tiles, and the counts the streaming pass has left for the tiles of this tensor before them (every tile strictly
  // between the tensor's first tile and this workgroup's lies wholly inside the tensor; the tensor's share of its
  // first tile is recounted from the mask words).
  const int tl = tid / kPerTile;
  const int piece = tid % kPerTile;
  const int64_t tile = first + tl;
  uint4 raw[4] = {};
  if (tile <= t1) {
    const uint4* __restrict__ m = reinterpret_cast<const uint4*>(a.mask + tile * 64 + 32 * (piece & 1));
#pragma unroll
    for (int k = 0; k < 4; ++k) raw[k] = m[k];
  }
  int pre = tile_counts_partial<kEmitThreads>(a.tile_count, t0 + 1, first, tid);
  if (first > t0 && wave == 0) pre += __popc(tensor_tile_word(a.mask, t0, lane, lo, hi));
  uint32_t bits[4];
  {
    const int row4 = 4 * (piece >> 1);
    auto byte_of = [&](uint32_t two) {  // the row's nibbles of two neighbouring mask words
      const uint32_t y = (two >> row4) & 0x000F000Fu;
      return y | (y >> 12);             // (bits 16 to 19 are left over)
    };
#pragma unroll
    for (int k = 0; k < 4; ++k)
      bits[k] = (byte_of(raw[k].x) & 0xFFu) | ((byte_of(raw[k].y) & 0xFFu) << 8) | ((byte_of(raw[k].z) & 0xFFu) << 16) |
                (byte_of(raw[k].w) << 24);
  }
  const int64_t e0 = tile * kWaveTile + piece * kOwn;  // the thread's first element
  if (e0 < lo || e0 + kOwn > hi) {                     // another tensor's elements, or behind the end
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t from = lo - (e0 + 32 * k), until = hi - (e0 + 32 * k);
      uint32_t keep = until >= 32 ? 0xFFFFFFFFu : until <= 0 ? 0u : (1u << (int)until) - 1u;
      if (from > 0) keep &= from >= 32 ? 0u : ~((1u << (int)from) - 1u);
      bits[k] &= keep;
    }
  }
  const int cnt = __popc(bits[0]) + __popc(bits[1]) + __popc(bits[2]) + __popc(bits[3]);
  const int incl = (int)wave_inclusive_sum((uint32_t)cnt);
  pre = (int)wave_sum((uint32_t)pre);
  if (lane == 63) sh.wave_tot[wave] = incl;
  if (lane == 0) sh.pre_tot[wave] = pre;
  __syncthreads();
  int before = 0, total = 0, base = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const int t = sh.wave_tot[w];
    if (w < wave) before += t;
    total += t;
    base += sh.pre_tot[w];
  }
  if (tid == 0 && (int)((first - t0) / kEmitTiles) == blk.tensor_blocks - 1) a.out_counts[j] = base + total;
  if (blockIdx.x == 0) clear_shares<kEmitThreads>(a, tid);
  if (total == 0) return;
  int pos = before + incl - cnt;  // slot of the thread's next element
  sh.start[tid] = pos;

  float* __restrict__ u = a.u;
  float* __restrict__ v = a.v;
  int32_t* __restrict__ part_idx = a.out_idx + region + base;
  float* __restrict__ part_val = a.out_val + region + base;
  const int64_t left = cap - base;
  const int room = left >= total ? total : left > 0 ? (int)left : 0;  // elements that find a slot
  const int32_t origin = (int32_t)(first * kWaveTile);
  bool overflow = false;
  // tiles that the streaming pass has not staged: shared with a neighbour tensor, or the ragged end
  const int first_shared = t0 * kWaveTile < lo || (t0 + 1) * kWaveTile > hi ? (int)(t0 - first) : -1;
  const int last_shared = (t1 + 1) * kWaveTile > hi || t1 * kWaveTile < lo ? (int)(t1 - first) : -1;
  auto is_staged = [&](int t) { return STAGED && t != first_shared && t != last_shared; };
  for (int win = 0; win < total; win += EmitOrderedShared<STAGED>::kWindow) {
    const int end = total - win < EmitOrderedShared<STAGED>::kWindow ? total : win + EmitOrderedShared<STAGED>::kWindow;
    if (win > 0) __syncthreads();
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      while (bits[k] != 0u && pos < end) {
        sh.list[pos - win] = (uint16_t)(tid * kOwn + 32 * k + (__ffs((int)bits[k]) - 1));
        bits[k] &= bits[k] - 1u;
        ++pos;
      }
    }
    __syncthreads();
    // neighbouring slots to neighbouring lanes, kBatch of them on their way at a time: loads, then stores
    constexpr int kBatch = 4;
    for (int s0 = win + tid; s0 < end; s0 += kBatch * kEmitThreads) {
      int32_t e[kBatch];
      float x[kBatch];
      bool parked[kBatch];
      int64_t at[kBatch];
#pragma unroll
      for (int k = 0; k < kBatch; ++k) {
        const int s = s0 + k * kEmitThreads;
        e[k] = -1;
        x[k] = 0.0f;
        parked[k] = false;
        at[k] = 0;
        if (s < end) {
          const int off = sh.list[s - win];
          const int t = off / kWaveTile;
          e[k] = origin + off;
          parked[k] = is_staged(t);
          if (STAGED && parked[k]) {
            at[k] = (first + t) * kWaveTile + (s - sh.start[t * kPerTile]);
            x[k] = a.stage_v[at[k]];
          } else if (s < room) {
            x[k] = v[e[k]];
          }
        }
      }
#pragma unroll
      for (int k = 0; k < kBatch; ++k) {
        if (e[k] < 0) continue;
        const int s = s0 + k * kEmitThreads;
        if (s < room) {
          if (STAGED) {
            __builtin_nontemporal_store(e[k], part_idx + s);
            __builtin_nontemporal_store(x[k], part_val + s);
          } else {
            part_idx[s] = e[k];
            part_val[s] = x[k];
          }
          if (!parked[k]) {  // u, v masked here
            v[e[k]] = 0.0f;
            if (a.factor_masking) u[e[k]] = 0.0f;
          }
        } else {  // region full: what was parked goes back to where the streaming pass took it from, the rest stays
          overflow = true;
          if (STAGED && parked[k]) {
            v[e[k]] = x[k];
            if (a.factor_masking && a.stage_u) u[e[k]] = a.stage_u[at[k]];
          }
        }
      }
    }
  }
  if (overflow) atomicOr(&a.state->flags, (uint32_t)DGC_DIAG_OVERFLOW);
}

// Emit pass after a SLOTTED streaming pass.  Four threads per tile of the workgroup's 32 tiles,
// two slots each: a thread asks for its slots' indices and values at once with the tile's count
// and the counts of the tensor's tiles before the workgroup (two wavefronts per workgroup: the
// parts of a 122 M-element set are all resident at once); a tile that lies wholly inside the tensor and selected
// at most kSlotsPerTile elements is a straight copy (its u and v are masked already; an element
// that finds the region full is put back).  The other tiles -- shared with a neighbour tensor, or
// with more selected elements than slots -- are taken by the wavefront that holds them, one after
// the other, from their mask words as in the plain pass: read v', write the pair, clear v and u.
// Order inside the workgroup's part: tile by tile, index order inside a tile (a record is in index
// order, and the tiles taken from mask words are placed by the votes of their rows), so the
// whole region ascends, and a full region keeps the lowest indices: this pass also serves
// DGC_FLAG_SORTED_OUTPUT.
struct EmitSlotsShared {
  uint16_t words[kEmitTiles * 64];  // mask words of the tiles that are not copied from slots
  int cnt[kEmitTiles];              // elements of every tile that belong to this tensor
  int pre_tot[kEmitSlotThreads / 64];
};

__global__ __launch_bounds__(kEmitSlotThreads) void emit_slots_kernel(EmitArgs a) {
  constexpr int kWaves = kEmitSlotThreads / 64;
  constexpr int kLanesPerTile = kEmitSlotThreads / kEmitTiles;
  constexpr int kPerLane = kSlotsPerTile / kLanesPerTile;
  static_assert(kPerLane == 2 && kLanesPerTile * kPerLane == kSlotsPerTile, "a thread takes two neighbouring slots");
  constexpr int kLaneWalk = 6;  // selected elements of one lane the short way takes
  constexpr int kTilesPerWave = 64 / kLanesPerTile;
  static_assert(kEmitTiles <= 32 && kTilesPerWave * kWaves == kEmitTiles, "tile counts are scanned by half a wavefront");
  __shared__ EmitSlotsShared sh;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const EmitBlock blk = a.blocks[blockIdx.x];
  const int j = blk.tensor;
  const int64_t region = a.out_offsets[j];  // asked for early: needed late
  const int64_t cap = a.out_offsets[j + 1] - region;
  const int64_t lo = blk.lo;
  const int64_t hi = blk.hi;
  const int64_t t0 = lo / kWaveTile;
  const int64_t t1 = (hi - 1) / kWaveTile;
  const int64_t first = blk.first_tile;

  const int tl = tid / kLanesPerTile;             // this thread's tile of the part ...
  const int s = (tid % kLanesPerTile) * kPerLane;  // ... and the first of its two slots of that tile
  const int64_t t = first + tl;
  const bool exists = t <= t1;
  const bool inside = exists && t * kWaveTile >= lo && (t + 1) * kWaveTile <= hi;
  const uint32_t c_raw = exists ? a.tile_count[t] : 0u;
  const uint32_t c_own = c_raw & kTileCountMask;
  int2 e_slot = make_int2(0, 0);
  int2 x_slot = make_int2(0, 0);  // bits of the values
  int2 y_slot = make_int2(0, 0);  // ... and of u', for what a settled threshold drops
  const int32_t* __restrict__ records = reinterpret_cast<const int32_t*>(a.mask);  // see the streaming pass
  if (inside) {  // (a record only if the count says so; loaded before the count is known)
    e_slot = *reinterpret_cast<const int2*>(records + t * kSlotRecord + s);
    x_slot = *reinterpret_cast<const int2*>(records + t * kSlotRecord + kSlotsPerTile + s);
    if (a.settled) y_slot = *reinterpret_cast<const int2*>(records + t * kSlotRecord + 2 * kSlotsPerTile + s);
  }
  // Slots taken by the tensor's tiles before the workgroup's first one.  The tensor's first tile
  // counts like the others when it lies wholly inside the tensor (its line may hold a record);
  // shared with the tensor before, it has mask words, from which the tensor's share is recounted.
  const bool first_shared = t0 * kWaveTile < lo;
  int pre = tile_counts_partial<kEmitSlotThreads>(a.tile_count, first_shared ? t0 + 1 : t0, first, tid);
  if (first > t0 && first_shared && wave == 0) pre += __popc(tensor_tile_word(a.mask, t0, lane, lo, hi));
  pre = (int)wave_sum((uint32_t)pre);
  if (lane == 0) sh.pre_tot[wave] = pre;

  const bool from_slots = inside && !(c_raw & kTileCountHasMask);
  // tiles of this wavefront that are taken from their mask words: one bit per tile, at its first lane
  const unsigned long long others = __ballot(exists && !from_slots && s == 0);
  if (from_slots && s == 0) sh.cnt[tl] = (int)c_own;
  if (!exists && s == 0) sh.cnt[tl] = 0;
  for (unsigned long long m = others; m; m &= m - 1) {
    const int k = wave * kTilesPerWave + (__ffsll((long long)m) - 1) / kLanesPerTile;
    const uint32_t w = tensor_tile_word(a.mask, first + k, lane, lo, hi);
    sh.words[k * 64 + lane] = (uint16_t)w;
    const int c = (int)wave_sum((uint32_t)__popc(w));
    if (lane == 0) sh.cnt[k] = c;
  }
  __syncthreads();
  int base = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) base += sh.pre_tot[w];
  // where every tile starts in the part: each wavefront scans the 32 counts for itself
  const int own = lane < kEmitTiles ? sh.cnt[lane] : 0;
  const int incl = (int)wave_inclusive_sum((uint32_t)own);
  const int total = __builtin_amdgcn_readlane(incl, kEmitTiles - 1);
  if (tid == 0 && (int)((first - t0) / kEmitTiles) == blk.tensor_blocks - 1) a.out_counts[j] = base + total;
  if (a.settled && blockIdx.x == 0 && tid == 0) a.state->crowded = 0;  // (nothing behind reads it)
  if (blockIdx.x == 0) clear_shares<kEmitSlotThreads>(a, tid);
  if (total == 0 && !a.settled) return;
  const int excl = incl - own;
  int32_t* __restrict__ out_idx = a.out_idx + region;
  float* __restrict__ out_val = a.out_val + region;
  float* __restrict__ u = a.u;
  float* __restrict__ v = a.v;
  bool overflow = false;
  {
    const int tile_start = __shfl(excl, tl & 31);
    // Where refine_kernel has settled the threshold, a record may hold more than is sent: the rest goes back to where
    // the streaming pass took it from, and what is sent closes ranks (places from the votes of the tile's lanes).
    int place[kPerLane] = {s, s + 1};
    bool goes[kPerLane] = {s < (int)c_own, s + 1 < (int)c_own};
    if (a.settled) {
      const int held = (int)((c_raw >> kTileCountHeldShift) & 0xFu);
      if (__ballot(from_slots && held > 0) != 0) {
        const uint32_t thr = __float_as_uint(a.settled[j]);
        const unsigned long long lower = ((1ull << (lane % kLanesPerTile)) - 1ull) << (lane & ~(kLanesPerTile - 1));
        const bool some = from_slots && held > 0;
        const bool keep0 = some && s < held && sent((uint32_t)x_slot.x & 0x7FFFFFFFu, thr);
        const bool keep1 = some && s + 1 < held && sent((uint32_t)x_slot.y & 0x7FFFFFFFu, thr);
        const unsigned long long votes0 = __ballot(keep0), votes1 = __ballot(keep1);
        if (some) {
          place[0] = __popcll(votes0 & lower) + __popcll(votes1 & lower);
          place[1] = place[0] + (keep0 ? 1 : 0);
          goes[0] = keep0;
          goes[1] = keep1;
          if (s < held && !keep0) {
            v[e_slot.x] = __int_as_float(x_slot.x);
            if (a.factor_masking) u[e_slot.x] = __int_as_float(y_slot.x);
          }
          if (s + 1 < held && !keep1) {
            v[e_slot.y] = __int_as_float(x_slot.y);
            if (a.factor_masking) u[e_slot.y] = __int_as_float(y_slot.y);
          }
        }
      }
      if (total == 0) return;
    }
#pragma unroll
    for (int q = 0; q < kPerLane; ++q) {
      const int32_t e_q = q == 0 ? e_slot.x : e_slot.y;
      const float x_q = __int_as_float(q == 0 ? x_slot.x : x_slot.y);
      if (from_slots && goes[q]) {
        const int64_t slot = (int64_t)base + tile_start + place[q];
        if (slot < cap) {
          out_idx[slot] = e_q;
          out_val[slot] = x_q;
        } else {  // region full: the element goes back to where the streaming pass took it from
          overflow = true;
          v[e_q] = x_q;
          if (a.factor_masking) u[e_q] = __int_as_float(records[t * kSlotRecord + 2 * kSlotsPerTile + s + q]);
        }
      }
    }
  }
  for (unsigned long long m = others; m; m &= m - 1) {
    const int k = wave * kTilesPerWave + (__ffsll((long long)m) - 1) / kLanesPerTile;
    const int64_t tk = first + k;
    const uint32_t w = sh.words[k * 64 + lane];
    const int64_t tile_slot = (int64_t)base + __shfl(excl, k);
    // Index order inside the tile is row (one 16-byte vector per lane), lane, component: an element's
    // position is the rows before it, plus the bits of its row in lower lanes, plus the lower bits of
    // its nibble.
    const int most = (int)wave_max((uint32_t)__popc(w));  // bits of the lane that has most (uniform)
    const int tile_count = __shfl(own, k);
    if (tile_count < 256 && most <= kLaneWalk) {
      // The usual case (a tile shared between tensors, or a dozen elements in one tile): positions
      // from one packed scan (the counts of the lane's four rows in the bytes of a word, as in the
      // staged pass), and every lane walks its own bits: all of the tile's reads of v are on their
      // way before the first store, one round trip to memory per tile instead of one per row.
      uint32_t xw = w - ((w >> 1) & 0x5555u);
      xw = (xw & 0x3333u) + ((xw >> 2) & 0x3333u);  // a count per nibble
      const uint32_t cnt = (xw & 0xFu) | ((xw & 0xF0u) << 4) | ((xw & 0xF00u) << 8) | ((xw & 0xF000u) << 12);
      const uint32_t inc = wave_inclusive_sum(cnt);
      const uint32_t tot = wave_last(inc);
      uint32_t next = (inc - cnt) + ((tot << 8) + (tot << 16) + (tot << 24));  // next position of each of the lane's rows
      const int32_t e_lane = (int32_t)tile_element(tk, lane, 0);
      uint32_t rem = w;
      int32_t e[kLaneWalk];
      int ps[kLaneWalk];
      float x[kLaneWalk];
#pragma unroll
      for (int i = 0; i < kLaneWalk; ++i) {
        e[i] = -1;
        ps[i] = 0;
        x[i] = 0.0f;
        if (i < most) {
          if (rem != 0u) {
            const int b = __ffs((int)rem) - 1;  // bit 4 r + c
            const int r8 = (b >> 2) * 8;
            ps[i] = (int)((next >> r8) & 0xFFu);
            next += 1u << r8;
            rem &= rem - 1u;
            if (tile_slot + ps[i] < cap) e[i] = e_lane + (b >> 2) * 256 + (b & 3);
            else overflow = true;  // region full: the element stays where it is
          }
          if (e[i] >= 0) x[i] = v[e[i]];
        }
      }
#pragma unroll
      for (int i = 0; i < kLaneWalk; ++i) {
        if (i < most && e[i] >= 0) {
          out_idx[tile_slot + ps[i]] = e[i];
          out_val[tile_slot + ps[i]] = x[i];
          v[e[i]] = 0.0f;
          if (a.factor_masking) u[e[i]] = 0.0f;
        }
      }
      continue;
    }
    // Otherwise row by row, positions from votes; a row's (up to four) elements of a lane are read together.
    int row_base = 0;
#pragma unroll
    for (int r = 0; r < kStreamUnroll; ++r) {
      const uint32_t nib = (w >> (4 * r)) & 0xFu;
      if (__ballot(nib != 0) == 0) continue;  // nothing in this row of the tile
      int lower = 0, row = 0;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const unsigned long long vote = __ballot((nib >> c) & 1u);
        lower += (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(vote >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)vote, 0u));
        row += __popcll(vote);
      }
      int pos = row_base + lower;
      int32_t e[4];
      int64_t at[4];
      float x[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        e[c] = -1;
        at[c] = tile_slot + pos;
        if ((nib >> c) & 1u) {
          if (at[c] < cap) e[c] = (int32_t)tile_element(tk, lane, 4 * r + c);
          else overflow = true;  // region full: the element stays where it is
          ++pos;
        }
        x[c] = e[c] >= 0 ? v[e[c]] : 0.0f;
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if (e[c] >= 0) {
          out_idx[at[c]] = e[c];
          out_val[at[c]] = x[c];
          v[e[c]] = 0.0f;
          if (a.factor_masking) u[e[c]] = 0.0f;
        }
      }
      row_base += row;
    }
  }
  if (overflow) atomicOr(&a.state->flags, (uint32_t)DGC_DIAG_OVERFLOW);
}

}  // namespace

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
hipError_t launch_clear_words(uint32_t* p, size_t words, hipStream_t stream) {
  if (words == 0) return hipSuccess;
  size_t blocks = (words + 255) / 256;
  if (blocks > 1024) blocks = 1024;
  hipLaunchKernelGGL(clear_words_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, p, words);
  return hipGetLastError();
}

int32_t norm_blocks(int64_t n) {
  int64_t blocks = ceil_div(n >> 2, (int64_t)kNormThreads * 8);
  if (blocks < 1) blocks = 1;
  if (blocks > kNormMaxBlocks) blocks = kNormMaxBlocks;
  return (int32_t)blocks;
}

hipError_t launch_norm(const float* g, int64_t n, double* partials, hipStream_t stream) {
  hipLaunchKernelGGL(norm_kernel, dim3((unsigned)norm_blocks(n)), dim3(kNormThreads), 0, stream, g, n, partials);
  return hipGetLastError();
}

int32_t norm_shares(int64_t n) {
  const int64_t shares = ceil_div(n >> 2, (int64_t)kSelectThreads * 4);
  return (int32_t)(shares < 1 ? 1 : shares > kNormMaxShares ? kNormMaxShares : shares);
}

template <bool NESTEROV, bool FUSED>
static void launch_select_mode(const SelectArgs& a, dim3 grid, hipStream_t stream) {
  const auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(kSelectThreads), 0, stream, a); };
  if (a.floor.in_pass) launch(select_kernel<NESTEROV, kSelectInPass, FUSED>);
  else if (a.bands) launch(select_kernel<NESTEROV, kSelectLists, FUSED>);
  else launch(select_kernel<NESTEROV, kSelectNoBands, FUSED>);
}

hipError_t launch_select(const SelectArgs& a, int32_t num_tensors, bool with_norm, hipStream_t stream) {
  const dim3 grid((unsigned)(num_tensors + (with_norm ? a.num_partials : 0)));
  if (a.nesterov) {
    if (with_norm) launch_select_mode<true, true>(a, grid, stream);
    else launch_select_mode<true, false>(a, grid, stream);
  } else {
    if (with_norm) launch_select_mode<false, true>(a, grid, stream);
    else launch_select_mode<false, false>(a, grid, stream);
  }
  return hipGetLastError();
}

hipError_t launch_band(const SelectArgs& a, const EmitBlock* blocks, int32_t num_blocks, int32_t num_tensors,
                       hipStream_t stream) {
  const dim3 grid((unsigned)(num_blocks * kBandsPerPart));
  if (a.nesterov) {
    hipLaunchKernelGGL(collect_band_kernel<true>, grid, dim3(kBandThreads), 0, stream, a, blocks);
    hipLaunchKernelGGL(rank_band_kernel<true>, dim3((unsigned)num_tensors), dim3(kSelectThreads), 0, stream, a);
  } else {
    hipLaunchKernelGGL(collect_band_kernel<false>, grid, dim3(kBandThreads), 0, stream, a, blocks);
    hipLaunchKernelGGL(rank_band_kernel<false>, dim3((unsigned)num_tensors), dim3(kSelectThreads), 0, stream, a);
  }
  return hipGetLastError();
}

// Dynamic LDS that nothing uses: it caps the workgroups a compute unit holds at `groups`.
constexpr size_t kStreamStaticLds = sizeof(float) * kStreamWaves * kWaveTile;  // mixed_thr of stream_kernel
static size_t stream_lds_pad(int groups, size_t static_lds) {
  const size_t per = kLdsPerComputeUnit / (size_t)groups - 2048;  // (2 KB of slack for the allocation granule)
  const size_t limit = 64 * 1024;                                  // a workgroup's LDS without a function attribute
  const size_t want = per < limit ? per : limit;
  return want > static_lds ? want - static_lds : 0;
}

template <bool NESTEROV, bool SCALED>
static void launch_stream_mode(const StreamArgs& a, int mode, int groups, dim3 grid, dim3 block, hipStream_t stream) {
  const size_t pad = stream_lds_pad(groups, kStreamStaticLds);
  if (mode == kStreamStaged) hipLaunchKernelGGL((stream_kernel<NESTEROV, SCALED, kStreamStaged>), grid, block, pad, stream, a);
  else if (mode == kStreamSlotted) hipLaunchKernelGGL((stream_kernel<NESTEROV, SCALED, kStreamSlotted>), grid, block, pad, stream, a);
  else if (mode == kStreamBand) hipLaunchKernelGGL((stream_kernel<NESTEROV, SCALED, kStreamBand>), grid, block, pad, stream, a);
  else hipLaunchKernelGGL((stream_kernel<NESTEROV, SCALED, kStreamPlain>), grid, block, pad, stream, a);
}

hipError_t launch_stream(const StreamArgs& a, hipStream_t stream) {
  const int64_t tiles = ceil_div(a.n, kWaveTile);
  const int64_t blocks = ceil_div(tiles, kStreamWaves);
  // scale is known to be exactly 1 when neither the norm kernel nor an override supplies it
  const bool scaled = a.scale_from_state != 0 || a.scale_const != 1.0f;
  const dim3 grid((unsigned)blocks), block(kStreamThreads);
  const int mode = a.stage_v ? kStreamStaged : a.floor.in_pass ? kStreamBand : a.slotted ? kStreamSlotted : kStreamPlain;
  // right after the norm pass part of g comes from the last-level cache, and more wavefronts pay
  const int groups = a.scale_from_state ? kStreamGroupsAfterNorm : kStreamResidentGroups;
  if (a.nesterov) {
    if (scaled) launch_stream_mode<true, true>(a, mode, groups, grid, block, stream);
    else launch_stream_mode<true, false>(a, mode, groups, grid, block, stream);
  } else {
    if (scaled) launch_stream_mode<false, true>(a, mode, groups, grid, block, stream);
    else launch_stream_mode<false, false>(a, mode, groups, grid, block, stream);
  }
  return hipGetLastError();
}

hipError_t launch_ceiling(const float* a, float* b, float* c, int64_t n, int groups, hipStream_t stream) {
  const int64_t tiles = n / kWaveTile;
  if (tiles < 1) return hipSuccess;
  if (groups < 1) groups = kStreamResidentGroups * kStreamWaves;
  hipLaunchKernelGGL(ceiling_kernel, dim3((unsigned)tiles), dim3(64), stream_lds_pad(groups, 0), stream, a, b, c, tiles);
  return hipGetLastError();
}

hipError_t launch_refine(const RefineArgs& a, int32_t num_tensors, hipStream_t stream) {
  hipLaunchKernelGGL(refine_kernel, dim3((unsigned)num_tensors), dim3(kRefineThreads), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_emit(const EmitArgs& a, int32_t num_blocks, hipStream_t stream) {
  if (a.stage_v)
    hipLaunchKernelGGL(emit_ordered_kernel<true>, dim3((unsigned)num_blocks), dim3(kEmitThreads), 0, stream, a);
  else if (a.slotted)
    hipLaunchKernelGGL(emit_slots_kernel, dim3((unsigned)num_blocks), dim3(kEmitSlotThreads), 0, stream, a);
  else
    hipLaunchKernelGGL(emit_ordered_kernel<false>, dim3((unsigned)num_blocks), dim3(kEmitThreads), 0, stream, a);
  return hipGetLastError();
}

}  // namespace dgc
