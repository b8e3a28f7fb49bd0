// HIP kernels of the receive side of the DGC hot path for gfx950 (wave64, CDNA4): the sum
// of N workers' sparse payloads into one dense vector, without float atomics on the paths
// that take payloads as dgc_compress writes them.

#include "dgc_device.h"
#include "dgc_internal.h"
#include "dgc_probe.h"

#include <type_traits>

namespace dgc {
namespace {

// ---------------------------------------------------------------------------
// Receive side (paper: the sum in Algorithm 3's all-reduce line)
// ---------------------------------------------------------------------------
// `scale` multiplies the value first in the two SGD modes (it is -learning rate there:
// theta - lr*x and theta + (-lr)*x round identically) and is ignored otherwise.
__device__ __forceinline__ void scatter_one(float* dense, int64_t n, int32_t i, float x, float scale,
                                            ScatterMode mode, uint32_t* diag_flags) {
  if (i < 0 || (int64_t)i >= n) {
    if (diag_flags) atomicOr(diag_flags, (uint32_t)DGC_DIAG_BAD_INDEX);
    return;
  }
  if (mode == kScatterAtomicSgd || mode == kScatterPlainSgd) x = scale * x;
  if (mode == kScatterAtomicAdd || mode == kScatterAtomicSgd) {
    unsafeAtomicAdd(dense + i, x);  // hardware float add at the L2 / memory side
  } else {
    dense[i] = dense[i] + x;
  }
}

// grid = (chunks, payloads)
__global__ __launch_bounds__(256) void scatter_pairs_kernel(float* dense, int64_t n, PairPayloads p,
                                                            int32_t first, ScatterMode mode,
                                                            float scale, uint32_t* diag_flags) {
  const int w = first + blockIdx.y;
  const int64_t count = p.count[w];
  const int32_t* __restrict__ idx = p.idx[w];
  const float* __restrict__ val = p.val[w];
  const int64_t stride = (int64_t)gridDim.x * 256;
  for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < count; q += stride)
    scatter_one(dense, n, idx[q], val[q], scale, mode, diag_flags);
}

// dense[idx] = 0 for the pairs of region-layout payloads, where a workgroup's number says which tensor it works on:
// grid = (tensors x per_tensor, payloads).  Bound by latency, the region and its count, then the indices, then the
// stores; clear_regions_kernel, which numbers the pairs through all tensors, has a scan and ten dependent LDS reads
// for every pair's tensor in front of its indices (launches included, in a graph: 23 tensors of 0.27 M elements, 1 % of four
// workers 7.2 -> 3.0 us, one of 1 M 7.5 -> 3.5, 150 of 3 M 8.7 -> 5.2).
__global__ __launch_bounds__(kFlatThreads) void clear_tensors_kernel(float* __restrict__ dense, int64_t n, RegionPayloads p,
                                                                     const int64_t* __restrict__ out_offsets,
                                                                     uint32_t per_tensor) {
  constexpr int kInFlight = kFlatPer;
  const uint32_t j = blockIdx.x / per_tensor;
  const int w = blockIdx.y;
  const int64_t region = out_offsets[j];
  const int64_t cap = out_offsets[j + 1] - region;
  int64_t count = p.counts[w][j];
  if (count > cap) count = cap;
  const int32_t* __restrict__ idx = p.idx[w] + region;
  const int64_t stride = (int64_t)per_tensor * kFlatChunk;
  for (int64_t q0 = (int64_t)(blockIdx.x % per_tensor) * kFlatChunk + threadIdx.x; q0 < count; q0 += stride) {
    int32_t i[kInFlight];
#pragma unroll
    for (int k = 0; k < kInFlight; ++k) {
      const int64_t q = q0 + k * kFlatThreads;
      i[k] = q < count ? idx[q] : -1;
    }
#pragma unroll
    for (int k = 0; k < kInFlight; ++k)
      if (i[k] >= 0 && (int64_t)i[k] < n) dense[i[k]] = 0.0f;
  }
}

// The same in sets whose tensors do not get a workgroup each: grid = (workgroups per payload, payloads).  The pairs of a payload are numbered
// through all its regions (tensor by tensor, only the filled part of each region), and a
// workgroup takes chunks of kFlatChunk consecutive numbers, grid-strided until the pairs
// run out, so that every thread that runs has a pair to move however unevenly the
// tensors are filled and however little of the capacity is used.  The numbering needs the prefix
// sum of the per-tensor counts: every workgroup forms it in LDS, kFlatTensors tensors at
// a time, and a thread finds the tensor of its pair by bisection there.  Bound by that walk over the tensors, a round trip
// to memory and a scan for every thousand of them (20000 tensors of 1500 elements, 0.1 % of sixteen workers, us: 556 with a round
// trip per tensor of a thread and a scan by way of LDS, 516 with one for its four and the scan in the vector unit; 9000 of
// 900, two workers: 23.2, 21.5; 40000 of 200: 212 either way).
__global__ __launch_bounds__(kFlatThreads) void clear_regions_kernel(float* __restrict__ dense, int64_t n, RegionPayloads p,
                                                                     const int64_t* __restrict__ out_offsets,
                                                                     int32_t num_tensors) {
  constexpr int kPerThread = kFlatTensors / kFlatThreads;  // tensors a thread stages per round
  __shared__ int64_t s_off[kFlatTensors];
  __shared__ uint32_t s_pre[kFlatTensors];   // pairs in the staged tensors before each one
  __shared__ uint32_t wave_sums[kFlatThreads / 64];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int w = blockIdx.y;
  const int32_t* __restrict__ counts = p.counts[w];
  const int32_t* __restrict__ idx = p.idx[w];
  int64_t carry = 0;                                    // pairs in the tensors before the staged ones
  for (int32_t c0 = 0; c0 < num_tensors; c0 += kFlatTensors) {
    uint32_t cnt[kPerThread];
    int64_t off[kPerThread], cap[kPerThread];
    int32_t held[kPerThread];
    uint32_t mine = 0;
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {  // (all asked for together: behind the last tensor, that one again)
      const int32_t j = c0 + tid * kPerThread + k < num_tensors ? c0 + tid * kPerThread + k : num_tensors - 1;
      off[k] = out_offsets[j];
      cap[k] = out_offsets[j + 1] - off[k];
      held[k] = counts[j];
    }
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
      int64_t c = c0 + tid * kPerThread + k < num_tensors ? held[k] : 0;
      if (c > cap[k]) c = cap[k];
      if (c < 0) c = 0;
      cnt[k] = (uint32_t)c;
      mine += cnt[k];
    }
    const uint32_t incl = wave_inclusive_sum(mine);
    if (lane == 63) wave_sums[wave] = incl;
    __syncthreads();
    uint32_t before = 0, staged = 0;
#pragma unroll
    for (int v = 0; v < kFlatThreads / 64; ++v) {
      const uint32_t t = wave_sums[v];
      if (v < wave) before += t;
      staged += t;
    }
    uint32_t run = before + incl - mine;
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
      s_pre[tid * kPerThread + k] = run;
      s_off[tid * kPerThread + k] = off[k];
      run += cnt[k];
    }
    __syncthreads();
    // chunks of this workgroup that reach into the staged tensors
    for (int64_t x0 = (int64_t)blockIdx.x * kFlatChunk; x0 < carry + (int64_t)staged;
         x0 += (int64_t)gridDim.x * kFlatChunk) {
      if (x0 + kFlatChunk <= carry) continue;
      int64_t slot[kFlatPer];
#pragma unroll
      for (int k = 0; k < kFlatPer; ++k) {
        const int64_t q = x0 + tid + k * kFlatThreads - carry;
        slot[k] = -1;
        if (q >= 0 && q < (int64_t)staged) {
          int lo = 0, hi = kFlatTensors - 1;  // largest i with s_pre[i] <= q
          while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if ((int64_t)s_pre[mid] <= q) lo = mid;
            else hi = mid - 1;
          }
          slot[k] = s_off[lo] + (q - (int64_t)s_pre[lo]);
        }
      }
      int32_t i[kFlatPer];
#pragma unroll
      for (int k = 0; k < kFlatPer; ++k) i[k] = slot[k] >= 0 ? idx[slot[k]] : -1;
#pragma unroll
      for (int k = 0; k < kFlatPer; ++k)
        if (i[k] >= 0 && (int64_t)i[k] < n) dense[i[k]] = 0.0f;
    }
    carry += staged;
    __syncthreads();
  }
}

// Receive side without float atomics: workers are added in the order given, so the
// result is that of the plain definition, bit for bit, in one launch.
//
// A workgroup owns a range of one tensor's elements that consists of whole parts of emit
// workgroups; in every payload's region those parts follow each other in index order
// (inside a part the order is free), so "index below the range's end" is monotone along
// a region and the payload's pairs inside the range are found by search: one wavefront
// per payload, both ends at once (from the same probes in the first round, half the lanes for each end from then on).
// Every thread then takes a few of the pairs into registers and marks their indices in
// an LDS bitmap of the range; a prefix sum over the bitmap numbers the distinct
// indices, which gives every index a slot in an LDS accumulator.  The slots start from
// dense[idx], the payloads are added one after the other with a barrier between them
// (inside one payload the indices are distinct), and the sums are stored.  Every index
// belongs to one workgroup, so plain loads and stores do.  (Float atomics complete at
// about 20 G/s on this part wherever they are executed, plain scattered stores at 80 G/s.)

// Positions of xa and xb (the first values not below them) in two lists at once, for lists in which "value < x" is
// monotone; `safe` is any readable word, read in place of a probe that has nothing left to ask.  The probes of
// both lists are in flight together.  In the first round all lanes probe for both bounds, so that up to 2112 values
// leave brackets of 32 and one more round, half the lanes to a bound, is the last; up to 4224 with two probes each
// (161 tensors, the longest of 2.36 M elements, sixteen payloads: 25.6 -> 24.2 us).  Longer lists take three rounds
// anyway, and the fewer the different sectors that the first one reads, the better: 62 tensors of up to 10 M
// elements, eight payloads, 32 probes 37 us, 64 probes 38, 128 probes 41.  The two lists of one payload choose for
// themselves: with one number for both, the longer list's, that set took 36.0 us and takes 35.3.
__device__ __forceinline__ void wave_equal_ranges(const int32_t* __restrict__ L0, int m0, const int32_t* __restrict__ L1,
                                                  int m1, const int32_t* __restrict__ safe, int32_t xa, int32_t xb,
                                                  int lane, int& lo_0, int& hi_0, int& lo_1, int& hi_1) {
  const int half = lane >> 5;  // 0: xa, 1: xb
  const int sub = lane & 31;
  const int32_t x = half ? xb : xa;
  const int32_t* __restrict__ A = m0 > 0 ? L0 : safe;
  const int32_t* __restrict__ B = m1 > 0 ? L1 : safe;
  int lo0, hi0, lo1, hi1;  // of the lane's half
  {
    const FirstRound r0(m0, first_round_shift(m0)), r1(m1, first_round_shift(m1));
    const bool twice = r0.probes > 64u || r1.probes > 64u;  // uniform
    const bool ask0 = r0.asks(lane), ask1 = r1.asks(lane), more0 = r0.asks(lane + 64), more1 = r1.asks(lane + 64);
    const int32_t v0 = A[r0.at(lane)], v1 = B[r1.at(lane)];
    int32_t w0 = 0, w1 = 0;
    if (twice) {
      w0 = A[r0.at(lane + 64)];
      w1 = B[r1.at(lane + 64)];
    }
    auto below = [&](int32_t bound, bool ask, int32_t v, bool more, int32_t w) {  // probes below the bound: a prefix
      return __popcll(__ballot(ask && v < bound)) + __popcll(__ballot(more && w < bound));
    };
    const int ca0 = below(xa, ask0, v0, more0, w0), cb0 = below(xb, ask0, v0, more0, w0);
    const int ca1 = below(xa, ask1, v1, more1, w1), cb1 = below(xb, ask1, v1, more1, w1);
    const int c0 = half ? cb0 : ca0, c1 = half ? cb1 : ca1;
    lo0 = r0.lo(c0);
    hi0 = r0.hi(c0);
    lo1 = r1.lo(c1);
    hi1 = r1.hi(c1);
  }
  while (__ballot(hi0 > lo0 || hi1 > lo1)) {
    const int span0 = hi0 - lo0, span1 = hi1 - lo1;
    const int step0 = (span0 + 31) >> 5, step1 = (span1 + 31) >> 5;
    const int pos0 = lo0 + sub * step0, pos1 = lo1 + sub * step1;
    const bool ask0 = span0 > 0 && pos0 < hi0, ask1 = span1 > 0 && pos1 < hi1;
    const int32_t v0 = A[ask0 ? pos0 : 0];
    const int32_t v1 = B[ask1 ? pos1 : 0];
    const unsigned long long votes0 = __ballot(ask0 && v0 < x);
    const unsigned long long votes1 = __ballot(ask1 && v1 < x);
    const int c0 = __popc((uint32_t)(votes0 >> (32 * half)));
    const int c1 = __popc((uint32_t)(votes1 >> (32 * half)));
    if (span0 > 0) {
      if (c0 == 0) {
        hi0 = lo0;
      } else {
        const int next = lo0 + c0 * step0;
        lo0 = lo0 + (c0 - 1) * step0 + 1;
        hi0 = next < hi0 ? next : hi0;
      }
    }
    if (span1 > 0) {
      if (c1 == 0) {
        hi1 = lo1;
      } else {
        const int next = lo1 + c1 * step1;
        lo1 = lo1 + (c1 - 1) * step1 + 1;
        hi1 = next < hi1 ? next : hi1;
      }
    }
  }
  lo_0 = __builtin_amdgcn_readlane(lo0, 0);
  hi_0 = __builtin_amdgcn_readlane(lo0, 32);
  lo_1 = __builtin_amdgcn_readlane(lo1, 0);
  hi_1 = __builtin_amdgcn_readlane(lo1, 32);
}

// begin[1 .. num] holds lengths; afterwards begin[w] is the sum of the lengths before w.  One wavefront.
static_assert(kMaxPayloads <= 64, "a payload per lane");
__device__ __forceinline__ void begins_from_lengths(int32_t* begin, int num, int lane) {
  const uint32_t sum = wave_inclusive_sum(lane < num ? (uint32_t)begin[lane + 1] : 0u);
  if (lane < num) begin[lane + 1] = (int32_t)sum;
  if (lane == 0) begin[0] = 0;
}

// Finds every payload's pairs inside [blk.begin, blk.end) and fills begin[], idx_at[] and
// val_at[] (in LDS: a payload's pointers looked up per pair in the kernel's argument block
// would put a load from memory in front of every pair load).  BOTH: of two sets of payloads at
// once (the new ones and the previous ones of a replacing merge); `total2` gets the second set's number
// of pairs, the first set's is returned.  Wavefront w looks after payload w; its number is uniform, and nothing
// is asked for conditionally, so that all its pointers come from one round of scalar loads and both counts from the
// next (a lane-wise payload number made six rounds of dependent loads of them).
template <bool BOTH, typename Shared, typename Shared2>
__device__ __forceinline__ int locate_pairs(Shared& sh, const RegionPayloads& p, int32_t num_payloads, Shared2& sh2,
                                            const RegionPayloads& p2, int32_t num_payloads2, const int64_t* __restrict__ out_offsets,
                                            const MergeBlock& blk, const int32_t* __restrict__ safe, int tid, int waves,
                                            int& total2) {
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int most = BOTH && num_payloads2 > num_payloads ? num_payloads2 : num_payloads;
  for (int w = wave; w < most; w += waves) {
    const bool have = w < num_payloads, have2 = BOTH && w < num_payloads2;
    const int at = have ? w : 0, at2 = have2 ? w : 0;
    const int32_t* __restrict__ idx = p.idx[at];
    const float* __restrict__ val = p.val[at];
    const int32_t* __restrict__ counts = p.counts[at];
    const int32_t* __restrict__ idx2 = BOTH ? p2.idx[at2] : idx;
    const int32_t* __restrict__ counts2 = BOTH ? p2.counts[at2] : counts;
    if (!have2) counts2 = counts;  // (there may be no second set at all)
    const int64_t region = out_offsets[blk.tensor];
    const int64_t cap = out_offsets[blk.tensor + 1] - region;
    const int32_t both = (lane & 1 ? counts2 : counts)[blk.tensor];  // one load for the two
    const int32_t count = __builtin_amdgcn_readlane(both, 0), count2 = __builtin_amdgcn_readlane(both, 1);
    const int64_t cnt = !have || count < 0 ? 0 : count > cap ? cap : count;
    const int64_t cnt2 = !have2 || count2 < 0 ? 0 : count2 > cap ? cap : count2;
    idx += region;
    idx2 += region;
    int lo = 0, hi = (int)cnt, lo2 = 0, hi2 = (int)cnt2;
    if (blk.begin != blk.lo || blk.end != blk.hi)  // (a range that is a whole tensor has all its pairs)
      wave_equal_ranges(idx, (int)cnt, idx2, (int)cnt2, safe, blk.begin, blk.end, lane, lo, hi, lo2, hi2);
    if (lane == 0) {
      if (have) {
        sh.idx_at[w] = in_global(idx + lo);
        sh.val_at[w] = in_global(val + region + lo);
        sh.begin[w + 1] = hi - lo;  // length for now
      }
      if (have2) {
        sh2.idx_at[w] = in_global(idx2 + lo2);
        sh2.begin[w + 1] = hi2 - lo2;
      }
    }
  }
  __syncthreads();
  if (tid < 64) begins_from_lengths(sh.begin, num_payloads, tid);
  if (BOTH && tid >= 64 && tid < 128) begins_from_lengths(sh2.begin, num_payloads2, tid - 64);
  __syncthreads();
  total2 = BOTH ? __builtin_amdgcn_readfirstlane(sh2.begin[num_payloads2]) : 0;  // (uniform, for the compiler as well)
  return __builtin_amdgcn_readfirstlane(sh.begin[num_payloads]);
}

// Largest w with begin[w] <= q.
__device__ __forceinline__ int payload_of(const int32_t* begin, int num_payloads, int q) {
  int w = 0, e = num_payloads;
  while (e - w > 1) {
    const int mid = (w + e) >> 1;
    if (begin[mid] <= q) w = mid;
    else e = mid;
  }
  return w;
}

// The same for the 64 neighbouring numbers q0, q0 + 1, ... of a wavefront's lanes, q0 below the number of all pairs: lane
// w of `own` holds begin[w] (behind the payloads: the largest number there is).  One vote says whose q0 is, and the payloads
// that start among the lanes, mostly one or none, are gone through, instead of a chain of reads from LDS in every lane.
// `last`: that of the last lane.
__device__ __forceinline__ int payloads_of(int32_t own, int num_payloads, int q0, int lane, int& first, int& last) {
  first = __popcll(__ballot(own <= q0)) - 1;
  int w = first;
  for (last = first; last + 1 < num_payloads; ++last) {
    const int32_t next = __builtin_amdgcn_readlane(own, last + 1);
    if (next > q0 + 63) break;
    w += q0 + lane >= next ? 1 : 0;
  }
  return w;
}
__device__ __forceinline__ uint64_t payload_bits(int first, int last) { return (~0ull >> (63 - last)) & (~0ull << first); }

template <int CAP>
struct MergeShared {
  alignas(16) uint32_t bitmap[kMergeMaxRange / 32];
  uint32_t prefix[kMergeMaxRange / 128];  // distinct indices before each group of four bitmap words
  float acc[CAP];
  uint32_t wave_sums[kMergeMaxThreads / 64];
  int32_t begin[kMaxPayloads + 1];  // number of pairs of the payloads before w inside the range
  global_ptr<int32_t> idx_at[kMaxPayloads];  // payload w's first pair inside the range
  global_ptr<float> val_at[kMaxPayloads];
};

// `scale` multiplies every value first (1 for the plain sum; -learning rate for the SGD
// apply, where `dense` is the parameter vector).
//
// REPLACE: `dense` becomes the sum of the payloads instead of growing by it.  It holds
// the sum of an earlier set of payloads (`old`: their index lists are all that is needed),
// i.e. zero wherever none of those has an index.  The accumulator then starts from zero,
// which saves the scattered reads of `dense`, and an index of the earlier set that is in
// none of the new payloads gets a zero: one launch instead of a clear and an accumulate.
struct OldLists {
  int32_t begin[kMaxPayloads + 1];
  global_ptr<int32_t> idx_at[kMaxPayloads];
};

// Number of the distinct index r (relative to the range) among those of the range: the indices
// marked before its group of 128 bits, plus the marked bits below it inside the group.
template <int CAP>
__device__ __forceinline__ int merge_slot(const MergeShared<CAP>& sh, int32_t r) {
  const uint4 g = reinterpret_cast<const uint4*>(sh.bitmap)[r >> 7];
  const int word = (r >> 5) & 3;
  const uint32_t own = word == 0 ? g.x : word == 1 ? g.y : word == 2 ? g.z : g.w;
  uint32_t c = (uint32_t)__popc(own & ((1u << (r & 31)) - 1u));
  c += word > 0 ? (uint32_t)__popc(g.x) : 0u;
  c += word > 1 ? (uint32_t)__popc(g.y) : 0u;
  c += word > 2 ? (uint32_t)__popc(g.z) : 0u;
  return (int)(sh.prefix[r >> 7] + c);
}

// THREADS: 512 when there are at most eight payloads (one wavefront searches one payload's region,
// and four workgroups of eight wavefronts fit a compute unit, LDS included: the 970 ranges of a
// 122 M-element set then run all at once instead of in two rounds), 1024 otherwise.  Bound by latency, the
// searches before all: replacing calls at 0.1 % 35.3 us on that set (37.5 with the pointers of a wavefront's payload fetched one after the
// other) and 24.2 on 25.6 M elements with sixteen payloads (25.5; 66 M with four 20.3 against 22.2, 1 M with four 8.9
// against 10.7).  (A first round of probes around the place that a range has if pairs are spread evenly took 34.9
// and 23.7, but 49.1 instead of 39.1 where the pairs crowd three tenths of one large tensor: every workgroup
// goes on from a bracket of its own, where the first rounds over the whole region read the same few sectors.
// Both sets of probes in one round: no gain where pairs are spread evenly.)  Behind the searches, the steps of the
// 346 ranges of the 25.6 M elements with sixteen payloads from their start, 19.9 -> 18.0 us, call 123.2 -> 121.3: pairs loaded through
// pointers that are known to be global (FLAT loads before), whose payload a vote tells (four dependent reads of LDS
// before), a wavefront that goes through its slots for payloads that it has pairs of only, and the wavefronts' sums read together.
// kMergeCap:
// pairs a workgroup takes into registers, slots of its LDS accumulator (a range with more takes
// the slow way at the end of the kernel).
template <bool REPLACE, int THREADS>
__global__ __launch_bounds__(THREADS) void merge_regions_kernel(float* __restrict__ dense, RegionPayloads p,
                                                                      int32_t num_payloads, RegionPayloads old,
                                                                      int32_t num_old,
                                                                      const int64_t* __restrict__ out_offsets,
                                                                      const MergeBlock* __restrict__ blocks,
                                                                      float scale, int32_t scaled) {
  constexpr int kMergeThreads = THREADS;
  constexpr int kMergeWaves = THREADS / 64;
  constexpr int kMergeCap = THREADS == 512 ? kMergeCapSmall : kMergeCapLarge;
  constexpr int kPerThread = kMergeCap / kMergeThreads;
  constexpr int kWordsPerThread = kMergeMaxRange / 32 / kMergeThreads;
  static_assert(kMergeCap % THREADS == 0 && kWordsPerThread % 4 == 0 && THREADS <= kMergeMaxThreads, "dealt evenly to threads");
  __shared__ MergeShared<kMergeCap> sh;
  __shared__ OldLists was;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const MergeBlock blk = blocks[blockIdx.x];
  const int32_t length = (int32_t)(blk.end - blk.begin);  // <= kMergeMaxRange
#pragma unroll
  for (int k = 0; k < kWordsPerThread; ++k) sh.bitmap[tid * kWordsPerThread + k] = 0;
  int old_total = 0;
  const int total = locate_pairs<REPLACE>(sh, p, num_payloads, was, old, num_old, out_offsets, blk,
                                          reinterpret_cast<const int32_t*>(blocks), tid, kMergeWaves, old_total);
  if (total == 0 && old_total == 0) return;
  // Whether the accumulator may start from zero: the earlier set's indices of this range fit
  // the registers too.  Otherwise they are cleared in `dense` first and the sum is added
  // to what `dense` holds then, as without REPLACE.
  const bool from_zero = REPLACE && total <= kMergeCap && old_total <= kMergeCap;
  if (REPLACE && !from_zero) {
    for (int q = tid; q < old_total; q += kMergeThreads) {
      const int w = payload_of(was.begin, num_old, q);
      const int64_t r = (int64_t)was.idx_at[w][q - was.begin[w]] - blk.begin;
      if (r >= 0 && r < length) dense[blk.begin + r] = 0.0f;
    }
    __syncthreads();  // the zeros are in place before any thread of the workgroup reads `dense`
  }
  if (total == 0 && !from_zero) return;

  if (total <= kMergeCap) {
    // the earlier set's indices of this range, asked for first and not looked at before the
    // new pairs are in: their loads are in flight together with those of the pairs
    int32_t was_idx[kPerThread];
    {
      const int32_t own = lane < num_old ? was.begin[lane] : INT32_MAX;
#pragma unroll
      for (int k = 0; k < kPerThread; ++k) {
        const int q0 = wave * 64 + k * kMergeThreads, q = q0 + lane;
        was_idx[k] = 0;
        if (from_zero && q0 < old_total) {  // uniform
          int first, last;
          const int w = payloads_of(own, num_old, q0, lane, first, last);
          if (q < old_total) was_idx[k] = was.idx_at[w][q - was.begin[w]];
        }
      }
    }
    // this thread's pairs: payload, index relative to the range (-1: none), value
    int pw[kPerThread];
    int32_t rel[kPerThread];
    float x[kPerThread];
    float held[kPerThread];  // what the element's slot starts from: asked for before the indices are numbered
    uint64_t mine = 0;  // payloads of the wavefront's pairs, a bit each (uniform)
    const int32_t own = lane < num_payloads ? sh.begin[lane] : INT32_MAX;
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
      const int q0 = wave * 64 + k * kMergeThreads, q = q0 + lane;
      rel[k] = -1;
      pw[k] = -1;
      x[k] = 0.0f;
      held[k] = 0.0f;
      if (q0 >= total) continue;  // uniform
      int first, last;
      const int w = payloads_of(own, num_payloads, q0, lane, first, last);
      mine |= payload_bits(first, last);
      if (q < total) {
        const int src = q - sh.begin[w];
        const int64_t r = (int64_t)sh.idx_at[w][src] - blk.begin;
        const float value = sh.val_at[w][src];
        x[k] = scaled ? scale * value : value;
        if (r >= 0 && r < length) {  // anything else can only come from a region that does not ascend
          pw[k] = w;
          rel[k] = (int32_t)r;
          if (!from_zero) held[k] = dense[blk.begin + r];
          atomicOr(&sh.bitmap[r >> 5], 1u << (r & 31));
        }
      }
    }
    __syncthreads();
    if (from_zero) {  // an index of the earlier set that no new payload has becomes zero
#pragma unroll
      for (int k = 0; k < kPerThread; ++k) {
        const int64_t r = (int64_t)was_idx[k] - blk.begin;
        if (tid + k * kMergeThreads < old_total && r >= 0 && r < length && !((sh.bitmap[r >> 5] >> (r & 31)) & 1u))
          dense[blk.begin + r] = 0.0f;
      }
      if (total == 0) return;
    }
    {
      uint32_t mine = 0, c[kWordsPerThread];
#pragma unroll
      for (int k = 0; k < kWordsPerThread; ++k) {
        c[k] = (uint32_t)__popc(sh.bitmap[tid * kWordsPerThread + k]);
        mine += c[k];
      }
      const uint32_t incl = wave_inclusive_sum(mine);
      if (lane == 63) sh.wave_sums[wave] = incl;
      __syncthreads();
      uint32_t run = incl - mine;
#pragma unroll
      for (int v = 0; v < kMergeWaves; ++v) {  // (all asked for together)
        const uint32_t t = sh.wave_sums[v];
        run += v < wave ? t : 0u;
      }
#pragma unroll
      for (int k = 0; k < kWordsPerThread; ++k) {
        if ((k & 3) == 0) sh.prefix[(tid * kWordsPerThread + k) >> 2] = run;
        run += c[k];
      }
    }
    __syncthreads();
    int id[kPerThread];
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
      id[k] = -1;
      if (rel[k] >= 0) {
        id[k] = merge_slot(sh, rel[k]);
        // pairs of several payloads with one index write the same
        sh.acc[id[k]] = held[k];
      }
    }
    __syncthreads();
    for (int w = 0; w < num_payloads; ++w) {  // payloads in the order given
      if ((mine >> w) & 1u) {
#pragma unroll
        for (int k = 0; k < kPerThread; ++k)
          if (pw[k] == w) sh.acc[id[k]] = sh.acc[id[k]] + x[k];
      }
      __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < kPerThread; ++k)
      if (id[k] >= 0) dense[blk.begin + rel[k]] = sh.acc[id[k]];
  } else {
    // More pairs than a thread's registers and the accumulator hold (many workers, or a
    // density above what this kernel is chosen for): the same steps with the pairs read
    // from the payloads' arrays each time, the distinct indices taken kMergeCap at a time.
    auto pair_of = [&](int q, int& w, int& src) {
      int lo_w = 0, e = num_payloads;  // largest w with begin[w] <= q
      while (e - lo_w > 1) {
        const int mid = (lo_w + e) >> 1;
        if (sh.begin[mid] <= q) lo_w = mid;
        else e = mid;
      }
      w = lo_w;
      src = q - sh.begin[w];
    };
    auto slot_of = [&](int64_t r) { return merge_slot(sh, (int32_t)r); };
    for (int q = tid; q < total; q += kMergeThreads) {
      int w;
      int src;
      pair_of(q, w, src);
      const int64_t r = (int64_t)sh.idx_at[w][src] - blk.begin;
      if (r >= 0 && r < length) atomicOr(&sh.bitmap[r >> 5], 1u << (r & 31));
    }
    __syncthreads();
    int distinct;
    {
      uint32_t mine = 0, c[kWordsPerThread];
#pragma unroll
      for (int k = 0; k < kWordsPerThread; ++k) {
        c[k] = (uint32_t)__popc(sh.bitmap[tid * kWordsPerThread + k]);
        mine += c[k];
      }
      const uint32_t incl = wave_inclusive_sum(mine);
      if (lane == 63) sh.wave_sums[wave] = incl;
      __syncthreads();
      uint32_t run = incl - mine, all = 0;
      for (int v = 0; v < kMergeWaves; ++v) {
        if (v < wave) run += sh.wave_sums[v];
        all += sh.wave_sums[v];
      }
      distinct = (int)all;
#pragma unroll
      for (int k = 0; k < kWordsPerThread; ++k) {
        if ((k & 3) == 0) sh.prefix[(tid * kWordsPerThread + k) >> 2] = run;
        run += c[k];
      }
    }
    __syncthreads();
    for (int first_slot = 0; first_slot < distinct; first_slot += kMergeCap) {
      for (int q = tid; q < total; q += kMergeThreads) {
        int w;
        int src;
        pair_of(q, w, src);
        const int64_t r = (int64_t)sh.idx_at[w][src] - blk.begin;
        if (r < 0 || r >= length) continue;
        const int id = slot_of(r) - first_slot;
        if (id >= 0 && id < kMergeCap) sh.acc[id] = dense[blk.begin + r];
      }
      __syncthreads();
      for (int w = 0; w < num_payloads; ++w) {  // payloads in the order given
        const int len = sh.begin[w + 1] - sh.begin[w];
        for (int q = tid; q < len; q += kMergeThreads) {
          const int64_t r = (int64_t)sh.idx_at[w][q] - blk.begin;
          if (r < 0 || r >= length) continue;
          const int id = slot_of(r) - first_slot;
          if (id >= 0 && id < kMergeCap) {
            const float value = sh.val_at[w][q];
            const float x = scaled ? scale * value : value;
            sh.acc[id] = sh.acc[id] + x;
          }
        }
        __syncthreads();
      }
      for (int q = tid; q < total; q += kMergeThreads) {
        int w;
        int src;
        pair_of(q, w, src);
        const int64_t r = (int64_t)sh.idx_at[w][src] - blk.begin;
        if (r < 0 || r >= length) continue;
        const int id = slot_of(r) - first_slot;
        if (id >= 0 && id < kMergeCap) dense[blk.begin + r] = sh.acc[id];
      }
      __syncthreads();
    }
  }
}

// Pairs of a part in the chunks that merge_parts_kernel takes (see there): a table of where they are, lane w looking after
// payload w, and rounds of a chunk for every wavefront.
typedef float fvec4u __attribute__((ext_vector_type(4), aligned(4)));  // a range starts anywhere
typedef int32_t ivec4 __attribute__((ext_vector_type(4)));
typedef int32_t ivec4u __attribute__((ext_vector_type(4), aligned(4)));

struct ChunkTable {
  const int32_t* idx;  // the lane's payload: start of the line that holds its first pair of the part
  const float* val;    // ... the value beside it
  int32_t pos;         // ... its place in the payload's arrays (may lie up to 31 before them)
  int head, end;       // its pairs are in slots [head, end) from there
  uint32_t chunk0;     // its first chunk among the part's
  uint32_t total;      // chunks of the part

  // `at` and `pairs`: the part's first pair of the lane's payload, and how many there are
  __device__ __forceinline__ ChunkTable(const int32_t* idx_of, const float* val_of, int32_t at, int32_t pairs, int num_payloads, int lane) {
    idx = idx_of + at;
    head = (int)((reinterpret_cast<uintptr_t>(idx) >> 2) & 31u);
    idx -= head;
    pos = at - head;
    val = val_of + at - head;
    const uint32_t until = (uint32_t)head + (uint32_t)pairs;  // (beyond 2^31 - 1: a foreign region)
    end = (int)(until < 0x7FFFFFFFu ? until : 0x7FFFFFFFu);
    const uint32_t own = pairs > 0 ? ((uint32_t)end + (uint32_t)kPartChunk - 1u) / (uint32_t)kPartChunk : 0u;
    const uint32_t upto = wave_inclusive_sum(own);
    total = wave_last(upto);
    chunk0 = lane < num_payloads ? upto - own : 0xFFFFFFFFu;
  }
  __device__ __forceinline__ int payload_at(uint32_t chunk) const { return __popcll(__ballot(chunk0 <= chunk)) - 1; }
};

struct ChunkRound {
  ivec4 idx;
  fvec4u x;
  int w;              // payload of the wavefront's chunk; -1: none
  int first, last;    // payloads of the whole round
  int part;           // -1: there is no round
  bool edge;          // the chunk holds slots that are no pairs of the part:
  uint32_t wanted;    // ... a bit for each of the lane's four that is one,
  int back;           // ... and how many places behind its own each was loaded

  // Asks for the next chunk of every one of `waves` wavefronts, of which there is one at least.
  __device__ __forceinline__ void fetch(const ChunkTable& t, uint32_t& cursor, uint32_t waves, int wave, int lane) {
    auto of_lane = [&](uint64_t x, int w) {
      return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, w) |
             (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), w) << 32;
    };
    const uint32_t until = t.total - cursor < waves ? t.total : cursor + waves;
    first = t.payload_at(cursor);
    last = t.payload_at(until - 1u);
    const uint32_t c = cursor + (uint32_t)wave;
    cursor = until;
    w = -1;
    edge = false;
    if (c >= until) return;  // uniform
    w = t.payload_at(c);
    const int slot0 = (int)(c - (uint32_t)__builtin_amdgcn_readlane((int)t.chunk0, w)) * kPartChunk;
    const int slot = slot0 + 4 * lane;
    const int head = __builtin_amdgcn_readlane(t.head, w), end = __builtin_amdgcn_readlane(t.end, w);
    // (known to be global: the sums' reads of LDS would wait for them, too, otherwise)
    const global_ptr<int32_t> from = (global_ptr<int32_t>)of_lane(reinterpret_cast<uint64_t>(t.idx), w);
    const global_ptr<float> values = (global_ptr<float>)of_lane(reinterpret_cast<uint64_t>(t.val), w);
    if (slot0 >= head && end - slot0 >= kPartChunk) {
      idx = __builtin_nontemporal_load((global_ptr<ivec4>)(from + slot));
      x = __builtin_nontemporal_load((global_ptr<fvec4u>)(values + slot));
    } else {
      // Slots before the first pair and behind the last hold other parts' pairs, or nothing that matters, or do not
      // exist.  (What is loaded is sorted out when the round is added: nothing here waits for it.)
      const EdgeFour four(slot, head, end, __builtin_amdgcn_readlane(t.pos, w) + slot);
      edge = true;
      wanted = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) wanted |= EdgeFour::wanted(slot + k, head, end) ? 1u << k : 0u;
      back = four.whole ? four.back : 0;
      if (four.whole) {
        idx = __builtin_nontemporal_load((global_ptr<ivec4u>)(from + slot - four.back));
        x = __builtin_nontemporal_load((global_ptr<fvec4u>)(values + slot - four.back));
      } else if (four.any) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if ((wanted >> k) & 1u) {
            idx[k] = from[slot + k];
            x[k] = values[slot + k];
          }
        }
      }
    }
  }
};

// Adds a round to a part's accumulator, behind whose elements there is a word per lane for what is no pair of it, and refills
// it by `fetch`.  `last_w`: payload that was added last (-1: none, the accumulator is being filled).  NAMED: `seen` gets
// a bit for every element that is added to, bit r / kSeenWords of word r % kSeenWords: neighbours are in words, and so
// in banks, of their own (1 M elements, 0.4 % of four workers in an eighth:
// 8.4 us without the bits, 10.5; 11.8 with 32 neighbours to a word).
constexpr int kSeenWords = kEmitElements / 32;
template <bool NAMED, typename Fetch>
__device__ __forceinline__ void add_round(ChunkRound& L, float* acc, uint32_t begin, uint32_t length, int32_t scaled, float scale,
                                          int& last_w, int lane, Fetch& fetch, uint32_t* seen) {
  uint32_t at[4];
  float x[4];
  if (L.edge) {  // uniform
    if (L.back & 1) {
      L.idx = ivec4{L.idx[1], L.idx[2], L.idx[3], L.idx[3]};
      L.x = fvec4u{L.x[1], L.x[2], L.x[3], L.x[3]};
    }
    if (L.back & 2) {
      L.idx = ivec4{L.idx[2], L.idx[3], L.idx[3], L.idx[3]};
      L.x = fvec4u{L.x[2], L.x[3], L.x[3], L.x[3]};
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (!((L.wanted >> k) & 1u)) L.idx[k] = INT32_MIN;  // outside every range
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t r = (uint32_t)L.idx[k] - begin;
    at[k] = r < length ? r : (uint32_t)(kEmitElements + lane);  // not a pair of the part, or of a foreign region
    x[k] = scaled ? scale * L.x[k] : L.x[k];
  }
  const int first = L.first, last = L.last, own = L.w;
  fetch(L);
  for (int w = first; w <= last; ++w) {  // payloads in the order given
    if (w != last_w) __syncthreads();    // the payload before is added (the first time: the accumulator is filled)
    last_w = w;
    if (own == w) {
      // the indices of one payload are distinct: all reads, then all writes, no barrier between its rounds
      float sum[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) sum[k] = acc[at[k]] + x[k];
#pragma unroll
      for (int k = 0; k < 4; ++k) acc[at[k]] = sum[k];
      if constexpr (NAMED) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (at[k] < length) atomicOr(&seen[at[k] % kSeenWords], 1u << (at[k] / kSeenWords));
      }
    }
  }
}

// Four consecutive elements of a range of `len`, from element e (a multiple of four) on.
__device__ __forceinline__ fvec4u load_quad(const float* src, int32_t len, int e) {
  fvec4u y = {0.0f, 0.0f, 0.0f, 0.0f};
  if (e + 4 <= len) {
    y = __builtin_nontemporal_load(reinterpret_cast<const fvec4u*>(src + e));
  } else {
#pragma unroll
    for (int c = 0; c < 3; ++c)
      if (e + c < len) y[c] = src[e + c];
  }
  return y;
}
__device__ __forceinline__ void store_quad(float* to, int32_t len, int e, const fvec4u& y) {
  if (e + 4 <= len) {
    __builtin_nontemporal_store(y, reinterpret_cast<fvec4u*>(to + e));
  } else {
#pragma unroll
    for (int c = 0; c < 3; ++c)
      if (e + c < len) to[e + c] = y[c];
  }
}

// The same sums where every emit workgroup's part of the set has a compute unit to itself: the part's range of `dense`
// then has a word of LDS for every element, and the pairs need no numbering (no bitmap, no prefix sum over it, no
// look-up of slots).  Only words of elements that occur are ever touched.  Parts are a quarter as long as the ranges
// above, so that a set of a few million elements keeps four times as many compute units busy.  A part that pairs crowd is
// taken as merge_parts_kernel takes it: all pairs of eight workers of 1 % in a fiftieth of 7 M elements 37.8 us (part kernels
// 45.9; each pair by itself, three times over, 297), of four of 0.8 % in an eighth of 1 M 9.4 (13.0; 22.2).
// Bound by latency, as the range kernel: launch included, in a graph, 0.1 % of four workers, replacing: 1 M elements 8.1
// -> 5.7 us, 7 M in two tensors 9.0 -> 6.9; of sixteen 14.8 -> 7.9 and 18.1 -> 12.8; accumulating 1 % of four workers,
// 23 tensors of 12 K 5.8 -> 4.5, 1 M 11.4 -> 6.7 (part kernels).
// REPLACE: the indices of the earlier payloads are elements that start from zero and get no pair: what the new ones
// share with them gets its sum, the others zero.
// NAMED: elements that no pair names are not stored, also where pairs crowd a part (they may be another stream's to update), which takes a
// crowded part longer: 0.4 % of eight workers in a fiftieth of 7 M elements 27.7 us, 20.2 written whole, 122 each pair by itself.
struct DirectShared {
  alignas(16) float acc[kEmitElements + 64];  // behind the part a word per lane for what is no pair of it
  int32_t begin[kMaxPayloads + 1];
  global_ptr<int32_t> idx_at[kMaxPayloads];
  global_ptr<float> val_at[kMaxPayloads];
};

template <bool REPLACE, bool NAMED, int THREADS>
__global__ __launch_bounds__(THREADS) void merge_direct_kernel(float* __restrict__ dense, RegionPayloads p,
                                                               int32_t num_payloads, RegionPayloads old,
                                                               int32_t num_old,
                                                               const int64_t* __restrict__ out_offsets,
                                                               const MergeBlock* __restrict__ blocks,
                                                               int32_t most, float scale, int32_t scaled) {
  __shared__ DirectShared sh;
  __shared__ alignas(16) uint32_t seen[NAMED ? kSeenWords : 4];
  __shared__ OldLists was;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const MergeBlock blk = blocks[blockIdx.x];
  const uint32_t length = (uint32_t)(blk.end - blk.begin);  // <= kEmitElements
  float* __restrict__ range = dense + blk.begin;
  int old_total = 0;
  const int total = locate_pairs<REPLACE>(sh, p, num_payloads, was, old, num_old, out_offsets, blk,
                                          reinterpret_cast<const int32_t*>(blocks), tid, THREADS / 64, old_total);
  if (total == 0 && old_total == 0) return;
  const uint32_t nowhere = 0xFFFFFFFFu;  // (an index outside the range: of a region that does not ascend)

  auto in_registers = [&](auto pairs) {  // up to `pairs` of either set, all loads on their way together
    constexpr int kPer = decltype(pairs)::value / THREADS;
    uint32_t old_rel[kPer], rel[kPer];
    int pw[kPer];
    float x[kPer];
    uint64_t mine = 0;  // payloads of the wavefront's pairs, a bit each (uniform)
    const int32_t own_old = REPLACE && lane < num_old ? was.begin[lane] : INT32_MAX;
    const int32_t own = lane < num_payloads ? sh.begin[lane] : INT32_MAX;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int q0 = wave * 64 + k * THREADS, q = q0 + lane;
      old_rel[k] = nowhere;
      if (!REPLACE || q0 >= old_total) continue;  // uniform
      int first, last;
      const int w = payloads_of(own_old, num_old, q0, lane, first, last);
      if (q < old_total) {
        const uint32_t r = (uint32_t)was.idx_at[w][q - was.begin[w]] - (uint32_t)blk.begin;
        old_rel[k] = r < length ? r : nowhere;
      }
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int q0 = wave * 64 + k * THREADS, q = q0 + lane;
      rel[k] = nowhere;
      pw[k] = -1;
      x[k] = 0.0f;
      if (q0 >= total) continue;  // uniform
      int first, last;
      const int w = payloads_of(own, num_payloads, q0, lane, first, last);
      mine |= payload_bits(first, last);
      if (q < total) {
        const int src = q - sh.begin[w];
        const uint32_t r = (uint32_t)sh.idx_at[w][src] - (uint32_t)blk.begin;
        const float value = sh.val_at[w][src];
        x[k] = scaled ? scale * value : value;
        if (r < length) {
          rel[k] = r;
          pw[k] = w;
        }
      }
    }
    float held[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      held[k] = 0.0f;
      if (!REPLACE && k * THREADS < total && rel[k] != nowhere) held[k] = range[rel[k]];
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      if (REPLACE && k * THREADS < old_total && old_rel[k] != nowhere) sh.acc[old_rel[k]] = 0.0f;
      if (k * THREADS < total && rel[k] != nowhere) sh.acc[rel[k]] = held[k];  // pairs of several payloads with one index write the same
    }
    __syncthreads();
    for (int w = 0; w < num_payloads; ++w) {  // payloads in the order given
      if ((mine >> w) & 1u) {
#pragma unroll
        for (int k = 0; k < kPer; ++k)
          if (pw[k] == w) sh.acc[rel[k]] = sh.acc[rel[k]] + x[k];
      }
      __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      if (k * THREADS < total && rel[k] != nowhere) range[rel[k]] = sh.acc[rel[k]];
      if (REPLACE && k * THREADS < old_total && old_rel[k] != nowhere) range[old_rel[k]] = sh.acc[old_rel[k]];
    }
  };
  if (total <= kDirectPairs && old_total <= kDirectPairs) {
    in_registers(std::integral_constant<int, kDirectPairs>{});
    return;
  }
  if (total <= most && old_total <= most) {
    in_registers(std::integral_constant<int, kDirectPairsMost>{});
    return;
  }

  // Pairs that crowd the part: as in merge_parts_kernel the whole of it is read (REPLACE: starts from zero; outside the earlier
  // payloads' indices it is zero anyway), the pairs are added in chunks, with rounds on their way, and the whole of it is written.
  constexpr int kWaves = THREADS / 64;
  constexpr int kRounds = 2 * kPartThreads / THREADS;  // as many pairs on their way as there
  constexpr int kQuads = kEmitElements / 4 / THREADS;
  const bool looks_after = lane < num_payloads;
  const ChunkTable t(looks_after ? p.idx[lane] : nullptr, looks_after ? p.val[lane] : nullptr,
                     looks_after ? (int32_t)(sh.idx_at[lane] - in_global(p.idx[lane])) : 0,
                     looks_after ? sh.begin[lane + 1] - sh.begin[lane] : 0, num_payloads, lane);
  uint32_t cursor = 0;  // next chunk
  auto fetch = [&](ChunkRound& L) {
    L.part = -1;
    if (cursor >= t.total) return;
    L.part = 0;
    L.fetch(t, cursor, kWaves, wave, lane);
  };
  ChunkRound rounds[kRounds];
#pragma unroll
  for (int i = 0; i < kRounds; ++i) fetch(rounds[i]);
  {
    fvec4u d[kQuads];
#pragma unroll
    for (int i = 0; i < kQuads; ++i) d[i] = load_quad(range, REPLACE ? 0 : (int32_t)length, 4 * (tid + i * THREADS));
#pragma unroll
    for (int i = 0; i < kQuads; ++i)
      *reinterpret_cast<float4*>(&sh.acc[4 * (tid + i * THREADS)]) = make_float4(d[i][0], d[i][1], d[i][2], d[i][3]);
  }
  if constexpr (NAMED) {
    for (int i = tid; i < kSeenWords; i += THREADS) seen[i] = 0;
  }
  int last_w = -1;
  for (bool more = true; more;) {
#pragma unroll
    for (int i = 0; i < kRounds; ++i) {
      if (rounds[i].part < 0) {
        more = false;
        break;
      }
      add_round<NAMED>(rounds[i], sh.acc, (uint32_t)blk.begin, length, scaled, scale, last_w, lane, fetch, seen);
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kQuads; ++i) {
    const int e = 4 * (tid + i * THREADS);
    const float4 y = *reinterpret_cast<const float4*>(&sh.acc[e]);
    const fvec4u four = {y.x, y.y, y.z, y.w};
    if constexpr (NAMED) {
      const uint4 q = *reinterpret_cast<const uint4*>(&seen[e % kSeenWords]);
      const uint32_t bit = 1u << (e / kSeenWords);
      if (q.x & q.y & q.z & q.w & bit) {
        store_quad(range, (int32_t)length, e, four);
      } else {
        if (q.x & bit) range[e] = four[0];
        if (q.y & bit) range[e + 1] = four[1];
        if (q.z & bit) range[e + 2] = four[2];
        if (q.w & bit) range[e + 3] = four[3];
      }
    } else {
      store_quad(range, (int32_t)length, e, four);
    }
  }
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

// One round of eight probes of a list of m values by as many neighbouring lanes: the probe of lane i, and
// after the vote the bracket [lo, hi] that the answer lies in.
struct ProbeRound {
  static constexpr int kProbes = 8;
  int start, step, last;  // probe i is at clamp(start + i * step, 0, last)
  // around a guess, four standard deviations to either side
  __device__ __forceinline__ ProbeRound(const Guess& g, int m)
      : start(g.place - kProbes / 2 * (g.sigma + 1)), step(g.sigma + 1), last(m - 1) {}
  // over the whole list
  __device__ __forceinline__ explicit ProbeRound(int m) : start(0), step((m + kProbes - 1) / kProbes), last(m - 1) {}
  __device__ __forceinline__ int at(int i) const {
    const int64_t p = (int64_t)start + (int64_t)i * step;
    return p < 0 ? 0 : p > last ? last : (int)p;
  }
  __device__ __forceinline__ void narrow(int below, int& lo, int& hi) const {  // `below` probes are less than x: a prefix
    if (below < kProbes && at(below) < hi) hi = at(below);
    if (below > 0 && at(below - 1) >= lo) lo = at(below - 1) + 1;
    if (lo > hi) lo = hi;
  }
};

// Receive side at warm-up densities (paper: Section 4, warm-up training -- 25 % down to
// 0.4 % of the elements are sent during the first epochs): with millions of pairs per
// payload, adding them one by one to `dense` costs a scattered read-modify-write each.
// Here a workgroup owns one emit workgroup's part of a tensor (at most kEmitElements
// elements, contiguous in index order in every payload's region, see above), keeps the
// whole range of `dense` in LDS, adds the payloads' pairs to it in the order of the
// payloads, and writes the range back: `dense` is read and written once, coalesced, four
// elements to a lane (one to a lane: 251 instead of 243 us on 122 M elements with eight
// payloads of 1.6 %), the pairs are read once, coalesced, and the sums are those of the
// plain definition, bit for bit.
//
// At these densities a region holds up to millions of pairs and the search for a part's
// pairs is several rounds of dependent loads: with one workgroup per compute unit (the
// accumulator fills LDS) nothing else would run meanwhile.  So the searches of all parts
// and payloads run first, spread over the chip, and leave (first pair, number of pairs)
// of every part in every payload's region in a table (a part ends where the next one of
// its tensor starts, so one bound per part is searched for).  The probes are what this
// launch costs (each one a 64-byte sector from HBM: 350 MB with 32 probes per round and
// two bounds per part), so eight lanes share a search: 8 probes per round, about seven
// rounds for a region of a million pairs, fewer where a first guess is close: 25.7 us on 122 M elements
// at 25 %, 30 with searches over the whole region.  The first round probes around the guess and over the
// whole region at once, so that a wrong guess (pairs that crowd a part of the tensor) costs no round.
__global__ __launch_bounds__(kFlatThreads) void locate_parts_kernel(RegionPayloads p, int32_t num_payloads,
                                                                    const int64_t* __restrict__ out_offsets,
                                                                    const MergeBlock* __restrict__ blocks,
                                                                    int32_t num_blocks, int2* __restrict__ found) {
  // A wavefront takes seven consecutive parts of one payload; its eighth group finds the
  // start of the part after them, which is where the seventh ends.
  const int lane = threadIdx.x & 63;
  const int group = lane >> 3;
  const int sub = lane & 7;
  const int waves_per_payload = (num_blocks + 6) / 7;
  const int64_t wave_id = (int64_t)blockIdx.x * (kFlatThreads / 64) + (threadIdx.x >> 6);
  const int w = (int)(wave_id / waves_per_payload);
  const int b = (int)(wave_id % waves_per_payload) * 7 + group;
  const bool valid = w < num_payloads && b < num_blocks;
  MergeBlock blk{};
  int64_t region = 0;
  const int32_t* __restrict__ list = nullptr;
  int32_t x = 0;
  int lo = 0, hi = 0;  // the answer lies in [lo, hi]
  int cnt = 0;
  bool last = true;    // the tensor's last part: it ends where the region's pairs end
  if (valid) {
    blk = blocks[b];
    region = out_offsets[blk.tensor];
    const int64_t cap = out_offsets[blk.tensor + 1] - region;
    int64_t c = p.counts[w][blk.tensor];
    if (c > cap) c = cap;
    if (c < 0) c = 0;
    cnt = (int)c;
    last = b + 1 >= num_blocks || blocks[b + 1].tensor != blk.tensor;
    list = p.idx[w] + region;
    x = blk.begin;
    hi = x > blk.lo ? cnt : 0;  // (a tensor's first part starts at the region's start)
  }
  // the first round around the place the part starts at if the pairs are spread evenly over the tensor, and
  // over the whole region
  if (__ballot(hi > 64)) {
    const ProbeRound near(Guess(cnt, x, blk.lo, blk.hi > blk.lo ? blk.hi : blk.lo + 1), cnt), all(cnt);
    const int32_t at_near = hi > 0 ? list[near.at(sub)] : 0, at_all = hi > 0 ? list[all.at(sub)] : 0;
    const unsigned long long votes = __ballot(hi > 0 && at_near < x), votes_all = __ballot(hi > 0 && at_all < x);
    if (hi > 0) {
      near.narrow(__popc((uint32_t)(votes >> (8 * group)) & 0xFFu), lo, hi);
      all.narrow(__popc((uint32_t)(votes_all >> (8 * group)) & 0xFFu), lo, hi);
    }
  }
  // first position whose index is not below x ("index < x" is monotone along a region)
  while (__ballot(hi > lo)) {
    const int span = hi - lo;
    const int step = (span + 7) >> 3;
    const int pos = lo + sub * step;
    const bool less = span > 0 && pos < hi && list[pos] < x;
    const unsigned long long votes = __ballot(less);
    const int c = __popc((uint32_t)(votes >> (8 * group)) & 0xFFu);  // probes below x form a prefix
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
  const int next_lo = __shfl(lo, (lane + 8) & 63);  // of the part after this one (group 7 does not use it)
  if (valid && group < 7 && sub == 0) {
    const int end = last ? cnt : next_lo;
    found[(int64_t)b * num_payloads + w] = make_int2((int)region + lo, end > lo ? end - lo : 0);
  }
}

// REPLACE: `dense` becomes the sum of the payloads: the accumulator starts from zero instead of
// the range of `dense`, and every range is written, also one that no pair falls into.
//
// The pairs of a part are taken in chunks of kPartChunk slots, a wavefront each and four consecutive slots to a
// lane, that start on 128-byte lines of the payload's index array (the slots before its first pair and behind its
// last stay empty, and no load goes beyond the last).  Two things bounded the kernel before: loads of a pair per lane that straddled lines (a bare
// read of eight payloads' pairs, 1.95 GB in parts of 8192: 284 us in whole lines, 338 half a line off), and
// instructions, sixteen wavefronts on four SIMDs (chunks of one pair per lane, lines or not: 535 us at 25 %).
// A round is a chunk for every wavefront, of one payload or of several in their order, and only a change of
// payload needs a barrier (the indices of one payload are distinct).  While a round is added, the next two are on
// their way, those of the next part included, so that neither the write-back nor the table look-up leaves the
// memory pipeline of the unit empty.  122 M elements, eight payloads: 497 -> 426 us at 25 % (2.56 GB, 6.0 TB/s),
// 242 -> 191 at 1.6 % as the SGD apply (1.1 GB, 5.7 TB/s); 25.6 M elements, sixteen payloads of 6.25 %: 103 -> 86.5
// (95 with the first and last loads of a part sorted out, and so waited for, when they are asked for),
// where 933 parts leave a fourth round of workgroups two thirds full.  Three rounds on their way: 442, 194, 100 against 426, 195, 95.
//
// SEARCH: every part has a workgroup of its own, which finds its payloads' pairs itself instead of reading them from the table of a
// launch before (see kPartSearches).  A wavefront takes up to four payloads, two at a time.
template <bool REPLACE, bool SEARCH>
__global__ __launch_bounds__(kPartThreads) void merge_parts_kernel(float* __restrict__ dense, RegionPayloads p,
                                                                   int32_t num_payloads,
                                                                   const int64_t* __restrict__ out_offsets,
                                                                   const MergeBlock* __restrict__ blocks,
                                                                   int32_t num_blocks,
                                                                   std::conditional_t<SEARCH, int2, const int2>* __restrict__ found,
                                                                   float scale, int32_t scaled) {
  constexpr int kQuads = kEmitElements / 4 / kPartThreads;
  constexpr int kWaves = kPartThreads / 64;
  __shared__ alignas(16) float acc[kEmitElements + 64];  // behind the range a word per lane for what is no pair of it
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  auto put_quad = [&](int i, const fvec4u& y) {
    *reinterpret_cast<float4*>(&acc[4 * (tid + i * kPartThreads)]) = make_float4(y[0], y[1], y[2], y[3]);
  };

  // The accumulator fills LDS, so a workgroup is alone on its compute unit: the grid is one
  // workgroup per compute unit and every workgroup takes parts b, b + grid, ...
  int b = blockIdx.x;
  if (b >= num_blocks) return;
  const int step = (int)gridDim.x;

  // Lane w looks after payload w.
  const int32_t* const idx_of = lane < num_payloads ? p.idx[lane] : nullptr;
  const float* const val_of = lane < num_payloads ? p.val[lane] : nullptr;
  __shared__ int2 own_entry[SEARCH ? kMaxPayloads : 1];
  if constexpr (SEARCH) {
    const MergeBlock blk = blocks[b];
    const int64_t region = out_offsets[blk.tensor];
    const int64_t cap = out_offsets[blk.tensor + 1] - region;
    for (int w = wave; w < num_payloads; w += 2 * kWaves) {  // uniform
      const bool two = w + kWaves < num_payloads;
      const int w2 = two ? w + kWaves : w;
      const int32_t* __restrict__ list = p.idx[w] + region;
      const int32_t* __restrict__ list2 = p.idx[w2] + region;
      const int32_t* __restrict__ counts = p.counts[w];
      const int32_t* __restrict__ counts2 = p.counts[w2];
      const int32_t both = (lane & 1 ? counts2 : counts)[blk.tensor];  // one load for the two
      const int32_t count = __builtin_amdgcn_readlane(both, 0), count2 = __builtin_amdgcn_readlane(both, 1);
      int lo = 0, hi = count < 0 ? 0 : count > cap ? (int)cap : count;
      int lo2 = 0, hi2 = !two || count2 < 0 ? 0 : count2 > cap ? (int)cap : count2;
      if (blk.begin != blk.lo || blk.end != blk.hi)  // (a part that is a whole tensor has all its pairs)
        wave_equal_ranges(list, hi, list2, hi2, reinterpret_cast<const int32_t*>(blocks), blk.begin, blk.end, lane, lo, hi, lo2, hi2);
      if (lane == 0) {  // (the table says the same after either way: a reader of the workspace can tell what of it is the part kernels')
        found[(int64_t)b * num_payloads + w] = own_entry[w] = make_int2((int)region + lo, hi > lo ? hi - lo : 0);
        if (two) found[(int64_t)b * num_payloads + w2] = own_entry[w2] = make_int2((int)region + lo2, hi2 > lo2 ? hi2 - lo2 : 0);
      }
    }
    __syncthreads();
  }
  auto entry_of = [&](int part) {
    if (SEARCH) return part == (int)blockIdx.x && lane < num_payloads ? own_entry[lane] : make_int2(0, 0);
    return part < num_blocks && lane < num_payloads ? found[(int64_t)part * num_payloads + lane] : make_int2(0, 0);
  };
  auto make_table = [&](const int2& f) { return ChunkTable(idx_of, val_of, f.x, f.y, num_payloads, lane); };
  int fb = b;            // the part that is being fetched
  ChunkTable t = make_table(entry_of(b));
  int2 next_entry = entry_of(b + step);
  uint32_t cursor = 0;   // next chunk of it
  auto fetch = [&](ChunkRound& L) {
    while (cursor >= t.total && fb + step < num_blocks) {
      fb += step;
      t = make_table(next_entry);
      next_entry = entry_of(fb + step);
      cursor = 0;
    }
    L.part = -1;
    if (cursor >= t.total) return;
    L.part = fb;
    L.fetch(t, cursor, kWaves, wave, lane);
  };

  ChunkRound A, B;
  bool a_next = true;  // which of the two is added next
  fetch(A);
  fetch(B);
  MergeBlock blk = blocks[b];
  {
    fvec4u d[kQuads];
#pragma unroll
    for (int i = 0; i < kQuads; ++i) d[i] = load_quad(dense + blk.begin, REPLACE ? 0 : (int32_t)(blk.end - blk.begin), 4 * (tid + i * kPartThreads));
#pragma unroll
    for (int i = 0; i < kQuads; ++i) put_quad(i, d[i]);
  }
  for (;;) {
    const bool more = b + step < num_blocks;
    const MergeBlock next = blocks[more ? b + step : b];
    const uint32_t begin = (uint32_t)blk.begin;
    const uint32_t length = (uint32_t)(blk.end - blk.begin);  // <= kEmitElements
    bool any = false;
    int last_w = -1;
    auto add = [&](ChunkRound& L) { add_round<false>(L, acc, begin, length, scaled, scale, last_w, lane, fetch, nullptr); };
    for (;;) {
      if (a_next) {
        if (A.part != b) break;
        add(A);
      } else {
        if (B.part != b) break;
        add(B);
      }
      a_next = !a_next;
      any = true;
    }
    // The range is written, and the accumulator takes the next part's: every thread its own elements.
    fvec4u d[kQuads];
#pragma unroll
    for (int i = 0; i < kQuads; ++i) d[i] = load_quad(dense + next.begin, (more && !REPLACE) ? (int32_t)(next.end - next.begin) : 0, 4 * (tid + i * kPartThreads));
    __syncthreads();
    float* __restrict__ range = dense + blk.begin;
#pragma unroll
    for (int k = 0; k < kQuads; ++k) {
      const float4 y = *reinterpret_cast<const float4*>(&acc[4 * (tid + k * kPartThreads)]);
      if (REPLACE || any) store_quad(range, (int32_t)length, 4 * (tid + k * kPartThreads), fvec4u{y.x, y.y, y.z, y.w});
    }
    if (!more) break;
#pragma unroll
    for (int k = 0; k < kQuads; ++k) put_quad(k, d[k]);
    b += step;
    blk = next;
    // (no barrier here: the first payload of the next part comes behind one)
  }
}

// The sparse clear at the same densities: the indices of all payloads inside the part
// are marked in an LDS bitmap and zeros stored where a bit is set, every element once.
// Bound by memory: 25.6 M elements, sixteen payloads of 6.25 %, 209 MB read (the indices, and the sectors, whose
// other elements are written back) and 102 MB written in 69 us, 4.5 TB/s; 83 us when the workgroup took one
// payload after the other, four indices per thread in flight.
__global__ __launch_bounds__(kPartClearThreads) void clear_parts_kernel(float* __restrict__ dense, RegionPayloads p,
                                                                        int32_t num_payloads,
                                                                        const MergeBlock* __restrict__ blocks,
                                                                        const int2* __restrict__ found) {
  constexpr int kWords = kEmitElements / 32 / kPartClearThreads;
  __shared__ uint32_t bitmap[kEmitElements / 32];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const MergeBlock blk = blocks[blockIdx.x];
  const int32_t length = (int32_t)(blk.end - blk.begin);
  // lane w looks after payload w
  const int2 entry = lane < num_payloads ? found[(int64_t)blockIdx.x * num_payloads + lane] : make_int2(0, 0);
#pragma unroll
  for (int k = 0; k < kWords; ++k) bitmap[tid + k * kPartClearThreads] = 0;
  if (__ballot(entry.y > 0) == 0) return;  // the same in every wavefront
  __syncthreads();
  // A wavefront takes payloads w, w + waves, ...: the order does not matter here, and no barrier separates
  // them.  Sixteen indices per lane are on their way at a time.
  {
    typedef int32_t vec4u __attribute__((ext_vector_type(4), aligned(4)));
    auto mark = [&](int32_t i) {
      const int64_t rr = (int64_t)i - blk.begin;  // outside the range: a foreign region
      if (rr >= 0 && rr < length) atomicOr(&bitmap[rr >> 5], 1u << (rr & 31));
    };
    for (int w = wave; w < num_payloads; w += kPartClearThreads / 64) {
      const int n = __builtin_amdgcn_readlane(entry.y, w);
      if (n == 0) continue;
      const int32_t* __restrict__ ip = p.idx[w] + __builtin_amdgcn_readlane(entry.x, w);
      const int quads = n >> 2;
      for (int first = lane; first < quads; first += 64 * kPartClearLoads) {
        vec4u r[kPartClearLoads];
#pragma unroll
        for (int k = 0; k < kPartClearLoads; ++k) {
          const int q = first + 64 * k;
          r[k] = __builtin_nontemporal_load(reinterpret_cast<const vec4u*>(ip + 4 * (q < quads ? q : 0)));
        }
#pragma unroll
        for (int k = 0; k < kPartClearLoads; ++k) {
          if (first + 64 * k < quads) {
#pragma unroll
            for (int c = 0; c < 4; ++c) mark(r[k][c]);
          }
        }
      }
      if (lane < (n & 3)) mark(ip[4 * quads + lane]);
    }
  }
  __syncthreads();
  float* __restrict__ range = dense + blk.begin;
  // Lane after lane along the range, four consecutive elements per lane.  A store of part
  // of a 64-byte sector costs the memory system a read-modify-write of its own, so a sector
  // with any element to clear is written whole by its four lanes, each of which reads its
  // 16 bytes first unless all of them are cleared.
  const bool aligned = ((reinterpret_cast<uintptr_t>(range) & 15) == 0);
  if (aligned) {
    typedef float fvec4 __attribute__((ext_vector_type(4)));
    constexpr int kGroups = kEmitElements / 4 / kPartClearThreads;
    constexpr int kBatch = 8;
    for (int i0 = 0; i0 < kGroups; i0 += kBatch) {
      uint32_t nib[kBatch];
      bool touch[kBatch];  // the lane's sector has an element to clear
      fvec4 old[kBatch];
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        const int e4 = tid + (i0 + i) * kPartClearThreads;
        const int e = e4 * 4;
        const uint32_t word = e < length ? bitmap[e4 >> 3] : 0u;
        nib[i] = (word >> ((e4 & 7) * 4)) & 15u;
        touch[i] = ((word >> ((e4 & 4) * 4)) & 0xFFFFu) != 0;
        old[i] = fvec4{0.0f, 0.0f, 0.0f, 0.0f};
        if (touch[i] && nib[i] != 15u && e + 4 <= length) old[i] = *reinterpret_cast<const fvec4*>(range + e);

      }
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        if (!touch[i]) continue;
        const int e = (tid + (i0 + i) * kPartClearThreads) * 4;
        if (e + 4 <= length) {
          fvec4 v = old[i];
#pragma unroll
          for (int c = 0; c < 4; ++c)
            if ((nib[i] >> c) & 1u) v[c] = 0.0f;
          *reinterpret_cast<fvec4*>(range + e) = v;

        } else {  // the last, incomplete group of the range
#pragma unroll
          for (int b = 0; b < 4; ++b)
            if (((nib[i] >> b) & 1u) && e + b < length) range[e + b] = 0.0f;
        }
      }
    }
  } else {
    for (int e4 = tid; e4 * 4 < length; e4 += kPartClearThreads) {
      const uint32_t nib = (bitmap[e4 >> 3] >> ((e4 & 7) * 4)) & 15u;
      const int e = e4 * 4;
#pragma unroll
      for (int b = 0; b < 4; ++b)
        if (((nib >> b) & 1u) && e + b < length) range[e + b] = 0.0f;
    }
  }
}

}  // namespace

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
int32_t compute_units() {
  static const int32_t units = [] {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
      n = 256;
    return (int32_t)n;
  }();
  return units;
}

hipError_t launch_scatter_pairs(float* dense, int64_t n, const PairPayloads& p, int32_t first,
                                int32_t num, int64_t max_count, ScatterMode mode, float scale,
                                uint32_t* diag_flags, hipStream_t stream) {
  if (num <= 0 || max_count <= 0) return hipSuccess;
  int64_t chunks = ceil_div(max_count, 256 * 4);
  if (chunks > 4096) chunks = 4096;
  hipLaunchKernelGGL(scatter_pairs_kernel, dim3((unsigned)chunks, (unsigned)num), dim3(256), 0, stream,
                     dense, n, p, first, mode, scale, diag_flags);
  return hipGetLastError();
}

hipError_t launch_clear_regions(float* dense, int64_t n, const RegionPayloads& p, int32_t num,
                                const int64_t* out_offsets_dev, int32_t num_tensors, int64_t total_capacity,
                                int64_t longest, hipStream_t stream) {
  if (num <= 0 || total_capacity <= 0) return hipSuccess;
  if ((int64_t)num_tensors * num <= kClearGroups) {
    const int64_t most = kClearGroups / 2 / ((int64_t)num_tensors * num), want = ceil_div(longest, kFlatChunk);
    const int64_t per = want < 1 || most < 1 ? 1 : want < most ? want : most;
    if (want <= kClearRounds * per) {
      hipLaunchKernelGGL(clear_tensors_kernel, dim3((unsigned)(num_tensors * per), (unsigned)num), dim3(kFlatThreads), 0,
                         stream, dense, n, p, out_offsets_dev, (uint32_t)per);
      return hipGetLastError();
    }
  }
  // a quarter of the capacity: regions sized as recommended hold eight times the expected
  // pairs, so most workgroups find one chunk; fuller regions make them loop
  int64_t chunks = ceil_div(total_capacity, 4 * kFlatChunk);
  if (chunks > 65536) chunks = 65536;
  hipLaunchKernelGGL(clear_regions_kernel, dim3((unsigned)chunks, (unsigned)num), dim3(kFlatThreads), 0, stream,
                     dense, n, p, out_offsets_dev, num_tensors);
  return hipGetLastError();
}

hipError_t launch_merge_regions(float* dense, const RegionPayloads& p, int32_t num, const RegionPayloads* old,
                                int32_t num_old, const int64_t* out_offsets_dev, const MergeBlock* blocks,
                                int32_t num_blocks, int64_t expected_pairs, bool scaled, float scale,
                                hipStream_t stream) {
  if (num <= 0 || num_blocks <= 0) return hipSuccess;
  const dim3 grid((unsigned)num_blocks);
  const int sc = scaled ? 1 : 0;
  // one wavefront per payload in a workgroup of eight, if the pairs a range can expect fit its accumulator
  const bool few = num <= 8 && num_old <= 8 && expected_pairs <= kMergeCapSmall;
  if (old) {  // dense becomes the sum (it holds the sum of `old` now)
    if (few)
      hipLaunchKernelGGL((merge_regions_kernel<true, 512>), grid, dim3(512), 0, stream, dense, p, num, *old, num_old,
                         out_offsets_dev, blocks, scale, sc);
    else
      hipLaunchKernelGGL((merge_regions_kernel<true, 1024>), grid, dim3(1024), 0, stream, dense, p, num, *old, num_old,
                         out_offsets_dev, blocks, scale, sc);
  } else {
    if (few)
      hipLaunchKernelGGL((merge_regions_kernel<false, 512>), grid, dim3(512), 0, stream, dense, p, num, p, 0,
                         out_offsets_dev, blocks, scale, sc);
    else
      hipLaunchKernelGGL((merge_regions_kernel<false, 1024>), grid, dim3(1024), 0, stream, dense, p, num, p, 0,
                         out_offsets_dev, blocks, scale, sc);
  }
  return hipGetLastError();
}

hipError_t launch_merge_direct(float* dense, const RegionPayloads& p, int32_t num, const RegionPayloads* old,
                               int32_t num_old, const int64_t* out_offsets_dev, const MergeBlock* parts,
                               int32_t num_parts, double expected_pairs, bool named_only, bool scaled,
                               float scale, hipStream_t stream) {
  if (num <= 0 || num_parts <= 0) return hipSuccess;
  const dim3 grid((unsigned)num_parts);
  const int sc = scaled ? 1 : 0;
  const int32_t most = num > 1 && expected_pairs > (double)kDirectPairs ? kDirectPairs : kDirectPairsMost;
  const auto launch = [&](auto kernel, int threads) {
    hipLaunchKernelGGL(kernel, grid, dim3((unsigned)threads), 0, stream, dense, p, num, old ? *old : p, old ? num_old : 0,
                       out_offsets_dev, parts, most, scale, sc);
  };
  if (num <= 8 && (!old || num_old <= 8)) {  // one wavefront per payload in a workgroup of eight
    old ? launch(merge_direct_kernel<true, false, 512>, 512)
        : named_only ? launch(merge_direct_kernel<false, true, 512>, 512) : launch(merge_direct_kernel<false, false, 512>, 512);
  } else {
    old ? launch(merge_direct_kernel<true, false, 1024>, 1024)
        : named_only ? launch(merge_direct_kernel<false, true, 1024>, 1024) : launch(merge_direct_kernel<false, false, 1024>, 1024);
  }
  return hipGetLastError();
}

static void launch_locate_parts(const RegionPayloads& p, int32_t num, const int64_t* out_offsets_dev,
                                const MergeBlock* parts, int32_t num_parts, int2* found, hipStream_t stream) {
  const int64_t waves = ceil_div(num_parts, 7) * num;  // seven parts of one payload per wavefront
  hipLaunchKernelGGL(locate_parts_kernel, dim3((unsigned)ceil_div(waves, kFlatThreads / 64)), dim3(kFlatThreads), 0,
                     stream, p, num, out_offsets_dev, parts, num_parts, found);
}

hipError_t launch_merge_parts(float* dense, const RegionPayloads& p, int32_t num, const int64_t* out_offsets_dev,
                              const MergeBlock* parts, int32_t num_parts, int64_t searched_tensors, void* found, bool replace,
                              bool scaled, float scale, hipStream_t stream) {
  if (num <= 0 || num_parts <= 0) return hipSuccess;
  const int units = compute_units();  // one workgroup of this kernel fits each
  const int grid = num_parts < units ? num_parts : units;
  const bool search = num_parts <= units && (int64_t)num_parts * num <= kPartSearches &&
                      (searched_tensors == 0 || (searched_tensors * num <= kPartSearchLists && num <= kPartSearchPayloads));
  if (!search) launch_locate_parts(p, num, out_offsets_dev, parts, num_parts, static_cast<int2*>(found), stream);
  const auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(kPartThreads), 0, stream, dense, p, num, out_offsets_dev,
                       parts, num_parts, static_cast<int2*>(found), scale, scaled ? 1 : 0);
  };
  if (search) launch(replace ? merge_parts_kernel<true, true> : merge_parts_kernel<false, true>);
  else launch(replace ? merge_parts_kernel<true, false> : merge_parts_kernel<false, false>);
  return hipGetLastError();
}

hipError_t launch_clear_parts(float* dense, const RegionPayloads& p, int32_t num, const int64_t* out_offsets_dev,
                              const MergeBlock* parts, int32_t num_parts, void* found, hipStream_t stream) {
  if (num <= 0 || num_parts <= 0) return hipSuccess;
  launch_locate_parts(p, num, out_offsets_dev, parts, num_parts, static_cast<int2*>(found), stream);
  hipLaunchKernelGGL(clear_parts_kernel, dim3((unsigned)num_parts), dim3(kPartClearThreads), 0, stream, dense, p, num,
                     parts, static_cast<const int2*>(found));
  return hipGetLastError();
}

}  // namespace dgc
