// HIP kernels of the wire format of the DGC payload for gfx950 (wave64, CDNA4): 32-bit
// values with 16-bit run lengths of zeros, both directions.

#include <cmath>

#include "dgc_device.h"
#include "dgc_internal.h"

namespace dgc {
namespace {

// ---------------------------------------------------------------------------
// Wire format (paper: Section 3.1 -- encode() packs the 32-bit nonzero values and
// 16-bit run lengths of zeros; footnote of Table 3)
// ---------------------------------------------------------------------------
// An entry (run, value) stands for `run` zeros followed by `value`, in the order of the
// flat index.  Sixteen bits hold a run of at most 65535, so a longer gap is bridged by
// entries (65535, 0.0f), each of which covers 65536 positions.  A pair whose
// predecessor in the whole set leaves `gap` zeros before it therefore takes
// 1 + (gap >> 16) entries, the last of them (gap & 0xFFFF, value).  Trailing zeros are
// not encoded.  Encoding needs every tensor's region in ascending index order
// (DGC_FLAG_SORTED_OUTPUT); regions follow each other in tensor order, which is index
// order.  Both directions are a prefix sum: block sums, their scan, write.

// Index of the last pair of the nearest non-empty region before tensor j, or -1.
// Called by one whole wavefront; every lane returns the same value.
__device__ __forceinline__ int32_t last_index_before(const EncodeArgs& a, int j) {
  const int lane = threadIdx.x & 63;
  for (int base = j - 1; base >= 0; base -= 64) {
    const int jj = base - lane;
    int64_t cnt = 0, region = 0;
    if (jj >= 0) {
      region = a.out_offsets[jj];
      const int64_t cap = a.out_offsets[jj + 1] - region;
      cnt = a.counts[jj];
      if (cnt > cap) cnt = cap;
    }
    const unsigned long long have = __ballot(cnt > 0);
    if (have) {
      const int src = __ffsll((long long)have) - 1;  // lowest lane = nearest tensor
      int32_t last = 0;
      if (lane == src) last = a.idx[region + cnt - 1];
      return __shfl(last, src);
    }
  }
  return -1;
}

// Tensor whose region holds workgroup slot `slot`: the last j with first_block[j] <= slot (a tensor with an
// empty region takes no slot and shares its number with the next one).  One round of loads and a vote for every 64 of up to
// 256 tensors; of more, the first wavefront searches, 64 probes a round, and the others learn it through LDS.
__device__ __forceinline__ int tensor_of_slot(const EncodeArgs& a, uint32_t slot, int* shared) {
  const int lane = threadIdx.x & 63;
  if (a.num_tensors <= 256) {
    uint32_t first[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) first[k] = lane + 64 * k < a.num_tensors ? a.first_block[lane + 64 * k] : 0xFFFFFFFFu;
    int before = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) before += __popcll(__ballot(first[k] <= slot));
    return before - 1;
  }
  if (threadIdx.x < 64) {
    int lo = 0, end = a.num_tensors;  // the first tensor that starts behind `slot` is in [lo, end]
    while (lo < end) {
      const int step = (end - lo + 63) >> 6;
      const int64_t at = lo + (int64_t)lane * step;
      const int c = __popcll(__ballot(at < end && a.first_block[at] <= slot));  // a prefix of the lanes
      if (c == 0) break;
      const int64_t next = lo + (int64_t)c * step;
      lo += (c - 1) * step + 1;
      end = next < end ? (int)next : end;
    }
    if (lane == 0) *shared = lo - 1;
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(*shared);
}

// Entries that the pairs of workgroup slot `slot` need, formed by the whole workgroup; every thread returns them.  `scratch`:
// two words of LDS.
__device__ __forceinline__ uint32_t need_of_slot(const EncodeArgs& a, uint32_t slot, uint32_t* scratch) {
  const int lane = threadIdx.x & 63;
  __syncthreads();  // (the scratch may be in use)
  if (threadIdx.x == 0) scratch[1] = 0;
  const int j = tensor_of_slot(a, slot, reinterpret_cast<int*>(scratch));
  const int64_t region = a.out_offsets[j];
  const int64_t cap = a.out_offsets[j + 1] - region;
  const int64_t count = a.counts[j] > cap ? cap : a.counts[j];
  const int64_t begin = (int64_t)(slot - a.first_block[j]) * kWireChunk;
  const int64_t end = count < begin + kWireChunk ? count : begin + kWireChunk;
  const int32_t* __restrict__ idx = a.idx + region;
  const int32_t first = begin == 0 && count > 0 ? last_index_before(a, j) : 0;
  uint32_t mine = 0;
  for (int64_t p = begin + threadIdx.x; p < end; p += kWireThreads) {
    const int32_t gap = idx[p] - (p > 0 ? idx[p - 1] : first) - 1;
    mine += 1u + (gap > 0 ? (uint32_t)gap >> 16 : 0u);
  }
  mine = wave_sum(mine);
  __syncthreads();
  if (lane == 0) atomicAdd(&scratch[1], mine);
  __syncthreads();
  return scratch[1];
}

// PASS 0: entries needed by the workgroup's pairs.  PASS 1: write them.  One workgroup per kWireChunk
// pairs a region can hold.  A wavefront takes 64 neighbouring pairs at a time, one per lane, so that
// every load and store is a straight run; its predecessor's index comes from the lane below, and only a
// round with a gap of 65536 or more needs a scan (a pair takes one entry otherwise).  With sixteen
// consecutive pairs per thread instead, 4.1 M pairs took 17 us to count and 71 us to write.
// ONCE: both in one launch.  A workgroup leaves its need in memory, with the number of the call, and looks for those of the
// workgroups before it for a while; what is missing then it forms itself, so that nothing waits without an end, whatever
// else runs.  The last workgroup to have them all counts the calls on.  161 tensors of 25.6 M elements, 0.1 %: 4.3 + 7.4 ->
// 8.8 us, the call and the decoding of sixteen streams after it 34.8 -> 32.4.
template <int PASS, bool ONCE>
__global__ __launch_bounds__(kWireThreads) void encode_kernel(EncodeArgs a) {
  constexpr int kWaves = kWireThreads / 64;
  __shared__ uint32_t scratch[2];
  __shared__ unsigned long long lacking[kWaves];
  const uint32_t call = ONCE ? a.state->wire_call : 0u;
  __shared__ uint32_t wave_need[kWaves];
  __shared__ uint32_t wave_before[kWaves];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  __shared__ int tensor;
  int j;
  uint32_t slot;
  if (a.per_tensor > 0) {
    j = (int)(blockIdx.x / (uint32_t)a.per_tensor);
    slot = a.first_block[j] + blockIdx.x % (uint32_t)a.per_tensor;
    if (slot >= a.first_block[j + 1]) return;
  } else {
    slot = blockIdx.x;
    j = tensor_of_slot(a, slot, &tensor);
  }
  const int64_t region = a.out_offsets[j];
  const int64_t cap = a.out_offsets[j + 1] - region;
  int64_t count = a.counts[j];
  if (count > cap) count = cap;
  const int64_t begin = (int64_t)(slot - a.first_block[j]) * kWireChunk;
  const bool last_slot = PASS == 1 && (ONCE || a.self_scan) && (int)slot == a.total_blocks - 1;  // knows how many entries there are
  auto leave_need = [&](uint32_t need) {
    __hip_atomic_store(a.needs + slot, (unsigned long long)(kWireCall | call) << 32 | need, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  auto arrive = [&]() {  // one thread; the workgroup has everything from the others
    if (__hip_atomic_fetch_add(&a.state->wire_arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)a.total_blocks - 1u) {
      a.state->wire_arrived = 0;
      a.state->wire_call = (call + 1u) & (kWireCall - 1u);
    }
  };
  if (begin >= count) {
    if (PASS == 0 && threadIdx.x == 0) a.sums[slot] = 0;
    if (!last_slot) {
      if (ONCE && threadIdx.x == 0) {
        leave_need(0);
        arrive();
      }
      return;
    }
  }
  const int32_t* __restrict__ idx = a.idx + region;
  const int64_t p0 = begin + wave * (64 * kWireRounds);  // the wavefront's first pair
  int32_t prev = -1;                                     // index of the pair before the round
  if (p0 > 0 && p0 <= count) prev = idx[p0 - 1];
  else if (p0 == 0 && count > 0) prev = last_index_before(a, j);
  const int64_t left = count - p0;
  const uint32_t pairs = left <= 0 ? 0u : left < 64 * kWireRounds ? (uint32_t)left : (uint32_t)(64 * kWireRounds);
  const bool one_round = pairs <= 64;  // uniform; small tensors have a pair or two each (20000 of them: 95 -> 60 us)
  int32_t mine[kWireRounds];
#pragma unroll
  for (int r = 0; r < kWireRounds; ++r) {
    if (r == 1 && one_round) break;
    const int64_t p = p0 + r * 64 + lane;
    mine[r] = p < count ? idx[p] : 0;
  }
  float x[PASS == 1 ? kWireRounds : 1];
  if (PASS == 1) {
    const float* __restrict__ val = a.val + region;
#pragma unroll
    for (int r = 0; r < kWireRounds; ++r) {
      if (r == 1 && one_round) break;
      const int64_t p = p0 + r * 64 + lane;
      x[r] = p < count ? val[p] : 0.0f;
    }
  }
  int32_t gap[kWireRounds];  // zeros before the lane's pair; not ascending: flagged, and encoded as if adjacent
  uint32_t fillers = 0;      // of the lane
  bool unsorted = false;
#pragma unroll
  for (int r = 0; r < kWireRounds; ++r) {
    if (r == 1 && one_round) break;
    const bool have = p0 + r * 64 + lane < count;
    int32_t before = __shfl_up(mine[r], 1);
    if (lane == 0) before = prev;
    prev = __builtin_amdgcn_readlane(mine[r], 63);
    gap[r] = have ? mine[r] - before - 1 : 0;
    if (gap[r] < 0) {
      gap[r] = 0;
      unsorted = true;
    }
    fillers += (uint32_t)gap[r] >> 16;
  }
  const uint32_t need = pairs + wave_sum(fillers);  // of the wavefront
  if (lane == 0) wave_need[wave] = need;
  if (PASS == 0) {
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t total = 0;
      for (int w = 0; w < kWaves; ++w) total += wave_need[w];
      a.sums[slot] = total;
    }
    if (unsorted) atomicOr(&a.state->flags, (uint32_t)DGC_DIAG_UNSORTED);
    return;
  }
  if (ONCE && unsorted) atomicOr(&a.state->flags, (uint32_t)DGC_DIAG_UNSORTED);
  uint32_t before_block = 0;
  if (ONCE) {
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t total = 0;
      for (int w = 0; w < kWaves; ++w) total += wave_need[w];
      leave_need(total);
    }
    unsigned long long word = 0;
    const bool mine_to_look = threadIdx.x < slot;
    if (mine_to_look) {
      const int looks = looks_for(a.looks, (int)threadIdx.x);
      for (int look = 0; look < looks && (uint32_t)(word >> 32) != (kWireCall | call); ++look) {
        if (look > 0) __builtin_amdgcn_s_sleep(1);
        word = __hip_atomic_load(a.needs + threadIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    const bool there = (uint32_t)(word >> 32) == (kWireCall | call);
    const unsigned long long votes = __ballot(mine_to_look && !there);
    const uint32_t seen = wave_sum(mine_to_look && there ? (uint32_t)word : 0u);
    if (lane == 0) {
      wave_before[wave] = seen;
      lacking[wave] = votes;
    }
    __syncthreads();
    unsigned long long any = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      before_block += wave_before[w];
      any |= lacking[w];
    }
    if (__builtin_amdgcn_readfirstlane(any != 0 ? 1 : 0)) {  // the same in every wavefront
      for (uint32_t t = 0; t < slot; ++t)
        if ((lacking[t >> 6] >> (t & 63u)) & 1u) before_block += need_of_slot(a, t, scratch);
    }
    if (threadIdx.x == 0) arrive();
  } else if (a.self_scan) {  // few block sums: every workgroup adds up those before its own
    uint32_t mine_before = 0;
    const uint4* __restrict__ four = reinterpret_cast<const uint4*>(a.sums);  // starts on a 256-byte boundary
    const uint32_t quads = slot >> 2;
    for (uint32_t i = threadIdx.x; i < quads; i += 4 * kWireThreads) {
      uint4 c[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) c[k] = i + k * kWireThreads < quads ? four[i + k * kWireThreads] : make_uint4(0, 0, 0, 0);
#pragma unroll
      for (int k = 0; k < 4; ++k) mine_before += (c[k].x + c[k].y) + (c[k].z + c[k].w);
    }
    if (threadIdx.x < (slot & 3u)) mine_before += a.sums[4 * quads + threadIdx.x];
    mine_before = wave_sum(mine_before);
    if (lane == 0) wave_before[wave] = mine_before;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWaves; ++w) before_block += wave_before[w];
  } else {
    __syncthreads();
    before_block = a.sums[slot];
  }
  int64_t pos = before_block;
  uint32_t block_total = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    if (w < wave) pos += wave_need[w];
    block_total += wave_need[w];
  }
  if (last_slot && threadIdx.x == 0) *a.num_entries = (int32_t)(before_block + block_total);
  bool overflow = false;
#pragma unroll
  for (int r = 0; r < kWireRounds; ++r) {
    const int64_t round_left = count - (p0 + r * 64);
    if (round_left <= 0) break;
    const bool have = lane < round_left;
    const uint32_t fill = (uint32_t)gap[r] >> 16;
    uint32_t incl = (uint32_t)lane + 1u;  // entries of the round up to and with this lane's
    uint32_t total = round_left < 64 ? (uint32_t)round_left : 64u;
    if (__ballot(fill != 0) != 0) {
      incl = wave_inclusive_sum(have ? 1u + fill : 0u);
      total = wave_last(incl);
    }
    if (have) {
      int64_t at = pos + incl - 1u;  // of the pair's own entry
      for (uint32_t f = fill; f > 0; --f) {
        if (at - f < a.capacity) {
          a.runs[at - f] = 0xFFFFu;
          a.vals[at - f] = 0.0f;
        } else {
          overflow = true;
        }
      }
      if (at < a.capacity) {
        a.runs[at] = (uint16_t)((uint32_t)gap[r] & 0xFFFFu);
        a.vals[at] = x[r];
      } else {
        overflow = true;
      }
    }
    pos += total;
  }
  if (overflow) atomicOr(&a.state->flags, (uint32_t)DGC_DIAG_OVERFLOW);
}

// In-place exclusive prefix sum of every segment of `sums`; one workgroup per segment.  Sums are formed in
// 64 bits and held at 2^31 - 1, which lies behind every element (a stream that covers more than it may
// cannot wrap round to a valid position).  `total_out` (may be null) receives the sum of segment 0;
// `diag_flags` (may be null) DGC_DIAG_BAD_INDEX if a segment's sum exceeds `limit`.
__global__ __launch_bounds__(kScanThreads) void scan_kernel(uint32_t* sums, ScanSegments seg, int32_t* total_out,
                                                            int64_t limit, uint32_t* diag_flags) {
  typedef uint32_t vec4u __attribute__((ext_vector_type(4), aligned(4)));
  static_assert(kScanPer % 4 == 0, "loads and stores of four");
  constexpr int kWaves = kScanThreads / 64;
  __shared__ uint64_t wave_sums[kWaves];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int32_t begin = seg.begin[blockIdx.x];
  const int32_t end = seg.begin[blockIdx.x + 1];
  uint64_t carry = 0;
  for (int64_t base = begin; base < end; base += kScanThreads * kScanPer) {
    const int64_t i0 = base + (int64_t)threadIdx.x * kScanPer;
    uint32_t x[kScanPer];
    uint64_t mine = 0;
    if (i0 + kScanPer <= end) {  // (one at a time, behind a condition each, they waited for each other: four segments of 8000 sums 8.9 us, now 4.8)
#pragma unroll
      for (int k = 0; k < kScanPer; k += 4) {
        const vec4u y = *reinterpret_cast<const vec4u*>(sums + i0 + k);
#pragma unroll
        for (int c = 0; c < 4; ++c) x[k + c] = y[c];
      }
    } else {
#pragma unroll
      for (int k = 0; k < kScanPer; ++k) x[k] = i0 + k < end ? sums[i0 + k] : 0u;
    }
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) mine += x[k];
    // (below 2^32 per thread: the two halves are scanned apart, which cannot overflow 32 bits)
    const uint64_t incl = (uint64_t)wave_inclusive_sum((uint32_t)mine & 0xFFFFu) +
                          ((uint64_t)wave_inclusive_sum((uint32_t)(mine >> 16)) << 16);
    if (lane == 63) wave_sums[wave] = incl;
    __syncthreads();
    uint64_t before = carry, total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const uint64_t t = wave_sums[w];
      if (w < wave) before += t;
      total += t;
    }
    uint64_t run = before + incl - mine;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
      const uint32_t own = x[k];
      x[k] = run < 0x7FFFFFFFull ? (uint32_t)run : 0x7FFFFFFFu;
      run += own;
    }
    if (i0 + kScanPer <= end) {
#pragma unroll
      for (int k = 0; k < kScanPer; k += 4) *reinterpret_cast<vec4u*>(sums + i0 + k) = vec4u{x[k], x[k + 1], x[k + 2], x[k + 3]};
    } else {
#pragma unroll
      for (int k = 0; k < kScanPer; ++k)
        if (i0 + k < end) sums[i0 + k] = x[k];
    }
    carry += total;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    if (total_out && blockIdx.x == 0) *total_out = (int32_t)carry;
    if (diag_flags && carry > (uint64_t)limit) atomicOr(diag_flags, (uint32_t)DGC_DIAG_BAD_INDEX);
  }
}

// ---- decoder ----------------------------------------------------------------
// A wavefront takes kDecodeBlock consecutive entries, kDecodePer per lane.
struct Entries {
  uint32_t runs[kDecodePer / 2];  // two to a word
  float val[kDecodePer];
  int have;                       // entries of this lane that exist
  __device__ __forceinline__ uint32_t run(int k) const { return (runs[k >> 1] >> (16 * (k & 1))) & 0xFFFFu; }
};

// Entries e0 .. e0 + kDecodePer - 1 of a payload of `count`; VALUES = false: the runs only.
template <bool VALUES>
__device__ __forceinline__ void load_entries(Entries& E, const uint16_t* __restrict__ runs, const float* __restrict__ vals,
                                             int64_t count, int64_t e0) {
  typedef float vec4u __attribute__((ext_vector_type(4), aligned(4)));
  static_assert(kDecodePer == 8, "one 16-byte load of runs, two of values");
  const int64_t left = count - e0;
  E.have = left <= 0 ? 0 : left < kDecodePer ? (int)left : kDecodePer;
#pragma unroll
  for (int k = 0; k < kDecodePer / 2; ++k) E.runs[k] = 0u;
#pragma unroll
  for (int k = 0; k < kDecodePer; ++k) E.val[k] = 0.0f;
  if (E.have == kDecodePer && (reinterpret_cast<uintptr_t>(runs) & 15) == 0) {  // e0 is a multiple of eight
    const uint4 r = *reinterpret_cast<const uint4*>(runs + e0);
    E.runs[0] = r.x;
    E.runs[1] = r.y;
    E.runs[2] = r.z;
    E.runs[3] = r.w;
  } else {
#pragma unroll
    for (int k = 0; k < kDecodePer; ++k)
      if (k < E.have) E.runs[k >> 1] |= (uint32_t)runs[e0 + k] << (16 * (k & 1));
  }
  if (!VALUES) return;
  if (E.have == kDecodePer) {
    const vec4u a = *reinterpret_cast<const vec4u*>(vals + e0);
    const vec4u b = *reinterpret_cast<const vec4u*>(vals + e0 + 4);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      E.val[k] = a[k];
      E.val[4 + k] = b[k];
    }
  } else {
#pragma unroll
    for (int k = 0; k < kDecodePer; ++k)
      if (k < E.have) E.val[k] = vals[e0 + k];
  }
}

// Positions the lane's entries cover.
__device__ __forceinline__ uint32_t covered(const Entries& E) {
  uint32_t span = (uint32_t)E.have;
#pragma unroll
  for (int k = 0; k < kDecodePer; ++k) span += E.run(k);
  return span;
}

// Positions covered by every block of every payload.  grid = (blocks / wavefronts, payloads)
__global__ __launch_bounds__(kWireThreads) void decode_sums_kernel(DecodeArgs a) {
  const int lane = threadIdx.x & 63;
  const int w = blockIdx.y;
  const int block = (int)blockIdx.x * (kWireThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (block >= a.seg.begin[w + 1] - a.seg.begin[w]) return;
  uint32_t sum = 0;
  for (int sub = 0; sub < 1 << a.block_shift; ++sub) {
    Entries E;
    load_entries<false>(E, a.runs[w], nullptr, a.count[w],
                        (((int64_t)block << a.block_shift) + sub) * kDecodeBlock + lane * kDecodePer);
    sum += covered(E);
  }
  sum = wave_sum(sum);
  if (lane == 0) a.sums[a.seg.begin[w] + block] = sum;
}

// Direct form: dense[position] += value, entry by entry.  grid = (blocks / wavefronts, payloads)
// Bound by the rate of the scattered additions: about 20 G/s as atomics wherever they are carried out.
template <bool ATOMIC>
__global__ __launch_bounds__(kWireThreads) void decode_direct_kernel(DecodeArgs a, int32_t first) {
  const int lane = threadIdx.x & 63;
  const int w = first + blockIdx.y;
  const int block = (int)blockIdx.x * (kWireThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int32_t slot0 = a.seg.begin[w];
  if (block >= a.seg.begin[w + 1] - slot0) return;
  Entries E;
  int64_t e0 = ((int64_t)block << a.block_shift) * kDecodeBlock + lane * kDecodePer;
  load_entries<true>(E, a.runs[w], a.vals[w], a.count[w], e0);
  uint64_t pos;
  if (a.scanned) {
    pos = a.sums[slot0 + block];
  } else {  // few blocks: the wavefront adds up those before its own
    uint32_t before = 0;
    for (int i = lane; i < block; i += 64) before += a.sums[slot0 + i];
    // (a block covers up to 2^25 positions: the two halves are summed apart)
    pos = (uint64_t)wave_sum(before & 0xFFFFu) + ((uint64_t)wave_sum(before >> 16) << 16);
  }
  bool bad = false;
  for (int sub = 0;;) {
    const uint32_t span = covered(E);
    const uint32_t incl = wave_inclusive_sum(span);
    uint64_t at = pos + (incl - span);
#pragma unroll
    for (int k = 0; k < kDecodePer; ++k) {
      at += E.run(k);
      if (k < E.have) {
        if (at < (uint64_t)a.n) {
          if (ATOMIC) unsafeAtomicAdd(a.dense + at, E.val[k]);
          else a.dense[at] = a.dense[at] + E.val[k];
        } else {
          bad = true;
        }
        ++at;
      }
    }
    if (++sub >= 1 << a.block_shift) break;
    pos += wave_last(incl);
    e0 += kDecodeBlock;
    load_entries<true>(E, a.runs[w], a.vals[w], a.count[w], e0);
  }
  if (bad && a.diag_flags) atomicOr(a.diag_flags, (uint32_t)DGC_DIAG_BAD_INDEX);
}

// Direct form of short payloads in one launch: a workgroup takes kDecodeGroup consecutive entries of a payload, a
// wavefront kDecodeBlock of them, and adds up what all the entries before its own cover for itself (two bytes each,
// kDecodeGroupsMax - 1 loads of eight per thread at most, all on their way together).  25.6 M elements, 0.1 % of
// sixteen workers: 3.3 + 24.4 us in two launches, 25.2 in one; 1 M, four workers: 2.7 + 4.3 and 5.0.
__global__ __launch_bounds__(kDecodeGroupThreads) void decode_short_kernel(DecodeArgs a) {
  constexpr int kWaves = kDecodeGroupThreads / 64;
  __shared__ uint64_t before[kWaves];
  __shared__ uint32_t own[kWaves];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int w = blockIdx.y;
  const int64_t count = a.count[w];
  const int64_t begin = (int64_t)blockIdx.x * kDecodeGroup;
  if (begin >= count) return;
  const uint16_t* __restrict__ runs = a.runs[w];
  Entries E;
  load_entries<true>(E, runs, a.vals[w], count, begin + tid * kDecodePer);
  uint64_t sum = 0;
#pragma unroll
  for (int k = 0; k < kDecodeGroupsMax - 1; ++k) {
    if (k < (int)blockIdx.x) {  // uniform; whole groups: every entry exists
      Entries P;
      load_entries<false>(P, runs, nullptr, count, (int64_t)k * kDecodeGroup + tid * kDecodePer);
      sum += covered(P);
    }
  }
  // (below 2^23 per thread: the two halves are summed over the lanes apart, which cannot overflow 32 bits)
  const uint64_t all = (uint64_t)wave_sum((uint32_t)sum & 0xFFFFu) + ((uint64_t)wave_sum((uint32_t)(sum >> 16)) << 16);
  const uint32_t span = covered(E);
  const uint32_t incl = wave_inclusive_sum(span);  // a wavefront's entries cover up to 2^25 positions
  if (lane == 63) {
    before[wave] = all;
    own[wave] = incl;
  }
  __syncthreads();
  uint64_t at = incl - span;
#pragma unroll
  for (int v = 0; v < kWaves; ++v) {
    at += before[v];
    if (v < wave) at += own[v];
  }
  bool bad = false;
#pragma unroll
  for (int k = 0; k < kDecodePer; ++k) {
    at += E.run(k);
    if (k < E.have) {
      if (at < (uint64_t)a.n) unsafeAtomicAdd(a.dense + at, E.val[k]);
      else bad = true;
      ++at;
    }
  }
  if (bad && a.diag_flags) atomicOr(a.diag_flags, (uint32_t)DGC_DIAG_BAD_INDEX);
}

// Range form: a workgroup owns kDecodeRange elements of `dense`.  One wavefront per payload finds, by
// search among the positions the blocks start at, the blocks of entries that reach into the range; the
// wavefronts take these blocks in turn, kDecodeTasks each at a time so that their loads are one wait, and
// add the entries inside the range in LDS, payload after payload with a barrier between them (positions of
// one payload are distinct).
// PLAIN: the accumulator starts from `dense`, and the elements that have changed are stored: the ordered
// sum, bit for bit.  Otherwise it starts from nothing (-0, which an element that no entry names still is at
// the end) and every element that occurs is added to `dense` by one atomic: callers may add to one vector
// from several streams at a time.  In neither form is an element stored that no entry names: it may be
// another stream's to update.  (Whole ranges, stored as whole sectors: 132 instead of 152 us for 66 M
// elements, 6.25 % of four workers, 182 instead of 192 at 25 % of two; 25.6 M, 0.1 % of sixteen: 78 and 77.)
// The atomics are what that form costs: 64 neighbouring elements go as four 64-byte
// requests, 20 G of which complete per second, 195 us for 66 M elements whose every sector is
// touched where plain stores take 75.
// MULTI: a block is several kDecodeBlocks (streams so long that the block sums did not fit otherwise).
template <bool PLAIN, bool MULTI>
__global__ __launch_bounds__(kDecodeThreads) void decode_range_kernel(DecodeArgs a) {
  constexpr int kWaves = kDecodeThreads / 64;
  constexpr int kEach = kDecodeRange / kDecodeThreads;
  constexpr int kBatch = kWaves * kDecodeTasks;
  __shared__ alignas(16) float acc[kDecodeRange];
  __shared__ int32_t first_block[kMaxPayloads];
  __shared__ int32_t blocks[kMaxPayloads];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t begin = (int64_t)blockIdx.x * kDecodeRange;
  const int32_t length = a.n - begin < kDecodeRange ? (int32_t)(a.n - begin) : kDecodeRange;
  float* __restrict__ range = a.dense + begin;

  float d[kEach];  // what the accumulator starts from
#pragma unroll
  for (int i = 0; i < kEach; ++i) {
    const int e = tid + i * kDecodeThreads;
    d[i] = PLAIN && e < length ? range[e] : -0.0f;
  }
  for (int w = wave; w < a.num; w += kWaves) {
    const int32_t slot0 = a.seg.begin[w];
    int lo = 0, hi = 0;
    // the last block that starts at or before the range's first element, up to the last that starts inside
    wave_equal_range(reinterpret_cast<const int32_t*>(a.sums) + slot0, a.seg.begin[w + 1] - slot0, (int32_t)begin + 1,
                            (int32_t)(begin + length), lane, lo, hi);
    if (lane == 0) {
      first_block[w] = lo - 1;
      blocks[w] = hi > lo - 1 && hi > 0 ? hi - (lo - 1) : 0;
    }
  }
#pragma unroll
  for (int i = 0; i < kEach; ++i) acc[tid + i * kDecodeThreads] = d[i];
  __syncthreads();

  // adds a block whose first entry's predecessors cover `pos` positions; returns what the block covers
  auto add = [&](const Entries& E, uint32_t pos) {
    uint32_t rel = pos - (uint32_t)begin;  // (positions stay below 2^32: see scan_kernel)
    float sum[kDecodePer];
    uint32_t at[kDecodePer];
#pragma unroll
    for (int k = 0; k < kDecodePer; ++k) {
      rel += E.run(k);
      at[k] = k < E.have && rel < (uint32_t)length ? rel : 0xFFFFFFFFu;
      sum[k] = at[k] != 0xFFFFFFFFu ? acc[at[k]] + E.val[k] : 0.0f;
      ++rel;
    }
#pragma unroll
    for (int k = 0; k < kDecodePer; ++k)
      if (at[k] != 0xFFFFFFFFu) acc[at[k]] = sum[k];
  };

  if (MULTI) {
    for (int w = 0; w < a.num; ++w) {
      for (int b = wave; b < blocks[w]; b += kWaves) {
        const int32_t block = first_block[w] + b;
        uint32_t pos = a.sums[a.seg.begin[w] + block];
        for (int sub = 0; sub < 1 << a.block_shift; ++sub) {
          Entries E;
          load_entries<true>(E, a.runs[w], a.vals[w], a.count[w],
                             (((int64_t)block << a.block_shift) + sub) * kDecodeBlock + lane * kDecodePer);
          const uint32_t span = covered(E);
          const uint32_t incl = wave_inclusive_sum(span);
          add(E, pos + incl - span);
          pos += wave_last(incl);
        }
      }
      __syncthreads();
    }
  } else {
    // tasks: the blocks of all payloads, one payload after the other
    const uint32_t own = lane < a.num ? (uint32_t)blocks[lane] : 0u;
    const uint32_t incl = wave_inclusive_sum(own);
    const int total = (int)wave_last(incl);
    if (total == 0) return;
    const uint32_t task0 = lane < a.num ? incl - own : 0xFFFFFFFFu;  // lane w: first task of payload w
    const int32_t block0 = lane < a.num ? first_block[lane] : 0;
    auto payload_of_task = [&](int t) { return __popcll(__ballot(task0 <= (uint32_t)t)) - 1; };
    for (int t0 = 0; t0 < total; t0 += kBatch) {
      Entries E[kDecodeTasks];
      uint32_t pos[kDecodeTasks];
      int wk[kDecodeTasks];
#pragma unroll
      for (int k = 0; k < kDecodeTasks; ++k) {
        const int t = t0 + k * kWaves + wave;
        wk[k] = -1;
        E[k].have = 0;
        pos[k] = 0;
        if (t < total) {  // uniform
          const int w = payload_of_task(t);
          const int32_t block = __builtin_amdgcn_readlane(block0, w) + t - __builtin_amdgcn_readlane((int)task0, w);
          wk[k] = w;
          pos[k] = a.sums[a.seg.begin[w] + block];
          load_entries<true>(E[k], a.runs[w], a.vals[w], a.count[w], (int64_t)block * kDecodeBlock + lane * kDecodePer);
        }
      }
#pragma unroll
      for (int k = 0; k < kDecodeTasks; ++k) {
        if (wk[k] >= 0) {
          const uint32_t span = covered(E[k]);
          pos[k] += wave_inclusive_sum(span) - span;
        }
      }
      const int w_first = payload_of_task(t0);
      const int w_last = payload_of_task(t0 + kBatch < total ? t0 + kBatch - 1 : total - 1);
      for (int w = w_first; w <= w_last; ++w) {
#pragma unroll
        for (int k = 0; k < kDecodeTasks; ++k)
          if (wk[k] == w) add(E[k], pos[k]);
        __syncthreads();
      }
    }
  }

  int own = tid;
  asm volatile("" : "+v"(own));  // (addresses and bounds formed anew: kept from the loads on, they cost a workgroup per compute unit)
#pragma unroll
  for (int i = 0; i < kEach; ++i) {
    const int e = own + i * kDecodeThreads;
    const float s = acc[e];
    if (e < length && __float_as_uint(s) != __float_as_uint(d[i])) {
      if (PLAIN) range[e] = s;
      else unsafeAtomicAdd(range + e, s);
    }
  }
}

}  // namespace

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
hipError_t launch_encode(EncodeArgs a, hipStream_t stream) {
  ScanSegments seg{};
  seg.begin[1] = a.total_blocks;
  if (a.total_blocks <= 0) {  // nothing can have been emitted
    hipLaunchKernelGGL(scan_kernel, dim3(1), dim3(kScanThreads), 0, stream, a.sums, seg, a.num_entries, (int64_t)0,
                       (uint32_t*)nullptr);
    return hipGetLastError();
  }
  a.self_scan = a.total_blocks <= kWireSelfScan ? 1 : 0;
  const bool once = a.needs != nullptr;
  // As many workgroups for every tensor if few of them stay idle, so that none has to search for its tensor
  // (20000 tensors of 1500 elements: 60 us, where a search of three dependent rounds of loads took 15 more and
  // a walk over the tensors, 64 at a time, 1200 more).
  const int64_t even = (int64_t)a.widest * a.num_tensors;
  a.per_tensor = even <= 2 * (int64_t)a.total_blocks ? a.widest : 0;
  const dim3 grid((unsigned)(a.per_tensor > 0 ? even : a.total_blocks));
  if (once) {
    hipLaunchKernelGGL((encode_kernel<1, true>), grid, dim3(kWireThreads), 0, stream, a);
    return hipGetLastError();
  }
  hipLaunchKernelGGL((encode_kernel<0, false>), grid, dim3(kWireThreads), 0, stream, a);
  if (!a.self_scan)
    hipLaunchKernelGGL(scan_kernel, dim3(1), dim3(kScanThreads), 0, stream, a.sums, seg, a.num_entries, (int64_t)0,
                       (uint32_t*)nullptr);
  hipLaunchKernelGGL((encode_kernel<1, false>), grid, dim3(kWireThreads), 0, stream, a);
  return hipGetLastError();
}

// Which form (times in us).  The direct one costs its additions, 20 G/s as atomics; in order they are plain,
// 40 G/s, and every payload has a launch of its own.  The range form costs an atomic request per 64-byte
// sector of `dense` that occurs, or in order one pass over `dense` at 5 TB/s, and decodes every block once for
// every range that it reaches into, about 1500 blocks per us.  Whole calls, encoder included, direct against
// range as atomics: 66 M elements, 1 % of two workers 89 against 165, 6 % in all of four 229 against 157,
// 25 % in all 950 against 267; 25.6 M elements, 0.4 % of sixteen workers 99 against 108.  In order, 25.6 M
// elements, 0.1 % of sixteen workers: 384 with three launches per payload against 94.
static bool use_range_form(const DecodeArgs& a, bool in_order) {
  double entries = 0.0;
  for (int32_t w = 0; w < a.num; ++w) entries += (double)a.count[w];
  const double n = (double)a.n;
  const double decode = (entries / kDecodeBlock + (double)a.num * n / kDecodeRange) / 1500.0;
  if (in_order) return 10.0 + n * 8.0 / 5e6 + decode < 8.0 * a.num + entries / 40e3;
  return n / 16.0 * (1.0 - std::exp(-16.0 * entries / n)) / 20e3 + decode < entries / 20e3;
}

hipError_t launch_decode(DecodeArgs a, bool in_order, hipStream_t stream) {
  int32_t most = 0;  // blocks
  for (int32_t w = 0; w < a.num; ++w) most = a.seg.begin[w + 1] - a.seg.begin[w] > most ? a.seg.begin[w + 1] - a.seg.begin[w] : most;
  const unsigned groups = (unsigned)ceil_div(most, kWireThreads / 64);
  const bool range = use_range_form(a, in_order);
  int64_t longest = 0;
  for (int32_t w = 0; w < a.num; ++w) longest = a.count[w] > longest ? a.count[w] : longest;
  if (!range && !in_order && longest <= (int64_t)kDecodeGroup * kDecodeGroupsMax) {
    hipLaunchKernelGGL(decode_short_kernel, dim3((unsigned)ceil_div(longest, kDecodeGroup), (unsigned)a.num),
                       dim3(kDecodeGroupThreads), 0, stream, a);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(decode_sums_kernel, dim3(groups, (unsigned)a.num), dim3(kWireThreads), 0, stream, a);
  a.scanned = range || most > kDecodeSelfScan || a.block_shift > 0 ? 1 : 0;
  if (a.scanned)  // (the direct form sees for itself which entries lie behind the end)
    hipLaunchKernelGGL(scan_kernel, dim3((unsigned)a.num), dim3(kScanThreads), 0, stream, a.sums, a.seg, (int32_t*)nullptr,
                       a.n, range ? a.diag_flags : nullptr);
  if (range) {
    const dim3 grid((unsigned)ceil_div(a.n, kDecodeRange)), block(kDecodeThreads);
    if (in_order && a.block_shift == 0) hipLaunchKernelGGL((decode_range_kernel<true, false>), grid, block, 0, stream, a);
    else if (in_order) hipLaunchKernelGGL((decode_range_kernel<true, true>), grid, block, 0, stream, a);
    else if (a.block_shift == 0) hipLaunchKernelGGL((decode_range_kernel<false, false>), grid, block, 0, stream, a);
    else hipLaunchKernelGGL((decode_range_kernel<false, true>), grid, block, 0, stream, a);
  } else if (in_order) {
    for (int32_t w = 0; w < a.num; ++w) {  // inside a payload every position is distinct
      const unsigned own = (unsigned)ceil_div(a.seg.begin[w + 1] - a.seg.begin[w], kWireThreads / 64);
      if (own > 0) hipLaunchKernelGGL(decode_direct_kernel<false>, dim3(own), dim3(kWireThreads), 0, stream, a, w);
    }
  } else {
    hipLaunchKernelGGL(decode_direct_kernel<true>, dim3(groups, (unsigned)a.num), dim3(kWireThreads), 0, stream, a, 0);
  }
  return hipGetLastError();
}

}  // namespace dgc
