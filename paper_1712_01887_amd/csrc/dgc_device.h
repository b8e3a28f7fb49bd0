// Device code shared by the kernels: wavefront scans, searches and exchange through LDS.
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

// In lane 0 the sum over the wavefront, every lane's value added to that of the lane half as far away as there are lanes
// left (32, 16, 8, 4, 2, 1).  Halves and rows change places in one instruction, the rest are shifts inside a row.
__device__ __forceinline__ double wave_sum_down(double x) {
  auto add = [&](auto move) {
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    const uint64_t o = (uint64_t)(uint32_t)move((int)(uint32_t)b) | (uint64_t)(uint32_t)move((int)(uint32_t)(b >> 32)) << 32;
    x += __longlong_as_double((long long)o);
  };
  add([](int v) { return (int)__builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false)[1]; });
  add([](int v) { return (int)__builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false)[1]; });
  add([](int v) { return __builtin_amdgcn_update_dpp(0, v, 0x108, 0xf, 0xf, false); });  // row_shl:8
  add([](int v) { return __builtin_amdgcn_update_dpp(0, v, 0x104, 0xf, 0xf, false); });
  add([](int v) { return __builtin_amdgcn_update_dpp(0, v, 0x102, 0xf, 0xf, false); });
  add([](int v) { return __builtin_amdgcn_update_dpp(0, v, 0x101, 0xf, 0xf, false); });
  return x;
}

// A pointer to global memory that the compiler cannot tell to be one, because it comes from LDS or was put together
// from registers.  Through a generic pointer every load is a FLAT one, which counts as an LDS operation, too: the next
// wait for LDS then waits for all such loads that are on their way.
template <typename T>
using global_ptr = const __attribute__((address_space(1))) T*;
template <typename T>
__device__ __forceinline__ global_ptr<T> in_global(const T* p) {
  return (global_ptr<T>)p;
}

// How often a workgroup looks for word `c` of those that other workgroups leave.  (Less than zero, which only tests ask for:
// as often for the even ones, and not at all for the odd ones.)
__device__ __forceinline__ int looks_for(int looks, int c) { return looks >= 0 ? looks : (c & 1) ? 0 : -looks; }

// Between stores to LDS by some lanes of a wavefront and loads of them by others.  The hardware carries out a
// wavefront's LDS operations in order; this keeps the compiler from moving them, and costs no instruction.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// Positions [lo, hi) of the list L[0, m) whose values lie in [xa, xb), for a list in which
// "value < xa" and "value < xb" are monotone; every lane of the wavefront takes part and
// gets the same answer.
__device__ __forceinline__ void wave_equal_range(const int32_t* __restrict__ L, int m, int32_t xa, int32_t xb,
                                                 int lane, int& out_lo, int& out_hi) {
  const int half = lane >> 5;  // 0: lower bound of xa, 1: lower bound of xb
  const int sub = lane & 31;
  const int32_t x = half ? xb : xa;
  int lo = 0, hi = m;  // the answer of this lane's half lies in [lo, hi]
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
