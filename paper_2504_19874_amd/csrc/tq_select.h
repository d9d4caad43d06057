// The k best of a workgroup's scores, shared by the top-k kernels (256 threads).
#pragma once
#include "tq_internal.h"

namespace tq {

__device__ __forceinline__ bool better(float va, int ia, float vb, int ib) {
  return va > vb || (va == vb && ia < ib);
}

// order-preserving map to the unsigned integers
__device__ __forceinline__ uint32_t ordered(float f) {
  const uint32_t b = __float_as_uint(f);
  return b & 0x80000000u ? ~b : b | 0x80000000u;
}
__device__ __forceinline__ float from_ordered(uint32_t b) { return __uint_as_float(b & 0x80000000u ? b & 0x7fffffffu : ~b); }

// the sum over groups of `lanes` (1, 2, 4, 8 or 16, uniform) neighbouring lanes, in every one of them; mirrored lanes hold the same
__device__ __forceinline__ int sum_of_lanes(int v, int lanes) {
  if (lanes >= 2) v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xf, 0xf, true);    // lane ^ 1
  if (lanes >= 4) v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xf, 0xf, true);    // lane ^ 2
  if (lanes >= 8) v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xf, 0xf, true);   // lane ^ 7
  if (lanes >= 16) v += __builtin_amdgcn_update_dpp(0, v, 0x140, 0xf, 0xf, true);  // lane ^ 15
  return v;
}

// a value that at least k of the workgroup's scores reach (-inf where there are fewer), close to the k-th largest: the k-th
// largest of the threads' own maxima `mx` (-inf: none).  keys [256], bar: LDS.
__device__ __forceinline__ float kth_of_maxima(float mx, int k, uint32_t* keys, uint32_t* bar, int tid) {
  uint32_t key = ordered(mx);
  if (k <= 16) {
    // of the 64 maxima of four threads: a sixteenth of the comparisons, and of 8192 scores 10.9 are expected to reach the bar for k = 10
    // and 18.4 for k = 16 (10.2 and 16.5 with a thread's own maxima)
    uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)key, 0xB1, 0xf, 0xf, true);
    key = o > key ? o : key;
    o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)key, 0x4E, 0xf, 0xf, true);
    key = o > key ? o : key;
    if ((tid & 3) == 0) keys[tid >> 2] = key;
    if (tid == 0) *bar = 0xffffffffu;
    __syncthreads();
    int above = 0;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const uint4 v = reinterpret_cast<const uint4*>(keys)[4 * (tid & 3) + t];
      above += (v.x > key ? 1 : 0) + (v.y > key ? 1 : 0) + (v.z > key ? 1 : 0) + (v.w > key ? 1 : 0);
    }
    above = sum_of_lanes(above, 4);
    if ((tid & 3) == 0 && above < k) atomicMin(bar, key);
    __syncthreads();
    return from_ordered(*bar);
  }
  keys[tid] = key;
  if (tid == 0) *bar = 0xffffffffu;
  __syncthreads();
  int above = 0;
  const uint4* m4 = reinterpret_cast<const uint4*>(keys);
#pragma unroll 8
  for (int t = 0; t < 64; ++t) {
    const uint4 o = m4[t];
    above += (o.x > key ? 1 : 0) + (o.y > key ? 1 : 0) + (o.z > key ? 1 : 0) + (o.w > key ? 1 : 0);
  }
  if (above < k) atomicMin(bar, key);  // the smallest of the k largest
  __syncthreads();
  return from_ordered(*bar);
}

}  // namespace tq
