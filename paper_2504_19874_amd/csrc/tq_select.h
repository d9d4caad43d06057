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

// a value that at least k of the workgroup's scores reach (-inf where there are fewer), close to the k-th largest: the k-th
// largest of the threads' own maxima `mx` (-inf: none).  keys [256], bar: LDS.
__device__ __forceinline__ float kth_of_maxima(float mx, int k, uint32_t* keys, uint32_t* bar, int tid) {
  const uint32_t key = ordered(mx);
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
