// The k best of a workgroup's scores, shared by the top-k kernels.
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

// a value that at least k of the workgroup's scores reach (-inf where there are fewer), close to the k-th largest: one that k, or an
// eighth more, of 256 maxima `mx` of T threads (-inf: none) reach, of 64 for k <= 16 (neighbouring threads' maxima joined; of 8192 scores
// 10.9 are expected to reach the 10th largest of 64, 10.2 that of 256).  keys [256], bar: LDS.  A wavefront halves the range between the
// smallest and the largest of them, some five steps of a comparison or four and as many counts.  (Ranked against each other in
// place of this: 600 instructions per wavefront for k > 16.)
template <int T>
__device__ __forceinline__ float kth_of_maxima(float mx, int k, uint32_t* keys, uint32_t* bar, int tid) {
  const auto larger = [](uint32_t x, uint32_t y) { return x > y ? x : y; };
  const auto smaller = [](uint32_t x, uint32_t y) { return x < y ? x : y; };
  uint32_t key = ordered(mx);
  const int lanes = k <= 16 ? T / 64 : T / 256;  // uniform
  if (lanes >= 2) key = larger(key, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)key, 0xB1, 0xf, 0xf, true));
  if (lanes >= 4) key = larger(key, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)key, 0x4E, 0xf, 0xf, true));
  if (lanes >= 8) key = larger(key, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)key, 0x141, 0xf, 0xf, true));
  if (lanes >= 16) key = larger(key, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)key, 0x140, 0xf, 0xf, true));
  if ((tid & (lanes - 1)) == 0) keys[tid / lanes] = key;
  __syncthreads();
  if (tid < 64) {
    constexpr uint32_t NONE = 0x007fffffu;  // ordered(-inf)
    uint4 v = k <= 16 ? make_uint4(keys[tid], NONE, NONE, NONE) : reinterpret_cast<const uint4*>(keys)[tid];
    const auto count = [&](uint32_t at) {
      const auto lanes_of = [](bool b) { return __builtin_popcountll(__builtin_amdgcn_ballot_w64(b)); };
      const int n = lanes_of(v.x >= at);
      return k <= 16 ? n : (n + lanes_of(v.y >= at)) + (lanes_of(v.z >= at) + lanes_of(v.w >= at));
    };
    // (threads without a score aside: their part of the range would be halved away in some ten steps)
    const auto some = [](uint32_t x) { return x > NONE ? x : 0xffffffffu; };
    uint32_t lo = over_wavefront(k <= 16 ? some(v.x) : smaller(smaller(some(v.x), some(v.y)), smaller(some(v.z), some(v.w))), smaller);
    uint32_t hi = over_wavefront(k <= 16 ? v.x : larger(larger(v.x, v.y), larger(v.z, v.w)), larger);
    lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)lo);
    hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)hi) + 1u;  // none reaches it (no score is as large as the largest integer)
    int n = lo < hi ? count(lo) : 0;  // that reach lo
    if (n < k) lo = NONE;
    while (n > k + k / 8 && hi - lo > 1u) {
      const uint32_t mid = lo + (hi - lo) / 2u;
      const int m = count(mid);
      if (m >= k) lo = mid, n = m;
      else hi = mid;
    }
    if (tid == 0) *bar = lo;
  }
  __syncthreads();
  return from_ordered(*bar);
}

}  // namespace tq
