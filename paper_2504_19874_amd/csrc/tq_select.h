// The k best of a workgroup's scores, shared by the top-k kernels.
#pragma once
#include "tq_internal.h"

namespace tq {

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
// eighth more (up to 8 for k < 8), of 256 maxima `mx` of T threads (-inf: none) reach, of 64 for k <= 16 (neighbouring threads' maxima joined; of 8192 scores
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
    if (k == 1) lo = hi - 1u, n = 1;  // the largest itself
    const int enough = k < 8 ? 8 : k + k / 8;
    while (n > enough && hi - lo > 1u) {
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

// more than this many are not ranked against each other as they are (two rows of 50001 equal scores, whole segments ranked:
// 144 ms)
constexpr int MANY = 512;

// a pair as an integer: larger ones come first.  Equal scores by index; zeros are equal, the sign of one in the lowest bit.
typedef unsigned long long pair;
__device__ __forceinline__ pair make_pair(float v, int i) {
  return (pair)ordered(v + 0.f) << 32 | (uint32_t)(0x7fffffff - i) << 1 | (v == 0.f ? __float_as_uint(v) >> 31 : 0u);
}
__device__ __forceinline__ int pair_index(pair p) { return 0x7fffffff - (int)((uint32_t)p >> 1); }
__device__ __forceinline__ float pair_score(pair p) {
  const float v = from_ordered((uint32_t)(p >> 32));
  return v == 0.f ? __uint_as_float((uint32_t)p << 31) : v;
}

// N scores per thread of T
template <int T, int N>
struct TopkLds {
  static constexpr int LIST = 64 + 64 * N * (T / 256) > MANY ? 64 + 64 * N * (T / 256) : MANY;  // the k best so far, and all that k groups of T / 256 threads hold
  pair list[LIST];
  pair best[64];
  pair groups[256];
  pair pair_bar;
  __attribute__((aligned(16))) uint32_t mx[256];
  uint32_t bar;
  int count;
};

// v[e]: this thread's scores of one segment, NaN where there is none; index_of(e): the e-th one's index.  kept: pairs in best so far
// (uniform).  Afterwards best holds the k best of all segments up to this one, and the number of them is returned.  few: so few scores in all
// that a bar costs more than it saves.
template <int T, int N, class Index>
__device__ int take_segment(TopkLds<T, N>& s, const float (&v)[N], Index index_of, int k, int kept, int tid, bool few = false) {
  constexpr int LIST = TopkLds<T, N>::LIST;
  float bar;
  if (tid == 0) s.count = kept;
  if (few) {  // uniform
    bar = -__builtin_inff();
    __syncthreads();
  } else if (kept < k) {
    float mx = -__builtin_inff();
#pragma unroll
    for (int e = 0; e < N; ++e) mx = fmaxf(mx, v[e]);  // ignores NaN
    bar = kth_of_maxima<T>(mx, k, s.mx, &s.bar, tid);
  } else {
    // the next larger value: an equal score of a later segment has a later index and does not beat a kept one
    bar = from_ordered((uint32_t)(s.best[k - 1] >> 32) + 1u);
    __syncthreads();
  }
  if (tid < kept) s.list[tid] = s.best[tid];
  // a wavefront's places are asked for together; most of its elements pass in no lane
  uint64_t pass[N];
  int passed = 0;
#pragma unroll
  for (int e = 0; e < N; ++e) {
    pass[e] = __builtin_amdgcn_ballot_w64(v[e] >= bar);
    passed += __builtin_popcountll(pass[e]);
  }
  if (passed != 0) {  // uniform
    int at = 0;
    if ((tid & 63) == 0) at = atomicAdd(&s.count, passed);
    at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
    for (int e = 0; e < N; ++e) {
      if (pass[e] == 0u) continue;
      const int pos = at + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(pass[e] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)pass[e], 0u));
      if (v[e] >= bar && pos < LIST) s.list[pos] = make_pair(v[e], index_of(e));
      at += __builtin_popcountll(pass[e]);
    }
  }
  __syncthreads();
  int n = s.count;
  if (n > MANY) {  // uniform
    pair key = 0;
#pragma unroll
    for (int e = 0; e < N; ++e)
      if (v[e] >= bar) {
        const pair o = make_pair(v[e], index_of(e));
        key = o > key ? o : key;
      }
    if (tid < 256) s.groups[tid] = 0;
    if (tid == 0) s.pair_bar = ~pair(0);
    __syncthreads();  // everyone has read the count, too
    atomicMax(&s.groups[tid / (T / 256)], key);
    if (tid == 0) s.count = kept;
    __syncthreads();
    if (tid < 256) {
      const pair own = s.groups[tid];
      int above = 0;
#pragma unroll 4
      for (int t = 0; t < 256; ++t) above += s.groups[t] > own ? 1 : 0;
      if (above < k) atomicMin(&s.pair_bar, own);
    }
    __syncthreads();
    const pair pair_bar = s.pair_bar;
    if (key >= pair_bar && key != 0)
#pragma unroll
      for (int e = 0; e < N; ++e)
        if (v[e] >= bar)
          if (const pair o = make_pair(v[e], index_of(e)); o >= pair_bar) s.list[atomicAdd(&s.count, 1)] = o;  // below LIST: at most k groups come here with any
    __syncthreads();
    n = s.count;
  }
  if (n == kept) return kept;  // uniform; nothing passed
  const int lanes = n * 16 <= T ? 16 : n * 8 <= T ? 8 : n * 4 <= T ? 4 : n * 2 <= T ? 2 : 1;  // that share a pair's comparisons
  for (int c = tid / lanes; c < n; c += T / lanes) {  // one round, or one lane each
    const pair own = s.list[c];
    int rank = 0;
#pragma unroll 4
    for (int o = tid & (lanes - 1); o < n; o += lanes) rank += s.list[o] > own ? 1 : 0;
    rank = sum_of_lanes(rank, lanes);
    if (rank < k) s.best[rank] = own;  // the lanes of a pair write the same
  }
  __syncthreads();
  return n < k ? n : k;
}

template <int T, int N>
__device__ __forceinline__ void write_best(const TopkLds<T, N>& s, int kept, int k, int none, int32_t* out_idx, float* out_val, int tid) {
  if (tid < k) {
    out_idx[tid] = tid < kept ? pair_index(s.best[tid]) : none;
    if (out_val != nullptr) out_val[tid] = tid < kept ? pair_score(s.best[tid]) : -__builtin_inff();
  }
}

}  // namespace tq
