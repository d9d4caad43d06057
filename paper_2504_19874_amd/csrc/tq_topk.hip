// Per-query top-k over a row of scores (the "return top-10" step of the nearest-neighbour configurations).
// Order: larger score first, equal scores by lower index; a NaN is never taken.
//
// A workgroup walks its part of a row in segments of 8192 scores, 32 per thread in registers, and keeps the k best pairs so
// far in LDS.  The first segment has no bar yet: the k-th largest of the 256 threads' own maxima is one (k threads hold a
// score that high), found by ranking the maxima against each other, and only scores that reach it, little more than k, are
// looked at again.  In later segments a score has to beat the k-th best pair, which a handful do.  The ones that pass are
// appended to a list and ranked against it.  Where they are many (equal scores, a row that rises), the k-th best of the
// threads' best PAIRS is the bar instead: pairs are never equal, so at most k threads have any that reach it.  A few long rows
// (one query against a million codes) are cut into chunks, one workgroup each, whose lists topk_merge_kernel joins in the same way.
// (Before: a sorted list per thread, k rounds of arg-max to join them.  4 rows of 10^6 scores, k = 10: 35 + 30 us for the
// chunks and the merge, 6.7 + 5.0 here; 2 rows of 300000, k = 64: 11.9 + 12.1.)
// What such a launch costs is a chain of latencies, so the comparisons are shared out: those of a few pairs over up to sixteen lanes each, those
// of the maxima over four (4 rows as above: 11.3 + 9.0 without).
#include "tq_select.h"

#include <type_traits>

namespace tq {
namespace {

constexpr int SEG = 8192;              // scores per segment
constexpr int PER = SEG / 256;         // per thread
constexpr int LIST = 64 + 64 * PER;    // the k best so far, and all that k threads hold
// more than this many are not ranked against each other as they are (two rows of 50001 equal scores, whole segments ranked:
// 144 ms; 54 us as it is, 39 for scores that differ, 163 for rising ones)
constexpr int MANY = 512;

struct TopkLds {
  float v[LIST];
  int i[LIST];
  float best_v[64];
  int best_i[64];
  uint32_t mx[256];
  uint32_t bar;
  int count;
  unsigned long long pair_bar;
  unsigned long long pairs[256];
};

// pairs in the order of better() as unsigned integers; 0 is below every one of them
__device__ __forceinline__ unsigned long long pair_key(float v, int i) {
  return (unsigned long long)ordered(v + 0.f) << 32 | (uint32_t)~i;  // + 0: a negative zero is equal to a positive one
}

// v[e]: this thread's scores of one segment, NaN where there is none; pair(e) fetches score and index of the e-th again (a
// handful are asked for, and a register array cannot be indexed).  kept: pairs in best so far (uniform).  Afterwards best
// holds the k best of all segments up to this one, and the number of them is returned.
// (Straight code for 32 elements would be 12 KB of instructions that a 10 us kernel has to fetch first: it is kept short.)
template <int N, class Pair>
__device__ int take_segment(TopkLds& s, const float (&v)[N], Pair pair, int k, int kept, int tid) {
  float bar;
  if (kept < k) {
    float mx = -__builtin_inff();
#pragma unroll
    for (int e = 0; e < N; ++e) mx = fmaxf(mx, v[e]);  // ignores NaN
    bar = kth_of_maxima(mx, k, s.mx, &s.bar, tid);
  } else {
    // the next larger value: an equal score of a later segment has a later index and does not beat a kept one
    bar = from_ordered(ordered(s.best_v[k - 1] + 0.f) + 1u);  // + 0: see pair_key
  }
  if (tid < kept) {
    s.v[tid] = s.best_v[tid];
    s.i[tid] = s.best_i[tid];
  }
  if (tid == 0) s.count = kept;
  __syncthreads();
  uint32_t pass = 0u;
#pragma unroll
  for (int e = N - 1; e >= 0; --e) pass = pass + pass + (v[e] >= bar ? 1u : 0u);
  if (pass != 0u) {
    int pos = atomicAdd(&s.count, __builtin_popcount(pass));
    for (uint32_t left = pass; left != 0u; left &= left - 1u, ++pos)
      if (pos < LIST) pair(__builtin_ctz(left), s.v[pos], s.i[pos]);
  }
  __syncthreads();
  int n = s.count;
  if (n > MANY) {  // uniform
    unsigned long long key = 0;
    for (uint32_t left = pass; left != 0u; left &= left - 1u) {
      float pv;
      int pi;
      pair(__builtin_ctz(left), pv, pi);
      const unsigned long long o = pair_key(pv, pi);
      key = o > key ? o : key;
    }
    s.pairs[tid] = key;
    if (tid == 0) s.pair_bar = ~0ull;
    __syncthreads();  // everyone has read the count, too
    int above = 0;
#pragma unroll 4
    for (int t = 0; t < 256; ++t) above += s.pairs[t] > key ? 1 : 0;
    if (above < k) atomicMin(&s.pair_bar, key);
    if (tid == 0) s.count = kept;
    __syncthreads();
    const unsigned long long pair_bar = s.pair_bar;
    if (key >= pair_bar)
      for (uint32_t left = pass; left != 0u; left &= left - 1u) {
        float pv;
        int pi;
        pair(__builtin_ctz(left), pv, pi);
        if (pair_key(pv, pi) >= pair_bar) {
          const int pos = atomicAdd(&s.count, 1);  // below LIST: at most k threads come here with any
          s.v[pos] = pv;
          s.i[pos] = pi;
        }
      }
    __syncthreads();
    n = s.count;
  }
  if (n == kept) return kept;  // uniform; nothing passed
  const int lanes = n <= 16 ? 16 : n <= 32 ? 8 : n <= 64 ? 4 : n <= 128 ? 2 : 1;  // that share a pair's comparisons
  for (int c = tid / lanes; c < n; c += 256) {  // one round, or one lane each
    const float cv = s.v[c];
    const int ci = s.i[c];
    int rank = 0;
#pragma unroll 8
    for (int o = tid & (lanes - 1); o < n; o += lanes) rank += better(s.v[o], s.i[o], cv, ci) ? 1 : 0;
    rank = sum_of_lanes(rank, lanes);
    if (rank < k) {  // the lanes of a pair write the same
      s.best_v[rank] = cv;
      s.best_i[rank] = ci;
    }
  }
  __syncthreads();
  return n < k ? n : k;
}

__device__ __forceinline__ void write_best(const TopkLds& s, int kept, int k, int none, int32_t* out_idx, float* out_val, int tid) {
  if (tid < k) {
    out_idx[tid] = tid < kept ? s.best_i[tid] : none;
    if (out_val != nullptr) out_val[tid] = tid < kept ? s.best_v[tid] : -__builtin_inff();
  }
}

// chunk_len > 0: workgroup (row, chunk) takes columns [c0, c0 + chunk_len) of the row (chunk_len is a multiple of
// 4, so a chunk is as aligned as the row) and writes k (value, index) pairs, -inf / INT_MAX where it has fewer
__global__ __launch_bounds__(256) void topk_kernel(const float* __restrict__ scores, const int64_t n_row, const int64_t ld, const int k,
                                                   const int vec4, int32_t* __restrict__ out_idx, float* __restrict__ out_val,
                                                   const int64_t chunk_len, const int32_t* __restrict__ flags) {
  if (flags != nullptr && flags[blockIdx.x] == 0) return;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  TopkLds& s = *reinterpret_cast<TopkLds*>(smem_raw);
  const int tid = threadIdx.x;
  const int64_t c0 = chunk_len > 0 ? (int64_t)blockIdx.y * chunk_len : 0;
  const int64_t n = chunk_len > 0 ? (n_row - c0 < chunk_len ? n_row - c0 : chunk_len) : n_row;
  const float* row = scores + (int64_t)blockIdx.x * ld + c0;
  const int64_t out_row = chunk_len > 0 ? (int64_t)blockIdx.x * gridDim.y + blockIdx.y : blockIdx.x;
  const float NONE = __builtin_nanf("");
  float v[PER];
  // element e of a thread: column 4 (tid + 256 (e / 4)) + e % 4 of the segment
  int kept = 0;
  for (int64_t seg = 0; seg < n; seg += SEG) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    if (vec4 && seg + SEG <= n) {  // uniform: all loads in flight together
#pragma unroll
      for (int u = 0; u < PER / 4; ++u) {
        const f32x4 w = *reinterpret_cast<const f32x4*>(row + seg + 4 * (tid + 256 * u));
#pragma unroll
        for (int e = 0; e < 4; ++e) v[4 * u + e] = w[e];
      }
    } else {
      const int left = (int)(n - seg < SEG ? n - seg : SEG);
      const float* const src = row + seg;
#pragma unroll
      for (int e = 0; e < PER; ++e) {
        const int c = 4 * (tid + 256 * (e >> 2)) + (e & 3);
        const float w = src[c < left ? c : left - 1];
        v[e] = c < left ? w : NONE;
      }
    }
    kept = take_segment(s, v, [&](int e, float& pv, int& pi) {
      const int64_t c = seg + 4 * (tid + 256 * (e >> 2)) + (e & 3);
      pv = row[c];
      pi = (int)(c0 + c);
    }, k, kept, tid);
  }
  write_best(s, kept, k, chunk_len > 0 ? 0x7fffffff : -1, out_idx + out_row * k, out_val != nullptr ? out_val + out_row * k : nullptr, tid);
}

// One workgroup per row: the k best of its cands <= 256 N pairs of score and index (index INT_MAX: no pair).
// They are sorted lists of k one behind the other, so a thread takes its pairs from ever other places of the lists: the threads' maxima are
// then alike, and few pairs beside the k best reach the k-th largest of them.  (37 lists of 64, a thread's pairs all of one place: 81 us.)
template <int N>
__global__ __launch_bounds__(256) void topk_merge_kernel(const float* __restrict__ part_val, const int32_t* __restrict__ part_idx,
                                                         const int cands, const int k, int32_t* __restrict__ out_idx,
                                                         float* __restrict__ out_val, const int32_t* __restrict__ flags) {
  if (flags != nullptr && flags[blockIdx.x] == 0) return;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  TopkLds& s = *reinterpret_cast<TopkLds*>(smem_raw);
  const int tid = threadIdx.x;
  const int64_t row = blockIdx.x;
  float v[N];
  auto place = [&](int e) { return e * 256 + ((tid + 37 * e) & 255); };  // 256 + 37 = 293, a prime: no k up to 64 divides it
#pragma unroll
  for (int e = 0; e < N; ++e) {
    const int c = place(e), cc = c < cands ? c : cands - 1;
    const float w = part_val[row * cands + cc];
    v[e] = c < cands && part_idx[row * cands + cc] != 0x7fffffff ? w : __builtin_nanf("");
  }
  const int kept = take_segment(s, v, [&](int e, float& pv, int& pi) {
    pv = part_val[row * cands + place(e)];
    pi = part_idx[row * cands + place(e)];
  }, k, 0, tid);
  write_best(s, kept, k, -1, out_idx + row * k, out_val != nullptr ? out_val + row * k : nullptr, tid);
}

}  // namespace

// Chunks per row when a call's rows are too few to fill the chip: 0 (one workgroup per row) unless the rows are
// few and longer than two segments; then chunks of a segment or more, about four workgroups per compute unit in all, and no more
// pairs per row than the joining kernel takes (4096).  A segment exactly where there could be more: cut into 122 parts, a row of
// 10^6 is a segment and eight columns each, two passes (4 rows, k = 10: 13.6 -> 10.8 us).  A workgroup takes 3 - 5 us per segment,
// more for k = 64, the joining 4.5 - 8.  us, one workgroup per row / chunks + joining:
//   1 row of 50000, k = 10    23.3 / 4.5 + 4.4
//   5 rows of 30000, k = 16   20.2 / 6.9 + 7.1
//   10 rows of 20000, k = 64  37.3 / 12.1 + 8.5
int topk_chunks(int64_t rows, int64_t n, int k) {
  if (k < 1 || rows < 1 || rows > 128 || n <= 2 * SEG) return 0;
  int64_t c = (4 * (int64_t)device_cu_count() + rows - 1) / rows;
  if (c > (n + SEG - 1) / SEG) c = (n + SEG - 1) / SEG;
  if (c > 4096 / k) c = 4096 / k;
  if (c > 65535) c = 65535;
  return c >= 2 ? (int)c : 0;
}

// chunks == 0: the rows' k best straight to out_idx / out_val.  chunks > 0 (from topk_chunks): the k best of every
// chunk to part_idx / part_val [rows][chunks][k], to be joined by launch_topk_merge.
hipError_t launch_topk(const float* scores, int64_t rows, int64_t n, int64_t ld, int k,
                       int32_t* out_idx, float* out_val, hipStream_t stream, int chunks, float* part_val,
                       int32_t* part_idx, const int32_t* flags) {
  if (rows == 0 || k == 0) return hipSuccess;
  if (k < 1 || k > 64 || rows > 0x7fffffff || n > 0x7fffffff) return hipErrorInvalidValue;
  if (chunks > 0 && (part_val == nullptr || part_idx == nullptr || chunks > 65535)) return hipErrorInvalidValue;
  const int vec4 = (ld % 4 == 0) && ((reinterpret_cast<uintptr_t>(scores) & 15u) == 0);
  int64_t chunk_len = chunks > 0 ? ((n + chunks - 1) / chunks + 3) / 4 * 4 : 0;
  if (chunks == (n + SEG - 1) / SEG) chunk_len = SEG;
  const dim3 grid((unsigned)rows, chunks > 0 ? (unsigned)chunks : 1u);
  if (chunks > 0) {
    out_idx = part_idx;
    out_val = part_val;
  }
  static LdsLimit lds_limit;
  if (const hipError_t e = raise_lds_limit(lds_limit, reinterpret_cast<const void*>(&topk_kernel), (int)sizeof(TopkLds)); e != hipSuccess) return e;
  hipLaunchKernelGGL(topk_kernel, grid, dim3(256), sizeof(TopkLds), stream, scores, n, ld, k, vec4, out_idx, out_val, chunk_len, flags);
  return hipGetLastError();
}

hipError_t launch_topk_merge(const float* part_val, const int32_t* part_idx, int64_t rows, int ranges, int k,
                             int32_t* out_idx, float* out_val, hipStream_t s, const int32_t* flags) {
  if (rows == 0) return hipSuccess;
  if (ranges < 1 || k < 1 || k > 64 || (int64_t)ranges * k > 4096 || rows > 0x7fffffff) return hipErrorInvalidValue;
  auto go = [&](auto n_c) {
    constexpr int N = decltype(n_c)::value;
    static LdsLimit lds_limit;
    if (const hipError_t e = raise_lds_limit(lds_limit, reinterpret_cast<const void*>(&topk_merge_kernel<N>), (int)sizeof(TopkLds)); e != hipSuccess) return e;
    hipLaunchKernelGGL((topk_merge_kernel<N>), dim3((unsigned)rows), dim3(256), sizeof(TopkLds), s, part_val, part_idx, ranges * k, k, out_idx, out_val, flags);
    return hipGetLastError();
  };
  if (ranges * k <= 1024) return go(std::integral_constant<int, 4>{});
  if (ranges * k <= 2048) return go(std::integral_constant<int, 8>{});
  return go(std::integral_constant<int, 16>{});
}

}  // namespace tq
