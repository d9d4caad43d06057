// Per-query top-k over a row of scores (the "return top-10" step of the nearest-neighbour configurations).
// Order: larger score first, equal scores by lower index; a NaN is never taken.
//
// A workgroup of 256 to 1024 threads walks its part of a row in segments of 16 scores per thread, in registers, and keeps the k best pairs so
// far in LDS, as integers that compare like pairs.  The first segment has no bar yet: what k of 64 or 256 groups of threads' maxima reach is
// one (kth_of_maxima), and only scores that reach it, little more than k, are looked at again.  In later segments a score has to beat
// the k-th best pair, which a handful do.  The ones that pass go from the registers to a list (a place for all of a wavefront's is
// asked for once; elements that pass in no lane are a branch) and are ranked against it.  Where they are many (equal scores, a row that
// rises), the k-th best of the groups' best PAIRS is the bar instead: pairs are never equal, so at most k groups have any that
// reach it.  A few long rows (one query against a million codes) are cut into chunks, one workgroup each, whose lists topk_merge_kernel
// joins in the same way.
// What such a launch costs is a chain of latencies: us, before (256 threads with 32 scores each, maxima ranked against each other,
// what passes fetched again from memory) and now: 3 rows of 12279, k = 64, 17.3 -> 5.8; 4 of 12969, k = 10, 6.5 -> 4.7; 45 of 16000,
// k = 64, 29.2 -> 6.1; 5 of 30000, k = 16, 13.4 -> 7.0; 4 of 10^6, k = 10, with the joining 9.9 -> 9.2; 14 of 84645, k = 64, 22.2 -> 11.2.
#include "tq_select.h"

#include <algorithm>
#include <type_traits>

namespace tq {
namespace {

constexpr int PER = 16;  // scores of a segment per thread
constexpr int THREADS = 1024;                 // of a workgroup at most; a segment has 16384 scores then
constexpr int SEG = THREADS * PER;
// chunk_len > 0: workgroup (row, chunk) takes columns [c0, c0 + chunk_len) of the row (chunk_len is a multiple of
// 4, so a chunk is as aligned as the row) and writes k (value, index) pairs, -inf / INT_MAX where it has fewer
template <int T>
__global__ __launch_bounds__(T) void topk_kernel(const float* __restrict__ scores, const int64_t n_row, const int64_t ld, const int k,
                                                 const int vec4, int32_t* __restrict__ out_idx, float* __restrict__ out_val,
                                                 const int64_t chunk_len, const int32_t* __restrict__ flags) {
  if (flags != nullptr && flags[blockIdx.x] == 0) return;
  __shared__ TopkLds<T, PER> s;
  const int tid = threadIdx.x;
  const int64_t c0 = chunk_len > 0 ? (int64_t)blockIdx.y * chunk_len : 0;
  const int64_t n = chunk_len > 0 ? (n_row - c0 < chunk_len ? n_row - c0 : chunk_len) : n_row;
  const float* row = scores + (int64_t)blockIdx.x * ld + c0;
  const int64_t out_row = chunk_len > 0 ? (int64_t)blockIdx.x * gridDim.y + blockIdx.y : blockIdx.x;
  const float NONE = __builtin_nanf("");
  float v[PER];
  // element e of a thread: column 4 (tid + T (e / 4)) + e % 4 of the segment, tid + T e of one that is not whole
  int kept = 0;
  for (int64_t seg = 0; seg < n; seg += T * PER) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    const bool whole = vec4 && seg + T * PER <= n;  // uniform
    if (whole) {
#pragma unroll
      for (int u = 0; u < PER / 4; ++u) {
        const f32x4 w = *reinterpret_cast<const f32x4*>(row + seg + 4 * (tid + T * u));
#pragma unroll
        for (int e = 0; e < 4; ++e) v[4 * u + e] = w[e];
      }
    } else {
      const int left = (int)(n - seg < T * PER ? n - seg : T * PER);
      const float* const src = row + seg;
#pragma unroll
      for (int e = 0; e < PER; ++e) {
        const int c = tid + T * e;  // (a few scores meet as many threads)
        const float w = src[c < left ? c : left - 1];
        v[e] = c < left ? w : NONE;
      }
    }
    const int first = (int)(c0 + seg) + (whole ? 4 * tid : tid);
    kept = take_segment<T, PER>(s, v, [&](int e) { return first + T * (whole ? 4 * (e >> 2) : e) + (whole ? e & 3 : 0); }, k, kept, tid);
  }
  write_best(s, kept, k, chunk_len > 0 ? 0x7fffffff : -1, out_idx + out_row * k, out_val != nullptr ? out_val + out_row * k : nullptr, tid);
}

// One workgroup per row: the k best of its cands <= 4 T pairs of score and index (index INT_MAX: no pair).
// They are sorted lists of k one behind the other, so a thread takes its pairs from ever other places of the lists: the threads' maxima are
// then alike, and few pairs beside the k best reach the k-th largest of them.  (37 lists of 64, a thread's pairs all of one place: 81 us.)
template <int T>
__global__ __launch_bounds__(T) void topk_merge_kernel(const float* __restrict__ part_val, const int32_t* __restrict__ part_idx,
                                                       const int cands, const int k, int32_t* __restrict__ out_idx,
                                                       float* __restrict__ out_val, const int32_t* __restrict__ flags) {
  constexpr int N = 4;
  if (flags != nullptr && flags[blockIdx.x] == 0) return;
  __shared__ TopkLds<T, N> s;
  const int tid = threadIdx.x;
  const int64_t row = blockIdx.x;
  float v[N];
  int idx[N];
#pragma unroll
  for (int e = 0; e < N; ++e) {
    const int c = e * T + ((tid + 37 * e) & (T - 1)), cc = c < cands ? c : cands - 1;  // 256 + 37 and 1024 + 37 are primes: no k up to 64 divides them
    const float w = part_val[row * cands + cc];
    idx[e] = part_idx[row * cands + cc];
    v[e] = c < cands && idx[e] != 0x7fffffff ? w : __builtin_nanf("");
  }
  const int kept = take_segment<T, N>(s, v, [&](int e) { return idx[e]; }, k, 0, tid);
  write_best(s, kept, k, -1, out_idx + row * k, out_val != nullptr ? out_val + row * k : nullptr, tid);
}

}  // namespace

// Chunks per row when a call's rows are too few to fill the chip: 0 (one workgroup per row) unless the rows are
// few and longer than three segments (two and a half for k > 16); then chunks of equal lengths, a segment at most (down to 4096 scores in chunks of 256 threads: no
// faster), and no more pairs per row than the joining kernel takes (4096).  A workgroup takes 4.7 us (k = 10) or 6 (64) for a segment and 2 for every further one, its lists joined 4.3 to 6.  us, one workgroup per
// row / chunks + joining:
//   10 rows of 20000, k = 64   8.2 / 10.8
//   2 rows of 49000, k = 64   10.7 / 10.4;  60: 12.0 / 10.9;  2 of 33000 9.1 / 10.3
//   2 rows of 49000, k = 10    8.0 /  8.1;  60: 8.5 / 8.7
//   100 rows of 41500, k = 64 11.5 / 13.9 (what more rows than compute units for their chunks lose; 23.6 before)
//   2 rows of 56430, k = 10    9.6 /  8.4
//   14 rows of 84645, k = 64  18.1 / 11.2
// More segments than compute units: as many chunks as make two workgroups of 512 threads for each, all of them at work at once, so that a second
// segment costs its 2 us only.  us, chunks of a segment / so (a workgroup per row):
//   32 rows of 400000, k = 10  22.4 / 16.8 (42);  64 of 10^6 72.0 / 43.4 (91);  128 of 300000 47.4 / 29.5 (37)
//   32 rows of 10^6, k = 64    50.6 / 34.3 (132);  128 of 200000 44.3 / 31.1 (37);  8 of 10^6, k = 10 12.5 / 10.9 (80)
int topk_chunks(int64_t rows, int64_t n, int k) {
  if (k < 1 || rows < 1 || rows > 128 || n <= (k <= 16 ? 3 * SEG : 5 * SEG / 2)) return 0;
  int64_t c = (n + SEG - 1) / SEG;
  if (const int64_t cus = device_cu_count(); rows * c > cus) c = std::min(c, 2 * cus / rows);
  if (c > 4096 / k) c = 4096 / k;
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
  const int64_t chunk_len = chunks > 0 ? ((n + chunks - 1) / chunks + 3) / 4 * 4 : 0;
  const dim3 grid((unsigned)rows, chunks > 0 ? (unsigned)chunks : 1u);
  if (chunks > 0) {
    out_idx = part_idx;
    out_val = part_val;
  }
  // As many threads as a row's first segment needs, but more rows at a time where there are more than the chip takes of the largest
  // workgroups (us, 256 / 512 / 1024 threads: 1000 rows of 9766, k = 10, 10.9 / 12.7 / 17.0; 871 of 16000, k = 64, 23.1 / 19.9 / 23.3;
  // 45 of 16000, k = 64, 17.0 / 9.5 / 6.1)
  const bool crowd = rows > 2 * (int64_t)device_cu_count();
  const int64_t len = chunks > 0 ? chunk_len : n;
  auto go = [&](auto t_c) {
    constexpr int T = decltype(t_c)::value;
    hipLaunchKernelGGL((topk_kernel<T>), grid, dim3(T), 0, stream, scores, n, ld, k, vec4, out_idx, out_val, chunk_len, flags);
    return hipGetLastError();
  };
  if (len <= 256 * PER || (crowd && k <= 16)) return go(std::integral_constant<int, 256>{});
  if (len <= 512 * PER || crowd || (chunks > 0 && rows * chunks > device_cu_count())) return go(std::integral_constant<int, 512>{});
  return go(std::integral_constant<int, THREADS>{});
}

hipError_t launch_topk_merge(const float* part_val, const int32_t* part_idx, int64_t rows, int ranges, int k,
                             int32_t* out_idx, float* out_val, hipStream_t s, const int32_t* flags) {
  if (rows == 0) return hipSuccess;
  if (ranges < 1 || k < 1 || k > 64 || (int64_t)ranges * k > 4096 || rows > 0x7fffffff) return hipErrorInvalidValue;
  auto go = [&](auto t_c) {
    constexpr int T = decltype(t_c)::value;
    hipLaunchKernelGGL((topk_merge_kernel<T>), dim3((unsigned)rows), dim3(T), 0, s, part_val, part_idx, ranges * k, k, out_idx, out_val, flags);
    return hipGetLastError();
  };
  return ranges * k <= 1024 ? go(std::integral_constant<int, 256>{}) : go(std::integral_constant<int, 1024>{});
}

}  // namespace tq
