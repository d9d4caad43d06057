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
// what passes fetched again from memory) and now: 3 rows of 12279, k = 64, 18.1 -> 6.0; 4 of 12969, k = 10, 6.8 -> 4.9; 45 of 16000,
// k = 64, 27.9 -> 6.2; 5 of 30000, k = 16, 13.2 -> 6.8; 4 of 10^6, k = 10, with the joining 9.9 -> 8.9; 14 of 84645, k = 64, 20.4 -> 10.8.
#include "tq_select.h"

#include <algorithm>
#include <type_traits>

namespace tq {
namespace {

constexpr int PER = 16;  // scores of a segment per thread
constexpr int THREADS = 1024;                 // of a workgroup at most; a segment has 16384 scores then
constexpr int SEG = THREADS * PER;
// Workgroups that a compute unit holds: left alone, the kernel takes 65 to 69 registers, seven wavefronts on a SIMD.  For two workgroups of 1024, or four of
// 512, the compiler is held to 64 (512 rows of 100000, k = 64: 47.5 -> 38.3 us); where fewer are at work that is 2 - 6 % slower.
constexpr int CU_256 = 7, CU_512 = 3, CU_1024 = 2;
// chunk_len > 0: workgroup (row, chunk) takes columns [c0, c0 + chunk_len) of the row (chunk_len is a multiple of
// 4, so a chunk is as aligned as the row) and writes k (value, index) pairs, -inf / INT_MAX where it has fewer
template <int T, int PER_CU>
__global__ __launch_bounds__(T, T / 256 * PER_CU) void topk_kernel(const float* __restrict__ scores, const int64_t n_row, const int64_t ld, const int k,
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

// Chunks per row when a call's rows are too few to fill the chip: 0 (one workgroup per row) unless the rows are few and longer than three
// segments of 1024 threads, two and a half for k > 16 (us, one workgroup per row / chunks: 128 rows of 41000, k = 10, 8.6 / 10.1; 128 of 49200 10.2 / 9.7; 100
// of 41000, k = 64, 12.6 / 12.8; 128 of 60000 15.6 / 13.5).  Then, while all of them are at work at once,
//   a segment of 1024 threads each, one workgroup to a compute unit   43 rows of 60000, k = 16, 8.7 (of 512 threads 9.4)
//   k <= 16: a segment of 512 threads each                            43 rows of 131072, k = 10, 8.8 (of 1024 9.1); 5 of 10^6 9.7 (10.0)
//   a segment of 1024 threads each, two to a compute unit             64 rows of 131072, k = 10, 9.9; 64 of 100000, k = 64, 13.2
//   the same by 512 threads in two steps                              65 rows of 131072, k = 10, 11.5; 86 13.9
// and beyond, two workgroups of 512 threads to a compute unit with as many segments as it takes (33 rows of 10^6, k = 10, 27.6; three of them 28.7).
// With segments of 1024 threads and then two workgroups of 512, whatever the row: 10.2, 10.9, 10.9 / 15.2, 13.4, 16.4; with 256 threads of 32 scores and
// up to four chunks to a compute unit, before that: 9.0, 10.2, 9.9 / 24.9, 11.6, 20.3, 35.3.  No more pairs per row than the joining kernel takes (4096).
int topk_chunks(int64_t rows, int64_t n, int k) {
  if (k < 1 || rows < 1 || rows > 128 || n <= (k <= 16 ? 3 * SEG : 5 * SEG / 2)) return 0;
  const int64_t cus = device_cu_count(), most = 4096 / k;
  auto of = [&](int64_t len) { return (n + len - 1) / len; };
  int64_t c = of(SEG);
  if (k <= 16 && rows * c > cus && rows * of(SEG / 2) <= CU_512 * cus) c = of(SEG / 2);
  if (rows * c > CU_512 * cus) c = 2 * cus / rows;
  c = std::min(c, most);
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
  const int64_t len = chunks > 0 ? chunk_len : n, cus = device_cu_count();
  auto go = [&](auto t_c, auto per_cu_c) {
    constexpr int T = decltype(t_c)::value;
    hipLaunchKernelGGL((topk_kernel<T, decltype(per_cu_c)::value>), grid, dim3(T), 0, stream, scores, n, ld, k, vec4, out_idx, out_val, chunk_len, flags);
    return hipGetLastError();
  };
  auto go_256 = [&] { return go(std::integral_constant<int, 256>{}, std::integral_constant<int, CU_256>{}); };
  auto go_512 = [&] { return go(std::integral_constant<int, 512>{}, std::integral_constant<int, CU_512>{}); };
  auto go_1024 = [&](int64_t workgroups) {
    return workgroups <= cus ? go(std::integral_constant<int, THREADS>{}, std::integral_constant<int, 1>{})
                             : go(std::integral_constant<int, THREADS>{}, std::integral_constant<int, CU_1024>{});
  };
  if (len <= 256 * PER) return go_256();
  // As many threads as a row's first segment needs, while all workgroups are at work at once
  if (chunks > 0) return len > 512 * PER && rows * chunks <= (len <= SEG ? CU_1024 : 1) * cus ? go_1024(rows * chunks) : go_512();
  // (us, 512 / 1024 threads: 512 rows of 8193, k = 16, 6.4 / 7.0, of 9766 7.0 / 6.8; 129 of 9766, k = 10, 5.9 / 5.2)
  if (rows <= CU_1024 * cus) return len <= (rows <= cus ? 512 : 576) * PER ? go_512() : go_1024(rows);
  // More rows: 512 threads; 256 for k <= 16 where those would need a second round or rows are short, and for the longest.  us, 256 / 512 / 512 threads held to 64 registers
  // (256 of 32 scores each, before):
  //   513 rows, k = 10, of 8192     6.4 /  5.2 /  5.4 (4.8);  of 16384 10.1 / 7.2 / 7.7 (7.4);  k = 16 of 100000 43.9 / 34.2 / 34.9 (36.1)
  //   513 rows, k = 1, of 300000    107 /  123 /  124 (125);  577 of 527352, k = 10, 211 / 231 (231)
  //   900 rows, k = 10, of 8192     7.3 /  7.3 /  6.4 (5.4);  of 16384 12.9 / 13.6 / 12.9 (12.3);  of 100000 64.2 / 73.6 / 70.1 (68.6)
  //   1024 rows, k = 64, of 40000  41.8 / 38.2 / 33.3 (57.1);  of 100000 89.9 / 95.3 / 85.5 (110)
  //   1200 rows, k = 10, of 9766   12.1 / 14.7 / 14.7 (15.5);  of 20000 18.7 / 20.0 / 21.0 (24.1)
  //   2000 rows, k = 10, of 40000  57.4 / 52.5 / 55.5 (58.7);  of 100000 142.8 / 138.5 / 145.3 (140.2)
  if (rows <= CU_512 * cus) return k <= 16 && len >= 12 * SEG ? go_256() : go_512();
  if (rows <= (CU_512 + 1) * cus) {
    if (k <= 16 && len > 512 * PER) return go_256();
    return go(std::integral_constant<int, 512>{}, std::integral_constant<int, CU_512 + 1>{});
  }
  return k <= 16 && len < 2 * SEG ? go_256() : go_512();
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
