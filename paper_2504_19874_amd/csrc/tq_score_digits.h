// Digits of a rotated query for tq_score_stream.hip and the score they are put together to.  Plain functions of integers,
// so that their range is checked on the host too (tests/host/score_digits.cpp).
#pragma once
#include <hip/hip_runtime.h>

namespace tq {

// The four balanced base-128 digits of Q 2^(7 - k) (negated for k = 7, where the mask byte reads as -128), |Q| <= 2^20:
// the first three in [-64, 63], the last in [-64, 64].
__host__ __device__ inline void stream_digits_of(int Q, int k, int (&dig)[4]) {
  int v = k == 7 ? -Q : Q * (1 << (7 - k));
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    dig[i] = ((v + 64) & 127) - 64;
    v = (v - dig[i]) >> 7;
  }
  dig[3] = v;
}

// (c0 + 2^7 c1 + 2^14 c2 + 2^21 c3) / 128, c0 a multiple of 128, rounded once.  A masked sum of up to 4096 values of up to
// 2^20 takes 34 bits (a query whose rotated coordinates are all alike comes to that), so it is never put together as one
// int: the lower three terms are at most 2^30.1, and what they carry over 2^14 goes to c3 (together at most 2^18.1, exact
// in fp32).
__host__ __device__ inline float stream_digits_sum(int c0, int c1, int c2, int c3) {
  const int lo = c2 * 128 + c1 + (c0 >> 7);
  return fmaf((float)(c3 + (lo >> 14)), 16384.f, (float)(lo & 16383));
}

}  // namespace tq
