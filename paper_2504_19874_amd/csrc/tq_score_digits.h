// Digits of a rotated query for tq_score_stream.hip and the score they are put together to.  Plain functions of integers,
// so that their range is checked on the host too (tests/host/score_digits.cpp, tests/host/mask_digits.cpp).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace tq {

// Four digits of Q = dig[0] + 49 dig[1] + 49^2 dig[2] + 49^3 dig[3], |Q| <= 2^20, all of them eighths of an fp6 value (e2m3): 0 .. 16 and
// the even numbers to 32, of either sign.  These are 49 residues modulo 49, each once: an odd 17 .. 31 is the even -32 .. -18.
__host__ __device__ inline void mask_digits_of(int Q, int (&dig)[4]) {
  float rest = (float)Q;  // integers up to 2^20: all of this is exact
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    float up = __builtin_rintf(rest * (1.f / 49.f));  // (49 is odd: never half way, and 2^20 / 49 leaves 9 bits for the fraction)
    int r = (int)__builtin_fmaf(-49.f, up, rest);     // -24 .. 24
    if ((r & 1) != 0 && (r > 16 || r < -16)) {
      up += r > 0 ? 1.f : -1.f;
      r -= r > 0 ? 49 : -49;
    }
    dig[i] = r;
    rest = up;
  }
  dig[3] = (int)rest;
}
// the fp6 value of a digit's eighths
__host__ __device__ inline uint32_t mask_digit_code(int d) {
  const uint32_t m = (uint32_t)(d < 0 ? -d : d);
  return (m <= 16 ? m : 8 + (m >> 1)) | (d < 0 ? 32u : 0u);
}

// The same as bytes, for masks with values 2^k (the host test of stream_digits_sum makes its sums from these; no kernel does): the four balanced base-128 digits of Q 2^(7 - k) (negated for k = 7, where the mask byte reads as -128), |Q| <= 2^20:
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

// c0 + 49 c1 + 49^2 c2 + 49^3 c3, rounded once: sums over at most 4096 coordinates, so the lower three terms come to at most 2^29, and
// 49^3 = 7 2^14 + 2961
__host__ __device__ inline float mask_digits_sum(int c0, int c1, int c2, int c3) {
  return stream_digits_sum(0, c0 + 49 * c1 + 2401 * c2 + 2961 * c3, 0, 7 * c3);
}

}  // namespace tq
