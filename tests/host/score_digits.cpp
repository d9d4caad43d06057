// The digit arithmetic of the few-query scoring kernel against 64-bit integers, at the ends of its range and in between:
// the sums that the matrix instructions make fit 32 bits, and the score they are joined to is the rounded exact one.
#include <cstdint>
#include <cstdio>
#include <random>
#include <vector>

#include "../../paper_2504_19874_amd/csrc/tq_score_digits.h"

static int check(const std::vector<int>& Q, const std::vector<bool>& mask, const char* what) {
  int64_t want = 0, c[4] = {0, 0, 0, 0};
  for (size_t j = 0; j < Q.size(); ++j) {
    const int k = (int)(j & 7);
    int dig[4];
    tq::stream_digits_of(Q[j], k, dig);
    for (int i = 0; i < 4; ++i) {
      if (dig[i] < -128 || dig[i] > 127) return std::printf("%s: digit %d of %d at bit %d is %d\n", what, i, Q[j], k, dig[i]), 1;
      if (mask[j]) c[i] += (int64_t)(int8_t)(1 << k) * dig[i];
    }
    if (mask[j]) want += Q[j];
  }
  for (int i = 0; i < 4; ++i)
    if (c[i] != (int32_t)c[i]) return std::printf("%s: sum %d is %lld\n", what, i, (long long)c[i]), 1;
  const float got = tq::stream_digits_sum((int)c[0], (int)c[1], (int)c[2], (int)c[3]);
  if (got != (float)want) return std::printf("%s: %.9g where the sum is %lld\n", what, got, (long long)want), 1;
  return 0;
}

int main() {
  std::mt19937 rng(5);
  int bad = 0;
  for (int d : {256, 2048, 3072, 4096}) {
    const std::vector<bool> all(d, true);
    for (int q : {1 << 20, -(1 << 20), 1 << 19, (1 << 20) - 1, 1038090, -1038090, 1, -1, 0, 8191, 8192, -8193}) bad += check(std::vector<int>(d, q), all, "equal values");
    for (int t = 0; t < 200; ++t) {
      std::vector<int> Q(d);
      std::vector<bool> m(d);
      std::uniform_int_distribution<int> u(t % 3 == 0 ? (1 << 20) - 1000 : -(1 << 20), 1 << 20);
      for (int j = 0; j < d; ++j) {
        Q[j] = t % 3 == 1 ? (rng() & 1 ? 1 << 20 : -(1 << 20)) : u(rng);
        m[j] = t % 5 == 0 || (rng() & 1);
      }
      bad += check(Q, m, "drawn values");
    }
  }
  if (bad == 0) std::puts("digits ok");
  return bad != 0;
}
