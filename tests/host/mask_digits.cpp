// The base-49 digits of the few-query scoring kernel: every one an fp6 value, together the number they came from; the sums that the
// matrix instructions make of them and of the masks' constant parts, and what these are joined to, against 64-bit integers.
#include <cstdint>
#include <cstdio>
#include <random>
#include <vector>

#include "../../paper_2504_19874_amd/csrc/tq_score_digits.h"

static float fp6(uint32_t c) {  // e2m3
  const int e = (c >> 3) & 3, m = c & 7;
  const float v = e == 0 ? m / 8.f : (8 + m) / 8.f * (1 << (e - 1));
  return c & 32 ? -v : v;
}

static int check(const std::vector<int>& Q, const std::vector<bool>& bit) {
  double acc[4] = {0, 0, 0, 0}, most = 0;
  int64_t want = 0;
  for (size_t j = 0; j < Q.size(); ++j) {
    const int v = (int)(j & 3);
    int dig[4];
    tq::mask_digits_of(v == 3 ? -Q[j] : Q[j], dig);
    const int64_t back = dig[0] + 49ll * dig[1] + 2401ll * dig[2] + 117649ll * dig[3];
    if (back != (v == 3 ? -Q[j] : Q[j])) return std::printf("%d came back as %lld\n", Q[j], (long long)back), 1;
    const float part = v == 0 ? 4 : v == 1 ? 2 : v == 2 ? 0 : 1, mask = v == 3 ? (bit[j] ? -1 : 1) : part + (bit[j] ? 2 : 0);
    double sum = 0;
    for (int i = 0; i < 4; ++i) {
      const uint32_t code = tq::mask_digit_code(dig[i]);
      if (code > 63 || 8 * fp6(code) != dig[i]) return std::printf("digit %d has code %u\n", dig[i], code), 1;
      acc[i] += (mask - part) * dig[i];
      sum += 6. * (dig[i] < 0 ? -dig[i] : dig[i]);
    }
    most += sum;
    if (bit[j]) want += Q[j];
  }
  if (most * 2 >= 16777216.) return std::printf("sums of up to %.0f\n", most), 1;  // exact in fp32 on the way
  const float got = tq::mask_digits_sum((int)(0.5 * acc[0]), (int)(0.5 * acc[1]), (int)(0.5 * acc[2]), (int)(0.5 * acc[3]));
  if (got != (float)want) return std::printf("%.9g where the sum is %lld\n", got, (long long)want), 1;
  return 0;
}

int main() {
  std::mt19937 rng(7);
  int bad = 0;
  for (int q = -(1 << 20); q <= 1 << 20 && bad == 0; q += q > -3000 && q < 3000 ? 1 : 37) bad += check({q, q, q, q}, {true, true, true, true});
  for (int d : {256, 2048, 4096}) {
    for (int q : {1 << 20, -(1 << 20), (1 << 20) - 1, 1 << 19, 117649 * 8 + 24 * 2450, 1, -1, 0}) bad += check(std::vector<int>(d, q), std::vector<bool>(d, true));
    for (int t = 0; t < 100; ++t) {
      std::vector<int> Q(d);
      std::vector<bool> m(d);
      std::uniform_int_distribution<int> u(t % 3 == 0 ? (1 << 20) - 1000 : -(1 << 20), 1 << 20);
      for (int j = 0; j < d; ++j) Q[j] = u(rng), m[j] = t % 5 == 0 || (rng() & 1);
      bad += check(Q, m);
    }
  }
  if (bad == 0) std::puts("digits ok");
  return bad != 0;
}
