// Attention read-out at d = 128 on the integer matrix cores: which kernel variant a call takes
// (the kernel itself is in tq_attend_128_kernel.h).
#include <algorithm>
#include <cstring>

#include "tq_attend_128_kernel.h"

namespace tq {

namespace {
// Keys per group up to which chunks of AT_KEYS[i] are taken, i = 0, 1.
// Short chunks where long ones would occupy at most half of the compute units: what a workgroup does besides its keys is then done by more of
// them, but its keys take a quarter of the time (8 heads of 1024 tokens, 4 queries each: 15.9 -> 10.6 us for the kernel).
// Of four wavefronts instead of eight for values of three planes or more, while every compute unit has one workgroup at most (beyond, two
// of them on a compute unit would fetch the matrices twice): their sums of signs then run on twice as many matrix cores.  A step, us,
// eight / four wavefronts: values of 4 bits, 8 heads of 1741 tokens 21.2 / 20.2; of 2 bits, 8 of 1024 17.0 / 17.6.
int64_t limit(int i, int n_groups, int q_per_group) {
  const int64_t others = (int64_t)n_groups * ((q_per_group + 3) / 4);
  if (others == 0) return 0;
  // (up to 64 chunks are joined by the quicker kernel)
  return i == 0 ? std::min<int64_t>(device_cu_count() / others, 64) * AT_KEYS[0] : device_cu_count() / 2 / others * AT_KEYS[2];
}

bool coefficients(const Codebook& cb, AttendCoefs* out) {
  if (!i8_coefficients(cb.bits, cb, out->c)) return false;
  double mean = 0.0;  // (0 and nothing else for a table symmetric about zero: the sums are exact)
  for (int i = 0; i < (1 << cb.bits); ++i) mean += cb.c[i];
  out->c[0] = (float)(mean / (1 << cb.bits));
  for (int v = 1; v < 16; ++v) out->c[v] = -out->c[v];
  return true;
}
}  // namespace
int attend128_keys(int64_t n, int n_groups, int q_per_group, int planes) {
  if (n > AT_KEYS[0] && n <= AT_KEYS[1] && n <= limit(1, n_groups, q_per_group)) return AT_KEYS[1];  // one chunk, which needs no joining
  if (attend128_takes_256(planes) && n <= limit(0, n_groups, q_per_group)) return AT_KEYS[0];
  return n <= limit(1, n_groups, q_per_group) ? AT_KEYS[1] : AT_KEYS[2];
}
int attend128_max_chunks(int64_t n, int n_groups, int q_per_group, int planes) {
  int most = attend128_chunks(n, AT_KEYS[2]);
  for (int i = attend128_takes_256(planes) ? 0 : 1; i < 2; ++i) {
    const int64_t lim = limit(i, n_groups, q_per_group);
    const int c = attend128_chunks(n < lim ? n : lim, AT_KEYS[i]);
    most = c > most ? c : most;
  }
  return most;
}

// value codes the kernel covers: d = 128, tables symmetric about zero; codes of Alg. 1 with 1..4 index bits,
// codes of Alg. 2 with 0..2, or two instances of Alg. 1 (cb_hi != NULL) with 1 + 2 or 2 + 3
bool attend128_applicable(int d, bool prod, const Codebook& cb, const Codebook* cb_hi) {
  float coef[16];
  if (d != 128 || !i8_coefficients(cb.bits, cb, coef)) return false;
  if (cb_hi != nullptr)
    return !prod && cb.bits >= 1 && cb.bits <= 2 && cb_hi->bits == cb.bits + 1 && i8_coefficients(cb_hi->bits, *cb_hi, coef);
  return cb.bits >= (prod ? 0 : 1) && cb.bits <= (prod ? 2 : 4);
}

// ka == nullptr: logits from a.scores; otherwise the scoring body runs in the same kernel on key codes of
// kb index bits (kprod: with the sign sketch)
hipError_t launch_attend128(int kb, bool kprod, const ScoreI8Args* ka, bool vprod, const AttendArgs& a, const AttendTables& t, int n_groups,
                            hipStream_t s) {
  if (a.nchunks == 0 || n_groups == 0 || a.q_per_group == 0) return hipSuccess;
  ScoreI8Args none;
  std::memset(&none, 0, sizeof(none));
  const ScoreI8Args& k = ka != nullptr ? *ka : none;
  if (ka == nullptr) kb = -1;
  AttendCoefs cf, cfh;
  std::memset(&cfh, 0, sizeof(cfh));
  if (a.d != 128 || !coefficients(t.cb, &cf)) return hipErrorInvalidValue;
  if (a.gs_hi > 0) {
    if (vprod || !coefficients(t.cb_hi, &cfh)) return hipErrorInvalidValue;
    switch (t.cb.bits) {
      case 1: return launch_attend128_s1(kb, kprod, k, a, cf, cfh, n_groups, s);
      case 2: return launch_attend128_s2(kb, kprod, k, a, cf, cfh, n_groups, s);
      default: return hipErrorInvalidValue;
    }
  }
  if (vprod) {
    switch (t.cb.bits) {
      case 0: return launch_attend128_p0(kb, kprod, k, a, cf, cfh, n_groups, s);
      case 1: return launch_attend128_p1(kb, kprod, k, a, cf, cfh, n_groups, s);
      case 2: return launch_attend128_p2(kb, kprod, k, a, cf, cfh, n_groups, s);
      default: return hipErrorInvalidValue;
    }
  }
  switch (t.cb.bits) {
    case 1: return launch_attend128_v1(kb, kprod, k, a, cf, cfh, n_groups, s);
    case 2: return launch_attend128_v2(kb, kprod, k, a, cf, cfh, n_groups, s);
    case 3: return launch_attend128_v3(kb, kprod, k, a, cf, cfh, n_groups, s);
    case 4: return launch_attend128_v4(kb, kprod, k, a, cf, cfh, n_groups, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace tq
