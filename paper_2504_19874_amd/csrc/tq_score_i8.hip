// Query preparation for the few-query scoring kernels on fixed-point digits (tq_score_stream.hip and, on the integer matrix cores,
// tq_score_i8_split.hip: what they compute is told there): rotate / sketch a query, choose its fixed-point scale, write the
// digit operands; and the Walsh coefficients of a centroid table.
//
// Fixed point: per query, Q_j = round(q_j * 2^e) with |Q_j| <= 2^20 in base 49 (tq_score_digits.h), 2^19 for split codes in balanced
// base 128, digits in [-64, 64] (valid signed bytes).  Integer arithmetic is exact; the only rounding is that of q, 2^-20 of the query's
// largest coordinate, far inside 1e-4.
#include <cstring>

#include "tq_score_digits.h"
#include "tq_score_i8.h"

namespace tq {

typedef float f32x4 __attribute__((ext_vector_type(4)));


// The operand of one rotated query ys [d] (LDS) for tq_score_stream.hip: 32 words per word group g, digit dg of its coordinates as 32 values
// of 6 bits, the first four words at 4 dg, the other two at 16 + 2 dg (24 words, here without the gap; written in bytes, which memory takes
// one by one and LDS does not: 7.0 -> 6.6 us at d = 3072).  Value 8 v + i is coordinate 32 g + 4 i + v, negated for v = 3.  A mask
// of bit b is 4 + 2 b, 2 + 2 b, 2 b or 1 - 2 b there (v = 0 .. 3); off_s[dg], zero before: what the parts without b come to.  A thread
// for four coordinates, d / 4 <= blockDim.x.
__device__ __forceinline__ void stream_digits(const float* ys, int d, float sc, uint32_t* img_s, int* off_s, int tid) {
  int off[4] = {0, 0, 0, 0};
  if (tid < d / 4) {  // eight threads of a group: four values = 24 bits of the 192 each
    const int g = tid >> 3, v = (tid >> 1) & 3, half = tid & 1;
    const int part = v == 0 ? 4 : v == 1 ? 2 : v == 2 ? 0 : 1;
    uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int Q = __float2int_rn(ys[32 * g + 16 * half + 4 * i + v] * sc);
      int dig[4];
      mask_digits_of(v == 3 ? -Q : Q, dig);
#pragma unroll
      for (int dg = 0; dg < 4; ++dg) {
        w[dg] |= mask_digit_code(dig[dg]) << (6 * i);
        off[dg] += part * dig[dg];
      }
    }
#pragma unroll
    for (int dg = 0; dg < 4; ++dg)
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const int at = 6 * v + 3 * half + k;  // of the lane's 24 bytes
        reinterpret_cast<uint8_t*>(img_s + g * 24 + (at < 16 ? dg * 4 : 16 + dg * 2 - 4))[at] = (uint8_t)(w[dg] >> (8 * k));
      }
  }
  // two sums to a word: a wavefront's are at most 64 x 4 x 56 each
  int o01 = off[0] + off[1] * 65536, o23 = off[2] + off[3] * 65536;
  const auto add = [](int x, int y) { return x + y; };
  o01 = over_wavefront(o01, add);
  o23 = over_wavefront(o23, add);
  if ((tid & 63) < 4) {
    const int both = (tid & 2) != 0 ? o23 : o01, low = (int)(int16_t)both;
    atomicAdd(off_s + (tid & 3), (tid & 1) != 0 ? (both - low) >> 16 : low);
  }
}

// Split codes (d = 128): rotate / sketch one query per workgroup (y = W q for W = Pi or S) and write its digits in the
// operand order of tq_score_i8_split.hip.  grid (nq, 1 or 2 matrices), 512 threads.  Row j of W is read by the 32 lanes
// of a half-wavefront, 16 bytes each, and reduced across them.
 // P = d / 128: 16-byte pieces per lane per row; a half-wavefront owns 8 P rows
__global__ __launch_bounds__(512) void prep_i8_kernel(const int d_hi, const float* __restrict__ W0,
                                                      const float* __restrict__ W1,
                                                      const float* __restrict__ x, const int64_t ldx,
                                                      uint4* __restrict__ img, float* __restrict__ scal) {
  constexpr int d = 128, P = d / 128;  // P: 16-byte pieces per lane per row; a half-wavefront owns 8 P rows
  __shared__ float ys[d];
  __shared__ float red_mx[8];
  __shared__ int red_tot[8], red_hi[8];
  const int tid = threadIdx.x;
  const int l32 = tid & 31, hw = tid >> 5;  // 16 half-wavefronts
  const int64_t q = blockIdx.x;
  const int mat = blockIdx.y;
  const float* W = mat == 0 ? W0 : W1;
  // this lane's share of the query, then 8 rows at a time, all their loads in flight together
  f32x4 xv[P];
#pragma unroll
  for (int c = 0; c < P; ++c) xv[c] = *reinterpret_cast<const f32x4*>(x + q * ldx + 128 * c + 4 * l32);
#pragma unroll 1
  for (int r0 = 0; r0 < 8 * P; r0 += 8) {
    f32x4 wv[8][P];
#pragma unroll
    for (int r = 0; r < 8; ++r)
#pragma unroll
      for (int c = 0; c < P; ++c)
        wv[r][c] = *reinterpret_cast<const f32x4*>(W + (int64_t)(hw + 16 * (r0 + r)) * d + 128 * c + 4 * l32);
    float part[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      float acc = 0.f;
#pragma unroll
      for (int c = 0; c < P; ++c) {
        acc = fmaf(wv[r][c].x, xv[c].x, acc); acc = fmaf(wv[r][c].y, xv[c].y, acc);
        acc = fmaf(wv[r][c].z, xv[c].z, acc); acc = fmaf(wv[r][c].w, xv[c].w, acc);
      }
      part[r] = acc;
    }
#pragma unroll
    for (int off = 16; off >= 1; off >>= 1)
#pragma unroll
      for (int r = 0; r < 8; ++r) part[r] += __shfl_xor(part[r], off);
#pragma unroll
    for (int r = 0; r < 8; ++r)
      if (l32 == r) ys[hw + 16 * (r0 + r)] = part[r];
  }
  __syncthreads();
  float mx = tid < d ? fabsf(ys[tid]) : 0.f;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
  if ((tid & 63) == 0) red_mx[tid >> 6] = mx;
  __syncthreads();
  mx = red_mx[0];
#pragma unroll
  for (int w = 1; w < 8; ++w) mx = fmaxf(mx, red_mx[w]);
  // power-of-two scale with |Q| <= 2^19
  int e = 0;
  if (mx > 0.f) (void)frexpf(mx, &e);  // mx = f * 2^e, f in [0.5, 1)
  const float sc = ldexpf(1.f, 19 - e);
  int tot = tid < d ? __float2int_rn(ys[tid] * sc) : 0;
  int tot_hi = tid < d_hi ? tot : 0;  // the first d_hi coordinates: instance hi of a split (Sec. 4.3)
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    tot += __shfl_xor(tot, off);
    tot_hi += __shfl_xor(tot_hi, off);
  }
  if ((tid & 63) == 0) {
    red_tot[tid >> 6] = tot;
    red_hi[tid >> 6] = tot_hi;
  }
  __syncthreads();
  if (tid == 0) {
    int t = 0, th = 0;
#pragma unroll
    for (int w = 0; w < 8; ++w) {
      t += red_tot[w];
      th += red_hi[w];
    }
    scal[(q * 2 + mat) * 4 + 0] = ldexpf(1.f, e - 19);
    scal[(q * 2 + mat) * 4 + 1] = (float)t * ldexpf(1.f, e - 19);
    scal[(q * 2 + mat) * 4 + 2] = (float)th * ldexpf(1.f, e - 19);
    scal[(q * 2 + mat) * 4 + 3] = (float)(t - th) * ldexpf(1.f, e - 19);
  }
  const int ks = d >> 6;
  for (int u = tid; u < ks * 16; u += 512) {  // unit = (k-step s, digit dg, k-chunk kq)
    const int kq = u & 3, dg = (u >> 2) & 3, s = u >> 4;
    const int c0 = i8_coord0(s, kq);
    uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      // balanced digits: D0, D1 in [-64, 63], D2 in [-64, 64]
      const int Q = __float2int_rn(ys[c0 + k] * sc);
      const int d0 = ((Q + 64) & 127) - 64;
      const int Q1 = (Q - d0) >> 7;
      const int d1 = ((Q1 + 64) & 127) - 64;
      const int d2 = (Q1 - d1) >> 7;
      const int dig = dg == 0 ? d0 : dg == 1 ? d1 : dg == 2 ? d2 : 0;
      w[k >> 2] |= ((uint32_t)dig & 0xFFu) << (8 * (k & 3));
    }
    img[((q * 2 + mat) * ks + s) * 16 + dg * 4 + kq] = make_uint4(w[0], w[1], w[2], w[3]);
  }
}

// Digits for tq_score_stream.hip, in place: the d floats of rotated query q, matrix mat (written by a matrix-vector kernel)
// become its digit words.  grid (nq, matrices), a thread for four of the d <= 4096 values.
__global__ __launch_bounds__(1024) void digitise_i8_kernel(const int d, const int mat0, uint32_t* img, float* __restrict__ scal) {
  __shared__ float ys[4096];
  __shared__ float red_mx[16];
  __shared__ long long red_tot[16];
  __shared__ int off_s[4];
  __shared__ uint32_t img_s[4096 / 32 * 24];
  const int tid = threadIdx.x;
  if (tid < 4) off_s[tid] = 0;
  const int64_t q = blockIdx.x;
  const int mat = mat0 + blockIdx.y;
  uint32_t* const own = img + (q * 2 + mat) * d;
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if (4 * tid < d) {
    v = *reinterpret_cast<const f32x4*>(own + 4 * tid);
    *reinterpret_cast<f32x4*>(ys + 4 * tid) = v;
  }
  float mx = fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3])));
  mx = over_wavefront(mx, [](float x, float y) { return fmaxf(x, y); });
  if ((tid & 63) == 0) red_mx[tid >> 6] = mx;
  __syncthreads();
  mx = red_mx[0];
  for (int w = 1; w < (int)(blockDim.x >> 6); ++w) mx = fmaxf(mx, red_mx[w]);
  int e = 0;
  if (mx > 0.f) (void)frexpf(mx, &e);  // mx = f * 2^e, f in [0.5, 1)
  const float sc = ldexpf(1.f, 20 - e);
  stream_digits(ys, d, sc, img_s, off_s, tid);
  int tot = 0;  // of a wavefront: 256 values of up to 2^20
#pragma unroll
  for (int k = 0; k < 4; ++k) tot += __float2int_rn(v[k] * sc);
  tot = over_wavefront(tot, [](int x, int y) { return x + y; });
  if ((tid & 63) == 0) red_tot[tid >> 6] = tot;
  __syncthreads();
  for (int i = tid; i < d / 32 * 24; i += blockDim.x) own[i / 24 * 32 + i % 24] = img_s[i];  // (everyone has read its floats)
  if (tid < 4) reinterpret_cast<float*>(own)[24 + tid] = (float)-off_s[tid];  // behind the first group's digits: where the sums start
  if (tid == 0) {
    long long t = 0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += red_tot[w];
    const float inv = ldexpf(1.f, e - 20);
    scal[(q * 2 + mat) * 4 + 0] = inv;
    scal[(q * 2 + mat) * 4 + 1] = (float)t * inv;
    scal[(q * 2 + mat) * 4 + 2] = 0.f;  // one instance
    scal[(q * 2 + mat) * 4 + 3] = (float)t * inv;
  }
}

// digit images and scalars of nq queries
size_t score_i8_workspace_bytes(int d, int64_t nq) { return (size_t)nq * 2 * ((size_t)(d >> 6) * 256 + 16) + 512; }

// Walsh coefficients of the centroid table over the bit planes of the index:
//   c[v] = sum_S w_S chi_S(v),  chi_S(v) = prod_{p in S} (2 v_p - 1) = sgn_S * (2 x_S(v) - 1),
// x_S(v) = XOR of the bits of v in S, sgn_S = +1 for odd |S| and -1 for even |S|.  Summed in
// pairs (v, K-1-v): for even |S| chi_S agrees on the pair, so a table with c[K-1-v] = -c[v]
// gives exactly zero there.
void i8_walsh(int bits, const Codebook& cb, double* w) {
  const int K = 1 << bits;
  for (int sset = 0; sset < K; ++sset) {
    double acc = 0.0;
    const int size = __builtin_popcount(sset);
    for (int v = 0; v < (K > 1 ? K / 2 : 1); ++v) {
      const int par = __builtin_popcount(v & sset) & 1;
      const double chi = ((size - par) & 1) ? -1.0 : 1.0;  // (-1)^(number of zero bits of v in S)
      if (K == 1) acc += cb.c[0];
      else if (size & 1) acc += chi * ((double)cb.c[v] - (double)cb.c[K - 1 - v]);
      else acc += chi * ((double)cb.c[v] + (double)cb.c[K - 1 - v]);
    }
    w[sset] = acc / K;
  }
}

// the d = 128 preparation kernel for the split variant (tq_score_i8_split.hip)
hipError_t launch_prep_i8_128(int d_hi, const float* Pi, const float* S, const float* q, int64_t ldq, int64_t nq,
                              bool prod, uint4* img, float* scal, hipStream_t stream) {
  hipLaunchKernelGGL(prep_i8_kernel, dim3((unsigned)nq, prod ? 2 : 1), dim3(512), 0, stream, d_hi, Pi, S, q, ldq,
                     img, scal);
  return hipGetLastError();
}

// sum_j q_j c[idx_j] = coef[0] * sum_j q_j + sum over the odd-sized plane subsets S of coef[S] * M_S, where M_S
// is the sum of q_j over the coordinates whose index bits in S XOR to 1.  False for a table that is not
// symmetric about zero (its even-sized subsets do not vanish).
bool i8_coefficients(int bits, const Codebook& cb, float* coef) {
  double w[16];
  i8_walsh(bits, cb, w);
  const int K = 1 << bits;
  double c0 = w[0];
  for (int v = 0; v < 16; ++v) coef[v] = 0.f;
  for (int sset = 1; sset < K; ++sset) {
    const double sgn = (__builtin_popcount(sset) & 1) ? 1.0 : -1.0;
    if (!i8_term(sset) && w[sset] != 0.0) return false;
    c0 -= sgn * w[sset];
    coef[sset] = (float)(2.0 * sgn * w[sset]);
  }
  coef[0] = (float)c0;
  return true;
}

bool score_i8_applicable(int bits, int d, const Codebook& cb) {
  if (bits < 0 || bits > 4 || d % 128 != 0 || d > I8_MAX_D) return false;
  double w[16];
  i8_walsh(bits, cb, w);
  for (int sset = 1; sset < (1 << bits); ++sset)
    if (!i8_term(sset) && w[sset] != 0.0) return false;  // not symmetric about zero
  return true;
}

// Arguments of the single-kernel d = 128 path (tq_score_i8_128_body.h) for callers that run it inside a
// kernel of their own; false when that path does not take these codes.
bool score128_args(int bits, bool prod, const float* PiT, const float* ST, const float* q, int64_t ldq,
                   const uint32_t* idx, const uint32_t* qjl, const float* gamma, const float* norm, int64_t n,
                   int n_groups, int q_per_group, float kappa, const Codebook& cb, int64_t group_stride, ScoreI8Args* a) {
  const auto al16 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; };
  if (bits < 0 || bits > 4 || !(bits > 0 || prod)) return false;
  if (bits > 0 && (PiT == nullptr || idx == nullptr || !al16(idx))) return false;
  if (prod && (ST == nullptr || qjl == nullptr || gamma == nullptr || !al16(qjl))) return false;
  std::memset(a, 0, sizeof(*a));
  a->PiT = PiT; a->ST = ST; a->x = q; a->ldx = ldq; a->idx = idx; a->qjl = qjl; a->gamma = gamma; a->norm = norm;
  a->n = n; a->group_stride = group_stride; a->total_rows = (int64_t)(n_groups - 1) * group_stride + n; a->d = 128; a->q_per_group = q_per_group; a->kappa = kappa;
  return i8_coefficients(bits, cb, a->coef);
}

hipError_t launch_score_i8(int bits, bool prod, const float* Pi, const float* S, const float* PiT, const float* ST,
                           const float* q, int64_t ldq,
                           void* workspace, const uint32_t* idx, const uint32_t* qjl, const float* gamma,
                           const float* norm, float* scores, int64_t lds, int64_t n, int d, int n_groups,
                           int q_per_group, float kappa, const Codebook& cb, hipStream_t stream) {
  if (n_groups == 0 || q_per_group == 0) return hipSuccess;
  if (bits < 0 || bits > 4 || d % 128 != 0 || d > I8_MAX_D) return hipErrorInvalidValue;
  const int64_t nq = (int64_t)n_groups * q_per_group;
  uint4* img = static_cast<uint4*>(workspace);
  float* scal = reinterpret_cast<float*>(static_cast<char*>(workspace) + (size_t)nq * 2 * (d >> 6) * 256);
  if (n == 0) return hipSuccess;
  ScoreI8Args a;
  a.img = img; a.scal = scal; a.PiT = PiT; a.ST = ST; a.x = q; a.ldx = ldq; a.idx = idx; a.qjl = qjl; a.gamma = gamma; a.norm = norm;
  a.scores = scores; a.lds = lds; a.n = n; a.total_rows = (int64_t)n_groups * n; a.group_stride = n; a.d = d; a.q_per_group = q_per_group; a.kappa = kappa;
  if (!i8_coefficients(bits, cb, a.coef)) return hipErrorInvalidValue;  // see score_i8_applicable
  // d = 128 with the transposed matrices at hand and 16-byte aligned codes: one kernel does it all
  const auto al16 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; };
  if (d == 128 && (bits > 0 || prod) && (bits == 0 || (PiT != nullptr && al16(idx))) &&
      (!prod || (ST != nullptr && al16(qjl))))
    return launch_score_i8_128(bits, prod, a, n_groups, stream);
  // the queries rotated into the places of their digits, then digitised there
  float* const y = static_cast<float*>(workspace);
  const bool r = bits > 0;
  if (const hipError_t e = r ? launch_matvec_rows(d, nq, Pi, prod ? S : nullptr, q, ldq, y, y + d, 2 * d, false, stream)
                             : launch_matvec_rows(d, nq, S, nullptr, q, ldq, y + d, nullptr, 2 * d, false, stream);
      e != hipSuccess)
    return e;
  hipLaunchKernelGGL(digitise_i8_kernel, dim3((unsigned)nq, r && prod ? 2 : 1), dim3((d / 4 + 63) / 64 * 64), 0, stream, d, r ? 0 : 1, static_cast<uint32_t*>(workspace), scal);
  if (const hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  return launch_score_stream(bits, prod, img, scal, idx, qjl, gamma, norm, scores, lds, n, d, n_groups, q_per_group, kappa, a.coef, stream);
}

}  // namespace tq
