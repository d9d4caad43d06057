// Scoring when only a few queries share each code (decode attention with
// grouped queries: 4 query heads per KV head).  There is no operand reuse to
// speak of, so the kernel is organised around the stream of codes:
//
//   lane = key.  A wavefront takes 64 consecutive keys, each lane loads its own
//   key's packed words for 128 coordinates at a time (16-byte loads, fully
//   coalesced across the wave), expands them coordinate by coordinate in
//   registers and feeds v_mfma_f32_4x4x1_16b_f32:  16 independent 4x4 blocks,
//   A = 4 query values (one per lane of a block), B = 4 key values (one per
//   lane of a block), so one instruction multiplies one coordinate of 64 keys
//   by 4 queries.  Lane l = 4*block + j ends up with D[i][j] in register i =
//   the score of query i against its own key.
//
// The rotated / sketched queries (Pi q, S q) come from a small matrix-vector
// kernel and sit in LDS laid out [k/4][query][k%4], so one 16-byte read gives a
// lane the values of its query (lane%4) for four consecutive coordinates.
#include "tq_internal.h"
#include "tq_h2.h"

#include <type_traits>

namespace tq {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int MV_Q = 4;  // vectors of a workgroup

// out[q][j] = sum_k W[j][k] x[q][k] for a handful of vectors; blockIdx.z selects (W0, out0) or (W1, out1), blockIdx.y a block of Q vectors.
// A wavefront takes R rows of the matrix at a time, 16 bytes per lane and load, against Q vectors that the
// workgroup has staged in LDS.  Bound by the matrix coming from memory; R = 4 shares the staging and the LDS reads over four
// rows where that still gives the chip enough workgroups.  The vectors go to LDS by direct loads, and the beginning of the rows is on
// its way before they are waited for; then two chunks of a row are loaded ahead (one with R = 4: two take 13.2 us instead of
// 11.8 for 50 vectors and 768 x 768).  us, vectors staged through registers one after the other and nothing ahead -> here:
//   3072, two matrices (75 MB)  4 vectors 21.9 -> 17.6 (57 with a row per wavefront, staged a float at a time), 12 33.3 -> 24.7
//   1536, one matrix            5 9.5 -> 7.5
//   384 / 128, one matrix       60 (a thread per row of the matrix) 15.0 / 6.2 -> 5.1 / 3.4
template <int Q, int R>
__global__ __launch_bounds__(256) void matvec_rows_kernel(const int d, const int nq, const float* __restrict__ W0,
                                                          const float* __restrict__ W1, const float* __restrict__ x,
                                                          const int64_t ldx, float* __restrict__ out0,
                                                          float* __restrict__ out1, const int64_t ldo, const int x_bf16) {
  extern __shared__ __attribute__((aligned(16))) float xs[];  // [Q][d]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q0 = blockIdx.y * Q;
  const int j0 = (blockIdx.x * 4 + (tid >> 6)) * R;
  const bool live = j0 < d;  // d is a multiple of 4 R: whole wavefronts
  const float4* w4 = reinterpret_cast<const float4*>((blockIdx.z == 0 ? W0 : W1) + (int64_t)(live ? j0 : 0) * d);
  const int n4 = d / 4;
  const uint32_t xs_lds = h2_lds_address(xs);
  constexpr int U = R == 4 ? 1 : 2;  // chunks of 64 x 16 bytes per row that are loaded ahead
  float4 w[U][R];
  auto load = [&](float4 (&o)[U][R], int k0) {  // past the rows' end: their last values again
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < R; ++i) o[u][i] = w4[i * n4 + min(k0 + 64 * u + lane, n4 - 1)];
  };
  // the vectors' way to LDS first, all of it, then the beginning of the matrix: both are under way together
  if (!x_bf16) {
#pragma unroll
    for (int r = 0; r < Q; ++r) {
      const float* const src = x + (q0 + r < nq ? q0 + r : nq - 1) * ldx;  // past the end: the last one again, not stored
      for (int k = wave * 64; k < n4; k += 256)
        if (k + lane < n4) h2_dma(src, (uint32_t)(k + lane) * 16, xs_lds + (uint32_t)(r * d + 4 * k) * 4);
    }
  }
  load(w, 0);
  if (x_bf16) {
#pragma unroll
    for (int r = 0; r < Q; ++r) {
      const uint2* src = reinterpret_cast<const uint2*>(reinterpret_cast<const uint16_t*>(x) + (q0 + r < nq ? q0 + r : nq - 1) * ldx);
      for (int k4 = tid; k4 < n4; k4 += 256) {
        const uint2 v = src[k4];
        reinterpret_cast<float4*>(xs + r * d)[k4] = make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u),
                                                                __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xffff0000u));
      }
    }
  }
  float acc[R][Q];
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int r = 0; r < Q; ++r) acc[i][r] = 0.f;
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int i = 0; i < R; ++i) asm volatile("" : "+v"(w[u][i].x), "+v"(w[u][i].y), "+v"(w[u][i].z), "+v"(w[u][i].w));
  h2_wait_barrier<0>();
  for (int k0 = 0; k0 < n4; k0 += 64 * U) {
    float4 next[U][R];
    if (k0 + 64 * U < n4) load(next, k0 + 64 * U);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k4 = k0 + 64 * u + lane;
      if (k4 < n4)
#pragma unroll
        for (int r = 0; r < Q; ++r) {
          const float4 v = reinterpret_cast<const float4*>(xs + r * d)[k4];
#pragma unroll
          for (int i = 0; i < R; ++i)
            acc[i][r] = fmaf(w[u][i].x, v.x, fmaf(w[u][i].y, v.y, fmaf(w[u][i].z, v.z, fmaf(w[u][i].w, v.w, acc[i][r]))));
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < R; ++i) w[u][i] = next[u][i];
  }
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int r = 0; r < Q; ++r) acc[i][r] = over_wavefront(acc[i][r], [](float x, float y) { return x + y; });
  if (!live) return;
  float* const out = blockIdx.z == 0 ? out0 : out1;
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int r = 0; r < Q; ++r)
      if (lane == i * Q + r && q0 + r < nq) out[(q0 + r) * ldo + j0 + i] = acc[i][r];
}

hipError_t launch_matvec_rows(int d, int64_t n, const float* W0, const float* W1, const float* x, int64_t ldx, float* out0,
                              float* out1, int64_t ldo, bool bf16, hipStream_t s) {
  if (n == 0) return hipSuccess;
  if (d % 32 != 0 || ldx % 4 != 0 || (size_t)MV_Q * d * sizeof(float) > 65536) return hipErrorInvalidValue;
  constexpr int64_t most = (int64_t)65535 * MV_Q;  // blocks of vectors are a grid dimension
  for (; n > most; n -= most) {
    if (const hipError_t e = launch_matvec_rows(d, most, W0, W1, x, ldx, out0, out1, ldo, bf16, s); e != hipSuccess) return e;
    x = bf16 ? reinterpret_cast<const float*>(reinterpret_cast<const uint16_t*>(x) + most * ldx) : x + most * ldx;
    out0 += most * ldo;
    out1 = out1 != nullptr ? out1 + most * ldo : nullptr;
  }
  const int nq = (int)n;
  const int mats = W1 != nullptr ? 2 : 1;
  auto go = [&](auto q_c, auto r_c) {
    constexpr int Q = decltype(q_c)::value, R = decltype(r_c)::value;
    hipLaunchKernelGGL((matvec_rows_kernel<Q, R>), dim3((d + 4 * R - 1) / (4 * R), (nq + Q - 1) / Q, mats), dim3(256),
                       (size_t)Q * d * sizeof(float), s, d, nq, W0, W1, x, ldx, out0, out1, ldo, bf16 ? 1 : 0);
    return hipGetLastError();
  };
  using std::integral_constant;
  const int64_t wide = (int64_t)(d / 16) * ((nq + 3) / 4) * mats, cus = device_cu_count();  // workgroups with R = 4
  const bool many = wide >= cus;
  if (nq == 1) return many ? go(integral_constant<int, 1>{}, integral_constant<int, 4>{}) : go(integral_constant<int, 1>{}, integral_constant<int, 1>{});
  // (one and a half workgroups per compute unit leave half of them with twice the work of the others: two rows per wavefront then. Four
  // vectors, two matrices of 3072: 24.1 -> 22.8 us, 16 and 768: 9.7 -> 8.2; with two workgroups and more the staging counts: 8 and 3072 19 / 24)
  if (many && wide < 2 * cus) return go(integral_constant<int, MV_Q>{}, integral_constant<int, 2>{});
  return many ? go(integral_constant<int, MV_Q>{}, integral_constant<int, 4>{}) : go(integral_constant<int, MV_Q>{}, integral_constant<int, 1>{});
}

// DeQuant of Alg. 1 / Alg. 2 for a handful of long vectors: x~[k] = nu (sum_j Pi^T[k][j] c[idx_j] + kappa gamma
// sum_j S^T[k][j] z_j), R output coordinates k per wavefront (rows of Pi^T and of S^T, 1 KB per load), the decoded
// codes of Q vectors in LDS (Alg. 2: their sign vectors behind them).  A thread decodes four neighbouring coordinates at a time; the rows' beginning is on
// its way meanwhile.  Many codes are bound by the decoding, which every workgroup does for itself: more rows per wavefront then.  (A row per wavefront, decoded
// a coordinate at a time, before -> now, us: 1536, 4 bits, 1 code 7.4 -> 5.6, 16 18.2 -> 8.9, 64 53.4 -> 14.7; 3072, 4 bits, 16 100 -> 16.9; 768, 3 + 1
// bits, 32 11.8 -> 6.2.)
template <int BITS, bool PROD, int Q, int R>
__global__ __launch_bounds__(256) void dequant_rows_kernel(const int d, const int n, const uint32_t* __restrict__ idx,
                                                           const uint32_t* __restrict__ qjl, const float* __restrict__ gamma,
                                                           const float* __restrict__ norm, const float* __restrict__ PiT,
                                                           const float* __restrict__ ST, const Codebook cb, const float kappa,
                                                           float* __restrict__ out, const int64_t ldo) {
  constexpr int NB = BITS > 0 ? BITS : 1;
  extern __shared__ __attribute__((aligned(16))) float ys[];  // [Q][d], then (PROD) [Q][d] of +-kappa gamma
  __shared__ float cent_s[16];
  float* const zs = ys + Q * d;
  const int tid = threadIdx.x, lane = tid & 63;
  const int q0 = blockIdx.y * Q;
  const int j0 = (blockIdx.x * 4 + (tid >> 6)) * R;
  const bool live = j0 < d;  // d is a multiple of 4 R: whole wavefronts
  const int n4 = d >> 2, groups = d >> 5;
  const float4* const w4 = reinterpret_cast<const float4*>(PiT + (int64_t)(live ? j0 : 0) * d);
  const float4* const s4 = PROD ? reinterpret_cast<const float4*>(ST + (int64_t)(live ? j0 : 0) * d) : nullptr;
  float4 w[R], sv[PROD ? R : 1];
  auto load = [&](float4 (&wo)[R], float4 (&so)[PROD ? R : 1], int k4) {  // past the rows' end: their last values again
#pragma unroll
    for (int i = 0; i < R; ++i) {
      wo[i] = w4[i * n4 + min(k4, n4 - 1)];
      if constexpr (PROD) so[i] = s4[i * n4 + min(k4, n4 - 1)];
    }
  };
  if (tid < 16) cent_s[tid] = cb.c[tid];
  float kg[Q];
#pragma unroll
  for (int r = 0; r < Q; ++r) kg[r] = PROD ? kappa * gamma[min(q0 + r, n - 1)] : 0.f;  // past the end: the last code again, not stored
  uint32_t word[Q][NB], sign[Q];
  auto fetch = [&](int e) {  // of four coordinates: their bits of the planes' words from bit 0 on
#pragma unroll
    for (int r = 0; r < Q; ++r) {
      const int64_t at = (int64_t)min(q0 + r, n - 1) * groups + (e >> 3);
#pragma unroll
      for (int pl = 0; pl < BITS; ++pl) word[r][pl] = idx[at * BITS + pl] >> 4 * (e & 7);
      if constexpr (PROD) sign[r] = qjl[at] >> 4 * (e & 7);
    }
  };
  fetch(min(tid, n4 - 1));
  load(w, sv, lane);
  __syncthreads();  // the table
  for (int e = tid; e < n4;) {
#pragma unroll
    for (int r = 0; r < Q; ++r) {
      float y[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        uint32_t code = 0;
#pragma unroll
        for (int pl = 0; pl < BITS; ++pl) code |= (word[r][pl] >> k & 1u) << pl;
        y[k] = cent_s[code];
      }
      reinterpret_cast<float4*>(ys + r * d)[e] = make_float4(y[0], y[1], y[2], y[3]);
      if constexpr (PROD)
        reinterpret_cast<float4*>(zs + r * d)[e] = make_float4((sign[r] & 1u) ? kg[r] : -kg[r], (sign[r] & 2u) ? kg[r] : -kg[r],
                                                               (sign[r] & 4u) ? kg[r] : -kg[r], (sign[r] & 8u) ? kg[r] : -kg[r]);
    }
    e += 256;
    if (e < n4) fetch(e);
  }
  __syncthreads();
  if (!live) return;  // the whole wavefront
  float acc[R][Q];
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int r = 0; r < Q; ++r) acc[i][r] = 0.f;
  for (int k0 = 0; k0 < n4; k0 += 64) {
    float4 wn[R], sn[PROD ? R : 1];
    if (k0 + 64 < n4) load(wn, sn, k0 + 64 + lane);
    const int k4 = k0 + lane;
    if (k4 < n4)
#pragma unroll
      for (int r = 0; r < Q; ++r) {
        const float4 v = reinterpret_cast<const float4*>(ys + r * d)[k4];
        float4 u = make_float4(0.f, 0.f, 0.f, 0.f);
        if constexpr (PROD) u = reinterpret_cast<const float4*>(zs + r * d)[k4];
#pragma unroll
        for (int i = 0; i < R; ++i) {
          acc[i][r] = fmaf(w[i].x, v.x, fmaf(w[i].y, v.y, fmaf(w[i].z, v.z, fmaf(w[i].w, v.w, acc[i][r]))));
          if constexpr (PROD) acc[i][r] = fmaf(sv[i].x, u.x, fmaf(sv[i].y, u.y, fmaf(sv[i].z, u.z, fmaf(sv[i].w, u.w, acc[i][r]))));
        }
      }
#pragma unroll
    for (int i = 0; i < R; ++i) {
      w[i] = wn[i];
      if constexpr (PROD) sv[i] = sn[i];
    }
  }
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int r = 0; r < Q; ++r) acc[i][r] = over_wavefront(acc[i][r], [](float x, float y) { return x + y; });
  float v = 0.f;
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int r = 0; r < Q; ++r) v = lane == r * R + i ? acc[i][r] : v;
  const int row = q0 + lane / R;
  if (lane < R * Q && row < n) out[(int64_t)row * ldo + j0 + lane % R] = (norm != nullptr ? norm[row] : 1.f) * v;
}

template <int BITS>
static hipError_t dequant_rows_bits(bool prod, int d, int n, const uint32_t* idx, const uint32_t* qjl, const float* gamma,
                                    const float* norm, const float* PiT, const float* ST, const Codebook& cb, float kappa,
                                    float* out, int64_t ldo, hipStream_t s) {
  auto go = [&](auto prod_c, auto q_c, auto r_c) {
    constexpr bool PROD = decltype(prod_c)::value;
    constexpr int Q = decltype(q_c)::value, R = decltype(r_c)::value, MOST = 64 * 1024;
    const int lds = (PROD ? 2 : 1) * Q * d * (int)sizeof(float);
    if (lds > MOST) return hipErrorInvalidValue;
    if (lds == MOST) {  // d = 2048: above the default limit with the table
      static LdsLimit limit;
      if (const hipError_t e = raise_lds_limit(limit, reinterpret_cast<const void*>(&dequant_rows_kernel<BITS, PROD, Q, R>), MOST); e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((dequant_rows_kernel<BITS, PROD, Q, R>), dim3((d + 4 * R - 1) / (4 * R), (n + Q - 1) / Q), dim3(256), lds, s, d, n, idx, qjl, gamma,
                       norm, PiT, ST, cb, kappa, out, ldo);
    return hipGetLastError();
  };
  using std::integral_constant;
  // One row per wavefront up to `once` workgroups per compute unit, two up to `twice`, else four (the decoding is shared by all of a
  // workgroup's); us with 1 / 2 / 4:
  //   4 bits, d = 1024      8 codes 5.0 / 5.5 / 6.4, 16 6.4 / 5.6 / 6.5, 32 9.9 / 7.2 / 6.8
  //   2 + 1 bits, d = 768   4 4.0 / 4.5 / 5.6, 16 5.3 / 5.1 / 5.8
  //   3 + 1 bits, d = 1536  32 27 / 17 / 13
  // Eight codes per workgroup, four with a sketch, while 64 KB beside the table hold them (d = 3072, 32 codes of 4 bits: 31 us, with 96 KB 48).
  const int64_t cus = device_cu_count();
  auto rows = [&](auto prod_c, auto q_c, int64_t once, int64_t twice) {
    const int64_t all = (int64_t)(d / 4) * ((n + decltype(q_c)::value - 1) / decltype(q_c)::value);
    if (all <= once * cus) return go(prod_c, q_c, integral_constant<int, 1>{});
    if (all <= twice * cus) return go(prod_c, q_c, integral_constant<int, 2>{});
    return go(prod_c, q_c, integral_constant<int, 4>{});
  };
  if (prod) {
    if (n <= 2 || d > 2048) return rows(std::true_type{}, integral_constant<int, 2>{}, 3, 6);
    return rows(std::true_type{}, integral_constant<int, 4>{}, 2, 6);
  }
  if (n <= 4 || d > 2048) return rows(std::false_type{}, integral_constant<int, 4>{}, 3, 3);
  return rows(std::false_type{}, integral_constant<int, 8>{}, 1, 2);
}

hipError_t launch_dequant_rows(int bits, bool prod, int d, int64_t n, const uint32_t* idx, const uint32_t* qjl,
                               const float* gamma, const float* norm, const float* PiT, const float* ST, const Codebook& cb,
                               float kappa, float* out, int64_t ldo, hipStream_t s) {
  if (n == 0) return hipSuccess;
  if (n > 65535 || d % 32 != 0 || d > 4096) return hipErrorInvalidValue;
  switch (bits) {
    case 0: return dequant_rows_bits<0>(prod, d, (int)n, idx, qjl, gamma, norm, PiT, ST, cb, kappa, out, ldo, s);
    case 1: return dequant_rows_bits<1>(prod, d, (int)n, idx, qjl, gamma, norm, PiT, ST, cb, kappa, out, ldo, s);
    case 2: return dequant_rows_bits<2>(prod, d, (int)n, idx, qjl, gamma, norm, PiT, ST, cb, kappa, out, ldo, s);
    case 3: return dequant_rows_bits<3>(prod, d, (int)n, idx, qjl, gamma, norm, PiT, ST, cb, kappa, out, ldo, s);
    case 4: return dequant_rows_bits<4>(prod, d, (int)n, idx, qjl, gamma, norm, PiT, ST, cb, kappa, out, ldo, s);
    default: return hipErrorInvalidValue;
  }
}

// ---------------------------------------------------------------------------
struct ScoreSmallArgs {
  const float* qr;  // [n_groups*q_per_group][d]  Pi q
  const float* qs;  // [n_groups*q_per_group][d]  S q   (prod only)
  const uint32_t* idx;
  const uint32_t* qjl;
  const float* gamma;
  const float* norm;  // nullable
  float* scores;
  int64_t lds;
  int64_t n;          // keys per group
  int d;
  int q_per_group;
  float kappa;
  Codebook cb;
};

template <int BITS, bool PROD, int KPL>
__global__ __launch_bounds__(256) void score_small_kernel(const ScoreSmallArgs a) {
  extern __shared__ __attribute__((aligned(16))) float q_s[];  // qr then qs, each d*4 floats
  __shared__ float cent_s[16];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int group = blockIdx.y;
  const int pass = blockIdx.z;           // queries 4*pass .. 4*pass+3 of the group
  const int d = a.d;
  const int q0 = pass * 4;
  const int nq_here = min(4, a.q_per_group - q0);

  if (tid < 16) cent_s[tid] = a.cb.c[tid];
  // stage the queries: element (row r, coordinate k) -> [(k/4)*4 + r]*4 + k%4
  for (int e = tid; e < 4 * d; e += 256) {
    const int r = e / d, k = e - r * d;
    const int64_t qrow = (int64_t)group * a.q_per_group + q0 + r;
    const int dst = (((k >> 2) * 4 + r) << 2) + (k & 3);
    q_s[dst] = (r < nq_here) ? a.qr[qrow * d + k] : 0.f;
    if (PROD) q_s[4 * d + dst] = (r < nq_here) ? a.qs[qrow * d + k] : 0.f;
  }
  __syncthreads();

  const int words_per_row = (d / 32) * BITS;
  const int qw_per_row = d / 32;
  const int64_t gbase = (int64_t)group * a.n;
  const float4* qr4 = reinterpret_cast<const float4*>(q_s);
  const float4* qs4 = reinterpret_cast<const float4*>(q_s + 4 * d);

  // a wavefront owns 64*KPL consecutive keys; lane l takes keys base + u*64 + l.
  // The KPL keys of a lane share every query read and give independent MFMA chains.
  const int64_t base = ((int64_t)blockIdx.x * 4 + wave) * (64 * KPL);
  if (base >= a.n) return;
  int64_t row[KPL];
  bool valid[KPL];
  floatx4 acc[KPL], acc2[KPL];
#pragma unroll
  for (int u = 0; u < KPL; ++u) {
    const int64_t key = base + u * 64 + lane;
    valid[u] = key < a.n;
    row[u] = gbase + (valid[u] ? key : 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) { acc[u][r] = 0.f; acc2[u][r] = 0.f; }
  }
  for (int c = 0; c < d / 128; ++c) {  // 128 coordinates = 4 groups of 32 at a time
    uint32_t w[KPL][4 * (BITS > 0 ? BITS : 1)];
    uint32_t zn[KPL][4];
#pragma unroll
    for (int u = 0; u < KPL; ++u) {
      if (BITS > 0) {
        const uint32_t* src = a.idx + row[u] * words_per_row + c * 4 * BITS;
#pragma unroll
        for (int v = 0; v < BITS; ++v) {  // 4*BITS words = BITS 16-byte loads
          const uint4 t = *reinterpret_cast<const uint4*>(src + 4 * v);
          w[u][4 * v] = t.x; w[u][4 * v + 1] = t.y; w[u][4 * v + 2] = t.z; w[u][4 * v + 3] = t.w;
        }
      }
      if (PROD) {
        const uint4 t = *reinterpret_cast<const uint4*>(a.qjl + row[u] * qw_per_row + c * 4);
        zn[u][0] = ~t.x; zn[u][1] = ~t.y; zn[u][2] = ~t.z; zn[u][3] = ~t.w;  // bit set = minus sign
      }
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) {
#pragma unroll
      for (int j4 = 0; j4 < 8; ++j4) {
        const float4 qa = qr4[((c * 32 + g * 8 + j4) << 2) + (lane & 3)];
        float4 qb = make_float4(0.f, 0.f, 0.f, 0.f);
        if (PROD) qb = qs4[((c * 32 + g * 8 + j4) << 2) + (lane & 3)];
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          const int j = j4 * 4 + jj;
          const float av = jj == 0 ? qa.x : jj == 1 ? qa.y : jj == 2 ? qa.z : qa.w;
          const float bv = jj == 0 ? qb.x : jj == 1 ? qb.y : jj == 2 ? qb.z : qb.w;
#pragma unroll
          for (int u = 0; u < KPL; ++u) {
            if (BITS > 0) {
              uint32_t code = 0;
#pragma unroll
              for (int pl = 0; pl < BITS; ++pl) code |= ((w[u][g * BITS + pl] >> j) & 1u) << pl;
              acc[u] = __builtin_amdgcn_mfma_f32_4x4x1f32(av, cent_s[code], acc[u], 0, 0, 0);
            }
            if (PROD) {
              // +-1.0f with the sign bit taken from bit j of the inverted word
              const uint32_t sb = zn[u][g] << (31 - j);
              const float val = __uint_as_float((sb & 0x80000000u) | 0x3f800000u);
              acc2[u] = __builtin_amdgcn_mfma_f32_4x4x1f32(bv, val, acc2[u], 0, 0, 0);
            }
          }
        }
      }
    }
  }
#pragma unroll
  for (int u = 0; u < KPL; ++u) {
    if (valid[u]) {
      const float nu = a.norm != nullptr ? a.norm[row[u]] : 1.f;
      const float kg = PROD ? a.kappa * a.gamma[row[u]] : 0.f;
      const int64_t key = base + u * 64 + lane;
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (r < nq_here)
          a.scores[((int64_t)group * a.q_per_group + q0 + r) * a.lds + key] = nu * (acc[u][r] + kg * acc2[u][r]);
    }
  }
}

template <int BITS, bool PROD>
static hipError_t launch_kpl(const ScoreSmallArgs& a, int n_groups, size_t smem, hipStream_t s) {
  // two keys per lane once there is enough work to keep every SIMD busy anyway
  const bool big = a.n * (int64_t)n_groups >= (int64_t)1 << 19;
  const int kpl = big ? 2 : 1;
  const dim3 grid((unsigned)((a.n + 256 * kpl - 1) / (256 * kpl)), n_groups, (a.q_per_group + 3) / 4);
  if (big)
    hipLaunchKernelGGL((score_small_kernel<BITS, PROD, 2>), grid, dim3(256), smem, s, a);
  else
    hipLaunchKernelGGL((score_small_kernel<BITS, PROD, 1>), grid, dim3(256), smem, s, a);
  return hipGetLastError();
}

template <int BITS>
static hipError_t launch_bits(const ScoreSmallArgs& a, bool prod, int n_groups, size_t smem, hipStream_t s) {
  return prod ? launch_kpl<BITS, true>(a, n_groups, smem, s) : launch_kpl<BITS, false>(a, n_groups, smem, s);
}

hipError_t launch_score_small(int bits, bool prod, const float* qr, const float* qs, const uint32_t* idx,
                              const uint32_t* qjl, const float* gamma, const float* norm, float* scores,
                              int64_t lds, int64_t n, int d, int n_groups, int q_per_group, float kappa,
                              const Codebook& cb, hipStream_t stream) {
  if (n == 0 || n_groups == 0 || q_per_group == 0) return hipSuccess;
  if (d % 128 != 0 || d > 1024) return hipErrorInvalidValue;
  ScoreSmallArgs a;
  a.qr = qr; a.qs = qs; a.idx = idx; a.qjl = qjl; a.gamma = gamma; a.norm = norm;
  a.scores = scores; a.lds = lds; a.n = n; a.d = d; a.q_per_group = q_per_group;
  a.kappa = kappa; a.cb = cb;
  const size_t smem = (size_t)(prod ? 2 : 1) * 4 * d * sizeof(float);  // <= 32 KB
  switch (bits) {
    case 0: return launch_bits<0>(a, prod, n_groups, smem, stream);
    case 1: return launch_bits<1>(a, prod, n_groups, smem, stream);
    case 2: return launch_bits<2>(a, prod, n_groups, smem, stream);
    case 3: return launch_bits<3>(a, prod, n_groups, smem, stream);
    case 4: return launch_bits<4>(a, prod, n_groups, smem, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace tq
