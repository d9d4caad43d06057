// Nearest-neighbour search by many queries: the k best codes of each, without a score matrix and at a third of the matrix
// work of evaluating every score to full precision.
//
// 1. prepare     every query's rotated coordinates as ONE fp16 piece, and a bound of what that leaves out: with the codes'
//                centroids as one piece too, a score is off by at most eps = |nu| (e1 + kappa |gamma| e2),
//                  e1 = (|q - q^| + r |q^|) sqrt(d) max |c|,   e2 = (|s - s^| + a |s|) sqrt(d)
//                (Cauchy-Schwarz; r: largest relative error of a centroid's piece, plus a for the fp32 sums).
// 2. sample      score - eps of some thousand codes, evenly spaced; the k-th best of a query is a bar that its k-th best
//                code reaches for certain (topk_kernel).
// 3. find        every score once with one matrix instruction per product instead of three; the codes whose
//                score + eps reaches the bar go to the query's list (expected: a thousand).
// 4. select      the k-th best of score - eps over the list is a better bar, which little more than k candidates pass;
//                those are scored with the pieces, products and order of tq_score_bf3.hip (the same bits), and ranked.
// A list that overflows (thousands of equal scores) flags its query: the caller runs the kernels that look at everything,
// which skip blocks of queries without a flag.
//
// 1000 queries, 10^6 codes, k = 10, d = 1536, 4 bits: 3.1 ms, 9.5 with every score from the exact kernel; 2.93 of it are
// the find kernel's.  500 queries, 30000 codes, k = 64, d = 512: 119 us (284 with 4096 codes in the sample: the gathering
// overflowed).
#include <algorithm>
#include <cmath>

#include "tq_bf3.h"
#include "tq_code_decode.h"
#include "tq_search.h"
#include "tq_select.h"

namespace tq {
namespace {

constexpr int CAP = 4096;  // candidates per query

struct SearchFactors {
  float c_rel;    // largest relative error of a centroid's leading piece
  float c_norm;   // sqrt(d) max |c|
  float acc_rel;  // fp32 sums of d products, here and in the exact kernel, and what that one's pieces leave out
  float sqrt_d;
  float s_rel;    // scale of the rotated queries' pieces over that of the sketched ones
};

// grid nq, 256 threads
__global__ __launch_bounds__(256) void search_prepare_kernel(const int d, const float* __restrict__ qr, const float* __restrict__ qs,
                                                             const SearchFactors f, uint32_t* __restrict__ r_pieces,
                                                             uint32_t* __restrict__ s_pieces, float* __restrict__ inv, float* __restrict__ e1,
                                                             float* __restrict__ e2, int32_t* __restrict__ count, int32_t* __restrict__ flags) {
  __shared__ float red[4][4];
  __shared__ float red_mx[4];
  const int tid = threadIdx.x, lane = tid & 63;
  const int64_t q = blockIdx.x;
  const float* const r = qr != nullptr ? qr + q * d : nullptr;
  const float* const z = qs != nullptr ? qs + q * d : nullptr;
  const float s_fac = 1.f / f.s_rel;
  float mx = 0.f;
  for (int k = tid; k < d; k += 256) {
    if (r != nullptr) mx = fmaxf(mx, fabsf(r[k]));
    if (z != nullptr) mx = fmaxf(mx, fabsf(z[k]) * s_fac);
  }
  mx = over_wavefront(mx, [](float x, float y) { return fmaxf(x, y); });
  if (lane == 0) red_mx[tid >> 6] = mx;
  __syncthreads();
  mx = fmaxf(fmaxf(red_mx[0], red_mx[1]), fmaxf(red_mx[2], red_mx[3]));
  float s, si;
  h2_scale(__float_as_uint(mx), s, si);
  float sum[4] = {0.f, 0.f, 0.f, 0.f};  // |q|^2, |q - q^|^2 of the two
  for (int u = tid; u < d / 4; u += 256) {
    const int g = u >> 3, k = u & 7;
    auto pieces = [&](const float* v, float scale, float back, float& n2, float& d2) {
      const float w[4] = {v[32 * g + k], v[32 * g + k + 16], v[32 * g + k + 8], v[32 * g + k + 24]};
      uint32_t o[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const f16x2 p = {(_Float16)(w[2 * e] * scale), (_Float16)(w[2 * e + 1] * scale)};
        const float a = w[2 * e] - (float)p[0] * back, b = w[2 * e + 1] - (float)p[1] * back;
        n2 = fmaf(w[2 * e], w[2 * e], fmaf(w[2 * e + 1], w[2 * e + 1], n2));
        d2 = fmaf(a, a, fmaf(b, b, d2));
        o[e] = h2_bits(p);
      }
      return make_uint2(o[0], o[1]);
    };
    const int64_t at = (int64_t)g * (search_step_bytes(gridDim.x) / 4) + q * 16 + k * 2;
    if (r != nullptr) *reinterpret_cast<uint2*>(r_pieces + at) = pieces(r, s, si, sum[0], sum[1]);
    if (z != nullptr) *reinterpret_cast<uint2*>(s_pieces + at) = pieces(z, s * s_fac, si * f.s_rel, sum[2], sum[3]);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) sum[i] = over_wavefront(sum[i], [](float x, float y) { return x + y; });
  if (lane == 0)
#pragma unroll
    for (int i = 0; i < 4; ++i) red[tid >> 6][i] = sum[i];
  __syncthreads();
  if (tid == 0) {
    float t[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i] = sqrtf((red[0][i] + red[1][i]) + (red[2][i] + red[3][i])) * 1.001f;
    inv[q] = si;
    e1[q] = 1.01f * (t[1] + (f.c_rel + f.acc_rel) * (t[0] + t[1])) * f.c_norm;
    e2[q] = 1.01f * (t[3] + f.acc_rel * t[2]) * f.sqrt_d;
    count[q * COUNT_STEP] = 0;
    flags[q] = 0;
  }
}

struct SelectArgs {
  const float *qr, *qs, *e1, *e2;
  int d, topk;
  const uint32_t *idx, *qjl;
  const float *gamma, *norm;
  float kappa;
  const float* list_u;
  const int32_t *list_i, *count;
  int32_t* flags;
  int32_t* out_idx;
  float* out_val;
  Codebook cb;
};

// grid nq, T threads.  HELD to the registers of four wavefronts a SIMD, where LDS admits four workgroups of 256 threads to a compute unit: a few registers more
// make it three (813 queries of 512 over 16000 codes of 4 bits, k = 10: 22.8 us, held 15.7).  Where LDS does not, holding only costs (2048: the whole search
// 4 to 8 %).
template <int BITS, bool PROD, int T, bool HELD>
__global__ __launch_bounds__(T, HELD ? 4 : 1) void search_select_kernel(const SelectArgs a) {
  constexpr int SEGS = (BITS > 0 ? 1 : 0) + (PROD ? 1 : 0);
  constexpr int NB = BITS > 0 ? BITS : 1;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  int* const cand = reinterpret_cast<int*>(smem);                                // [CAP] codes that are scored again
  float* const score = reinterpret_cast<float*>(cand + CAP);                     // [CAP]
  unsigned short* const qp = reinterpret_cast<unsigned short*>(score + CAP);     // [segment][2 pieces][d]
  __shared__ __attribute__((aligned(16))) uint32_t keys[256];
  __shared__ uint32_t bar_s;
  __shared__ int n_s;
  __shared__ uint2 table_s[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t q = blockIdx.x;
  const int d = a.d, k = a.topk;
  const int total = a.count[q * COUNT_STEP];
  if (total > CAP) {
    if (tid == 0) a.flags[q] = 1;
    return;
  }
  if (tid < 16) {
    uint32_t p1, p2, p3;
    split3(a.cb.c[tid], p1, p2, p3);
    table_s[tid] = make_uint2(p1 | (p2 << 16), p3);
  }
  if (tid == 0) n_s = 0;
  // the query's pieces, as the scoring kernel stages them
  for (int e = tid; e < d / 4; e += T) {
    int seg = 0;
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      if (m == 0 ? BITS == 0 : !PROD) continue;
      const f32x4 v = *reinterpret_cast<const f32x4*>((m == 0 ? a.qr : a.qs) + q * d + 4 * e);
      uint32_t lo[3], hi[3];
      split3_pair(f32x2{v[0], v[1]}, lo[0], lo[1], lo[2]);
      split3_pair(f32x2{v[2], v[3]}, hi[0], hi[1], hi[2]);
#pragma unroll
      for (int pc = 0; pc < 2; ++pc) *reinterpret_cast<uint2*>(qp + (seg * 2 + pc) * d + 4 * e) = make_uint2(lo[pc], hi[pc]);
      ++seg;
    }
  }
  // candidates: score + eps from the list, eps again from the code's scalars
  constexpr int N = CAP / T;
  const float e1 = a.e1[q], e2 = a.e2[q];
  float mx = -__builtin_inff();
  float top[N];
#pragma unroll
  for (int i0 = 0; i0 < N; i0 += 4) {
#pragma unroll
    for (int i = i0; i < i0 + 4; ++i) top[i] = __builtin_nanf("");
    if (i0 * T >= total) continue;  // uniform
    // (four of a thread's at a time: one by one they are two trips to memory each)
    int64_t row[4];
    float nu[4], ga[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int c = (i0 + i) * T + tid, cc = c < total ? c : total - 1;
      row[i] = a.list_i[q * CAP + cc];
      top[i0 + i] = a.list_u[q * CAP + cc];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      nu[i] = a.norm != nullptr ? a.norm[row[i]] : 1.f;
      ga[i] = PROD ? a.gamma[row[i]] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float eps = fabsf(nu[i]) * e1;
      if (PROD) eps = fmaf(fabsf(nu[i] * (a.kappa * ga[i])), e2, eps);
      if ((i0 + i) * T + tid >= total) top[i0 + i] = __builtin_nanf("");
      mx = fmaxf(mx, fmaf(-2.f, eps, top[i0 + i]));
    }
  }
  const float bar = kth_of_maxima<T>(mx, k, keys, &bar_s, tid);
  uint32_t pass = 0u;
#pragma unroll
  for (int i = N - 1; i >= 0; --i) pass = pass + pass + (top[i] >= bar ? 1u : 0u);
  while (pass != 0u) {
    const int i = __builtin_ctz(pass);
    pass &= pass - 1u;
    cand[atomicAdd(&n_s, 1)] = a.list_i[q * CAP + i * T + tid];
  }
  __syncthreads();
  const int n = n_s;

  // scores as tq_score_bf3.hip makes them: 32 candidates of a wavefront are the columns, every row is the query
  const int gw = d >> 5, h = lane >> 5;
  for (int b = wave; b * 32 < n; b += T / 64) {
    const int s = b * 32 + (lane & 31);
    const int64_t row = cand[s < n ? s : n - 1];
    const uint32_t* const wi = a.idx + row * ((int64_t)gw * BITS);
    const uint32_t* const wz = PROD ? a.qjl + row * gw : nullptr;
    floatx16 acc1, acc2;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc1[r] = acc2[r] = 0.f;
    // The words of four groups at a time, four to eight ahead of their use: a lane's row is somewhere in memory.  (With one group ahead and
    // the list above entry by entry: d = 3072, 4 bits, 203163 codes, 70 queries 105 us, 86 so, the whole search 515 -> 444; bound by
    // the decoding of a wavefront.  Four that decode for one that multiplies, through LDS: the same; eight per query: 72 us there, but 44
    // for 27 at d = 512 and 972 queries.)
    constexpr int AHEAD = 4;  // d is a multiple of 128
    uint32_t w[AHEAD][NB], z[AHEAD], wn[AHEAD][NB], zn[AHEAD];
    auto load = [&](int g) {
      const int gg = g < gw ? g : gw - AHEAD;
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) {
        if constexpr (BITS > 0) load_plane_words<BITS>(wi + (gg + u) * BITS, wn[u]);
        if (PROD) zn[u] = wz[gg + u];
      }
    };
    auto signs = [&](uint32_t bits) -> bf16x8 {
      uint32_t v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = 0xBF80BF80u ^ (((bits >> (2 * e)) & 1u) << 15) ^ (((bits >> (2 * e + 1)) & 1u) << 31);
      const u32x4 o = u32x4{v[0], v[1], v[2], v[3]};
      return *reinterpret_cast<const bf16x8*>(&o);
    };
    load(0);
    for (int g0 = 0; g0 < gw; g0 += AHEAD) {
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) {
#pragma unroll
        for (int pl = 0; pl < BITS; ++pl) w[u][pl] = wn[u][pl];
        z[u] = PROD ? zn[u] : 0u;
      }
      load(g0 + AHEAD);
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) {
        const int g = g0 + u;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          const int off = 16 * half + 8 * h, at = 32 * g + off;
          auto piece = [&](int seg, int pc) { return *reinterpret_cast<const bf16x8*>(qp + (seg * 2 + pc) * d + at); };
          if (BITS == 1) {
            const bf16x8 f = signs(w[u][0] >> off);
            acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(piece(0, 1), f, acc1, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(piece(0, 0), f, acc1, 0, 0, 0);
          } else if (BITS > 1) {
            uint32_t lv[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
              lv[e] = 0u;
#pragma unroll
              for (int pl = 0; pl < BITS; ++pl) lv[e] |= ((((w[u][pl] >> (off + 4 * e)) & 0xFu) * 0x00204081u) & 0x01010101u) << pl;
            }
            u32x4 v1, v2;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const uint2 lo = table_s[(lv[e >> 1] >> (16 * (e & 1))) & 0xFFu], hi = table_s[(lv[e >> 1] >> (16 * (e & 1) + 8)) & 0xFFu];
              v1[e] = __builtin_amdgcn_perm(hi.x, lo.x, 0x05040100u);
              v2[e] = __builtin_amdgcn_perm(hi.x, lo.x, 0x07060302u);
            }
            const bf16x8 f1 = *reinterpret_cast<const bf16x8*>(&v1), f2 = *reinterpret_cast<const bf16x8*>(&v2);
            const bf16x8 a1 = piece(0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(piece(0, 1), f1, acc1, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, f2, acc1, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, f1, acc1, 0, 0, 0);
          }
          if (PROD) {
            const bf16x8 f = signs(z[u] >> off);
            acc2 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(piece(SEGS - 1, 1), f, acc2, 0, 0, 0);
            acc2 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(piece(SEGS - 1, 0), f, acc2, 0, 0, 0);
          }
        }
      }
    }
    const float c1 = BITS == 1 ? a.cb.c[1] : 1.f;
    const float nu = a.norm != nullptr ? a.norm[row] : 1.f;
    const float kg = PROD ? a.kappa * a.gamma[row] : 0.f;
    if (h == 0 && s < n) score[s] = nu * fmaf(kg, PROD ? acc2[0] : 0.f, c1 * acc1[0]);
  }
  __syncthreads();
  // the k best of them, in the scores' place (three workgroups per compute unit for four where they have one behind the pieces: 1000 queries of
  // 768, 3 bits, 30.0 us for 19.1); a NaN is not returned
  TopkLds<T, N>& best = *reinterpret_cast<TopkLds<T, N>*>(score);
  static_assert(sizeof(TopkLds<T, N>) <= CAP * 4, "room");
  float v[N];
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = i * T + tid < n ? score[i * T + tid] : __builtin_nanf("");
  __syncthreads();
  const int kept = take_segment<T, N>(best, v, [&](int i) { return cand[i * T + tid]; }, k, 0, tid, n <= 64);
  write_best(best, kept, k, -1, a.out_idx + q * k, a.out_val != nullptr ? a.out_val + q * k : nullptr, tid);
}

size_t align256(size_t v) { return (v + 255) / 256 * 256; }

// codes of the sample: of n codes about k n / m reach the k-th best of m sampled ones.  The lists are sized for four times
// the thousand that this aims at (the number is a sum of k exponentials: for k >= 8 more than four times its mean does not
// happen; below, the sample is that for k = 8).  And a tile of 256 x 256 (tq_search_gemm.hip) gathers 512 of its 65536 scores:
// half of that is what 250 k codes in the sample lead to; a workgroup of tq_search_few.hip gathers 256 of 4096 to 16384.
int64_t sample_codes(int64_t n, int topk) {
  const int64_t k = topk < 8 ? 8 : topk;
  int64_t m = n * k / (CAP / 4);
  if (m < 250 * k) m = 250 * k;
  if (m < 4096) m = 4096;
  return m < n ? m : n;
}

struct SearchSpace {
  size_t r, s, sample, list_u, list_i, top_v, top_i, inv, e1, e2, count, total;
  SearchSpace(int d, int64_t n, int64_t nq, int topk) {
    size_t at = 0;
    auto take = [&](size_t bytes) {
      const size_t o = at;
      at += align256(bytes);
      return o;
    };
    r = take((size_t)search_step_bytes((int)nq) * (d / 32));
    s = take((size_t)search_step_bytes((int)nq) * (d / 32));
    sample = take((size_t)nq * ((sample_codes(n, topk) + 3) / 4 * 4) * 4);
    list_u = take((size_t)nq * CAP * 4);
    list_i = take((size_t)nq * CAP * 4);
    top_v = take((size_t)nq * topk * 4);
    top_i = take((size_t)nq * topk * 4);
    inv = take((size_t)nq * 4);
    e1 = take((size_t)nq * 4);
    e2 = take((size_t)nq * 4);
    count = take((size_t)nq * COUNT_STEP * 4);
    total = at;
  }
};

// Queries per block: their lists (78 KB a query at k = 10 and 10^6 codes, of which 40 the sample's scores) stay below
// 512 MB, 1000 queries at k = 64 and 10^6 codes among it; at least 64, and blocks of about the same size.
int64_t block_queries(int d, int64_t n, int64_t nq, int topk) {
  const int64_t one = (int64_t)SearchSpace(d, n, 64, topk).total / 64 + 1;
  const int64_t most = std::max<int64_t>(64, (int64_t(512) << 20) / one / 128 * 128);
  if (nq <= most) return nq;
  const int64_t blocks = (nq + most - 1) / most;
  return std::min(most, ((nq + blocks - 1) / blocks + 127) / 128 * 128);
}

int select_lds(int segs, int d) { return CAP * 8 + segs * 2 * d * 2; }

template <int BITS, bool PROD, int T, bool HELD>
hipError_t launch_select_t(const SelectArgs& a, int nq, hipStream_t s) {
  static LdsLimit lds_limit;  // per instantiation: the limit is raised once per device
  if (const hipError_t e = raise_lds_limit(lds_limit, reinterpret_cast<const void*>(&search_select_kernel<BITS, PROD, T, HELD>), 80 * 1024); e != hipSuccess)
    return e;
  hipLaunchKernelGGL((search_select_kernel<BITS, PROD, T, HELD>), dim3((unsigned)nq), dim3(T), select_lds((BITS > 0 ? 1 : 0) + (PROD ? 1 : 0), a.d), s, a);
  return hipGetLastError();
}

template <int BITS, bool PROD>
hipError_t launch_select(const SelectArgs& a, int nq, hipStream_t s) {
  // Eight wavefronts per query where a compute unit has no other (us, 4 / 8 / 16 of them: 44 queries of 1536, 1 bit, k = 64, 24 / 15.0 / 14.7;
  // 200 of 768, 4 bits, k = 10, 17.0 / 14.9 / 19.3); long codes, whose decoding they would be in each other's way for, keep four (39 of
  // 3072, 3 + 1 bits, k = 64: 54 / 65 / 66, 48 now).
  if (nq <= device_cu_count() && a.d <= 2048) return launch_select_t<BITS, PROD, 512, false>(a, nq, s);
  // (a kilobyte and a quarter of LDS beside what is counted here)
  const bool four = 4 * (select_lds((BITS > 0 ? 1 : 0) + (PROD ? 1 : 0), a.d) + 1280) <= 160 * 1024;
  return four ? launch_select_t<BITS, PROD, 256, true>(a, nq, s) : launch_select_t<BITS, PROD, 256, false>(a, nq, s);
}

hipError_t launch_block(const SearchArgs& a, const Codebook& cb, char* base, int32_t* flags, hipStream_t s) {
  const SearchSpace sp(a.d, a.n, a.nq, a.topk);
  auto at = [&](size_t o) { return static_cast<void*>(base + o); };
  const float sqrt_d = std::sqrt((float)a.d);
  SearchFactors f;
  f.c_rel = f.c_norm = 0.f;
  for (int i = 0; i < (1 << a.bits); ++i) {
    const float c = std::fabs(cb.c[i]);
    f.c_norm = std::fmax(f.c_norm, c * sqrt_d);
  }
  if (a.bits > 1) f.c_rel = code_table_error(a.bits, cb);
  // A matrix instruction adds its 16 products to the accumulator with an error of at most 2^-24 (2.02 |accumulator| + 8 sum of
  // |products|), measured with operands of one size, of widely different ones and with a few large ones (2.01 and 7.2 were the
  // largest; a chain of them makes 2.02 2^-24 per instruction of all magnitudes together, and the second term once).  The
  // chains are d / 16 instructions here and 3 d / 16 in the exact kernel, whose two bf16 pieces of a factor leave out 2^-17
  // of it and their smallest product 2^-16; the score's own three roundings are far below.
  f.acc_rel = ((float)a.d * (4.f / 16.f * 2.04f) + 16.f) * 0x1p-24f + 0x1p-15f;
  f.sqrt_d = sqrt_d;
  f.s_rel = std::exp2(std::round(std::log2(sqrt_d)));
  hipLaunchKernelGGL(search_prepare_kernel, dim3((unsigned)a.nq), dim3(256), 0, s, a.d, a.bits > 0 ? a.qr : nullptr, a.prod ? a.qs : nullptr, f,
                     static_cast<uint32_t*>(at(sp.r)), static_cast<uint32_t*>(at(sp.s)), static_cast<float*>(at(sp.inv)),
                     static_cast<float*>(at(sp.e1)), static_cast<float*>(at(sp.e2)), static_cast<int32_t*>(at(sp.count)),
                     flags);
  if (const hipError_t e = hipGetLastError(); e != hipSuccess) return e;

  const int64_t m = sample_codes(a.n, a.topk), ld = (m + 3) / 4 * 4;
  CodeSearch c;
  c.r_pieces = at(sp.r); c.s_pieces = at(sp.s); c.nq = a.nq;
  c.inv = static_cast<const float*>(at(sp.inv)); c.e1 = static_cast<const float*>(at(sp.e1)); c.e2 = static_cast<const float*>(at(sp.e2));
  c.bar = static_cast<const float*>(at(sp.top_v)) + a.topk - 1; c.bar_step = a.topk; c.s_rel = f.s_rel;
  c.sample = static_cast<float*>(at(sp.sample)); c.ld_sample = ld;
  c.list_u = nullptr; c.list_i = static_cast<int32_t*>(at(sp.list_i)); c.count = static_cast<int32_t*>(at(sp.count)); c.cap = CAP;
  if (const hipError_t e = launch_code_search(a.bits, a.prod, c, a.d, a.idx, a.qjl, a.gamma, a.norm, m, a.n / m, a.kappa, cb, s); e != hipSuccess) return e;
  if (const hipError_t e = launch_topk(c.sample, a.nq, m, ld, a.topk, static_cast<int32_t*>(at(sp.top_i)), static_cast<float*>(at(sp.top_v)), s);
      e != hipSuccess)
    return e;
  c.list_u = static_cast<float*>(at(sp.list_u));
  if (const hipError_t e = launch_code_search(a.bits, a.prod, c, a.d, a.idx, a.qjl, a.gamma, a.norm, a.n, 1, a.kappa, cb, s); e != hipSuccess) return e;

  SelectArgs g;
  g.qr = a.qr; g.qs = a.qs; g.e1 = c.e1; g.e2 = c.e2; g.d = a.d; g.topk = a.topk; g.idx = a.idx; g.qjl = a.qjl; g.gamma = a.gamma; g.norm = a.norm;
  g.kappa = a.kappa; g.list_u = c.list_u; g.list_i = c.list_i; g.count = c.count; g.flags = flags;
  g.out_idx = a.topk_idx; g.out_val = a.topk_val; g.cb = cb;
  switch (a.bits * 2 + (a.prod ? 1 : 0)) {
    case 1: return launch_select<0, true>(g, a.nq, s);
    case 2: return launch_select<1, false>(g, a.nq, s);
    case 3: return launch_select<1, true>(g, a.nq, s);
    case 4: return launch_select<2, false>(g, a.nq, s);
    case 5: return launch_select<2, true>(g, a.nq, s);
    case 6: return launch_select<3, false>(g, a.nq, s);
    case 7: return launch_select<3, true>(g, a.nq, s);
    case 8: return launch_select<4, false>(g, a.nq, s);
    case 9: return launch_select<4, true>(g, a.nq, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

bool search_applicable(int bits, bool prod, int d, int64_t n, int nq, int topk, const Codebook& cb) {
  return topk >= 1 && topk <= 64 && nq > 0 && n >= 8192 && n <= 0x7fffffff && d % 128 == 0 && d <= 4096 && (bits > 0 || prod) && code_gemm_serves(bits, cb);
}

size_t search_workspace_bytes(int d, int64_t n, int64_t nq, int topk) {
  return align256((size_t)nq * 4) + SearchSpace(d, n, block_queries(d, n, nq, topk), topk).total;
}

hipError_t launch_search(const SearchArgs& a, const Codebook& cb, void* workspace, const int32_t** flags, hipStream_t s) {
  int32_t* const all_flags = static_cast<int32_t*>(workspace);  // [nq], then the space of a block
  *flags = all_flags;
  const int64_t block = block_queries(a.d, a.n, a.nq, a.topk);
  for (int64_t q0 = 0; q0 < a.nq; q0 += block) {
    SearchArgs b = a;
    b.nq = (int)std::min(block, a.nq - q0);
    if (a.qr != nullptr) b.qr += q0 * a.d;
    if (a.qs != nullptr) b.qs += q0 * a.d;
    b.topk_idx += q0 * a.topk;
    if (a.topk_val != nullptr) b.topk_val += q0 * a.topk;
    if (const hipError_t e = launch_block(b, cb, static_cast<char*>(workspace) + align256((size_t)a.nq * 4), all_flags + q0, s); e != hipSuccess)
      return e;
  }
  return hipSuccess;
}

}  // namespace tq
