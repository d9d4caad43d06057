// Few queries per code at d = 128 when the code is a pair of instances over a
// split of the rotated coordinates (Sec. 4.3: outlier channels with one more
// bit).  Coordinate group g < gs_hi (32 coordinates each) belongs to instance
// hi with BITS + 1 index planes and its own codebook, the others to instance lo
// with BITS planes; each instance has its own norm, residual norm and sketch
// scale, so the score is
//     nu_hi * (mse_hi + kappa_hi gamma_hi qjl_hi) + nu_lo * (mse_lo + kappa_lo gamma_lo qjl_lo)
// with the four inner sums taken over the instance's own coordinates only.
//
// Masked sums of fixed-point query digits, Walsh terms of the symmetric codebooks.
// "Sum over one instance only" is an A operand with the other instance's
// coordinate groups zeroed: every mask is made once and fed to two matrix
// instructions, one per instance.
// Queries are prepared inside the kernel while the code words are in flight
// (FUSED, needs the transposed matrices; see tq_score_i8_prep.h), or by
// prep_i8_kernel beforehand; either leaves the per-instance sums of the rounded
// query coordinates.
#include "tq_score_i8_prep.h"

namespace tq {

struct SplitArgs {
  int gs_hi;
  float kappa_hi;   // sqrt(pi/2) / d_hi; ScoreI8Args::kappa is that of instance lo
  float coef_hi[16];  // Walsh form of the hi codebook; ScoreI8Args::coef is that of lo
};

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Tiles of 16 keys whose codes are asked for together, a round ahead of their use: with four, two workgroups have no room on a compute unit
// (8 x 91627 keys, 4 queries each, 1 + 1 and 2 + 1 bits 21.2 us, 18.6 with two)
constexpr int SPLIT_ROUND = 2;
constexpr int SPLIT_LDS = I8_PART_FLOATS * 4 + 2 * 2048 + 2 * 4 * 4 * 4;  // partial sums, digits, scalars

// What the two instances share: digits of the rounded coordinates Q of query qi's rotation (m = 0) or sketch (m = 1), and their sums
// -> scal_s[m][qi][0: 1/scale, 2: sum over instance hi, 3: over lo].  Wavefront w takes (matrix w / 4, query w % 4).
template <bool PROD>
__device__ __forceinline__ void split_digitise(const ScoreI8Args& a, int q0, int wave, int lane, int d_hi, const float* part_s, unsigned char* dig_s,
                                               float* scal_s) {
  const int m = wave >> 2, qi = wave & 3;
  if (m == 1 && !PROD) return;
  const bool live = q0 + qi < a.q_per_group;
  float y[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int c = lane + 64 * u;
    y[u] = live ? part_s[((m * 2 + 0) * 4 + qi) * 128 + c] + part_s[((m * 2 + 1) * 4 + qi) * 128 + c] : 0.f;
  }
  const float mx = wave_max(fmaxf(fabsf(y[0]), fabsf(y[1])));
  int e = 0;
  if (mx > 0.f) (void)frexpf(mx, &e);  // mx = f * 2^e, f in [0.5, 1): |Q| <= 2^19
  const float sc = ldexpf(1.f, 19 - e);
  const int Q[2] = {__float2int_rn(y[0] * sc), __float2int_rn(y[1] * sc)};
  const int tot = wave_sum(Q[0] + Q[1]);
  const int tot_hi = wave_sum((lane < d_hi ? Q[0] : 0) + (lane + 64 < d_hi ? Q[1] : 0));
#pragma unroll
  for (int u = 0; u < 2; ++u) put_mask_digits(dig_s, m, qi, lane + 64 * u, (float)Q[u]);
  if (lane == 0) {
    const float inv = ldexpf(1.f, e - 19);
    scal_s[(m * 4 + qi) * 4 + 0] = inv;
    scal_s[(m * 4 + qi) * 4 + 2] = (float)tot_hi * inv;
    scal_s[(m * 4 + qi) * 4 + 3] = (float)(tot - tot_hi) * inv;
  }
}

// The masked sums on v_mfma_f32_16x16x128_f8f6f4 as in tq_score_i8_128_body.h: a stored word ANDed with 0x11111111 << v is eight fp4 operands, the
// digits are integers and every sum is exact, so the scores are those of the integer instructions bit for bit.  Bytes from a table of 64 KB in LDS,
// written by every workgroup, left room for one workgroup on a compute unit, three in turn.  64 channels at 2 + 1 bits and 64 at 1 + 1, us: 8 x
// 91627 keys, 4 queries each, 26.8 / 18.6 so, 8 x 65536 18.0 / 11.7, 8 x 16384 9.4 / 6.6; 16 x 131072, 8 queries, a bit more 144 / 85 (bound
// by the codes' intake, as one parameter set is).
template <int BITS, bool PROD, bool FUSED, int TILES>
__global__ __launch_bounds__(512, 4) void score_i8_split_kernel(const ScoreI8Args a, const SplitArgs sp) {
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn_s[];
  float* const part_s = reinterpret_cast<float*>(dyn_s);                                      // [2][2][4][128]
  unsigned char* const dig_s = reinterpret_cast<unsigned char*>(part_s + I8_PART_FLOATS);     // [2][4][4][128]
  float* const scal_s = reinterpret_cast<float*>(dig_s + 2 * 2048);                           // [2][4][4]
  constexpr int NP = BITS + 1;                     // planes of instance hi
  constexpr int NMH = (1 << NP) - 1;               // plane subsets of hi
  constexpr int NML = (1 << BITS) - 1;             // plane subsets of lo (a prefix of hi's)
  constexpr int RT = SPLIT_ROUND, ROUNDS = TILES / RT;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15;   // key within a tile / row of A
  const int kq = lane >> 4;    // coordinate group of this lane's words; also the query whose sums this lane receives
  const int group = blockIdx.y;
  const int q0 = blockIdx.z * 4;
  const int gs = sp.gs_hi;
  const bool g_hi = kq < gs;   // this lane's words belong to instance hi

  I8Prep<true, PROD> prep;
  if (FUSED) prep.load(a, group, q0, wave, tid);  // this thread's column of the transposed matrix, before anything else

  // ---- code words of this wavefront's keys: plane words of the lane's own group, a round ahead ----
  const int wpr = 4 * BITS + gs;  // idx words per row
  const int woff = g_hi ? kq * NP : gs * NP + (kq - gs) * BITS;
  const int64_t gbase = (int64_t)group * a.n;
  const int64_t wave_key0 = ((int64_t)blockIdx.x * 8 + wave) * (16 * TILES);
  struct Round {
    uint32_t pw[RT][NP], zw[RT];
    float kgh[RT], kgl[RT], nuh[RT], nul[RT];
  };
  Round codes[2];
  auto load_round = [&](int r, Round& c) {
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const int64_t key = wave_key0 + (r * RT + t) * 16 + col;
      const int64_t row = gbase + (key < a.n ? key : a.n - 1);  // clamped: results of such lanes are not stored
      const uint32_t* const pi = a.idx + row * wpr + woff;
#pragma unroll
      for (int pl = 0; pl < BITS; ++pl) c.pw[t][pl] = pi[pl];
      c.pw[t][BITS] = g_hi ? pi[BITS] : 0u;  // a lo group has no such plane: an all-zero mask changes nothing
      c.zw[t] = PROD ? a.qjl[row * 4 + kq] : 0u;
      c.kgh[t] = PROD ? a.gamma[2 * row] : 0.f;
      c.kgl[t] = PROD ? a.gamma[2 * row + 1] : 0.f;
      c.nuh[t] = a.norm[2 * row];
      c.nul[t] = a.norm[2 * row + 1];
    }
  };
  load_round(0, codes[0]);
  __builtin_amdgcn_sched_barrier(0);

  // ---- digits and scalars of this workgroup's queries ------------------------------------------------
  if constexpr (FUSED) {
    prep.matvec(part_s);
    __syncthreads();
    split_digitise<PROD>(a, q0, wave, lane, 32 * gs, part_s, dig_s, scal_s);
  } else {  // prepared by prep_i8_kernel, as base-128 digits
    const int qi = tid >> 7, c = tid & 127;
    const int64_t row = (int64_t)group * a.q_per_group + (q0 + qi < a.q_per_group ? q0 + qi : q0);
    const signed char* const img = reinterpret_cast<const signed char*>(a.img);
#pragma unroll
    for (int m = 0; m < (PROD ? 2 : 1); ++m) {
      auto digit = [&](int i) { return (int)img[(((row * 2 + m) * 2 + ((c >> 4) & 1)) * 16 + i * 4 + (c >> 5)) * 16 + (c & 15)]; };
      put_mask_digits(dig_s, m, qi, c, (float)(digit(0) + 128 * digit(1) + 16384 * digit(2)));
      if (c < 4) scal_s[(m * 4 + qi) * 4 + c] = a.scal[(row * 2 + m) * 4 + c];
    }
  }
  __syncthreads();

  // ---- A operands: lane = row + 16 kq, row = 4 * query + digit; of an fp8 operand a lane has 16 bytes of one coordinate group and 16 of another
  // (mask_slot), so that an instance's operand is the digits with the other instance's groups zeroed
  const int a_query = col >> 2, a_digit = col & 3;
  const v4i zero = v4i{0, 0, 0, 0};
  v8i ar[2], az[2];  // [instance: 0 lo, 1 hi]
  auto a_read = [&](int m, v8i (&o)[2]) {
    const unsigned char* const row = dig_s + ((m * 4 + a_query) * 4 + a_digit) * 128 + 16 * kq;
    const v4i d0 = *reinterpret_cast<const v4i*>(row), d1 = *reinterpret_cast<const v4i*>(row + 64);
    const bool h0 = (kq >> 1) < gs, h1 = 2 + (kq >> 1) < gs;
    o[1] = __builtin_shufflevector(h0 ? d0 : zero, h1 ? d1 : zero, 0, 1, 2, 3, 4, 5, 6, 7);
    o[0] = __builtin_shufflevector(h0 ? zero : d0, h1 ? zero : d1, 0, 1, 2, 3, 4, 5, 6, 7);
  };
  a_read(0, ar);
  if (PROD) a_read(1, az);
  const float r_inv = scal_s[kq * 4], r_sum_hi = scal_s[kq * 4 + 2], r_sum_lo = scal_s[kq * 4 + 3];
  const float s_inv = PROD ? scal_s[(4 + kq) * 4] : 0.f, s_sum_hi = PROD ? scal_s[(4 + kq) * 4 + 2] : 0.f, s_sum_lo = PROD ? scal_s[(4 + kq) * 4 + 3] : 0.f;

  auto masks = [&](uint32_t w) -> v8i {  // fp4: four registers
    const v4i b = v4i{(int)(w & 0x11111111u), (int)(w & 0x22222222u), (int)(w & 0x44444444u), (int)((w >> 3) & 0x11111111u)};
    return __builtin_shufflevector(b, b, 0, 1, 2, 3, -1, -1, -1, -1);
  };
  auto product = [&](const v8i& d, const v8i& b) -> f32x4 {
    return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(d, b, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 4, 0, 127, 0, 127);
  };
  auto digits_sum = [&](const f32x4& acc) -> float {  // D0 + 2^5 D1 + 2^10 D2 + 2^15 D3, the inner sums exact
    return fmaf(fmaf(acc[3], 32.f, acc[2]), 1024.f, fmaf(acc[1], 32.f, acc[0]));
  };

  // per-lane constants of the final combination
  float crh[NMH], crl[NML > 0 ? NML : 1];
#pragma unroll
  for (int m = 1; m <= NMH; ++m) crh[m - 1] = sp.coef_hi[m] * r_inv;
#pragma unroll
  for (int m = 1; m <= NML; ++m) crl[m - 1] = a.coef[m] * r_inv;
  const float base_hi = sp.coef_hi[0] * r_sum_hi, base_lo = a.coef[0] * r_sum_lo;
  const float zs = 2.f * s_inv;
  const bool out_live = q0 + kq < a.q_per_group;
  float* const out0 = a.scores + ((int64_t)group * a.q_per_group + (out_live ? q0 + kq : 0)) * a.lds + wave_key0 + col;

  if (wave_key0 >= a.n) return;  // uniform over the wavefront; no barrier follows
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    if (TILES == 4 && wave_key0 + r * (RT * 16) >= a.n) break;  // uniform (with more tiles a test costs 2 - 3 % of a long list)
    const Round& c = codes[r & 1];
    if (r + 1 < ROUNDS) load_round(r + 1, codes[(r + 1) & 1]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      float th = base_hi, tl = base_lo;
#pragma unroll
      for (int m = 1; m <= NMH; ++m) {
        if (!i8_term(m)) continue;
        uint32_t w = 0u;
#pragma unroll
        for (int pl = 0; pl < NP; ++pl)
          if (m & (1 << pl)) w ^= c.pw[t][pl];
        const v8i b = masks(w);
        th = fmaf(crh[m - 1], digits_sum(product(ar[1], b)), th);
        if (m <= NML) tl = fmaf(crl[m - 1], digits_sum(product(ar[0], b)), tl);
      }
      if (PROD) {
        const v8i b = masks(c.zw[t]);
        th = fmaf(sp.kappa_hi * c.kgh[t], fmaf(zs, digits_sum(product(az[1], b)), -s_sum_hi), th);
        tl = fmaf(a.kappa * c.kgl[t], fmaf(zs, digits_sum(product(az[0], b)), -s_sum_lo), tl);
      }
      float total = fmaf(c.nuh[t], th, c.nul[t] * tl);
      // (formed here whether it is stored or not: behind a branch of its own this compiler loses sight of the waits that the registers of the
      // matrix instructions above need)
      asm volatile("" : "+v"(total));
      if (out_live && wave_key0 + (r * RT + t) * 16 + col < a.n) out0[(r * RT + t) * 16] = total;
    }
  }
}

template <int BITS, bool PROD, bool FUSED, int TILES>
static hipError_t launch_split_one(const ScoreI8Args& a, const SplitArgs& sp, int n_groups, hipStream_t s) {
  static_assert(SPLIT_LDS <= 64 * 1024, "no limit to raise");
  const int64_t per_wg = 8 * 16 * TILES;
  const dim3 grid((unsigned)((a.n + per_wg - 1) / per_wg), n_groups, (a.q_per_group + 3) / 4);
  hipLaunchKernelGGL((score_i8_split_kernel<BITS, PROD, FUSED, TILES>), grid, dim3(512), SPLIT_LDS, s, a, sp);
  return hipGetLastError();
}

// Keys per workgroup as in tq_score_i8_128.hip: 2048, fewer while that leaves compute units without one (1024 of more keys than the chip takes at
// once: 8 x 61687, 8 queries each, 19.3 -> 23.5 us).  But no more than the tiles of 8 wavefronts that a short cache fills, however many groups there are:
// 3 bits, 32 groups of 32 queries, us, 16 tiles to a wavefront / as few as hold the keys: one key 12.0 / 5.5, 512 keys 12.8 / 7.6, 1024 13.6 / 10.7.
template <int BITS, bool PROD, bool FUSED>
static hipError_t launch_split_tiles(const ScoreI8Args& a, const SplitArgs& sp, int n_groups, hipStream_t s) {
  const int64_t others = (int64_t)n_groups * ((a.q_per_group + 3) / 4), cus = device_cu_count();
  if (a.n <= 512 || ((a.n + 1023) / 1024) * others <= cus / 2) return launch_split_one<BITS, PROD, FUSED, 4>(a, sp, n_groups, s);
  if (a.n <= 1024 || ((a.n + 2047) / 2048) * others <= cus / 2) return launch_split_one<BITS, PROD, FUSED, 8>(a, sp, n_groups, s);
  return launch_split_one<BITS, PROD, FUSED, 16>(a, sp, n_groups, s);
}

template <int BITS, bool PROD>
static hipError_t launch_split(const ScoreI8Args& a, const SplitArgs& sp, int n_groups, bool fused, hipStream_t s) {
  return fused ? launch_split_tiles<BITS, PROD, true>(a, sp, n_groups, s) : launch_split_tiles<BITS, PROD, false>(a, sp, n_groups, s);
}

// c[v] = sum_S w_S chi_S(v) rewritten over masked sums (see tq_score_i8.hip):
//   sum_j q_j c[idx_j] = (w_0 - sum_S sgn_S w_S) * sum_j q_j + sum_S 2 sgn_S w_S M_S
static bool walsh_coefficients(int bits, const Codebook& cb, float* coef) {
  double w[16];
  i8_walsh(bits, cb, w);
  const int K = 1 << bits;
  double c0 = w[0];
  for (int v = 0; v < 16; ++v) coef[v] = 0.f;
  for (int sset = 1; sset < K; ++sset) {
    const double sgn = (__builtin_popcount(sset) & 1) ? 1.0 : -1.0;
    if (!i8_term(sset) && w[sset] != 0.0) return false;  // not symmetric about zero
    c0 -= sgn * w[sset];
    coef[sset] = (float)(2.0 * sgn * w[sset]);
  }
  coef[0] = (float)c0;
  return true;
}

bool score_i8_split_applicable(int bits_lo, const Codebook& cb_lo, const Codebook& cb_hi) {
  float tmp[16];
  return bits_lo >= 0 && bits_lo <= 3 && cb_hi.bits == bits_lo + 1 && walsh_coefficients(bits_lo, cb_lo, tmp) &&
         walsh_coefficients(bits_lo + 1, cb_hi, tmp);
}

hipError_t launch_score_i8_split(int bits_lo, bool prod, const float* Pi, const float* S, const float* PiT,
                                 const float* ST, const float* q, int64_t ldq,
                                 void* workspace, const uint32_t* idx, const uint32_t* qjl, const float* gamma,
                                 const float* norm, float* scores, int64_t lds, int64_t n, int n_groups,
                                 int q_per_group, int gs_hi, float kappa_lo, float kappa_hi, const Codebook& cb_lo,
                                 const Codebook& cb_hi, hipStream_t stream) {
  if (n_groups == 0 || q_per_group == 0 || n == 0) return hipSuccess;
  if (gs_hi < 1 || gs_hi > 3 || bits_lo < 0 || bits_lo > 3) return hipErrorInvalidValue;
  const int64_t nq = (int64_t)n_groups * q_per_group;
  uint4* img = static_cast<uint4*>(workspace);
  float* scal = reinterpret_cast<float*>(static_cast<char*>(workspace) + (size_t)nq * 2 * 2 * 256);
  // with the transposed matrices at hand the scoring kernel prepares the queries itself
  const bool fused = PiT != nullptr && (!prod || ST != nullptr);
  if (!fused) {
    hipError_t e = launch_prep_i8_128(32 * gs_hi, Pi, S, q, ldq, nq, prod, img, scal, stream);
    if (e != hipSuccess) return e;
  }
  ScoreI8Args a;
  a.img = img; a.scal = scal; a.PiT = PiT; a.ST = ST; a.x = q; a.ldx = ldq; a.idx = idx; a.qjl = qjl;
  a.gamma = gamma; a.norm = norm; a.scores = scores; a.lds = lds; a.n = n; a.total_rows = (int64_t)n_groups * n;
  a.d = 128; a.q_per_group = q_per_group; a.kappa = kappa_lo;
  SplitArgs sp;
  sp.gs_hi = gs_hi;
  sp.kappa_hi = kappa_hi;
  if (!walsh_coefficients(bits_lo, cb_lo, a.coef) || !walsh_coefficients(bits_lo + 1, cb_hi, sp.coef_hi))
    return hipErrorInvalidValue;
  switch (bits_lo * 2 + (prod ? 1 : 0)) {
    case 0: return launch_split<0, false>(a, sp, n_groups, fused, stream);
    case 1: return launch_split<0, true>(a, sp, n_groups, fused, stream);
    case 2: return launch_split<1, false>(a, sp, n_groups, fused, stream);
    case 3: return launch_split<1, true>(a, sp, n_groups, fused, stream);
    case 4: return launch_split<2, false>(a, sp, n_groups, fused, stream);
    case 5: return launch_split<2, true>(a, sp, n_groups, fused, stream);
    case 6: return launch_split<3, false>(a, sp, n_groups, fused, stream);
    case 7: return launch_split<3, true>(a, sp, n_groups, fused, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace tq
