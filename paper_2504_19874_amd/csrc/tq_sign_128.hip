// DeQuant at d = 128 of codes whose table is a sum of signs (tq_sign.h).
//
// A wavefront owns 32 output coordinates and keeps its digits of both matrices in registers (60 each, copied from the
// image at the start, or made there, see OWN); it walks blocks of 32 codes, whose words it reads as they lie: no LDS, no barrier, and few codes are simply
// few wavefronts.  One accumulator per kind of sign, the small digits first, joined with the codes' factors in the end: a sum meets two
// roundings at its full size where pieces met ten times as many.
//
// Bound by the stores (131072 codes: 67 MB, 11.2 us alone) and the instructions together: per block and wavefront 10 - 30 matrix instructions and
// about 170 others, which the stores cover in part (codes asked for two blocks ahead: 5 % slower).  3 bits in all, one call, us, with the images, before -> now: 8 codes 8.5 -> 3.4, 4096 9.5 -> 4.2, 16384
// 10.3 -> 5.5, 131072 23.8 -> 19.3, 524288 84 -> 65; 2 bits without a sketch 131072 17.4 -> 14.1.  Error against 64 bits, of a
// coordinate's root mean square: above 8192 codes 2.5 - 3.8e-6 -> 1.55e-6, up to them 0.92 - 1.17e-7 -> 0.69 - 0.78e-7.
#include <type_traits>

#include "tq_sign.h"

namespace tq {
namespace {

struct Sign128Args {
  const uint32_t* idx;
  const uint32_t* qjl;
  const float* gamma;
  const float* norm;  // nullable
  const unsigned char* image;  // OWN: not looked at
  const float* Pi;             // OWN: the matrices themselves
  const float* S;
  float* out;
  int64_t ldo, n;
  float kappa;
  SignCoefs c;
};

// The largest magnitude of 16 values and of a column, from those of the 8 parts that its 128 entries are read in
__device__ __forceinline__ float largest16(const float (&v)[16]) {
  float mx = 0.f;
#pragma unroll
  for (int e = 0; e < 16; ++e) mx = sign_larger(fabsf(v[e]), mx);
  return mx;
}
__device__ __forceinline__ float largest_part(const float (&max_s)[8][32], int l) {
  float mx = max_s[0][l];
#pragma unroll
  for (int k = 1; k < 8; ++k) mx = sign_larger(max_s[k][l], mx);
  return mx;
}
// half of a lane's 32 values of a digit: words 0..3 of a lane lie together, words 4 and 5 behind those of all lanes
__device__ __forceinline__ void put_digit(unsigned char* f, int lane, int half, const uint32_t (&w)[3]) {
  uint32_t* const lo = reinterpret_cast<uint32_t*>(f + lane * 16);
  if (half == 0) {
    lo[0] = w[0], lo[1] = w[1], lo[2] = w[2];
  } else {
    lo[3] = w[0];
    *reinterpret_cast<uint2*>(f + 1024 + lane * 8) = make_uint2(w[1], w[2]);
  }
}
// (an entry that is not finite makes its whole column NaN, as it does in a sum of pieces)
__device__ __forceinline__ float column_unit(float largest) { return largest <= 3.4e38f ? sign_unit(largest) : __builtin_nanf(""); }

// DIG: the leading digits that are used.  OWN: no images; the four wavefronts of a workgroup own the same outputs, each makes a quarter
// of their digits from the matrices, the same ones as sign128_image_kernel, and they cross through LDS: nothing outside the call's
// own output is written, so that calls on several streams may share their parameters.
template <int BITS, bool PROD, int DIG, bool OWN>
__global__ __launch_bounds__(256, 2) void sign128_dequant_kernel(const Sign128Args a) {
  __shared__ __attribute__((aligned(16))) float row_s[4][2][32];  // by wavefront: the factors of its block's codes
  constexpr int J0 = SIGN_DIGITS - DIG;
  constexpr int MATS = (BITS > 0 ? 1 : 0) + (PROD ? 1 : 0), NPL = BITS > 0 ? BITS : 1;
  typedef uint32_t w2 __attribute__((ext_vector_type(2), aligned(4)));
  typedef uint32_t w4 __attribute__((ext_vector_type(4), aligned(4)));
  const int lane = threadIdx.x & 63, l = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int id = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)));
  const int ct = OWN ? blockIdx.x & 3 : id & 3;
  const int64_t blocks = (a.n + 31) / 32, step = (gridDim.x * (blockDim.x >> 6)) >> 2;

  SignFrag frag[MATS][SIGN_DIGITS][2];
  float pi_unit = 0.f, s_unit = 0.f;  // (minus: see minus_sign_bits)
  if constexpr (OWN) {
    __shared__ __attribute__((aligned(16))) unsigned char own_s[MATS][2][DIG][SIGN_FRAG_BYTES];
    __shared__ float max_s[MATS][8][32];
    const int st = wave >> 1, half = wave & 1;
    float v[MATS][16];
#pragma unroll
    for (int m = 0; m < MATS; ++m) {
      const float* const col = (BITS > 0 && m == 0 ? a.Pi : a.S) + 32 * ct + l;
#pragma unroll
      for (int e = 0; e < 16; ++e) v[m][e] = col[(32 * (2 * h + st) + 4 * (e & 7) + 2 * half + (e >> 3)) * 128];
    }
#pragma unroll
    for (int m = 0; m < MATS; ++m) max_s[m][2 * wave + h][l] = largest16(v[m]);
    __syncthreads();
#pragma unroll
    for (int m = 0; m < MATS; ++m) {
      const float mx = largest_part(max_s[m], l);
      (BITS > 0 && m == 0 ? pi_unit : s_unit) = -column_unit(mx);
#pragma unroll
      for (int j = J0; j < SIGN_DIGITS; ++j) {
        uint32_t w[3];
        sign_digit(v[m], sign_unit(mx), j, w);
        put_digit(own_s[m][st][j - J0], lane, half, w);
      }
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < MATS; ++m)
#pragma unroll
      for (int j = J0; j < SIGN_DIGITS; ++j)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          const unsigned char* const f = own_s[m][s][j - J0];
          frag[m][j][s].a = *reinterpret_cast<const u32x4*>(f + lane * 16);
          frag[m][j][s].b = *reinterpret_cast<const uint2*>(f + 1024 + lane * 8);
        }
  } else {
#pragma unroll
    for (int m = 0; m < MATS; ++m)
#pragma unroll
      for (int j = J0; j < SIGN_DIGITS; ++j)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          const unsigned char* const f = a.image + (BITS > 0 && m == 0 ? 0 : SIGN128_BYTES) + ((s * 4 + ct) * SIGN_DIGITS + j) * SIGN_FRAG_BYTES;
          frag[m][j][s].a = *reinterpret_cast<const u32x4*>(f + lane * 16);
          frag[m][j][s].b = *reinterpret_cast<const uint2*>(f + 1024 + lane * 8);
        }
    const unsigned char* const units = a.image + sign_image_bytes(128) + (32 * ct + l) * 4;
    if constexpr (BITS > 0) pi_unit = -*reinterpret_cast<const float*>(units);
    if constexpr (PROD) s_unit = -*reinterpret_cast<const float*>(units + SIGN128_BYTES);
  }
  // the two factors in two parts each: rounded once they would be off for every code alike
  const double alpha_d = a.c.alpha * (double)pi_unit, beta_d = a.c.beta * (double)pi_unit;
  const float alpha = (float)alpha_d, beta = (float)beta_d, alpha_lo = (float)(alpha_d - (double)alpha), beta_lo = (float)(beta_d - (double)beta);

  uint32_t w[2][NPL], z[2];  // of steps 0 and 1
  float nu, nk;              // norm, norm kappa gamma of this lane's code
  auto load = [&](int64_t blk) {
    const int64_t i = blk * 32 + l, row = i < a.n ? i : a.n - 1;  // past the end: not stored
    if constexpr (BITS == 2) {
      const w4 v = *reinterpret_cast<const w4*>(a.idx + row * 8 + 4 * h);
      w[0][0] = v[0], w[0][1] = v[1], w[1][0] = v[2], w[1][1] = v[3];
    } else if constexpr (BITS == 1) {
      const w2 v = *reinterpret_cast<const w2*>(a.idx + row * 4 + 2 * h);
      w[0][0] = v[0], w[1][0] = v[1];
    }
    if constexpr (PROD) {
      const w2 v = *reinterpret_cast<const w2*>(a.qjl + row * 4 + 2 * h);
      z[0] = v[0], z[1] = v[1];
    }
    nu = a.norm != nullptr ? a.norm[row] : 1.f;
    nk = PROD ? a.gamma[row] : 0.f;
  };
  const floatx16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const uint32_t row_bytes = (uint32_t)a.ldo * 4u;
  const uint32_t lane_off = 4u * (uint32_t)h * row_bytes + 4u * (uint32_t)l;
  const uint32_t two = sign_two();
  int64_t blk = OWN ? (int64_t)(blockIdx.x >> 2) * 4 + wave : id >> 2;
  if (blk < blocks) load(blk);
  for (; blk < blocks; blk += step) {
    v8i_t sw[2][NPL], sz[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      if constexpr (BITS > 0)
#pragma unroll
        for (int p = 0; p < BITS; ++p) sw[s][p] = minus_sign_bits(w[s][p], two);
      if constexpr (PROD) sz[s] = minus_sign_bits(z[s], two);
    }
    float (&row_f)[2][32] = row_s[(threadIdx.x >> 6) & 3];
    row_f[0][l] = nu;
    if constexpr (PROD) row_f[1][l] = nu * (a.kappa * nk);
    if (blk + step < blocks) load(blk + step);  // the next block's codes travel during this one
    floatx16 acc[NPL], accz;
    auto digit = [&](auto j_c) {
      constexpr int j = decltype(j_c)::value;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        if constexpr (PROD) accz = sign_mfma<j>(sz[s], sign_operand(frag[MATS - 1][j][s]), j == J0 && s == 0 ? zero : accz);
        if constexpr (BITS > 0)
#pragma unroll
          for (int p = 0; p < BITS; ++p) acc[p] = sign_mfma<j>(sw[s][p], sign_operand(frag[0][j][s]), j == J0 && s == 0 ? zero : acc[p]);
      }
    };
    if constexpr (J0 == 0) digit(std::integral_constant<int, 0>{});
    digit(std::integral_constant<int, 1>{});
    digit(std::integral_constant<int, 2>{});
    digit(std::integral_constant<int, 3>{});
    digit(std::integral_constant<int, 4>{});
    // register r is code 8 (r / 4) + 4 h + r % 4 of the block
    float o[16];
    uint32_t off = lane_off;
    asm volatile("" : "+v"(off));  // the rows' offsets are made again in every round: kept they would be 16 registers
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const f32x4 fn = *reinterpret_cast<const f32x4*>(&row_f[0][8 * k + 4 * h]);
      f32x4 fk = fn;
      if constexpr (PROD) fk = *reinterpret_cast<const f32x4*>(&row_f[1][8 * k + 4 * h]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = 4 * k + e;
        float c = 0.f;
        if constexpr (BITS == 1) c = DIG == 5 ? fmaf(alpha, acc[0][r], alpha_lo * acc[0][r]) : alpha * acc[0][r];
        if constexpr (BITS == 2)
          c = fmaf(alpha, acc[1][r], DIG == 5 ? fmaf(beta, acc[0][r], fmaf(alpha_lo, acc[1][r], beta_lo * acc[0][r])) : beta * acc[0][r]);
        if constexpr (BITS > 0 && PROD) o[r] = fmaf(fk[e], s_unit * accz[r], fn[e] * c);
        else if constexpr (PROD) o[r] = fk[e] * (s_unit * accz[r]);
        else o[r] = fn[e] * c;
        // (formed here, not behind the branches of the stores: see settled() in tq_q128_few.hip)
        asm volatile("" : "+v"(o[r]));
      }
    }
    // the next codes have arrived by now; waited for behind the stores they would be waited for with those
    if constexpr (BITS > 0)
#pragma unroll
      for (int p = 0; p < BITS; ++p) asm volatile("" : "+v"(w[0][p]), "+v"(w[1][p]));
    if constexpr (PROD) asm volatile("" : "+v"(z[0]), "+v"(z[1]), "+v"(nk));
    asm volatile("" : "+v"(nu));
    const int64_t v0 = blk * 32;
    char* const base = reinterpret_cast<char*>(a.out + v0 * a.ldo + 32 * ct);
    if (v0 + 32 <= a.n) {  // uniform
#pragma unroll
      for (int r = 0; r < 16; ++r)
        __builtin_nontemporal_store(o[r], reinterpret_cast<float*>(base + (off + (uint32_t)(8 * (r >> 2) + (r & 3)) * row_bytes)));
    } else {
      const int left = (int)(a.n - v0);
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (8 * (r >> 2) + (r & 3) + 4 * h < left)
          __builtin_nontemporal_store(o[r], reinterpret_cast<float*>(base + (off + (uint32_t)(8 * (r >> 2) + (r & 3)) * row_bytes)));
    }
  }
}

// A workgroup per matrix, tile of 32 outputs and digit; a wavefront per step and half of a lane's 32 values (3 of a fragment's
// 6 words).
__global__ __launch_bounds__(256) void sign128_image_kernel(const float* Pi, const float* S, unsigned char* image) {
  __shared__ float max_s[8][32];
  const int j = blockIdx.x % SIGN_DIGITS, ct = (blockIdx.x / SIGN_DIGITS) & 3, m = blockIdx.x / (4 * SIGN_DIGITS);
  const int tid = threadIdx.x, lane = tid & 63, st = tid >> 7, half = (tid >> 6) & 1, l = lane & 31, h = lane >> 5, g = 2 * h + st;
  const float* const col = (m == 0 ? Pi : S) + 32 * ct + l;
  float v[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) v[e] = col[(32 * g + 4 * (e & 7) + 2 * half + (e >> 3)) * 128];
  max_s[2 * (tid >> 6) + h][l] = largest16(v);
  __syncthreads();
  const float mx = largest_part(max_s, l);
  image += m * SIGN128_BYTES;
  if (j == 0 && tid < 32) reinterpret_cast<float*>(image + sign_image_bytes(128))[32 * ct + l] = column_unit(mx);
  uint32_t w[3];
  sign_digit(v, sign_unit(mx), j, w);
  put_digit(image + ((st * 4 + ct) * SIGN_DIGITS + j) * SIGN_FRAG_BYTES, lane, half, w);
}

// Four of the five digits (20 bits: 2^-18.6 of an entry in the root mean square) where two bf16 pieces of both factors served before
// (2^-17.8 of a term), all five in place of the fp32 instructions.
template <int BITS, bool PROD, bool OWN>
hipError_t launch_digits(const Sign128Args& a, hipStream_t s) {
  // eight wavefronts per compute unit and four per block of codes; while there are fewer, each is a workgroup (OWN: four that share
  // their digits, always)
  const int64_t blocks = (a.n + 31) / 32, cu = device_cu_count();
  const int waves = !OWN && blocks * 4 <= cu ? 1 : 4;
  const int64_t groups = OWN ? (blocks + 3) / 4 * 4 : blocks * 4 / waves, most = (8 * cu / waves + 3) / 4 * 4;
  const dim3 grid((unsigned)(groups < most ? groups : most)), block(64 * waves);
  if (a.n > kBf3DequantRows) hipLaunchKernelGGL((sign128_dequant_kernel<BITS, PROD, 4, OWN>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((sign128_dequant_kernel<BITS, PROD, 5, OWN>), grid, block, 0, s, a);
  return hipGetLastError();
}

template <int BITS, bool PROD>
hipError_t launch_one(const Sign128Args& a, hipStream_t s) {
  return a.image != nullptr ? launch_digits<BITS, PROD, false>(a, s) : launch_digits<BITS, PROD, true>(a, s);
}

}  // namespace

bool sign_table(int bits, const Codebook& cb, SignCoefs* c) {
  if (bits < 0 || bits > 2) return false;
  c->alpha = c->beta = 0.;
  if (bits == 0) return true;
  const double top = cb.c[(1 << bits) - 1];
  for (int i = 0; i < 1 << bits; ++i)
    if (cb.c[i] != -cb.c[(1 << bits) - 1 - i]) return false;
  if (!(top > 1e-30 && top < 1e30)) return false;
  c->alpha = bits == 1 ? top : 0.5 * (top + cb.c[2]);
  c->beta = bits == 1 ? 0. : 0.5 * (top - cb.c[2]);
  return bits == 1 || (cb.c[2] >= 0.f && c->beta > 1e-6 * c->alpha);
}

hipError_t launch_sign128_images(const float* Pi, const float* S, void* images, hipStream_t s) {
  hipLaunchKernelGGL(sign128_image_kernel, dim3((S != nullptr ? 8 : 4) * SIGN_DIGITS), dim3(256), 0, s, Pi, S, static_cast<unsigned char*>(images));
  return hipGetLastError();
}

hipError_t launch_sign128_dequant(int bits, bool prod, const uint32_t* idx, const uint32_t* qjl, const float* gamma, const float* norm,
                                  const void* images, const float* Pi, const float* S, float* out, int64_t ldo, int64_t n, float kappa,
                                  const SignCoefs& c, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (images == nullptr && ((bits > 0 && Pi == nullptr) || (prod && S == nullptr))) return hipErrorInvalidValue;
  if (ldo < 128 || ldo > (1 << 22)) return hipErrorInvalidValue;  // 32 rows are addressed with 32-bit byte offsets
  const Sign128Args a{idx, qjl, gamma, norm, static_cast<const unsigned char*>(images), Pi, S, out, ldo, n, kappa, c};
  switch (bits * 2 + (prod ? 1 : 0)) {
    case 1: return launch_one<0, true>(a, s);
    case 2: return launch_one<1, false>(a, s);
    case 3: return launch_one<1, true>(a, s);
    case 4: return launch_one<2, false>(a, s);
    case 5: return launch_one<2, true>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace tq
