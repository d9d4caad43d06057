// DeQuant of codes whose table is a sum of signs (tq_sign.h) at d = 256, 384, ...: signs against digits, a stream of products per kind of sign.
//
// The sketch goes first, then the planes from the lower one up: between two streams the sums are multiplied by what the units of the
// one are in units of the next (per code and output after the sketch), so that one set of accumulators does.  The digits of 64
// contraction indices of the workgroup's outputs lie in LDS, the next ones on their way by direct loads; a code's signs come out of its words in
// registers, seven instructions per 32 of them, and serve all five digits and two tiles of outputs.
//
// Workgroup: four wavefronts of TW tiles of 32 codes, 64 outputs: few outputs for many codes, so that little comes through L2 (256 codes x 256
// outputs, eight wavefronts: 115 us where this takes 87), and two workgroups per compute unit, of which one multiplies while the other
// waits at its barrier.  Two steps of 64 contraction indices per barrier, fragments asked for one digit ahead.
//
// Bound by the matrix instructions: at their rate in registers, which the chip's power sets (6.6 PFLOP/s with signs against digits), 20011
// codes of 768, 2 + 1 bits, take 55 us, their stores 13.  Before -> now, us: that 106 -> 87, 1 + 1 bits 84 -> 57, 1 bit 50 -> 34; 3000 codes
// of 1536, 2 + 1 bits 159 -> 75; 100000 of 384 218 -> 115; 20011 of 3072 1594 -> 1340.  Error against 64 bits, of a
// coordinate's root mean square: d = 768, 2 + 1 bits 3.5e-7 -> 1.7e-7; 3072 6.9e-7 -> 3.2e-7.
#include <type_traits>

#include "tq_sign.h"

namespace tq {
namespace {

constexpr int XCDS = 8;

// Behind a tile's digits of a step: 32 floats for the largest magnitudes of its outputs in 64 rows, and at step 0 32 more, the units.
// Output of lane l of tile t: 64 (t / 2) + 2 l + t % 2.
constexpr int LARGEST = SIGN_DIGITS * SIGN_FRAG_BYTES, UNITS = LARGEST + 128;
static_assert(UNITS + 128 <= SIGN_STEP_BYTES, "space behind the digits");

struct SignGemmArgs {
  const unsigned char* pi;
  const unsigned char* s;
  const uint32_t* idx;
  const uint32_t* qjl;
  const float* gamma;
  const float* norm;  // nullable
  float* out;
  int64_t ldo, n;
  int d, tiles_m, tiles_n, per_xcd;
  float kappa;
  SignCoefs c;
};

template <int BITS, bool PROD, int TW, int WC>
__global__ __launch_bounds__(64 * WC, 2) void sign_gemm_kernel(const SignGemmArgs a) {
  constexpr int TC = WC * TW * 32, TO = 64, STEP = 2 * SIGN_STEP_BYTES, BUF = 2 * STEP, LOADS = 16 / WC;
  constexpr int STREAMS = BITS + (PROD ? 1 : 0);
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
  float* const first_s = reinterpret_cast<float*>(lds + 2 * BUF);  // [TC] of the sketch sums
  float* const last_s = first_s + TC;                              // [TC] of everything

  const int total = a.tiles_m * a.tiles_n;
  const int logical = (int)(blockIdx.x % XCDS) * a.per_xcd + (int)(blockIdx.x / XCDS);
  if (logical >= total) return;
  const int tile_m = logical % a.tiles_m, tile_n = logical / a.tiles_m;
  const int tid = threadIdx.x, lane = tid & 63, l = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int S = a.d >> 6, G = a.d >> 5;  // S even
  const int64_t n0 = (int64_t)tile_n * TC;
  const int rows = (int)(a.n - n0 < TC ? a.n - n0 : TC);

  // ---- digits: direct loads ------------------------------------------
  uint32_t voff[LOADS];
#pragma unroll
  for (int j = 0; j < LOADS; ++j) {
    const int kb = wave * LOADS + j;
    voff[j] = (uint32_t)(2 * tile_m) * SIGN_STEP_BYTES + kb * 1024 + lane * 16;
  }
  const uint32_t lds0 = h2_lds_address(lds);
  const size_t step_bytes = (size_t)G * SIGN_STEP_BYTES;
  int ask_stream = 0, ask_step = 0;
  const unsigned char* ask = PROD ? a.s : a.pi;
  auto dma = [&](int buf) {
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int j = 0; j < LOADS; ++j) h2_dma(ask + k * step_bytes, voff[j], lds0 + buf * BUF + k * STEP + (wave * LOADS + j) * 1024);
    ask_step += 2;
    if (ask_step < S) {
      ask += 2 * step_bytes;
    } else if (ask_stream + 1 < STREAMS) {
      ++ask_stream;
      ask_step = 0;
      ask = a.pi;
    } else {
      ask_step -= 2;  // the last steps are asked for again
    }
  };

  // ---- codes: the words of two steps -----------------------------------------------------------------------
  struct Pair {
    uint32_t w[TW][2];
  };
  int64_t row[TW];
#pragma unroll
  for (int t = 0; t < TW; ++t) {
    const int r = (wave * TW + t) * 32 + l;
    row[t] = n0 + (r < rows ? r : rows - 1);  // past the end: not stored
  }
  int word_stream = 0, word_step = 0;
  auto load = [&](Pair& p) {
    const bool sketch = PROD && word_stream == 0;  // uniform
    const uint32_t* const base = sketch ? a.qjl : a.idx + (word_stream - (PROD ? 1 : 0));
    const int per = sketch ? 1 : BITS;  // words of a group
#pragma unroll
    for (int t = 0; t < TW; ++t) {
      const uint32_t* const w = base + (row[t] * G + h * S + word_step) * per;
      p.w[t][0] = w[0];
      p.w[t][1] = w[per];
    }
    word_step += 2;
    if (word_step == S) {
      if (word_stream + 1 < STREAMS) {
        ++word_stream;
        word_step = 0;
      } else {
        word_step -= 2;
      }
    }
  };
  auto arrived = [&](Pair& p) {
#pragma unroll
    for (int t = 0; t < TW; ++t) asm volatile("" : "+v"(p.w[t][0]), "+v"(p.w[t][1]));
  };

  floatx16 acc[TW][2];
#pragma unroll
  for (int t = 0; t < TW; ++t)
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[t][u][r] = 0.f;
  const uint32_t two = sign_two();
  // ten products of a digit: the next one's fragments are on their way from LDS during each
  auto compute = [&](int buf, const Pair& p) {
    auto fragments = [&](int i, SignFrag (&f)[2]) {  // i: digit + 5 step
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const unsigned char* const at = lds + buf * BUF + (i / SIGN_DIGITS) * STEP + u * SIGN_STEP_BYTES + (i % SIGN_DIGITS) * SIGN_FRAG_BYTES;
        f[u].a = *reinterpret_cast<const u32x4*>(at + lane * 16);
        f[u].b = *reinterpret_cast<const uint2*>(at + 1024 + lane * 8);
      }
    };
    v8i_t sg[TW];
    SignFrag f[2][2];
    fragments(0, f[0]);
    auto digit = [&](auto i_c) {
      constexpr int i = decltype(i_c)::value, j = i % SIGN_DIGITS;
      if constexpr (i + 1 < 2 * SIGN_DIGITS) fragments(i + 1, f[(i + 1) & 1]);
      if constexpr (j == 0)
#pragma unroll
        for (int t = 0; t < TW; ++t) sg[t] = minus_sign_bits(p.w[t][i / SIGN_DIGITS], two);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int t = 0; t < TW; ++t) acc[t][u] = sign_mfma<j>(sg[t], sign_operand(f[i & 1][u]), acc[t][u]);
      __builtin_amdgcn_sched_barrier(0);
    };
    digit(std::integral_constant<int, 0>{});
    digit(std::integral_constant<int, 1>{});
    digit(std::integral_constant<int, 2>{});
    digit(std::integral_constant<int, 3>{});
    digit(std::integral_constant<int, 4>{});
    digit(std::integral_constant<int, 5>{});
    digit(std::integral_constant<int, 6>{});
    digit(std::integral_constant<int, 7>{});
    digit(std::integral_constant<int, 8>{});
    digit(std::integral_constant<int, 9>{});
  };

  Pair cur, nxt;
  int buf = 0;
  load(nxt);
  dma(0);
  float pi_unit[2], s_unit[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const size_t at = (size_t)(2 * tile_m + u) * SIGN_STEP_BYTES + UNITS + l * 4;
    pi_unit[u] = BITS > 0 ? *reinterpret_cast<const float*>(a.pi + at) : 1.f;
    s_unit[u] = PROD ? *reinterpret_cast<const float*>(a.s + at) : 1.f;
  }
  for (int c = tid; c < TC; c += 64 * WC) {
    const int64_t r = n0 + (c < rows ? c : rows - 1);
    const float nu = a.norm != nullptr ? a.norm[r] : 1.f, kg = PROD ? a.kappa * a.gamma[r] : 1.f;
    first_s[c] = kg;
    last_s[c] = BITS > 0 ? nu : nu * kg;
  }
  // what a unit of the sums stands for in the planes' first stream and in the last
  const double first_c = BITS == 2 ? a.c.beta : a.c.alpha;
#pragma unroll
  for (int k = 0; k < STREAMS; ++k) {
#pragma unroll 1
    for (int s = 0; s < S; s += 2) {
      h2_wait_barrier<0>();
      arrived(nxt);
      cur = nxt;
      dma(buf ^ 1);
      load(nxt);
      compute(buf, cur);
      buf ^= 1;
    }
    if (PROD && BITS > 0 && k == 0) {
      float per[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) per[u] = (float)((double)s_unit[u] / (first_c * (double)pi_unit[u]));
#pragma unroll
      for (int t = 0; t < TW; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 f = *reinterpret_cast<const f32x4*>(first_s + (wave * TW + t) * 32 + 8 * q + 4 * h);
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int u = 0; u < 2; ++u) acc[t][u][4 * q + e] *= f[e] * per[u];
        }
    } else if (k + 1 < STREAMS) {
      const float per = (float)(a.c.beta / a.c.alpha);
#pragma unroll
      for (int t = 0; t < TW; ++t)
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[t][u][r] *= per;
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // nothing of this workgroup's is under way to LDS when it ends

  // ---- a lane has 16 codes of two neighbouring outputs, a half-wave stores 256 bytes of a row ----------------
  float per[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) per[u] = -(BITS > 0 ? (float)(a.c.alpha * (double)pi_unit[u]) : s_unit[u]);  // (minus: see minus_sign_bits)
  const int m = tile_m * TO + 2 * l;
  typedef float f32x2 __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int t = 0; t < TW; ++t)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int c = (wave * TW + t) * 32 + 8 * q + 4 * h;
      const f32x4 f = *reinterpret_cast<const f32x4*>(last_s + c);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        f32x2 o = {f[e] * (per[0] * acc[t][0][4 * q + e]), f[e] * (per[1] * acc[t][1][4 * q + e])};
        asm volatile("" : "+v"(o));  // (formed here, not behind the branch of its store)
        if (c + e < rows) __builtin_nontemporal_store(o, reinterpret_cast<f32x2*>(a.out + (n0 + c + e) * a.ldo + m));
      }
    }
}

template <int BITS, bool PROD, int TW, int WC>
hipError_t launch_tile(SignGemmArgs a, hipStream_t s) {
  constexpr int TC = WC * TW * 32, LDS = 8 * SIGN_STEP_BYTES + 2 * TC * 4;
  a.tiles_m = a.d / 64;
  const int64_t tiles_n = (a.n + TC - 1) / TC;
  if (tiles_n * a.tiles_m > (int64_t)1 << 30) return hipErrorInvalidValue;
  a.tiles_n = (int)tiles_n;
  a.per_xcd = (a.tiles_m * a.tiles_n + XCDS - 1) / XCDS;
  static LdsLimit lds_limit;  // per instantiation: the limit is raised once per device
  if (const hipError_t e = raise_lds_limit(lds_limit, reinterpret_cast<const void*>(&sign_gemm_kernel<BITS, PROD, TW, WC>), LDS); e != hipSuccess)
    return e;
  hipLaunchKernelGGL((sign_gemm_kernel<BITS, PROD, TW, WC>), dim3(a.per_xcd * XCDS), dim3(64 * WC), LDS, s, a);
  return hipGetLastError();
}

template <int BITS, bool PROD>
hipError_t launch_one(const SignGemmArgs& a, hipStream_t s) {
  // 512 codes per workgroup where that gives three quarters of the chip's two per compute unit, else 256 (20011 codes of 768 87 / 93 us; 3000 of
  // 1536 93 / 75)
  if ((int64_t)(a.d / 64) * ((a.n + 511) / 512) * 2 >= 3 * device_cu_count()) return launch_tile<BITS, PROD, 4, 4>(a, s);
  return launch_tile<BITS, PROD, 2, 4>(a, s);
}

// a workgroup for 64 rows and two tiles
__global__ __launch_bounds__(256) void sign_gemm_largest_kernel(const float* __restrict__ W, const int d, unsigned char* image) {
  __shared__ float max_s[4][64];
  const int st = blockIdx.x, pair = blockIdx.y, c = threadIdx.x & 63, part = threadIdx.x >> 6;
  const float* const at = W + (int64_t)(64 * st + 16 * part) * d + 64 * pair + c;
  float v[16], mx = 0.f;
#pragma unroll
  for (int j = 0; j < 16; ++j) v[j] = fabsf(at[(int64_t)j * d]);
#pragma unroll
  for (int j = 0; j < 16; ++j) mx = sign_larger(v[j], mx);
  max_s[part][c] = mx;
  __syncthreads();
  if (part != 0) return;
#pragma unroll
  for (int k = 1; k < 4; ++k) mx = sign_larger(max_s[k][c], mx);
  reinterpret_cast<float*>(image + ((size_t)st * (d >> 5) + 2 * pair + (c & 1)) * SIGN_STEP_BYTES + LARGEST)[c >> 1] = mx;
}

// a workgroup per step and tile, a wavefront per digit (two tiles each, their 8 bytes in one load, were a longer chain: 3072 x 3072 39 us
// against 30)
__global__ __launch_bounds__(64 * SIGN_DIGITS) void sign_gemm_image_kernel(const float* __restrict__ W, const int d, unsigned char* image) {
  const int st = blockIdx.x, t = blockIdx.y, lane = threadIdx.x & 63, j = threadIdx.x >> 6, l = lane & 31, h = lane >> 5;
  const int S = d >> 6, g = h * S + st;
  const size_t step_bytes = (size_t)(d >> 5) * SIGN_STEP_BYTES;
  unsigned char* const tile = image + (size_t)t * SIGN_STEP_BYTES;
  const float* const col = W + 64 * (t >> 1) + 2 * l + (t & 1);
  float v[32], mx = 0.f;
#pragma unroll
  for (int e = 0; e < 32; ++e) v[e] = col[(int64_t)(32 * g + 4 * (e & 7) + (e >> 3)) * d];
#pragma unroll 4
  for (int k = 0; k < S; ++k) mx = sign_larger(reinterpret_cast<const float*>(tile + k * step_bytes + LARGEST)[l], mx);
  int e2;
  (void)frexpf(fmaxf(sign_unit(mx), 1e-20f), &e2);  // the unit 2^e2: the digits below are exact in fp32
  // (an entry that is not finite makes its whole output NaN, as it does in a sum of pieces)
  if (st == 0 && j == 0 && h == 0) reinterpret_cast<float*>(tile + UNITS)[l] = mx <= 3.4e38f ? ldexpf(1.f, e2) : __builtin_nanf("");
  const float scale = ldexpf(1.f, -20 - e2);
  uint32_t w[6] = {0u, 0u, 0u, 0u, 0u, 0u};
#pragma unroll
  for (int e = 0; e < 32; ++e) {
    float x = v[e] * scale, digit = rintf(x);  // from the leading digit down
    for (int k = SIGN_DIGITS - 1; k > j; --k) {
      x = (x - digit) * 32.f;
      digit = rintf(x);
    }
    const int q = (int)fminf(fmaxf(digit, -16.f), 16.f);
    const uint32_t code = q < 0 ? 32u - (uint32_t)q : (uint32_t)q;
    const int at = 6 * e;
    w[at >> 5] |= code << (at & 31);
    if ((at & 31) > 26) w[(at >> 5) + 1] |= code >> (32 - (at & 31));
  }
  unsigned char* const f = tile + st * step_bytes + j * SIGN_FRAG_BYTES;
  *reinterpret_cast<uint4*>(f + lane * 16) = make_uint4(w[0], w[1], w[2], w[3]);
  *reinterpret_cast<uint2*>(f + 1024 + lane * 8) = make_uint2(w[4], w[5]);
}

}  // namespace

bool sign_gemm_images(int d) { return d >= 256 && d % 128 == 0; }

// Two bits without a sketch are two streams, ten products of a digit, where fp16 pieces take three products of twice the steps' length each:
// below 2^20 coordinates these have the smaller tiles (768 coordinates: 100 codes 14.9 us, 16.4 here; 1000 16.8, 17.0; 3000 24.2, 18.1).
// Everything else is faster here from the first code on (1 + 1 bits: 65 codes of 256 8.8 -> 8.1, of 3072 97 -> 53).
bool sign_gemm_serves(int bits, bool prod, int d, int64_t n) { return sign_gemm_images(d) && (prod || bits != 2 || n * d >= 1 << 20); }

hipError_t launch_sign_gemm_image(const float* W, int d, void* image, hipStream_t s) {
  if (d < 256 || d % 128 != 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(sign_gemm_largest_kernel, dim3(d / 64, d / 64), dim3(256), 0, s, W, d, static_cast<unsigned char*>(image));
  hipLaunchKernelGGL(sign_gemm_image_kernel, dim3(d / 64, d / 32), dim3(64 * SIGN_DIGITS), 0, s, W, d, static_cast<unsigned char*>(image));
  return hipGetLastError();
}

hipError_t launch_sign_gemm(int bits, bool prod, const void* pi_image, const void* s_image, int d, const uint32_t* idx, const uint32_t* qjl,
                            const float* gamma, const float* norm, int64_t n, float* out, int64_t ldo, float kappa, const SignCoefs& c, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (d < 256 || d % 128 != 0 || d > 16384) return hipErrorInvalidValue;
  SignGemmArgs a{};
  a.pi = static_cast<const unsigned char*>(pi_image); a.s = static_cast<const unsigned char*>(s_image); a.idx = idx; a.qjl = qjl; a.gamma = gamma;
  a.norm = norm; a.out = out; a.ldo = ldo; a.n = n; a.d = d; a.kappa = kappa; a.c = c;
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
