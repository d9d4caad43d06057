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

// Up to one workgroup of sign_few_kernel per compute unit, two where there is more than one stream of products, which is not enough for one bit with a
// sketch while the contraction is a step per wavefront or less.  us, sign_gemm_kernel / here:
//   2 + 1 bits           d = 256 1 code 10.0 / 3.8, 2000 11.0 / 6.0; 768 64 22.8 / 8.0, 1000 24.0 / 15.7, 1500 (2.25 workgroups) 24.4 / 22.8; 1536 200 41.8 / 12.6
//   1 + 1 bits           256 2048 (1 workgroup) 8.4 / 5.7, 2900 (1.4) 8.6 / 9.5, 4096 (2) 8.7 / 9.9; 512 1300 (1.3) 12.5 / 12.4, 2000 (2) 12.4 / 12.8; 768 1300 (2)
//                        16.5 / 14.8; 3072 64 52.2 / 24.3, 400 (2.6) 52.9 / 58.9
//   one stream           512 1000 8.1 / 5.6, 1500 (1.5) 8.3 / 9.5
//   2 bits (tq_code_gemm.hip / here)  256 4096 (2) 8.8 / 7.8; 1536 200 29.4 / 8.8, 1000 (3) 31.8 / 23.9, 1500 (4.5) 35.0 / 38.5
bool few_serves(int bits, bool prod, int d, int64_t n) {
  const int streams = bits + (prod ? 1 : 0), most = streams > 2 || streams == 2 && (!prod || d > 512) ? 2 : 1;
  return (d / 32) * ((n + 63) / 64) <= (int64_t)most * device_cu_count();
}

template <int BITS, bool PROD>
hipError_t launch_one(const SignGemmArgs& a, hipStream_t s) {
  // 512 codes per workgroup where that gives three quarters of the chip's two per compute unit, else 256 (20011 codes of 768 87 / 93 us; 3000 of
  // 1536 93 / 75)
  if (a.n <= 32) return launch_few<BITS, PROD, 1>(a, s);
  if (few_serves(BITS, PROD, a.d, a.n)) return launch_few<BITS, PROD, 2>(a, s);
  if ((int64_t)(a.d / 64) * ((a.n + 511) / 512) * 2 >= 3 * device_cu_count()) return launch_tile<BITS, PROD, 4, 4>(a, s);
  return launch_tile<BITS, PROD, 2, 4>(a, s);
}

// Few codes: a tile of 32 outputs and up to 64 codes per workgroup, the contraction split over its eight wavefronts.  Each takes every eighth step, digits
// straight into registers and one step ahead, and keeps a sum of its own per stream; the eight meet in LDS.  Bound by latency: a wavefront has d / 512 steps, and
// the matrices come once from memory for all of the chip, d <= 1536 within three trips (sign_gemm_kernel goes through the whole contraction step by step in d / 64
// workgroups: 64 codes of 1536, 2 + 1 bits, 41.7 us, here 13.0; few_serves has more).  Error of a coordinate's root mean square against 64 bits, d = 1536, 300 codes,
// sign_gemm_kernel / here: 2 + 1 bits 2.2e-7 / 1.3e-7, 1 bit 1.7e-7 / 1.2e-7; 2 bits, tq_code_gemm.hip / here: 4.4e-7 / 1.3e-7.
template <int BITS, bool PROD, int TW>
__global__ __launch_bounds__(512, 2) void sign_few_kernel(const SignGemmArgs a) {
  constexpr int NW = 8, TC = TW * 32, KINDS = (BITS > 0 ? 1 : 0) + (PROD ? 1 : 0);
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  float* const sum_s = reinterpret_cast<float*>(lds);  // [kind][wavefront][TW][16][64]
  // two neighbouring tiles, whose outputs alternate, on one XCD
  const int k8 = (int)blockIdx.x / XCDS, item = (k8 >> 1) * XCDS + (int)blockIdx.x % XCDS, pairs = a.tiles_m >> 1;
  if (item >= pairs * a.tiles_n) return;
  const int tile = 2 * (item % pairs) + (k8 & 1);
  const int tid = threadIdx.x, lane = tid & 63, l = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int S = a.d >> 6, G = a.d >> 5;
  const int64_t n0 = (int64_t)(item / pairs) * TC;
  const int rows = (int)(a.n - n0 < TC ? a.n - n0 : TC);
  const size_t step_bytes = (size_t)G * SIGN_STEP_BYTES;
  const uint32_t* at_idx[TW];
  const uint32_t* at_qjl[TW];
#pragma unroll
  for (int t = 0; t < TW; ++t) {
    const int r = t * 32 + l;
    const int64_t first = (n0 + (r < rows ? r : rows - 1)) * G + h * S;  // past the end: not stored
    at_idx[t] = BITS > 0 ? a.idx + first * BITS : nullptr;
    at_qjl[t] = PROD ? a.qjl + first : nullptr;
  }
  struct Step {
    SignFrag z[PROD ? SIGN_DIGITS : 1], p[BITS > 0 ? SIGN_DIGITS : 1];
    uint32_t zw[TW], pw[TW][BITS > 0 ? BITS : 1];
  };
  auto digits = [&](const unsigned char* image, int s, SignFrag (&o)[SIGN_DIGITS]) {
    const unsigned char* const at = image + s * step_bytes + (size_t)tile * SIGN_STEP_BYTES;
#pragma unroll
    for (int j = 0; j < SIGN_DIGITS; ++j) {
      o[j].a = *reinterpret_cast<const u32x4*>(at + j * SIGN_FRAG_BYTES + lane * 16);
      o[j].b = *reinterpret_cast<const uint2*>(at + j * SIGN_FRAG_BYTES + 1024 + lane * 8);
    }
  };
  auto load_sketch = [&](Step& f, int s) {
    if constexpr (PROD) {
#pragma unroll
      for (int t = 0; t < TW; ++t) f.zw[t] = at_qjl[t][s];
      digits(a.s, s, f.z);
    }
  };
  auto load_planes = [&](Step& f, int s) {
    if constexpr (BITS > 0) {
#pragma unroll
      for (int t = 0; t < TW; ++t)
#pragma unroll
        for (int b = 0; b < BITS; ++b) f.pw[t][b] = at_idx[t][s * BITS + b];
      digits(a.pi, s, f.p);
    }
  };
  floatx16 accz[TW], accp[BITS > 0 ? BITS : 1][TW];
#pragma unroll
  for (int t = 0; t < TW; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      accz[t][r] = 0.f;
#pragma unroll
      for (int b = 0; b < BITS; ++b) accp[b][t][r] = 0.f;
    }
  const uint32_t two = sign_two();
  auto products = [&](const v8i_t& sg, const SignFrag (&f)[SIGN_DIGITS], floatx16& acc) {
    acc = sign_mfma<0>(sg, sign_operand(f[0]), acc);
    acc = sign_mfma<1>(sg, sign_operand(f[1]), acc);
    acc = sign_mfma<2>(sg, sign_operand(f[2]), acc);
    acc = sign_mfma<3>(sg, sign_operand(f[3]), acc);
    acc = sign_mfma<4>(sg, sign_operand(f[4]), acc);
  };
  auto sketch = [&](const Step& f) {
    if constexpr (PROD)
#pragma unroll
      for (int t = 0; t < TW; ++t) products(minus_sign_bits(f.zw[t], two), f.z, accz[t]);
  };
  auto planes = [&](const Step& f) {
    if constexpr (BITS > 0)
#pragma unroll
      for (int b = 0; b < BITS; ++b)
#pragma unroll
        for (int t = 0; t < TW; ++t) products(minus_sign_bits(f.pw[t][b], two), f.p, accp[b][t]);
  };
  const size_t unit_at = (size_t)tile * SIGN_STEP_BYTES + UNITS + l * 4;
  const float pi_unit = BITS > 0 ? *reinterpret_cast<const float*>(a.pi + unit_at) : 1.f;
  const float s_unit = PROD ? *reinterpret_cast<const float*>(a.s + unit_at) : 1.f;
  if (wave < S) {
    // past the last step: it once more, not multiplied
    if constexpr (PROD && BITS > 0 && TW == 2) {  // one kind of sign ahead: registers
      Step f;
      load_sketch(f, wave);
      load_planes(f, wave);
      for (int s = wave; s < S; s += NW) {
        const int next = s + NW < S ? s + NW : s;
        __builtin_amdgcn_sched_barrier(0);
        sketch(f);
        __builtin_amdgcn_sched_barrier(0);
        load_sketch(f, next);
        __builtin_amdgcn_sched_barrier(0);
        planes(f);
        __builtin_amdgcn_sched_barrier(0);
        load_planes(f, next);
      }
    } else {
      Step f0, f1;
      auto load = [&](Step& f, int s) {
        load_sketch(f, s < S ? s : s - NW);
        load_planes(f, s < S ? s : s - NW);
        __builtin_amdgcn_sched_barrier(0);
      };
      load(f0, wave);
      for (int s = wave;; s += 2 * NW) {
        load(f1, s + NW);
        sketch(f0);
        planes(f0);
        __builtin_amdgcn_sched_barrier(0);
        if (s + NW >= S) break;
        load(f0, s + 2 * NW);
        sketch(f1);
        planes(f1);
        __builtin_amdgcn_sched_barrier(0);
        if (s + 2 * NW >= S) break;
      }
    }
  }
  // ---- (minus: see minus_sign_bits) ----
  const float upper = -(float)(a.c.alpha * (double)pi_unit), lower = -(float)(a.c.beta * (double)pi_unit);
  auto put = [&](int kind, int t, int r, float v) { sum_s[(((kind * NW + wave) * TW + t) * 16 + r) * 64 + lane] = v; };
#pragma unroll
  for (int t = 0; t < TW; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      if constexpr (BITS == 1) put(0, t, r, upper * accp[0][t][r]);
      if constexpr (BITS == 2) put(0, t, r, fmaf(upper, accp[1][t][r], lower * accp[0][t][r]));
      if constexpr (PROD) put(KINDS - 1, t, r, -s_unit * accz[t][r]);
    }
  __syncthreads();
  const int m = 64 * (tile >> 1) + (tile & 1) + 2 * l;
  for (int e = wave; e < TW * 16; e += NW) {
    const int t = e >> 4, r = e & 15, c = 32 * t + 8 * (r >> 2) + 4 * h + (r & 3);
    float v[KINDS];
#pragma unroll
    for (int kind = 0; kind < KINDS; ++kind) {
      v[kind] = sum_s[(kind * NW * TW * 16 + e) * 64 + lane];
#pragma unroll
      for (int w = 1; w < NW; ++w) v[kind] += sum_s[((kind * NW + w) * TW * 16 + e) * 64 + lane];
    }
    if (c < rows) {
      const float nu = a.norm != nullptr ? a.norm[n0 + c] : 1.f, kg = PROD ? a.kappa * a.gamma[n0 + c] : 0.f;
      const float sum = !PROD ? v[0] : BITS > 0 ? fmaf(kg, v[KINDS - 1], v[0]) : kg * v[0];
      a.out[(n0 + c) * a.ldo + m] = nu * sum;
    }
  }
}

template <int BITS, bool PROD, int TW>
hipError_t launch_few(SignGemmArgs a, hipStream_t s) {
  constexpr int LDS = ((BITS > 0 ? 1 : 0) + (PROD ? 1 : 0)) * 8 * TW * 16 * 64 * 4;
  a.tiles_m = a.d / 32;  // even
  a.tiles_n = (int)((a.n + 32 * TW - 1) / (32 * TW));
  static LdsLimit lds_limit;  // per instantiation: the limit is raised once per device
  if (const hipError_t e = raise_lds_limit(lds_limit, reinterpret_cast<const void*>(&sign_few_kernel<BITS, PROD, TW>), LDS); e != hipSuccess) return e;
  const dim3 grid((a.tiles_m / 2 * a.tiles_n + XCDS - 1) / XCDS * 2 * XCDS);
  hipLaunchKernelGGL((sign_few_kernel<BITS, PROD, TW>), grid, dim3(512), LDS, s, a);
  return hipGetLastError();
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
// between few codes and 2^20 coordinates these have the smaller tiles (768 coordinates: 1000 codes 16.8 us, 17.0 with sign_gemm_kernel; 3000 24.2, 18.1).
bool sign_gemm_serves(int bits, bool prod, int d, int64_t n) {
  return sign_gemm_images(d) && (prod || bits != 2 || few_serves(bits, prod, d, n) || n * d >= 1 << 20);
}

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
