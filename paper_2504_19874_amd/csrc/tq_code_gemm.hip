// Packed codes against the rows of a fixed operand, both as fp16 pieces (tq_h2.h), on v_mfma_f32_32x32x16_f16.
//
// The fixed operand (rows of Pi^T and S^T as two pieces each, or queries as one) comes in the contraction's own order and moves to
// LDS by direct loads.  The codes are decoded on their way there: a thread has the plane words of one code and one half of a
// group of 32 coordinates; the bits of four coordinates (same bit position of the four bytes of a word) make four table
// selectors, v_perm_b32 looks the bytes of the centroids' pieces up in registers, the sign is the top plane, and two more
// permutes join bytes to fp16 values: 13 instructions per four coordinates and piece pair, no table in memory.  Signs (and a
// 1-bit table) are +-1 with one piece.
//
// Two-stage codes need one accumulator set: the sketch segment goes first, its sums are multiplied by the code's
// kappa gamma (in units of the other segment), and the centroid segment is added on top.
//
// Tile TM x TN per workgroup of WM x WN wavefronts (256 x 256: 64 x 128 per wavefront, twelve 16-byte LDS reads feed 24
// matrix instructions with two pieces on both sides), k in steps of 32 through NS buffers, one barrier per step.
#include <cmath>
#include <cstring>

#include "tq_code_decode.h"
#include "tq_d128_tile.h"

#include <type_traits>

namespace tq {
namespace {

constexpr int XCDS = 8;

struct CodeGemmArgs {
  const unsigned char* WS;  // sketch segment (PROD), centroid segment
  const unsigned char* WP;
  const float* ws_inv;      // device: 1 / scale of the two images
  const float* wp_inv;
  int M, d;
  const uint32_t* idx;
  const uint32_t* qjl;
  const float* gamma;
  const float* norm;
  int64_t n;
  float kappa;
  CodeTable tab;
  float* out;
  int64_t ldo;
  int tiles_m, tiles_n, per_xcd;
};

template <int BITS, bool PROD, int TW, int WM, int WN, int NBUF>
struct CodeCfg {
  static constexpr int UW = WM;  // so that every thread decodes half a group of one code per step
  static constexpr int THREADS = 64 * WM * WN, TM = WM * TW * 32, TN = WN * UW * 32;
  static constexpr int NPA = 2, NPB = BITS >= 2 ? 2 : 1;
  static constexpr int A_BYTES = TM * 64 * NPA, B_BYTES = TN * 64 * NPB;
  static constexpr int NS = NBUF;
  static constexpr int LDS = NS * (A_BYTES + B_BYTES) + 2 * TN * 4;
  static constexpr int LOADERS = A_BYTES / 1024 < WM * WN ? A_BYTES / 1024 : WM * WN;  // wavefronts that load the fixed operand
  static constexpr int AL = A_BYTES / 1024 / LOADERS;                                  // their direct loads per step
  static_assert(THREADS == 2 * TN && AL * LOADERS * 1024 == A_BYTES, "roles");
};

template <int BITS, bool PROD, int TW, int WM, int WN, int NBUF>
__global__ __launch_bounds__(64 * WM * WN, 2) void code_gemm_kernel(const CodeGemmArgs a) {
  using C = CodeCfg<BITS, PROD, TW, WM, WN, NBUF>;
  constexpr int UW = C::UW, TM = C::TM, TN = C::TN, NPA = C::NPA, NPB = C::NPB, NS = C::NS, AL = C::AL;
  constexpr bool HAVE_P = BITS > 0, HAVE_S = PROD;
  constexpr int NW = BITS > 0 ? BITS : 1;
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
  float* const first_s = reinterpret_cast<float*>(lds + NS * (C::A_BYTES + C::B_BYTES));  // [TN] factor of the sketch sums
  float* const last_s = first_s + TN;                                                     // [TN] factor of everything

  const int total = a.tiles_m * a.tiles_n;
  const int logical = (int)(blockIdx.x % XCDS) * a.per_xcd + (int)(blockIdx.x / XCDS);
  if (logical >= total) return;
  const int tile_m = logical % a.tiles_m, tile_n = logical / a.tiles_m;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int l32 = lane & 31, h = lane >> 5;
  const int m0 = tile_m * TM;
  const int64_t n0 = (int64_t)tile_n * TN;
  const int rows_m = min(TM, a.M - m0);
  const int rows_n = (int)min((int64_t)TN, a.n - n0);
  const int G = a.d >> 5;
  const int n_s = HAVE_S ? G : 0, n_steps = n_s + (HAVE_P ? G : 0);

  // ---- fixed operand: direct loads -------------------------------------------------------------------
  const uint32_t row_a = (uint32_t)a.d * (2u * NPA);
  const unsigned char* const gP = a.WP + (int64_t)m0 * row_a;
  const unsigned char* gA = HAVE_S ? a.WS + (int64_t)m0 * row_a : gP;
  uint32_t va[AL];
  {
    const int l8 = lane >> 3, slot = lane & 7;
#pragma unroll
    for (int j = 0; j < AL; ++j) {
      const int line = (wave * AL + j) * 8 + l8;
      const int r = NPA == 2 ? line : 2 * line + (slot >> 2);
      va[j] = (uint32_t)min(r, rows_m - 1) * row_a + h2_chunk<NPA>(r, slot) * 16;
    }
  }
  const uint32_t lds0 = h2_lds_address(lds);
  int a_step = 0;
  auto dma = [&](int buf) {
    if (C::LOADERS == WM * WN || wave < C::LOADERS)  // (a wavefront without loads waits for fewer than it may: nothing to wait for)
#pragma unroll
      for (int j = 0; j < AL; ++j) h2_dma(gA, va[j], lds0 + buf * C::A_BYTES + (wave * AL + j) * 1024);
    if (a_step + 1 < n_steps) {  // the last step is requested again and again
      ++a_step;
      gA += 64 * NPA;
      if (HAVE_S && HAVE_P && a_step == n_s) gA = gP;
    }
  };

  // ---- codes -----------------------------------------------------------------------------------------
  // (the two threads of a code side by side: its words are then one request, not two from wavefronts that meet the line apart: 551204 codes
  // of 768, 3 + 1 bits 2698 -> 2664 us, 413072 of 256, 4 bits 210 -> 205)
  const int code = tid >> 1, half = tid & 1;
  const int64_t row = n0 + min(code, rows_n - 1);  // codes past the end: the last one again, not stored
  const uint32_t* const widx = HAVE_P ? a.idx + row * G * BITS : nullptr;
  const uint32_t* const wz = HAVE_S ? a.qjl + row * G : nullptr;
  uint32_t words[NS][NW];
  int w_step = 0;
  // in_s: the step that is under way belongs to the sketch segment (later ones may not)
  auto load_step = [&](uint32_t (&w)[NW], auto in_s) {
    const int j = w_step < n_steps ? w_step : n_steps - 1;
    if (decltype(in_s)::value && (!HAVE_P || j < n_s)) w[0] = wz[j];
    else if constexpr (HAVE_P) load_plane_words<BITS>(widx + (j - n_s) * BITS, w);
    ++w_step;
  };
  const uint32_t b_at = h2_place<NPB>(code, 2 * half);
  int b_step = 0;
  auto decode_step = [&](int buf, const uint32_t (&w)[NW], auto in_s) {
    unsigned char* const bb = lds + NS * C::A_BYTES + buf * C::B_BYTES;
    if (decltype(in_s)::value && (!HAVE_P || b_step < n_s)) {
      uint32_t v[1][8];
      decode16<1, 1>(w, half, a.tab, v);
      *reinterpret_cast<uint4*>(bb + b_at) = make_uint4(v[0][0], v[0][1], v[0][2], v[0][3]);
      *reinterpret_cast<uint4*>(bb + (b_at ^ 16)) = make_uint4(v[0][4], v[0][5], v[0][6], v[0][7]);
    } else if constexpr (HAVE_P) {
      uint32_t v[NPB][8];
      decode16<BITS, NPB>(w, half, a.tab, v);
#pragma unroll
      for (int p = 0; p < NPB; ++p) {
        *reinterpret_cast<uint4*>(bb + (b_at ^ (64 * p))) = make_uint4(v[p][0], v[p][1], v[p][2], v[p][3]);
        *reinterpret_cast<uint4*>(bb + (b_at ^ (64 * p) ^ 16)) = make_uint4(v[p][4], v[p][5], v[p][6], v[p][7]);
      }
    }
    ++b_step;
  };

  // ---- fragments and products --------------------------------------------------------------------------
  const unsigned char *pa[NPA][2], *pb[NPB][2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
#pragma unroll
    for (int p = 0; p < NPA; ++p) pa[p][s] = lds + h2_place<NPA>(wm * TW * 32 + l32, p * 4 + s * 2 + h);
#pragma unroll
    for (int p = 0; p < NPB; ++p) pb[p][s] = lds + NS * C::A_BYTES + h2_place<NPB>(wn * UW * 32 + l32, p * 4 + s * 2 + h);
  }
  floatx16 acc[TW][UW];
#pragma unroll
  for (int t = 0; t < TW; ++t)
#pragma unroll
    for (int u = 0; u < UW; ++u)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[t][u][r] = 0.f;
  auto compute = [&](int buf, auto np_c) {
    constexpr int NP = decltype(np_c)::value;  // pieces of the code side in this segment
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      f16x8 fa[TW][NPA], fb[UW][NP];
      auto read_a = [&](int p) {
#pragma unroll
        for (int t = 0; t < TW; ++t) fa[t][p] = *reinterpret_cast<const f16x8*>(pa[p][s] + buf * C::A_BYTES + t * (2048 * NPA));
      };
      auto read_b = [&](int p) {
#pragma unroll
        for (int u = 0; u < UW; ++u) fb[u][p] = *reinterpret_cast<const f16x8*>(pb[p][s] + buf * C::B_BYTES + u * (2048 * NPB));
      };
      auto product = [&](int p, int q) {
#pragma unroll
        for (int t = 0; t < TW; ++t)
#pragma unroll
          for (int u = 0; u < UW; ++u)
            acc[t][u] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fb[u][q], fa[t][p], acc[t][u], 0, 0, 0);
      };
      if (NPA == 2) read_a(NPA - 1);
      read_b(0);
      read_a(0);
      if (NP == 2) read_b(NP - 1);
      if (NPA == 2) product(NPA - 1, 0);
      if (NP == 2) product(0, NP - 1);
      product(0, 0);
    }
  };

  // ---- the pipeline ------------------------------------------------------------------------------------
#pragma unroll
  for (int i = 0; i < NS; ++i) load_step(words[i], std::bool_constant<HAVE_S>{});
#pragma unroll
  for (int i = 0; i + 1 < NS; ++i) dma(i);
  {
    const float pi = HAVE_P ? a.wp_inv[0] * a.tab.inv : 1.f;
    const float si = HAVE_S ? a.ws_inv[0] : 1.f;
    for (int c = tid; c < TN; c += C::THREADS) {
      const int64_t r = n0 + min(c, rows_n - 1);
      const float nu = a.norm != nullptr ? a.norm[r] : 1.f;
      const float kg = HAVE_S ? a.kappa * a.gamma[r] : 0.f;
      first_s[c] = HAVE_P ? kg * si / pi : 1.f;
      last_s[c] = HAVE_P ? nu * pi : nu * (kg * si);
    }
  }
  decode_step(0, words[0], std::bool_constant<HAVE_S>{});
  h2_wait_barrier<0>();
  auto scale = [&] {  // the sketch sums in units of the centroid segment
#pragma unroll
    for (int u = 0; u < UW; ++u)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float4 f = *reinterpret_cast<const float4*>(first_s + wn * UW * 32 + u * 32 + 8 * k + 4 * h);
#pragma unroll
        for (int t = 0; t < TW; ++t) {
          acc[t][u][4 * k] *= f.x;
          acc[t][u][4 * k + 1] *= f.y;
          acc[t][u][4 * k + 2] *= f.z;
          acc[t][u][4 * k + 3] *= f.w;
        }
      }
  };
  auto step = [&](auto buf_c, auto in_s) {
    constexpr int buf = decltype(buf_c)::value;
    dma((buf + NS - 1) % NS);
    load_step(words[buf], in_s);
    decode_step((buf + 1) % NS, words[(buf + 1) % NS], in_s);
    compute(buf, std::integral_constant<int, decltype(in_s)::value ? 1 : NPB>{});
    h2_wait_barrier<(NS - 2) * (AL + 1) + 1>();
  };
  // (two loops: with the segments' products in two arms of one loop the accumulators are copied between them)
  auto round = [&](auto in_s) {  // one step in each buffer
    step(std::integral_constant<int, 0>{}, in_s);
    step(std::integral_constant<int, 1>{}, in_s);
    if constexpr (NS == 4) {
      step(std::integral_constant<int, 2>{}, in_s);
      step(std::integral_constant<int, 3>{}, in_s);
    }
  };
  int left = HAVE_P ? G : 0;
  if constexpr (HAVE_S) {
    int st = 0;
    for (; st + NS <= n_s; st += NS) round(std::true_type{});
    if constexpr (NS == 2)  // with four buffers the number of groups is a multiple of four
      if (st < n_s) step(std::integral_constant<int, 0>{}, std::true_type{});
    if constexpr (HAVE_P) {
      scale();
      if constexpr (NS == 2)
        if (st < n_s) {
          step(std::integral_constant<int, 1>{}, std::false_type{});
          --left;
        }
    }
  }
  if constexpr (HAVE_P) {
    for (; left >= NS; left -= NS) round(std::false_type{});
    if constexpr (NS == 2)
      if (left > 0) step(std::integral_constant<int, 0>{}, std::false_type{});
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // nothing of this workgroup's is under way to LDS when it ends

  // ---- x~ = nu acc: a lane has 16 codes of one coordinate, a half-wave stores 128 bytes of a row ----------
#pragma unroll
  for (int u = 0; u < UW; ++u)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int c = wn * UW * 32 + u * 32 + 8 * k + 4 * h;
      const float4 f = *reinterpret_cast<const float4*>(last_s + c);
      const float fe[4] = {f.x, f.y, f.z, f.w};
#pragma unroll
      for (int t = 0; t < TW; ++t) {
        const int m = (wm * TW + t) * 32 + l32;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (c + e < rows_n && m < rows_m) a.out[(n0 + c + e) * a.ldo + m0 + m] = acc[t][u][4 * k + e] * fe[e];
      }
    }
}

template <int BITS, bool PROD, int TW, int WM, int WN, int NBUF>
hipError_t launch_tile(CodeGemmArgs a, hipStream_t s) {
  using C = CodeCfg<BITS, PROD, TW, WM, WN, NBUF>;
  a.tiles_m = (a.M + C::TM - 1) / C::TM;
  const int64_t tiles_n = (a.n + C::TN - 1) / C::TN;
  if (tiles_n * a.tiles_m > (int64_t)1 << 30) return hipErrorInvalidValue;
  a.tiles_n = (int)tiles_n;
  a.per_xcd = (a.tiles_m * a.tiles_n + XCDS - 1) / XCDS;
  static LdsLimit lds_limit;  // per instantiation: the limit is raised once per device
  if (const hipError_t e = raise_lds_limit(lds_limit, reinterpret_cast<const void*>(&code_gemm_kernel<BITS, PROD, TW, WM, WN, NBUF>), C::LDS);
      e != hipSuccess)
    return e;
  hipLaunchKernelGGL((code_gemm_kernel<BITS, PROD, TW, WM, WN, NBUF>), dim3(a.per_xcd * XCDS), dim3(C::THREADS), C::LDS, s, a);
  return hipGetLastError();
}

// The large tile while it gives most compute units one (its reads per product are half those of the next); below that
// smaller ones, whose steps are shorter than a load's latency: four buffers then, where d is a multiple of 128.  Matrices
// of up to 64 rows have a tile of their own.
template <int BITS, bool PROD>
hipError_t launch_dequant(const CodeGemmArgs& a, hipStream_t s) {
  const int64_t cus = device_cu_count();
  auto count = [&](int tm, int tn) { return (int64_t)((a.M + tm - 1) / tm) * ((a.n + tn - 1) / tn); };
  const bool four = a.d % 128 == 0;
  if (a.M <= 64) return launch_tile<BITS, PROD, 1, 2, 4, 2>(a, s);
  const bool wide = (a.M + 255) / 256 * 256 * 5 < (a.M + 127) / 128 * 128 * 6;  // little more padding than the next tile
  if (wide && count(256, 256) * 4 >= cus * 3) return launch_tile<BITS, PROD, 2, 4, 2, 2>(a, s);
  if (count(128, 128) * 2 >= cus || !four) return four ? launch_tile<BITS, PROD, 2, 2, 2, 4>(a, s) : launch_tile<BITS, PROD, 2, 2, 2, 2>(a, s);
  return launch_tile<BITS, PROD, 1, 2, 1, 4>(a, s);
}

// ---- images ----------------------------------------------------------------------------------------------

// rows of the transpose, 32 x 32 values at a time through LDS
__global__ __launch_bounds__(256) void code_image_kernel(const float* __restrict__ W, const int d, const uint32_t* max_bits, float* w_inv,
                                                         unsigned char* out) {
  __shared__ float tile[32][33];
  float s, inv;
  h2_scale(*max_bits, s, inv);
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *w_inv = inv;
  const int r0 = blockIdx.y * 32, g = blockIdx.x;  // rows of the transpose, group of 32 along it
  for (int e = threadIdx.x; e < 1024; e += 256) tile[e >> 5][e & 31] = W[(int64_t)(32 * g + (e >> 5)) * d + r0 + (e & 31)] * s;
  __syncthreads();
  const int r = threadIdx.x >> 3, q = threadIdx.x & 7;  // row, quad of positions 4 q .. 4 q + 3
  const float v[4] = {tile[q][r], tile[q + 16][r], tile[q + 8][r], tile[q + 24][r]};
  uint32_t hi[2], lo[2];
  h2_split(v[0], v[1], hi[0], lo[0]);
  h2_split(v[2], v[3], hi[1], lo[1]);
  unsigned char* const p = out + ((int64_t)(r0 + r) * (d >> 5) + g) * 128 + q * 8;
  *reinterpret_cast<uint2*>(p) = make_uint2(hi[0], hi[1]);
  *reinterpret_cast<uint2*>(p + 64) = make_uint2(lo[0], lo[1]);
}

uint16_t half_bits(float f) {
  const _Float16 h = (_Float16)f;
  uint16_t b;
  std::memcpy(&b, &h, 2);
  return b;
}

}  // namespace

bool code_gemm_serves(int bits, const Codebook& cb) { return bits >= 0 && bits <= 4 && (bits == 0 || codebook_symmetric(cb, bits)); }

CodeTable make_code_table(int bits, const Codebook& cb) {
  CodeTable t;
  std::memset(&t, 0, sizeof(t));
  t.inv = bits == 1 ? cb.c[1] : 1.f;
  if (bits < 2) return t;
  const int H = 1 << (bits - 1);
  int e = 0;
  (void)std::frexp(cb.c[2 * H - 1], &e);          // the largest magnitude: f 2^e, f in [0.5, 1)
  const float s = std::ldexp(1.f, 15 - e);
  t.inv = std::ldexp(1.f, e - 15);
  for (int m = 0; m < H; ++m) {
    const float v = cb.c[H + m] * s;
    const uint16_t hi = half_bits(v);
    const uint16_t lo = half_bits(v - (float)(_Float16)v);
    const int w = m >> 2, sh = 8 * (m & 3);
    t.hh[w] |= (uint32_t)(hi >> 8) << sh;
    t.hl[w] |= (uint32_t)(hi & 255) << sh;
    t.lh[w] |= (uint32_t)(lo >> 8) << sh;
    t.ll[w] |= (uint32_t)(lo & 255) << sh;
  }
  return t;
}

float code_table_error(int bits, const Codebook& cb) {
  const int H = 1 << (bits - 1);
  int e = 0;
  (void)std::frexp(cb.c[2 * H - 1], &e);
  const float s = std::ldexp(1.f, 15 - e);
  float worst = 0.f;
  for (int m = 0; m < H; ++m) {
    const float v = cb.c[H + m] * s;
    if (v > 0.f) worst = std::fmax(worst, std::fabs(v - (float)(_Float16)v) / v);
  }
  return worst;
}

hipError_t launch_code_image(const float* W, int d, void* image, float* w_inv, hipStream_t s) {
  if (d <= 0 || d % 32 != 0) return hipErrorInvalidValue;
  uint32_t* const max_bits = reinterpret_cast<uint32_t*>(w_inv) + 1;
  if (const hipError_t e = launch_h2_max(W, d, d, d, max_bits, s); e != hipSuccess) return e;
  hipLaunchKernelGGL(code_image_kernel, dim3(d / 32, d / 32), dim3(256), 0, s, W, d, max_bits, w_inv, static_cast<unsigned char*>(image));
  return hipGetLastError();
}

hipError_t launch_code_dequant(int bits, bool prod, const void* pit_image, const float* pit_inv, const void* st_image, const float* st_inv,
                               int d, const uint32_t* idx, const uint32_t* qjl, const float* gamma, const float* norm, int64_t n,
                               float* out, int64_t ldo, float kappa, const Codebook& cb, hipStream_t s) {
  CodeGemmArgs a;
  std::memset(&a, 0, sizeof(a));
  a.WP = static_cast<const unsigned char*>(pit_image); a.WS = static_cast<const unsigned char*>(st_image);
  a.wp_inv = pit_inv; a.ws_inv = st_inv; a.M = d; a.d = d; a.idx = idx; a.qjl = qjl; a.gamma = gamma; a.norm = norm; a.n = n;
  a.kappa = kappa; a.tab = make_code_table(bits, cb); a.out = out; a.ldo = ldo;
  TQ_CODE_BITS(launch_dequant)
}

}  // namespace tq
