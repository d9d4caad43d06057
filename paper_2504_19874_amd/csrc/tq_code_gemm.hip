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

#include "tq_code_gemm.h"
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
  // search (M queries): inverse scale and error bound factors of each, lists of candidates
  const float* q_inv;
  const float* e1;
  const float* e2;
  const float* bar;
  int bar_step;
  float* list_u;
  int32_t* list_i;
  int32_t* count;
  int cap;
  int64_t code_step;  // sample pass: code i is row i * code_step
  float s_rel;        // sketch segment: scale of the queries' first image over that of their second
  int tiles_m, tiles_n, per_xcd;
};

enum CodeMode {
  M_DEQUANT,  // two pieces on both sides, out[code][row]
  M_SAMPLE,   // one piece on both sides, out[row][code] = score - its error bound
  M_FIND      // ... scores that may reach the query's bar, appended to its list
};

// 16 of a group's 32 values (bit positions 4 half .. 4 half + 3 of the four bytes), as they lie along the contraction
template <int BITS, int NP>
__device__ __forceinline__ void decode16(const uint32_t* w, int half, const CodeTable& tab, uint32_t (&out)[NP][8]) {
  const int sh = 4 * half;
  if constexpr (BITS == 1) {
    const uint32_t n = ~w[0] >> sh;  // bit set: negative
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      out[0][2 * k] = ((n << (15 - k)) & 0x80008000u) | 0x3C003C00u;
      out[0][2 * k + 1] = ((n << (7 - k)) & 0x80008000u) | 0x3C003C00u;
    }
  } else {
    // magnitude bits: the low planes, complemented where the top plane says negative
    uint32_t u[BITS > 1 ? BITS - 1 : 1];
#pragma unroll
    for (int p = 0; p < BITS - 1; ++p) u[p] = ~(w[p] ^ w[BITS - 1]) >> sh;
    const uint32_t n = ~w[BITS - 1] >> sh;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      uint32_t sel = 0u;
#pragma unroll
      for (int p = 0; p < BITS - 1; ++p) sel |= (k >= p ? u[p] >> (k - p) : u[p] << (p - k)) & (0x01010101u << p);
      const uint32_t neg = (n << (7 - k)) & 0x80808080u;
#pragma unroll
      for (int pc = 0; pc < NP; ++pc) {
        const uint32_t* th = pc == 0 ? tab.hh : tab.lh;
        const uint32_t* tl = pc == 0 ? tab.hl : tab.ll;
        const uint32_t hi = (BITS == 4 ? __builtin_amdgcn_perm(th[1], th[0], sel) : __builtin_amdgcn_perm(th[0], th[0], sel)) ^ neg;
        const uint32_t lo = BITS == 4 ? __builtin_amdgcn_perm(tl[1], tl[0], sel) : __builtin_amdgcn_perm(tl[0], tl[0], sel);
        out[pc][2 * k] = __builtin_amdgcn_perm(hi, lo, 0x06020400u);
        out[pc][2 * k + 1] = __builtin_amdgcn_perm(hi, lo, 0x07030501u);
      }
    }
  }
}

template <int BITS>
__device__ __forceinline__ void load_plane_words(const uint32_t* p, uint32_t (&w)[BITS]) {
  typedef uint32_t v2 __attribute__((ext_vector_type(2), aligned(4)));
  typedef uint32_t v3 __attribute__((ext_vector_type(3), aligned(4)));
  typedef uint32_t v4 __attribute__((ext_vector_type(4), aligned(4)));
  if constexpr (BITS == 1) w[0] = *p;
  if constexpr (BITS == 2) { const v2 v = *reinterpret_cast<const v2*>(p); w[0] = v[0]; w[1] = v[1]; }
  if constexpr (BITS == 3) { const v3 v = *reinterpret_cast<const v3*>(p); w[0] = v[0]; w[1] = v[1]; w[2] = v[2]; }
  if constexpr (BITS == 4) { const v4 v = *reinterpret_cast<const v4*>(p); w[0] = v[0]; w[1] = v[1]; w[2] = v[2]; w[3] = v[3]; }
}

template <int MODE, int BITS, bool PROD, int TW, int WM, int WN, int NBUF>
struct CodeCfg {
  static constexpr int UW = WM;  // so that every thread decodes half a group of one code per step
  static constexpr int THREADS = 64 * WM * WN, TM = WM * TW * 32, TN = WN * UW * 32;
  static constexpr int NPA = MODE == M_DEQUANT ? 2 : 1, NPB = MODE == M_DEQUANT && BITS >= 2 ? 2 : 1;
  static constexpr int A_BYTES = TM * 64 * NPA, B_BYTES = TN * 64 * NPB;
  static constexpr int NS = NBUF;
  static constexpr int LDS = NS * (A_BYTES + B_BYTES) + 4 * TN * 4 + (MODE == M_DEQUANT ? 0 : 4 * TM * 4);
  static constexpr int LOADERS = A_BYTES / 1024 < WM * WN ? A_BYTES / 1024 : WM * WN;  // wavefronts that load the fixed operand
  static constexpr int AL = A_BYTES / 1024 / LOADERS;                                  // their direct loads per step
  static_assert(THREADS == 2 * TN && AL * LOADERS * 1024 == A_BYTES, "roles");
};

template <int MODE, int BITS, bool PROD, int TW, int WM, int WN, int NBUF>
__global__ __launch_bounds__(64 * WM * WN, 2) void code_gemm_kernel(const CodeGemmArgs a) {
  using C = CodeCfg<MODE, BITS, PROD, TW, WM, WN, NBUF>;
  constexpr int UW = C::UW, TM = C::TM, TN = C::TN, NPA = C::NPA, NPB = C::NPB, NS = C::NS, AL = C::AL;
  constexpr bool HAVE_P = BITS > 0, HAVE_S = PROD;
  constexpr int NW = BITS > 0 ? BITS : 1;
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
  float* const first_s = reinterpret_cast<float*>(lds + NS * (C::A_BYTES + C::B_BYTES));  // [TN] factor of the sketch sums
  float* const last_s = first_s + TN;                                                     // [TN] factor of everything
  float* const nu_s = last_s + TN;   // search: [TN] norm, norm kappa gamma
  float* const nk_s = nu_s + TN;
  float* const qi_s = nk_s + TN;     // search: [TM] inverse scale, error factors, bar

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
  const int code = tid % TN, half = __builtin_amdgcn_readfirstlane(tid / TN);
  const int64_t row = (n0 + min(code, rows_n - 1)) * (MODE == M_SAMPLE ? a.code_step : 1);  // codes past the end: the last one again, not stored
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
            acc[t][u] = MODE == M_DEQUANT ? __builtin_amdgcn_mfma_f32_32x32x16_f16(fb[u][q], fa[t][p], acc[t][u], 0, 0, 0)
                                          : __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[t][p], fb[u][q], acc[t][u], 0, 0, 0);
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
    const float pi = HAVE_P ? (MODE == M_DEQUANT ? a.wp_inv[0] : 1.f) * a.tab.inv : 1.f;
    const float si = HAVE_S ? (MODE == M_DEQUANT ? a.ws_inv[0] : a.s_rel) : 1.f;
    for (int c = tid; c < TN; c += C::THREADS) {
      const int64_t r = (n0 + min(c, rows_n - 1)) * (MODE == M_SAMPLE ? a.code_step : 1);
      const float nu = a.norm != nullptr ? a.norm[r] : 1.f;
      const float kg = HAVE_S ? a.kappa * a.gamma[r] : 0.f;
      first_s[c] = HAVE_P ? kg * si / pi : 1.f;
      last_s[c] = HAVE_P ? nu * pi : nu * (kg * si);
      if (MODE != M_DEQUANT) {
        nu_s[c] = c < rows_n ? nu : __builtin_nanf("");  // a code past the end compares false
        nk_s[c] = nu * kg;
      }
    }
    if (MODE != M_DEQUANT)
      for (int m = tid; m < TM; m += C::THREADS) {
        const int q = m0 + min(m, rows_m - 1);
        qi_s[m] = a.q_inv[q];
        qi_s[TM + m] = a.e1[q];
        qi_s[2 * TM + m] = a.e2[q];
        if (MODE == M_FIND) qi_s[3 * TM + m] = m < rows_m ? a.bar[(int64_t)q * a.bar_step] : __builtin_inff();
      }
  }
  decode_step(0, words[0], std::bool_constant<HAVE_S>{});
  h2_wait_barrier<0>();
  auto scale = [&] {  // the sketch sums in units of the centroid segment
    if constexpr (MODE != M_DEQUANT) {
#pragma unroll
      for (int u = 0; u < UW; ++u) {
        const float f = first_s[wn * UW * 32 + u * 32 + l32];
#pragma unroll
        for (int t = 0; t < TW; ++t)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[t][u][r] *= f;
      }
      return;
    }
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

  if constexpr (MODE != M_DEQUANT) {
    // a lane has 16 queries of one code per tile
#pragma unroll
    for (int u = 0; u < UW; ++u) {
      const int c = wn * UW * 32 + u * 32 + l32;
      const float last = last_s[c], nu = nu_s[c], nk = nk_s[c];
#pragma unroll
      for (int t = 0; t < TW; ++t)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int m = (wm * TW + t) * 32 + 8 * k + 4 * h;
          __builtin_amdgcn_sched_barrier(0);  // one quad's factors at a time (registers)
          const float4 qi = *reinterpret_cast<const float4*>(qi_s + m), e1 = *reinterpret_cast<const float4*>(qi_s + TM + m);
          const float4 e2 = HAVE_S ? *reinterpret_cast<const float4*>(qi_s + 2 * TM + m) : e1;
          const float qe[4] = {qi.x, qi.y, qi.z, qi.w}, e1e[4] = {e1.x, e1.y, e1.z, e1.w}, e2e[4] = {e2.x, e2.y, e2.z, e2.w};
          float bar[4] = {0.f, 0.f, 0.f, 0.f};
          if (MODE == M_FIND) {
            const float4 b = *reinterpret_cast<const float4*>(qi_s + 3 * TM + m);
            bar[0] = b.x, bar[1] = b.y, bar[2] = b.z, bar[3] = b.w;
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float eps = nu * e1e[e];
            if (HAVE_S) eps = fmaf(nk, e2e[e], eps);
            const float v = acc[t][u][4 * k + e] * last;
            if constexpr (MODE == M_SAMPLE) {
              if (c < rows_n && m + e < rows_m) a.out[(int64_t)(m0 + m + e) * a.ldo + n0 + c] = fmaf(v, qe[e], -eps);
            } else {
              const float top = fmaf(v, qe[e], eps);
              if (top >= bar[e]) {
                const int q = m0 + m + e;
                const int pos = atomicAdd(a.count + q, 1);
                if (pos < a.cap) {
                  a.list_u[(int64_t)q * a.cap + pos] = top;
                  a.list_i[(int64_t)q * a.cap + pos] = (int)(n0 + c);
                }
              }
            }
          }
        }
    }
    return;
  }

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

template <int MODE, int BITS, bool PROD, int TW, int WM, int WN, int NBUF>
hipError_t launch_tile(CodeGemmArgs a, hipStream_t s) {
  using C = CodeCfg<MODE, BITS, PROD, TW, WM, WN, NBUF>;
  a.tiles_m = (a.M + C::TM - 1) / C::TM;
  const int64_t tiles_n = (a.n + C::TN - 1) / C::TN;
  if (tiles_n * a.tiles_m > (int64_t)1 << 30) return hipErrorInvalidValue;
  a.tiles_n = (int)tiles_n;
  a.per_xcd = (a.tiles_m * a.tiles_n + XCDS - 1) / XCDS;
  static LdsLimit lds_limit;  // per instantiation: the limit is raised once per device
  if (const hipError_t e = raise_lds_limit(lds_limit, reinterpret_cast<const void*>(&code_gemm_kernel<MODE, BITS, PROD, TW, WM, WN, NBUF>), C::LDS);
      e != hipSuccess)
    return e;
  hipLaunchKernelGGL((code_gemm_kernel<MODE, BITS, PROD, TW, WM, WN, NBUF>), dim3(a.per_xcd * XCDS), dim3(C::THREADS), C::LDS, s, a);
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
  if (a.M <= 64) return launch_tile<M_DEQUANT, BITS, PROD, 1, 2, 4, 2>(a, s);
  const bool wide = (a.M + 255) / 256 * 256 * 5 < (a.M + 127) / 128 * 128 * 6;  // little more padding than the next tile
  if (wide && count(256, 256) * 4 >= cus * 3) return launch_tile<M_DEQUANT, BITS, PROD, 2, 4, 2, 2>(a, s);
  if (count(128, 128) * 2 >= cus || !four) return four ? launch_tile<M_DEQUANT, BITS, PROD, 2, 2, 2, 4>(a, s) : launch_tile<M_DEQUANT, BITS, PROD, 2, 2, 2, 2>(a, s);
  return launch_tile<M_DEQUANT, BITS, PROD, 1, 2, 1, 4>(a, s);
}

// Search: the query tile that holds the queries, 256 codes; four buffers (with one piece a step is a third of the dequantiser's)
template <int MODE, int BITS, bool PROD, int NBUF>
hipError_t launch_search_tile(const CodeGemmArgs& a, hipStream_t s) {
  if (a.M > 128) return launch_tile<MODE, BITS, PROD, 2, 4, 2, NBUF>(a, s);
  if (a.M > 64) return launch_tile<MODE, BITS, PROD, 2, 2, 4, NBUF>(a, s);
  if (a.M > 32) return launch_tile<MODE, BITS, PROD, 1, 2, 4, NBUF>(a, s);
  return launch_tile<MODE, BITS, PROD, 1, 1, 8, NBUF>(a, s);
}

template <int BITS, bool PROD>
hipError_t launch_search(const CodeGemmArgs& a, hipStream_t s) {
  if (a.list_u == nullptr)
    return a.d % 128 == 0 ? launch_search_tile<M_SAMPLE, BITS, PROD, 4>(a, s) : launch_search_tile<M_SAMPLE, BITS, PROD, 2>(a, s);
  return a.d % 128 == 0 ? launch_search_tile<M_FIND, BITS, PROD, 4>(a, s) : launch_search_tile<M_FIND, BITS, PROD, 2>(a, s);
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
#define TQ_CODE_BITS(F)                       \
  switch (bits * 2 + (prod ? 1 : 0)) {        \
    case 1: return F<0, true>(a, s);          \
    case 2: return F<1, false>(a, s);         \
    case 3: return F<1, true>(a, s);          \
    case 4: return F<2, false>(a, s);         \
    case 5: return F<2, true>(a, s);          \
    case 6: return F<3, false>(a, s);         \
    case 7: return F<3, true>(a, s);          \
    case 8: return F<4, false>(a, s);         \
    case 9: return F<4, true>(a, s);          \
    default: return hipErrorInvalidValue;     \
  }
  TQ_CODE_BITS(launch_dequant)
}

hipError_t launch_code_search(int bits, bool prod, const CodeSearch& q, int d, const uint32_t* idx, const uint32_t* qjl, const float* gamma,
                              const float* norm, int64_t n, int64_t code_step, float kappa, const Codebook& cb, hipStream_t s) {
  CodeGemmArgs a;
  std::memset(&a, 0, sizeof(a));
  a.WP = static_cast<const unsigned char*>(q.r_pieces); a.WS = static_cast<const unsigned char*>(q.s_pieces);
  a.M = q.nq; a.d = d; a.idx = idx; a.qjl = qjl; a.gamma = gamma; a.norm = norm; a.n = n; a.kappa = kappa; a.tab = make_code_table(bits, cb);
  a.q_inv = q.inv; a.e1 = q.e1; a.e2 = q.e2; a.bar = q.bar; a.bar_step = q.bar_step; a.out = q.sample; a.ldo = q.ld_sample; a.code_step = code_step;
  a.list_u = q.list_u; a.list_i = q.list_i; a.count = q.count; a.cap = q.cap; a.s_rel = q.s_rel;
  TQ_CODE_BITS(launch_search)
#undef TQ_CODE_BITS
}

}  // namespace tq
