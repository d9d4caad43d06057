// The pass of a search over all codes (tq_search.hip says what for): scores of M queries from one fp16 piece of every factor.
//
// The codes are decoded on their way to LDS as in tq_code_gemm.hip (leading piece only), the queries' pieces come by direct
// loads; a score takes one v_mfma_f32_32x32x16_f16 per 16 coordinates.  A workgroup keeps its tile of queries and walks a
// range of code tiles: requests for the next tile's words and query pieces run on across the border, so that a tile costs
// its steps and its comparisons and no round trip to memory (128 coordinates are only four steps).  Within a step the
// fragments of the next 16 k are read, and the codes of the next step decoded, between the matrix instructions, in pinned order.
//
// A score is compared as it lies in the accumulator: nu (acc A + E1 + kappa |gamma| E2) >= bar is acc >= (bar / nu - E1 -
// kappa |gamma| E2) / A for nu > 0 (the others pass to the second test), two or three instructions per score and no multiplication of the score itself; what passes is
// evaluated and tested again before it goes to the query's list.  That is a round trip to a counter in memory, with dozens
// per tile more than a short tile itself takes: they are gathered in LDS, the counters are asked for all of them at once at
// the end of the next tile, and the pairs stored at the end of the one after that (d = 128, 10^6 codes, 1000
// queries: 605 us, was 1037 with a trip each).
//
// Bound by the power of the matrix cores and, at 3 and 4 bits, by the decoding's vector instructions (10^6 codes, 1000 queries: d = 1536, 4 bits
// 2.93 ms, 1.05 PFLOP/s (3.05 with the planes joined position by position); d = 3072, 1 + 1 bits 9.1 ms, 1.35; d = 128, 4 bits 0.55 ms, 0.46; in registers 1.62).  With the loading and the decoding
// given to four wavefronts each it was no faster at d = 3072 and slower elsewhere (registers).
#include <cstring>

#include "tq_search_gemm.h"

#include <type_traits>

namespace tq {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int XCDS = 8;

template <int TW, int WM, int WN>
struct SearchCfg {
  static constexpr int UW = WM;  // so that every thread decodes a group of one code in two steps
  static constexpr int THREADS = 64 * WM * WN, TM = WM * TW * 32, TN = WN * UW * 32;
  static constexpr int A_BYTES = TM * 64, B_BYTES = TN * 64, NS = 4;
  static constexpr int LOADERS = A_BYTES / 1024 < WM * WN ? A_BYTES / 1024 : WM * WN;  // wavefronts that load query pieces
  static constexpr int AL = A_BYTES / 1024 / LOADERS;                                  // their direct loads per step
  static constexpr int CODE_F = 4, QUERY_F = 7;  // floats kept per code (two tiles' worth) and per query
  static constexpr int FOUND = THREADS;          // candidates of a tile that are gathered (two tiles' worth): one per thread
  static constexpr int LDS = NS * (A_BYTES + B_BYTES) + 2 * CODE_F * TN * 4 + QUERY_F * TM * 4 + 2 * FOUND * 12;
  static_assert(THREADS == 2 * TN && AL * LOADERS * 1024 == A_BYTES && TN % 64 == 0, "roles");
};

template <bool FIND, int BITS, bool PROD, int TW, int WM, int WN>
__global__ __launch_bounds__(64 * WM * WN, 2) void search_gemm_kernel(const SearchGemmArgs a) {
  using C = SearchCfg<TW, WM, WN>;
  constexpr int UW = C::UW, TM = C::TM, TN = C::TN, NS = C::NS, AL = C::AL;
  constexpr bool HAVE_P = BITS > 0, HAVE_S = PROD;
  constexpr int NW = BITS > 0 ? BITS : 1;
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
  // per code of a tile (two parities): factor of the sketch sums / of everything, norm, kappa gamma
  float* const code_s = reinterpret_cast<float*>(lds + NS * (C::A_BYTES + C::B_BYTES));
  // per query: bar / A, E1 / A, E2 / A (for the first test), 1 / scale, E1, E2, bar
  float* const query_s = code_s + 2 * C::CODE_F * TN;
  int* const found_s = reinterpret_cast<int*>(query_s + C::QUERY_F * TM);  // [parity][query, code, score + eps][FOUND]
  __shared__ int found_n[4];                                              // by tile number

  const int logical = (int)(blockIdx.x % XCDS) * a.per_xcd + (int)(blockIdx.x / XCDS);
  if (logical >= a.qblocks * a.ranges) return;
  // the query blocks of one range of codes follow each other on an XCD and share its L2
  const int qb = __builtin_amdgcn_readfirstlane(logical % a.qblocks), range = __builtin_amdgcn_readfirstlane(logical / a.qblocks);
  const int tile0 = __builtin_amdgcn_readfirstlane((int)((int64_t)range * a.tiles / a.ranges));
  const int tile1 = __builtin_amdgcn_readfirstlane((int)((int64_t)(range + 1) * a.tiles / a.ranges));
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int l32 = lane & 31, h = lane >> 5;
  const int m0 = qb * TM;
  const int rows_m = min(TM, a.M - m0);
  const int G = a.d >> 5;
  const int n_s = HAVE_S ? G : 0, n_steps = n_s + (HAVE_P ? G : 0);

  // ---- query pieces: direct loads, round and round -----------------------------------------------------
  const uint32_t step_a = search_step_bytes(a.M);
  const unsigned char* const gP = a.R + m0 * 64;
  const unsigned char* const gS = HAVE_S ? a.S + m0 * 64 : gP;
  const unsigned char* gA = gS;
  uint32_t va[AL];
  {
    const int l8 = lane >> 3, slot = lane & 7;
#pragma unroll
    for (int j = 0; j < AL; ++j) {
      const int r = 2 * ((wave * AL + j) * 8 + l8) + (slot >> 2);
      va[j] = (uint32_t)min(r, rows_m - 1) * 64 + h2_chunk<1>(r, slot) * 16;
    }
  }
  const uint32_t lds0 = h2_lds_address(lds);
  int a_step = 0;
  auto dma = [&](int buf) {
    // (pinned to scalar registers: the compiler does not always see that these are the same for all lanes)
    const uint64_t g = (uint64_t)gA;
    const uint32_t g_lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)g);  // (unsigned: the halves are joined)
    const uint32_t g_hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(g >> 32));
    const void* const base = reinterpret_cast<const void*>((uint64_t)g_hi << 32 | g_lo);
    const uint32_t to = (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds0 + buf * C::A_BYTES + wave * (AL * 1024)));
    if (C::LOADERS == WM * WN || wave < C::LOADERS)  // (a wavefront without loads waits for fewer than it may: nothing to wait for)
#pragma unroll
      for (int j = 0; j < AL; ++j) h2_dma(base, va[j], to + j * 1024);
    ++a_step;
    gA += step_a;
    if (HAVE_S && HAVE_P && a_step == n_s) gA = gP;
    if (a_step == n_steps) a_step = 0, gA = gS;
  };

  // ---- codes: the words of four steps at a time, tile after tile ------------------------------------------
  // Two neighbouring lanes share a code: one has the groups of even steps, the other those of odd ones, each decoded over
  // two steps.  A lane's two groups of a round are asked for together, so that a line of codes is met once in four steps:
  // 256 codes are as many lines as the cache beside the compute unit has, and words asked for step by step came from L2 once
  // for every step and half group, 646 requests a step with the queries' 128 (d = 1536, 4 bits, 10^6 codes, 1000 queries,
  // the whole search: 3.49 -> 3.23 ms; d = 3072, 3 bits 1.17 times faster).
  const int code = tid >> 1, odd = tid & 1;
  auto code_row = [&](int tile, int c) {  // codes past the end: the last one again
    const int64_t i = (int64_t)tile * TN + c;
    return (i < a.n ? i : a.n - 1) * (FIND ? 1 : a.code_step);
  };
  const uint32_t *wi = nullptr, *wz = nullptr;
  int w_step = 0, w_tile = tile0;
  auto point = [&] {
    const int64_t row = code_row(w_tile, code);
    if (HAVE_P) wi = a.idx + (row * G + odd) * BITS;
    if (HAVE_S) wz = a.qjl + row * G + odd;
  };
  point();
  uint32_t words[2][NW], next_words[2][NW];  // [pair of steps]
  auto load_round = [&] {
    if (HAVE_S && (!HAVE_P || w_step < n_s)) {
#pragma unroll
      for (int j = 0; j < 2; ++j) next_words[j][0] = wz[w_step + 2 * j];
    } else if constexpr (HAVE_P) {
      uint32_t w0[NW], w1[NW];  // (loaded into the array itself, one of the two branches would leave it in memory)
      load_plane_words<BITS>(wi + (w_step - n_s) * BITS, w0);
      load_plane_words<BITS>(wi + (w_step - n_s + 2) * BITS, w1);
#pragma unroll
      for (int p = 0; p < NW; ++p) next_words[0][p] = w0[p], next_words[1][p] = w1[p];
    }
    w_step += NS;
    if (w_step == n_steps) {
      w_step = 0;
      ++w_tile;
      point();
    }
  };
  auto advance = [&] {
    // (moves that the compiler can not put off to the end of its loop, where it would wait for the loads behind them)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int p = 0; p < NW; ++p) asm volatile("v_mov_b32 %0, %1" : "=v"(words[j][p]) : "v"(next_words[j][p]));
    __builtin_amdgcn_sched_barrier(0);
    load_round();
  };
  // the two store into the buffers of both steps of a pair at once: the odd one has its two halves exchanged, for the banks
  const uint32_t b_at = h2_place<1>(code, 2 * odd) + odd * C::B_BYTES;
  auto store_codes = [&](int pair, int chunk, const uint32_t* v) {
    *reinterpret_cast<uint4*>(lds + NS * C::A_BYTES + 2 * pair * C::B_BYTES + (b_at ^ (16 * chunk))) = make_uint4(v[0], v[1], v[2], v[3]);
  };

  const unsigned char *pa[2], *pb[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    pa[s] = lds + h2_place<1>(wm * TW * 32 + l32, s * 2 + h);
    pb[s] = lds + NS * C::A_BYTES + h2_place<1>(wn * UW * 32 + l32, s * 2 + h);
  }
  floatx16 acc[TW][UW];
  const PlaneTable tab(a.tab);
  constexpr int KEPT = BITS == 4 ? 4 : BITS == 3 ? 2 : BITS == 2 ? 1 : 0;
  uint32_t kept[1 + KEPT];  // of a group's planes from its first step to its second
  auto clear = [&] {
#pragma unroll
    for (int t = 0; t < TW; ++t)
#pragma unroll
      for (int u = 0; u < UW; ++u)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][u][r] = 0.f;
  };

  // ---- per-code scalars of a tile: requested a tile ahead, stored behind the tile before ------------------
  float next_nu = 1.f, next_kg = 0.f;
  auto request_scalars = [&](int tile) {
    if (tid < TN) {
      const int64_t r = code_row(tile, tid);
      next_nu = a.norm != nullptr ? a.norm[r] : 1.f;
      next_kg = HAVE_S ? a.gamma[r] : 0.f;
    }
  };
  auto store_scalars = [&](int tile) {
    if (tid < TN) {
      float* const c = code_s + (tile & 1) * C::CODE_F * TN + tid;
      const float pi = HAVE_P ? a.tab.inv : 1.f;
      const float kg = a.kappa * next_kg, nu = (int64_t)tile * TN + tid < a.n ? next_nu : __builtin_nanf("");
      c[0] = HAVE_P ? kg * a.s_rel / pi : 1.f;
      c[TN] = HAVE_P ? pi : kg * a.s_rel;
      c[2 * TN] = nu;
      c[3 * TN] = kg;
    }
  };

  struct Frag {
    f16x8 a[TW], b[UW];
  };
  constexpr int NR = TW + UW, NM = TW * UW;
  auto read_one = [&](Frag& f, int buf, int s, int i) {
    if (i < TW) f.a[i] = *reinterpret_cast<const f16x8*>(pa[s] + buf * C::A_BYTES + i * 2048);
    else f.b[i - TW] = *reinterpret_cast<const f16x8*>(pb[s ^ (buf & 1)] + buf * C::B_BYTES + (i - TW) * 2048);
  };
  Frag f0, f1;
  // of_p: the pair of steps that is decoded meanwhile (the one after this step's pair) belongs to the centroid segment
  auto step = [&](auto buf_c, auto of_p) __attribute__((always_inline)) {  // (called, it would keep the accumulators in memory)
    constexpr int buf = decltype(buf_c)::value, nbuf = (buf + 1) % NS;
    constexpr int half = buf & 1, pair = (buf / 2 + 1) % 2;  // half of the group, and which pair of the round
    Planes<decltype(of_p)::value ? NW : 1> codes;
    if constexpr (half == 0) {
      codes.set(words[pair], tab);
      kept[0] = codes.s;
#pragma unroll
      for (int i = 0; i < KEPT; ++i) kept[1 + i] = codes.n[i];
    } else {
      codes.s = kept[0];
#pragma unroll
      for (int i = 0; i < KEPT; ++i) codes.n[i] = kept[1 + i];
    }
    uint32_t v[8];
    auto from = [](int i) { return 2 * i * NR / NM < NR ? 2 * i * NR / NM : NR; };  // reads go into the first half of a half-step
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NM; ++i) {
      acc[i / UW][i % UW] = __builtin_amdgcn_mfma_f32_32x32x16_f16(f0.a[i / UW], f0.b[i % UW], acc[i / UW][i % UW], 0, 0, 0);
#pragma unroll
      for (int r = from(i); r < from(i + 1); ++r) read_one(f1, buf, 1, r);
#pragma unroll
      for (int k = 4 * i / NM; k < 4 * (i + 1) / NM; ++k) {
        codes.quad(4 * half + k, tab, v[2 * k], v[2 * k + 1]);
        if (k & 1) store_codes(pair, 2 * half + k / 2, v + 2 * (k - 1));
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0), so that the compiler knows the fragments have arrived
    // everyone has read this step; the next one is there (younger than its query pieces: the loads of the two steps after
    // it and, in the second pair, the words requested in front of those of step 1)
    h2_wait_barrier<(NS - 2) * AL + (buf >= 2 ? 2 : 0)>();
#pragma unroll
    for (int i = 0; i < NM; ++i) {
      acc[i / UW][i % UW] = __builtin_amdgcn_mfma_f32_32x32x16_f16(f1.a[i / UW], f1.b[i % UW], acc[i / UW][i % UW], 0, 0, 0);
#pragma unroll
      for (int r = from(i); r < from(i + 1); ++r) read_one(f0, nbuf, 0, r);
      if (i == NM - 1) {
        // (the words are waited for with all that is under way: in front of this step's loads, which would be the youngest)
        if constexpr (buf == 1) advance();
        dma(buf);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto round = [&](auto this_p, auto next_p) __attribute__((always_inline)) {
    step(std::integral_constant<int, 0>{}, this_p);
    step(std::integral_constant<int, 1>{}, this_p);
    step(std::integral_constant<int, 2>{}, next_p);
    step(std::integral_constant<int, 3>{}, next_p);
  };

  // ---- candidates ------------------------------------------------------------------------------------------
  int pend_q = -1, pend_code = 0, pend_pos = 0;
  float pend_top = 0.f;
  auto store_pending = [&] {
    if (pend_q >= 0 && pend_pos < a.cap) {
      a.list_u[(int64_t)pend_q * a.cap + pend_pos] = pend_top;
      a.list_i[(int64_t)pend_q * a.cap + pend_pos] = pend_code;
    }
    pend_q = -1;
  };
  auto ask_for = [&](int tile) {  // places for what was found in that tile
    const int* const f = found_s + (tile & 1) * 3 * C::FOUND;
    if (tid < found_n[tile & 3] && tid < C::FOUND) {
      pend_q = f[tid];
      pend_code = f[C::FOUND + tid];
      pend_top = __int_as_float(f[2 * C::FOUND + tid]);
      pend_pos = atomicAdd(a.count + (int64_t)pend_q * COUNT_STEP, 1);
    }
  };

  // ---- before the first tile -------------------------------------------------------------------------------
  request_scalars(tile0);
  load_round();
  advance();
#pragma unroll
  for (int i = 0; i < NS; ++i) dma(i);
  for (int m = tid; m < TM; m += C::THREADS) {
    const int q = m0 + min(m, rows_m - 1);
    const float inv = a.q_inv[q], e1 = a.e1[q], e2 = a.e2[q], bar = FIND ? (m < rows_m ? a.bar[(int64_t)q * a.bar_step] : __builtin_inff()) : 0.f;
    const float A = HAVE_P ? inv * a.tab.inv : inv;
    query_s[m] = bar / A;
    query_s[TM + m] = e1 / A;
    query_s[2 * TM + m] = e2 / A;
    query_s[3 * TM + m] = inv;
    query_s[4 * TM + m] = e1;
    query_s[5 * TM + m] = e2;
    query_s[6 * TM + m] = m < rows_m ? bar : __builtin_nanf("");  // past the last query: not reached by a score that is infinite either
  }
  store_scalars(tile0);
  if (tid < 4) found_n[tid] = 0;
  auto decode_half = [&](auto half_c) {  // of the first pair of steps
    constexpr int half = decltype(half_c)::value;
    Planes<HAVE_S ? 1 : NW> codes;
    codes.set(words[0], tab);
    uint32_t v[8];
#pragma unroll
    for (int k = 0; k < 4; ++k) codes.quad(4 * half + k, tab, v[2 * k], v[2 * k + 1]);
    store_codes(0, 2 * half, v);
    store_codes(0, 2 * half + 1, v + 4);
  };
  decode_half(std::integral_constant<int, 0>{});
  decode_half(std::integral_constant<int, 1>{});
  h2_wait_barrier<0>();
#pragma unroll
  for (int i = 0; i < NR; ++i) read_one(f0, 0, 0, i);

  for (int tile = tile0; tile < tile1; ++tile) {
    request_scalars(tile + 1 < tile1 ? tile + 1 : tile);
    clear();
    // (a tile's last pair of steps decodes the first pair of the next one: of the sketch where there is one)
    if constexpr (HAVE_S && !HAVE_P) {
      for (int st = 0; st < n_s; st += NS) round(std::false_type{}, std::false_type{});
    } else {
      if constexpr (HAVE_S) {
        for (int st = NS; st < n_s; st += NS) round(std::false_type{}, std::false_type{});
        round(std::false_type{}, std::true_type{});
        int sl = l32;
        asm volatile("" : "+v"(sl));
        const float* const fs = code_s + (tile & 1) * C::CODE_F * TN + wn * UW * 32 + sl;
#pragma unroll
        for (int u = 0; u < UW; ++u) {  // the sketch sums in units of the centroid segment
          const float f = fs[u * 32];
#pragma unroll
          for (int t = 0; t < TW; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[t][u][r] *= f;
        }
      }
      for (int st = HAVE_S ? NS : 0; st < G; st += NS) round(std::true_type{}, std::true_type{});
      if constexpr (HAVE_S) round(std::true_type{}, std::false_type{});
    }

    // ---- comparisons: a lane has 16 queries of one code per 32 x 32 tile ------------------------------------
    // (what is derived from the lane is made again here: kept from before the loop it would take registers all through it)
    int el = l32, eh = h, par = (tile & 1) * C::CODE_F * TN;
    asm volatile("" : "+v"(el), "+v"(eh), "+s"(par));
    const float* const cs = code_s + par;
    const int64_t n0 = (int64_t)tile * TN;
    if (FIND) {
      // (every wavefront has met barriers since it added to what is read, and will before it adds to what is cleared)
      store_pending();
      if (tile > tile0) ask_for(tile - 1);
      if (tid == 0) found_n[(tile + 2) & 3] = 0;
    }
    const int c0 = wn * UW * 32 + el;
    // the first test divides by what the score is multiplied with; where that is not a positive number it lets everything through
    float inv[UW], kg[UW], rest[UW];
#pragma unroll
    for (int u = 0; u < UW; ++u) {
      const float nu = cs[2 * TN + c0 + 32 * u], fac = HAVE_P ? 1.f : cs[TN + c0 + 32 * u];
      kg[u] = HAVE_S ? cs[3 * TN + c0 + 32 * u] : 0.f;
      const float per = nu * fac;
      inv[u] = per > 0.f ? 1.f / per : __builtin_nanf("");
      rest[u] = HAVE_P ? 1.f : 1.f / fabsf(fac);
    }
#pragma unroll
    for (int t = 0; t < TW; ++t)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int m = (wm * TW + t) * 32 + 8 * k + 4 * eh;
        __builtin_amdgcn_sched_barrier(0);  // one quad of queries at a time (registers)
        auto quad = [&](int f, float (&o)[4]) {
          const float4 v = *reinterpret_cast<const float4*>(query_s + f * TM + m);
          o[0] = v.x, o[1] = v.y, o[2] = v.z, o[3] = v.w;
        };
        auto exact = [&](int u, int e, float sign) {  // score + sign * its error bound
          const float* const q = query_s + m + e;
          const float nu = cs[2 * TN + c0 + 32 * u], fac = cs[TN + c0 + 32 * u];
          float eps = HAVE_P ? fabsf(nu) * q[4 * TM] : 0.f;  // (without centroids that factor is zero, and a norm may be infinite)
          if (HAVE_S) eps = fmaf(fabsf(nu * kg[u]), q[5 * TM], eps);
          return fmaf(acc[t][u][4 * k + e] * (nu * fac), q[3 * TM], sign * eps);
        };
        if constexpr (!FIND) {
#pragma unroll
          for (int u = 0; u < UW; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (n0 + c0 + 32 * u < a.n && m + e < rows_m)
                a.sample[(int64_t)(m0 + m + e) * a.ld_sample + n0 + c0 + 32 * u] = exact(u, e, -1.f);
        } else {
          float b[4], d1[4], d2[4] = {0.f, 0.f, 0.f, 0.f};
          quad(0, b);
          quad(1, d1);
          if (HAVE_S) quad(2, d2);
#pragma unroll
          for (int u = 0; u < UW; ++u) {
            uint64_t maybe[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              float bound = HAVE_S ? fmaf(d2[e], fabsf(kg[u]), d1[e]) : d1[e];
              if (!HAVE_P) bound *= rest[u];
              maybe[e] = __builtin_amdgcn_ballot_w64(!(acc[t][u][4 * k + e] < fmaf(b[e], inv[u], -bound)));
            }
            if ((maybe[0] | maybe[1] | maybe[2] | maybe[3]) == 0u) continue;  // four scores of every lane behind one branch
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              if (maybe[e] == 0u) continue;
              const float top = exact(u, e, 1.f);
              if (((maybe[e] >> lane) & 1u) != 0u && top >= query_s[6 * TM + m + e]) {
                const int q = m0 + m + e, code_i = (int)n0 + c0 + 32 * u;
                const int at = atomicAdd(&found_n[tile & 3], 1);
                if (at < C::FOUND) {
                  int* const f = found_s + (tile & 1) * 3 * C::FOUND + at;
                  f[0] = q;
                  f[C::FOUND] = code_i;
                  f[2 * C::FOUND] = __float_as_int(top);
                } else if (const int pos = atomicAdd(a.count + (int64_t)q * COUNT_STEP, 1); pos < a.cap) {
                  a.list_u[(int64_t)q * a.cap + pos] = top;
                  a.list_i[(int64_t)q * a.cap + pos] = code_i;
                }
              }
            }
          }
        }
      }
    store_scalars(tile + 1);
  }
  if (FIND) {
    __syncthreads();
    store_pending();
    if (tile1 > tile0) ask_for(tile1 - 1);
    store_pending();
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // nothing of this workgroup's is under way to LDS when it ends
}

template <bool FIND, int BITS, bool PROD, int TW, int WM, int WN>
hipError_t launch_tile(SearchGemmArgs a, int per_cu, hipStream_t s) {
  using C = SearchCfg<TW, WM, WN>;
  a.qblocks = (a.M + C::TM - 1) / C::TM;
  a.tiles = (int)((a.n + C::TN - 1) / C::TN);
  // (rounded up, the last few workgroups would be a second round of the chip: 703 queries, three blocks, 530278 codes of 1536, 1 bit, the whole
  // search 1867 us, 1050 so; 699 queries, 35872 codes of 512, 2 bits 99.9 -> 95.9)
  int64_t r = (int64_t)per_cu * device_cu_count() / a.qblocks;
  r = r < 1 ? 1 : r > a.tiles ? a.tiles : r;
  a.ranges = (int)r;
  a.per_xcd = (a.qblocks * a.ranges + XCDS - 1) / XCDS;
  static LdsLimit lds_limit;  // per instantiation: the limit is raised once per device
  if (const hipError_t e = raise_lds_limit(lds_limit, reinterpret_cast<const void*>(&search_gemm_kernel<FIND, BITS, PROD, TW, WM, WN>), C::LDS);
      e != hipSuccess)
    return e;
  hipLaunchKernelGGL((search_gemm_kernel<FIND, BITS, PROD, TW, WM, WN>), dim3(a.per_xcd * XCDS), dim3(C::THREADS), C::LDS, s, a);
  return hipGetLastError();
}

// 256 codes per tile; as many queries per tile as still give most compute units one
template <bool FIND, int BITS, bool PROD>
hipError_t launch_fits(const SearchGemmArgs& a, hipStream_t s) {
  const int64_t cus = device_cu_count(), cols = (a.n + 255) / 256;
  // (half of them: a tile of half the queries decodes every code twice as often.  More than 128 queries: fewer go to tq_search_few.hip)
  auto fills = [&](int tm) { return (a.M + tm - 1) / tm * cols * 2 >= cus; };
  if (fills(256)) return launch_tile<FIND, BITS, PROD, 2, 4, 2>(a, 1, s);
  if (fills(128)) return launch_tile<FIND, BITS, PROD, 2, 2, 4>(a, 1, s);
  if (fills(64)) return launch_tile<FIND, BITS, PROD, 1, 2, 4>(a, 1, s);
  return launch_tile<FIND, BITS, PROD, 1, 1, 8>(a, 2, s);
}
template <int BITS, bool PROD>
hipError_t launch_one(const SearchGemmArgs& a, hipStream_t s) {
  return a.list_u != nullptr ? launch_fits<true, BITS, PROD>(a, s) : launch_fits<false, BITS, PROD>(a, s);
}

}  // namespace

hipError_t launch_code_search(int bits, bool prod, const CodeSearch& q, int d, const uint32_t* idx, const uint32_t* qjl, const float* gamma,
                              const float* norm, int64_t n, int64_t code_step, float kappa, const Codebook& cb, hipStream_t s) {
  if (d % 128 != 0) return hipErrorInvalidValue;
  SearchGemmArgs a;
  std::memset(&a, 0, sizeof(a));
  a.R = static_cast<const unsigned char*>(q.r_pieces); a.S = static_cast<const unsigned char*>(q.s_pieces);
  a.M = q.nq; a.d = d; a.idx = idx; a.qjl = qjl; a.gamma = gamma; a.norm = norm; a.n = n; a.kappa = kappa; a.tab = make_code_table(bits, cb);
  a.q_inv = q.inv; a.e1 = q.e1; a.e2 = q.e2; a.bar = q.bar; a.bar_step = q.bar_step; a.sample = q.sample; a.ld_sample = q.ld_sample;
  a.code_step = code_step; a.list_u = q.list_u; a.list_i = q.list_i; a.count = q.count; a.cap = q.cap; a.s_rel = q.s_rel;
  if (search_few_serves(bits, prod, q.nq, d, n)) return launch_search_few(bits, prod, a, s);
  TQ_CODE_BITS(launch_one)
}

}  // namespace tq
