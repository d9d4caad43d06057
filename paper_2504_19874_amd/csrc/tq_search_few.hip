// The pass of a search over codes (tq_search.hip says what for) for few queries: scores from one fp16 piece of every
// factor as in tq_search_gemm.hip, product for product in the same order, so that both give the same bits.
//
// There the codes go through LDS, since four wavefronts multiply what one decodes.  With up to 128 queries a tile of codes is multiplied by
// one wavefront only: 48 KB in and out of LDS per step and a barrier for two to four matrix instructions, 350 - 420 ns a step of 32 coordinates,
// whether the words came from memory or from L2 (21 queries, 105293 codes of 3072, 2 + 1 bits: 147 us, 70 here; 57, 275068 of 512, 1 + 1 bits
// 81 / 51).  Here a lane decodes what it multiplies: lane (c, h) of a fragment holds the positions 16 s + 8 h .. + 7 of code c, which are bit
// positions 4 s + 2 h and the next of the group's bytes, so that the words moved right by 2 h give every lane its values with the same constants.  Only the queries' pieces go through LDS, CH steps at a time in two buffers: one wait and one
// barrier a chunk, for requests made a chunk before.  A code's scalars are the lane's own.
#include "tq_search_gemm.h"

#include <type_traits>

namespace tq {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int XCDS = 8;

// TW x 32 queries, a wavefront's 32 codes.  (Chunks of eight steps: no faster, and a lane has twice the words.)
constexpr int WAVES = 4, CH = 4;
template <int TW>
struct FewCfg {
  static constexpr int THREADS = 64 * WAVES, TM = 32 * TW, TN = 32 * WAVES;
  static constexpr int STEP_BYTES = TM * 64, CHUNK_BYTES = CH * STEP_BYTES;
  static constexpr int AL = CHUNK_BYTES / 1024 / WAVES;  // a wavefront's direct loads per chunk
  static constexpr int QUERY_F = 7;
  static constexpr int FOUND = THREADS;
  static constexpr int LDS = 2 * CHUNK_BYTES + QUERY_F * TM * 4 + 2 * FOUND * 12;
  static_assert(AL * 1024 * WAVES == CHUNK_BYTES, "roles");
};

template <bool FIND, int BITS, bool PROD, int TW>
__global__ __launch_bounds__(64 * WAVES, 2) void search_few_kernel(const SearchGemmArgs a) {
  using C = FewCfg<TW>;
  constexpr int TM = C::TM, TN = C::TN, AL = C::AL;
  constexpr bool HAVE_P = BITS > 0, HAVE_S = PROD;
  constexpr int NW = BITS > 0 ? BITS : 1;
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
  // per query: bar / A, E1 / A, E2 / A (for the first test), 1 / scale, E1, E2, bar
  float* const query_s = reinterpret_cast<float*>(lds + 2 * C::CHUNK_BYTES);
  int* const found_s = reinterpret_cast<int*>(query_s + C::QUERY_F * TM);  // [parity][query, code, score + eps][FOUND]
  __shared__ int found_n[4];                                              // by tile number

  const int logical = (int)(blockIdx.x % XCDS) * a.per_xcd + (int)(blockIdx.x / XCDS);
  if (logical >= a.qblocks * a.ranges) return;
  const int qb = __builtin_amdgcn_readfirstlane(logical % a.qblocks), range = __builtin_amdgcn_readfirstlane(logical / a.qblocks);
  const int tile0 = __builtin_amdgcn_readfirstlane((int)((int64_t)range * a.tiles / a.ranges));
  const int tile1 = __builtin_amdgcn_readfirstlane((int)((int64_t)(range + 1) * a.tiles / a.ranges));
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, h = lane >> 5;
  const int m0 = qb * TM;
  const int rows_m = min(TM, a.M - m0);
  const int G = a.d >> 5;
  const int n_s = HAVE_S ? G / CH : 0, n_chunks = n_s + (HAVE_P ? G / CH : 0);

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
      const int at = wave * AL + j, step = at / (2 * TW), r = 2 * (at % (2 * TW) * 8 + l8) + (slot >> 2);
      va[j] = (uint32_t)min(r, rows_m - 1) * 64 + step * step_a + h2_chunk<1>(r, slot) * 16;
    }
  }
  const uint32_t lds0 = h2_lds_address(lds);
  int a_chunk = 0, buf = 0;
  auto dma = [&](int to_buf) {
    const uint64_t g = (uint64_t)gA;
    const uint32_t g_lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)g);
    const uint32_t g_hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(g >> 32));
    const void* const base = reinterpret_cast<const void*>((uint64_t)g_hi << 32 | g_lo);
    const uint32_t to = (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds0 + to_buf * C::CHUNK_BYTES + wave * (AL * 1024)));
#pragma unroll
    for (int j = 0; j < AL; ++j) h2_dma(base, va[j], to + j * 1024);
    ++a_chunk;
    gA += (int64_t)step_a * CH;
    if (HAVE_S && HAVE_P && a_chunk == n_s) gA = gP;
    if (a_chunk == n_chunks) a_chunk = 0, gA = gS;
  };

  // ---- codes: a chunk's words at a time, tile after tile --------------------------------------------------
  auto code_row = [&](int tile) {  // codes past the end: the last one again
    const int64_t i = (int64_t)tile * TN + wave * 32 + l32;
    return (i < a.n ? i : a.n - 1) * (FIND ? 1 : a.code_step);
  };
  const uint32_t *wi = nullptr, *wz = nullptr;
  int w_chunk = 0, w_tile = tile0;
  auto point = [&] {
    const int64_t row = code_row(w_tile);
    if (HAVE_P) wi = a.idx + row * G * BITS;
    if (HAVE_S) wz = a.qjl + row * G;
  };
  point();
  uint32_t words[CH * NW], next_words[CH * NW];
  auto load_chunk = [&] {
    typedef uint32_t v4 __attribute__((ext_vector_type(4), aligned(4)));
    if (HAVE_S && (!HAVE_P || w_chunk < n_s)) {
      uint32_t w[CH];
#pragma unroll
      for (int j = 0; j < CH; j += 4) {
        const v4 v = *reinterpret_cast<const v4*>(wz + w_chunk * CH + j);
#pragma unroll
        for (int e = 0; e < 4; ++e) w[j + e] = v[e];
      }
#pragma unroll
      for (int j = 0; j < CH; ++j) next_words[j] = w[j];
    } else if constexpr (HAVE_P) {
      uint32_t w[CH * NW];
#pragma unroll
      for (int j = 0; j < CH * NW; j += 4) {
        const v4 v = *reinterpret_cast<const v4*>(wi + (w_chunk - n_s) * (CH * BITS) + j);
#pragma unroll
        for (int e = 0; e < 4; ++e) w[j + e] = v[e];
      }
#pragma unroll
      for (int j = 0; j < CH * NW; ++j) next_words[j] = w[j];
    }
    if (++w_chunk == n_chunks) {
      w_chunk = 0;
      ++w_tile;
      point();
    }
  };

  floatx16 acc[TW];
  const PlaneTable tab(a.tab);
  constexpr int AHEAD = 2;
  const unsigned char* const pa[2] = {lds + h2_place<1>(l32, h), lds + h2_place<1>(l32, 2 + h)};
  // of_p: the chunk belongs to the centroid segment
  auto chunk = [&](auto of_p) __attribute__((always_inline)) {  // (called, it would keep the accumulators in memory)
    constexpr int B = decltype(of_p)::value ? NW : 1;
    // what was asked for a chunk ago is there, moved right by the lane's half (a move that the compiler can not put off to behind the loads below)
#pragma unroll
    for (int j = 0; j < CH * B; ++j) asm volatile("v_lshrrev_b32 %0, %1, %2" : "=v"(words[j]) : "v"(2 * h), "v"(next_words[j]));
    h2_wait_barrier<0>();
    __builtin_amdgcn_sched_barrier(0);
    load_chunk();
    dma(buf ^ 1);
    __builtin_amdgcn_sched_barrier(0);
    // half a step at a time: the fragments of the queries AHEAD half-steps before their products, the codes' one before, between the products
    constexpr int HALVES = 2 * CH;
    const int at = buf * C::CHUNK_BYTES;
    f16x8 f[AHEAD + 1][TW];
    uint32_t v[2][4];
    auto read = [&](int i) {
#pragma unroll
      for (int t = 0; t < TW; ++t)
        f[i % (AHEAD + 1)][t] = *reinterpret_cast<const f16x8*>(pa[i & 1] + at + (i >> 1) * C::STEP_BYTES + t * 2048);
    };
    auto decode = [&](int i, int j) {  // one of the two quads of a half-step
      Planes<B> codes;
      codes.set(words + (i >> 1) * B, tab);
      codes.quad(4 * (i & 1) + j, tab, v[i & 1][2 * j], v[i & 1][2 * j + 1]);
    };
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) read(i);
    decode(0, 0);
    decode(0, 1);
#pragma unroll
    for (int i = 0; i < HALVES; ++i) {
      __builtin_amdgcn_sched_barrier(0);
      if (i + AHEAD < HALVES) read(i + AHEAD);
      const uint4 b4 = make_uint4(v[i & 1][0], v[i & 1][1], v[i & 1][2], v[i & 1][3]);
      const f16x8 b = *reinterpret_cast<const f16x8*>(&b4);
#pragma unroll
      for (int t = 0; t < TW; ++t) {
        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(f[i % (AHEAD + 1)][t], b, acc[t], 0, 0, 0);
        if (i + 1 < HALVES) {
#pragma unroll
          for (int j = 2 * t / TW; j < 2 * (t + 1) / TW; ++j) decode(i + 1, j);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    buf ^= 1;
  };

  // ---- candidates: gathered in LDS, places for them asked for a tile later, stored another tile later ------
  int pend_q = -1, pend_code = 0, pend_pos = 0;
  float pend_top = 0.f;
  auto store_pending = [&] {
    if (pend_q >= 0 && pend_pos < a.cap) {
      a.list_u[(int64_t)pend_q * a.cap + pend_pos] = pend_top;
      a.list_i[(int64_t)pend_q * a.cap + pend_pos] = pend_code;
    }
    pend_q = -1;
  };
  auto ask_for = [&](int tile) {
    const int* const f = found_s + (tile & 1) * 3 * C::FOUND;
    if (tid < found_n[tile & 3]) {
      pend_q = f[tid];
      pend_code = f[C::FOUND + tid];
      pend_top = __int_as_float(f[2 * C::FOUND + tid]);
      pend_pos = atomicAdd(a.count + (int64_t)pend_q * COUNT_STEP, 1);
    }
  };

  // ---- before the first tile -------------------------------------------------------------------------------
  dma(0);
  load_chunk();
  float next_nu = 1.f, next_ga = 0.f;
  auto request_scalars = [&](int tile) {
    const int64_t r = code_row(tile);
    next_nu = a.norm != nullptr ? a.norm[r] : 1.f;
    next_ga = HAVE_S ? a.gamma[r] : 0.f;
  };
  request_scalars(tile0);
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
  if (tid < 4) found_n[tid] = 0;

  for (int tile = tile0; tile < tile1; ++tile) {
    const float pi = HAVE_P ? a.tab.inv : 1.f;
    const float kg = HAVE_S ? a.kappa * next_ga : 0.f;
    const float nu = (int64_t)tile * TN + wave * 32 + l32 < a.n ? next_nu : __builtin_nanf("");  // past the end: reaches nothing
    const float fac_s = HAVE_P ? kg * a.s_rel / pi : 1.f, fac = HAVE_P ? pi : kg * a.s_rel;
#pragma unroll
    for (int t = 0; t < TW; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
    if constexpr (HAVE_S) {
      for (int c = 0; c < n_s; ++c) chunk(std::false_type{});
      if constexpr (HAVE_P) {  // the sketch sums in units of the centroid segment
#pragma unroll
        for (int t = 0; t < TW; ++t)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[t][r] *= fac_s;
      }
    }
    if constexpr (HAVE_P)
      for (int c = n_s; c < n_chunks; ++c) chunk(std::true_type{});

    // ---- comparisons: a lane has 16 queries of one code per 32 x 32 tile ------------------------------------
    // (what is derived from the lane is made again here: kept from before the loop, sums of it would take hundreds of registers all through it)
    int eh = h;
    asm volatile("" : "+v"(eh));
    request_scalars(tile + 1 < tile1 ? tile + 1 : tile);
    if (FIND) {
      // (every wavefront has met a barrier since it added to what is read, and will before it adds to what is cleared)
      store_pending();
      if (tile > tile0) ask_for(tile - 1);
      if (tid == 0) found_n[(tile + 2) & 3] = 0;
    }
    const int64_t code_i = (int64_t)tile * TN + wave * 32 + l32;
    // the first test divides by what the score is multiplied with; where that is not a positive number it lets everything through
    const float per = HAVE_P ? nu : nu * fac;
    const float inv = per > 0.f ? 1.f / per : __builtin_nanf(""), rest = HAVE_P ? 1.f : 1.f / fabsf(fac);
#pragma unroll
    for (int t = 0; t < TW; ++t)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int m = t * 32 + 8 * k + 4 * eh;
        __builtin_amdgcn_sched_barrier(0);  // one quad of queries at a time (registers)
        auto exact = [&](int e, float sign) {  // score + sign * its error bound
          const float* const q = query_s + m + e;
          float eps = HAVE_P ? fabsf(nu) * q[4 * TM] : 0.f;  // (without centroids that factor is zero, and a norm may be infinite)
          if (HAVE_S) eps = fmaf(fabsf(nu * kg), q[5 * TM], eps);
          return fmaf(acc[t][4 * k + e] * (nu * fac), q[3 * TM], sign * eps);
        };
        if constexpr (!FIND) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (code_i < a.n && m + e < rows_m) a.sample[(int64_t)(m0 + m + e) * a.ld_sample + code_i] = exact(e, -1.f);
        } else {
          auto quad = [&](int f) { return *reinterpret_cast<const float4*>(query_s + f * TM + m); };
          const float4 b4 = quad(0), d14 = quad(1), d24 = HAVE_S ? quad(2) : make_float4(0.f, 0.f, 0.f, 0.f);
          const float b[4] = {b4.x, b4.y, b4.z, b4.w}, d1[4] = {d14.x, d14.y, d14.z, d14.w}, d2[4] = {d24.x, d24.y, d24.z, d24.w};
          uint64_t maybe[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float bound = HAVE_S ? fmaf(d2[e], fabsf(kg), d1[e]) : d1[e];
            if (!HAVE_P) bound *= rest;
            maybe[e] = __builtin_amdgcn_ballot_w64(!(acc[t][4 * k + e] < fmaf(b[e], inv, -bound)));
          }
          if ((maybe[0] | maybe[1] | maybe[2] | maybe[3]) == 0u) continue;  // four scores of every lane behind one branch
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if (maybe[e] == 0u) continue;
            const float top = exact(e, 1.f);
            if (((maybe[e] >> lane) & 1u) != 0u && top >= query_s[6 * TM + m + e]) {
              const int q = m0 + m + e;
              const int at = atomicAdd(&found_n[tile & 3], 1);
              if (at < C::FOUND) {
                int* const f = found_s + (tile & 1) * 3 * C::FOUND + at;
                f[0] = q;
                f[C::FOUND] = (int)code_i;
                f[2 * C::FOUND] = __float_as_int(top);
              } else if (const int pos = atomicAdd(a.count + (int64_t)q * COUNT_STEP, 1); pos < a.cap) {
                a.list_u[(int64_t)q * a.cap + pos] = top;
                a.list_i[(int64_t)q * a.cap + pos] = (int)code_i;
              }
            }
          }
        }
      }
  }
  if (FIND) {
    __syncthreads();
    store_pending();
    if (tile1 > tile0) ask_for(tile1 - 1);
    store_pending();
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // nothing of this workgroup's is under way to LDS when it ends
}

template <bool FIND, int BITS, bool PROD, int TW>
hipError_t launch_tile(SearchGemmArgs a, hipStream_t s) {
  using C = FewCfg<TW>;
  a.qblocks = (a.M + C::TM - 1) / C::TM;
  a.tiles = (int)((a.n + C::TN - 1) / C::TN);
  // Four workgroups a compute unit for up to 32 queries, where codes are little more than decoded (21 of 3072, 2 + 1 bits, 105293 codes: 79 -> 70 us);
  // two beyond, each of which walks twice the codes (57 of 512, 1 + 1 bits, 275068 codes: 51 us, 57 with four).
  const int per_cu = TW == 1 ? 4 : 2;
  int64_t r = (int64_t)per_cu * device_cu_count() / a.qblocks;
  r = r < 1 ? 1 : r > a.tiles ? a.tiles : r;
  a.ranges = (int)r;
  a.per_xcd = (a.qblocks * a.ranges + XCDS - 1) / XCDS;
  static LdsLimit lds_limit;  // per instantiation: the limit is raised once per device
  if (const hipError_t e = raise_lds_limit(lds_limit, reinterpret_cast<const void*>(&search_few_kernel<FIND, BITS, PROD, TW>), C::LDS);
      e != hipSuccess)
    return e;
  hipLaunchKernelGGL((search_few_kernel<FIND, BITS, PROD, TW>), dim3(a.per_xcd * XCDS), dim3(C::THREADS), C::LDS, s, a);
  return hipGetLastError();
}

template <bool FIND, int BITS, bool PROD>
hipError_t launch_fits(const SearchGemmArgs& a, hipStream_t s) {
  // As many queries per workgroup as there are, but 32 of them while the list is so short that the chip is not full with more (of long codes, whose decoding
  // is then done two to four times, twice over for up to 64 queries and for more than 128, four times between).  The whole search, us, 32 / 64 / 96 / 128
  // (through LDS): 128 queries of 128, 3 bits, 11000 codes 33.0 / 35.6 / 39.0 / 42.4 (40.5); 96 of 768, 2 + 1 bits, 36000 80.8 / 90.4 / 90.4 (108), 60000
  // 96.5 / 94.9 / 92.1; 128 of 3072, 1 + 1 bits, 16000 160 / 164 / 179 / 197 (243), 60000 235 / 222 / 260 / 233; 64 of 1536, 4 bits, 8192 69 / 76, 60000 94.0 /
  // 87.8; 200 of 2048, 4 bits, k = 64, 16000 143, 121 with 128.
  const int full = a.d < 1024 ? 5 : a.M <= 64 || a.M > 128 ? 2 : BITS >= 3 && !PROD ? 3 : 4;
  if ((a.n + 127) / 128 * ((a.M + 31) / 32) <= full * (int64_t)device_cu_count()) return launch_tile<FIND, BITS, PROD, 1>(a, s);
  if (a.M > 96) return launch_tile<FIND, BITS, PROD, 4>(a, s);
  if (a.M > 64) return launch_tile<FIND, BITS, PROD, 3>(a, s);
  if (a.M > 32) return launch_tile<FIND, BITS, PROD, 2>(a, s);
  return launch_tile<FIND, BITS, PROD, 1>(a, s);
}
template <int BITS, bool PROD>
hipError_t launch_one(const SearchGemmArgs& a, hipStream_t s) {
  return a.list_u != nullptr ? launch_fits<true, BITS, PROD>(a, s) : launch_fits<false, BITS, PROD>(a, s);
}

}  // namespace

// Up to 128 queries; and long codes where tiles of 256 queries and codes would leave half of the chip idle, whose steps follow each other
// at the latency of a step.  Beyond, a code that is decoded once for 256 queries is cheaper (1000 queries' sample 57 us, 100 here; 200 queries,
// 500000 codes of 768 381 us, 420), and 3 and 4 bits without a sketch, whose steps all have the dearest decoding, from a quarter on.  The whole search, us, 250 queries
// of 3072, through LDS / here: 28000 codes, 1 bit 140 / 134, 2 bits 167 / 163, 2 + 1 bits 299 / 276, 3 + 1 bits 307 / 288; 43000, 1 + 1 bits 311 / 325;
// 4 bits: 10000 codes 163 / 161, 19000 177 / 182, 49000 214 / 250.
bool search_few_serves(int bits, bool prod, int M, int d, int64_t n) {
  return M <= 128 || (d >= 2048 && (M + 255) / 256 * ((n + 255) / 256) * (bits >= 3 && !prod ? 4 : 2) <= (int64_t)device_cu_count());
}

hipError_t launch_search_few(int bits, bool prod, const SearchGemmArgs& a, hipStream_t s) {
  TQ_CODE_BITS(launch_one)
}

}  // namespace tq
