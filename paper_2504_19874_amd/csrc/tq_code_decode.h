// Packed codes into fp16 operands of the matrix cores (tq_code_gemm.hip, tq_search.hip, tq_search_gemm.hip, tq_search_few.hip).
#pragma once
#include "tq_code_gemm.h"

namespace tq {

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

// F<BITS, PROD>(a, s) for the kind of code that `bits` and `prod` name
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

}  // namespace tq
