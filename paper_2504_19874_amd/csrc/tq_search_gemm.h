// What the two kernels share that pass over all codes of a search (tq_search_gemm.hip, tq_search_few.hip).
#pragma once
#include "tq_code_decode.h"

namespace tq {

struct SearchGemmArgs {
  const unsigned char* R;  // pieces of the rotated and of the sketched queries
  const unsigned char* S;
  int M, d;
  const uint32_t* idx;
  const uint32_t* qjl;
  const float* gamma;
  const float* norm;
  int64_t n, code_step;
  float kappa, s_rel;
  CodeTable tab;
  const float *q_inv, *e1, *e2, *bar;
  int bar_step;
  float* sample;
  int64_t ld_sample;
  float* list_u;
  int32_t* list_i;
  int32_t* count;
  int cap;
  int qblocks, ranges, tiles, per_xcd;
};

// Constants that the compiler is not to see through: as literals they would cost an instruction where they are a third operand
struct PlaneTable {
  uint32_t hh[2], hl[2];  // bytes of the magnitudes' pieces, the high ones negated
  uint32_t top16, top8, one16, odd_bits, pairs, threes, sevens;
  __device__ __forceinline__ explicit PlaneTable(const CodeTable& t) {
#pragma unroll
    for (int i = 0; i < 2; ++i) hh[i] = t.hh[i] ^ 0x80808080u, hl[i] = t.hl[i];
    top16 = 0x80008000u, top8 = 0x80808080u, one16 = 0x3C003C00u, odd_bits = 0x55555555u, pairs = 0x33333333u, threes = 0x03030303u, sevens = 0x07070707u;
    asm volatile("" : "+s"(top16), "+s"(top8), "+v"(one16), "+s"(odd_bits), "+s"(pairs), "+s"(threes), "+s"(sevens));
  }
};

// Words of a group of 32 values into fp16 operands, four values (bit position p of the four bytes) at a time as in tq_code_decode.h, with the low
// planes of several positions joined at once: vector instructions are paid in matrix time.  A lane that takes 16 values of a group: 42 / 36 / 33 / 16
// instructions at 4 / 3 / 2 / 1 bits, 75 / 58 / 43 / 25 position by position.
template <int BITS>
struct Planes {
  uint32_t s, n[4];
  __device__ __forceinline__ void set(const uint32_t* w, const PlaneTable& t) {
    auto pick = [](uint32_t m, uint32_t a, uint32_t b) { return __builtin_amdgcn_bitop3_b32(m, a, b, 0xCA); };  // a where m, else b
    s = w[BITS - 1];
    if constexpr (BITS == 2) n[0] = ~(w[0] ^ s);
    if constexpr (BITS > 2) {
      const uint32_t x0 = ~(w[0] ^ s), x1 = ~(w[1] ^ s);
      const uint32_t even = pick(t.odd_bits, x0, x1 << 1), odd = pick(t.odd_bits, x0 >> 1, x1);
      if constexpr (BITS == 3) n[0] = even, n[1] = odd;
      if constexpr (BITS == 4) {  // n[i]: positions i and i + 4 as the halves of bytes
        const uint32_t x2 = ~(w[2] ^ s);
        n[0] = pick(t.pairs, even, x2 << 2);
        n[1] = pick(t.pairs, odd, x2 << 1);
        n[2] = pick(t.pairs, even >> 2, x2);
        n[3] = pick(t.pairs, odd >> 2, x2 >> 1);
      }
    }
  }
  __device__ __forceinline__ void quad(int p, const PlaneTable& t, uint32_t& a, uint32_t& b) const {
    if constexpr (BITS == 1) {
      a = __builtin_amdgcn_bitop3_b32(s << (15 - p), t.top16, t.one16, 0xAE);  // (~s & top) | one
      b = __builtin_amdgcn_bitop3_b32(s << (7 - p), t.top16, t.one16, 0xAE);
    } else {
      const uint32_t sel = BITS == 4 ? (n[p & 3] >> (p & 4)) & t.sevens : BITS == 3 ? (n[p & 1] >> (p & 6)) & t.threes : (n[0] >> p) & 0x01010101u;
      const uint32_t up = BITS == 4 ? __builtin_amdgcn_perm(t.hh[1], t.hh[0], sel) : __builtin_amdgcn_perm(t.hh[0], t.hh[0], sel);
      const uint32_t hi = __builtin_amdgcn_bitop3_b32(s << (7 - p), t.top8, up, 0x6A);  // (s & top) ^ up
      const uint32_t lo = BITS == 4 ? __builtin_amdgcn_perm(t.hl[1], t.hl[0], sel) : __builtin_amdgcn_perm(t.hl[0], t.hl[0], sel);
      a = __builtin_amdgcn_perm(hi, lo, 0x06020400u);
      b = __builtin_amdgcn_perm(hi, lo, 0x07030501u);
    }
  }
};

// Few queries (tq_search_few.hip); the number of query blocks and ranges is its own
bool search_few_serves(int bits, bool prod, int M, int d, int64_t n);
hipError_t launch_search_few(int bits, bool prod, const SearchGemmArgs& a, hipStream_t s);

}  // namespace tq
