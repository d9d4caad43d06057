// Dense contractions of fp32 factors on the fp16 matrix cores, two fp16 pieces per factor.
//
// Every fp32 value is taken as x = (hi + lo) / s with s a power of two that brings the largest magnitude of its row (of
// the whole matrix for the fixed operand) into [2^14, 2^15), hi = fp16(s x), lo = fp16(s x - hi).  What is left out is
// below 2^-22 |x| (2^-24.5 in the root mean square), or below 2^-39 of the row's largest value where that is more (the
// end of the subnormal range).  A product of two pieces is exact in fp32; hi hi + hi lo + lo hi are summed in the fp32
// accumulator of v_mfma_f32_32x32x16_f16 and lo lo (2^-22 of the product at most) is dropped.  That is three matrix
// instructions per fp32 product at the accuracy of an fp32 evaluation to within its own rounding; three bf16 pieces
// need five for less.  A bf16 vector is one exact piece: two products.
//
// Layout.  Both operands are rows of pieces, [row][k / 32][piece][32 k]: with two pieces a row's k-step is one line of
// 128 bytes.  A workgroup copies its tiles from memory straight into LDS (global_load_lds_dwordx4: no registers, no
// vector instructions), eight lanes per line, and the lanes take the line's eight 16-byte chunks in the order
// slot ^ (row % 8), so that the LDS rows need no padding and a fragment read (32 rows, one chunk each) meets every bank
// equally often.
#pragma once
#include "tq_internal.h"

namespace tq {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

constexpr int kH2ImageHeader = 256;  // bytes before an image built in scratch memory: its scale

// scale of a row (or matrix) whose largest magnitude has the bit pattern `maxbits`: s = 2^e with s * max in [2^14, 2^15),
// as bits of s and of 1 / s (kept away from the ends of the exponent range; infinities and NaN take s = 1)
__device__ __forceinline__ void h2_scale(uint32_t maxbits, float& s, float& inv) {
  const int e = (int)(maxbits >> 23);
  int se = 268 - e;
  se = se > 252 ? 252 : se;
  se = e >= 255 ? 127 : se;
  s = __uint_as_float((uint32_t)se << 23);
  inv = __uint_as_float((uint32_t)(254 - se) << 23);
}

__device__ __forceinline__ uint32_t h2_bits(f16x2 v) { return *reinterpret_cast<const uint32_t*>(&v); }

// two scaled values as their hi and lo pieces (packed pairs)
__device__ __forceinline__ void h2_split(float a, float b, uint32_t& hi, uint32_t& lo) {
  typedef float f2 __attribute__((ext_vector_type(2)));
  const f16x2 h = __builtin_convertvector(f2{a, b}, f16x2);
  const f16x2 l = __builtin_convertvector(f2{a - (float)h[0], b - (float)h[1]}, f16x2);
  hi = h2_bits(h);
  lo = h2_bits(l);
}

// 64 lanes x 16 bytes from memory into LDS at `lds` (uniform, bytes) + 16 * lane; the compiler does not know of it, so
// whoever reads the data waits for it explicitly (h2_wait_barrier)
__device__ __forceinline__ void h2_dma(const void* base, uint32_t voff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base), "s"(lds) : "memory");
}
__device__ __forceinline__ uint32_t h2_lds_address(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}
template <int VM>
__device__ __forceinline__ void h2_wait_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(VM) : "memory");
}

// LDS image of a tile: a row's k-step is NP * 4 chunks of 16 bytes; with one piece two rows share a line of 128 bytes.
// h2_place: byte address of chunk c of row r; h2_chunk: the chunk that the slot of r's line holds.
template <int NP>
__device__ __forceinline__ uint32_t h2_place(int r, int c) {
  if (NP == 2) return r * 128 + ((c ^ ((r >> 1) & 7)) << 4);
  return (r >> 1) * 128 + ((((r & 1) << 2) | (c ^ ((r >> 2) & 3))) << 4);
}
template <int NP>
__device__ __forceinline__ uint32_t h2_chunk(int r, int slot) {
  return NP == 2 ? slot ^ ((r >> 1) & 7) : (slot & 3) ^ ((r >> 2) & 3);
}

// ---- host side -------------------------------------------------------------------------------------------------------

// the quantiser's two contractions (tq_gemm_h2.hip)
struct H2Quant {
  const void* W;         // image of the fixed matrix (two pieces), M = d rows
  const float* w_inv;    // device: 1 / scale of that image
  const void* X;         // pieces of the vectors
  int npx;               // pieces per vector value: 2, or 1 for bf16 vectors
  int d;
  int64_t n;
  const float* fac;      // [n] accumulator -> rotated coordinate of the (unit-normalised) vector
  const float* esc;      // [n] power of two for the residual's pieces
  float* out;            // launch_h2_store: the products, [n][d]
  uint32_t* words;       // packed indices or signs
  void* E;               // residual pieces out (two), nullable
  float* part;           // [ceil(d / tile)][n] partial squared residual norms: out with E, in for the sketch
  int part_tiles;        // in for the sketch: how many of them
  float* gamma;          // sketch: the residual norms out
};
bool h2_codebook_serves(int bits, const Codebook& cb);
size_t h2_image_bytes(int M, int d);                         // pieces only
hipError_t launch_h2_image(const float* W, int64_t ldw, int M, int d, void* image, float* w_inv, hipStream_t s);
hipError_t launch_h2_max(const float* W, int64_t ldw, int M, int d, uint32_t* max_bits, hipStream_t s);  // bits of the largest magnitude
// rows of x as pieces, their norms and factors; w_inv: of the matrix they will meet.  cut (the quantiser): an fp32 value is
// first rounded to its two leading bf16 pieces, 17 bits, the reading of fp32 vectors that the contraction on bf16 pieces
// (tq_gemm.hip) has: batches on either side of the line between the two, and calls with and without workspace, then decide alike,
// and codes stay what they have been (with all 22 bits the mean error of a rotated coordinate falls from 1.9e-6 to 0.1 -
// 0.3e-6 sigma; of 10^6 vectors at d = 3072, 1 + 1 bits, 1e-3 of the sign words change).  The pieces here hold it exactly.
hipError_t launch_h2_split(const void* x, bool bf16, bool cut, int64_t ldx, int64_t n, int d, bool normalise, const float* w_inv, void* pieces,
                           float* norm, float* fac, float* esc, hipStream_t s);
int h2_part_tiles(int d, int64_t n);                         // rows of H2Quant::part
int64_t h2_full_rows(int d, int64_t rows);                   // the largest useful pass over at most `rows` vectors
hipError_t launch_h2_quant(int bits, const H2Quant& a, const Codebook& cb, hipStream_t s);
hipError_t launch_h2_sign(const H2Quant& a, hipStream_t s);
hipError_t launch_h2_store(const H2Quant& a, hipStream_t s);  // out = W X^T as it is

}  // namespace tq
