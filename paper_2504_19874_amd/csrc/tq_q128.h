// Shared by the d = 128 quantisers on the fp16 matrix cores: tq_q128_bf3.hip (large batches, the matrices resident in LDS) and
// tq_q128_few.hip (small ones, the matrices in registers).  Both read the same image of the matrices.
#pragma once
#include "tq_bf3.h"
#include "tq_h2.h"

namespace tq {

constexpr int MAT_ELEMS = 128 * 128;  // one piece of one matrix
constexpr int PI_ELEMS = 2 * MAT_ELEMS;
constexpr int W_ELEMS = 2 * MAT_ELEMS;

// The residual is carried 64-fold, and so are the tables that it comes from: its two fp16 pieces then have room on both sides
// (for a unit vector; 2^-30 |e| at the lower end).
constexpr float Q128_RES = 64.f;
// Tables that the kernels take: others (no unit vector comes near such centroids) go to the fp32 instructions
constexpr float Q128_TABLE_MAX = 64.f;
inline bool q128_table(const Codebook& cb, int bits) {
  for (int i = 0; i < 1 << bits; ++i)
    if (!(cb.c[i] >= -Q128_TABLE_MAX && cb.c[i] <= Q128_TABLE_MAX)) return false;
  return true;
}
// Rows that are taken as given may be of any length: the power of two that brings a vector's 64-fold residual into the range of
// fp16, 1 for every unit vector.  inv: accumulator -> 64-fold coordinate; an accumulator is a sum of 128 products of values
// below 2^15, and a residual is at most a coordinate and a centroid.  (The sketch keeps signs only: no one undoes this.)
__device__ __forceinline__ float q128_room(float inv) {
  const float most = fmaf(inv, 0x1p37f, Q128_RES * Q128_TABLE_MAX);
  const uint32_t e = __float_as_uint(most) >> 23;  // (NaN and infinity: 255)
  return most <= 65000.f ? 1.f : __uint_as_float((268u - e) << 23);  // most in [2^(e - 127), 2^(e - 126)): below 2^15 then
}
inline Codebook q128_scaled(Codebook cb) {
  for (float& v : cb.c) v *= Q128_RES;
  for (float& v : cb.t) v *= Q128_RES;
  return cb;
}

// element offset of column col (a multiple of 4) of row `row` inside a piece: chunk (col / 8) xor (row % 16)
__device__ __forceinline__ int q128_at(int row, int col) { return row * 128 + ((((col >> 3) ^ row) & 15) << 3) + (col & 7); }

// position of column j inside its run of 16 in the image of S Pi^T: the two middle groups of four change
// places (the order in which a 32 x 32 accumulator tile enumerates them)
__device__ __forceinline__ int q128_w_col(int j) { return (j & ~12) | ((j & 4) << 1) | ((j & 8) >> 1); }

// sum of the squares of two bf16 values added to acc: one two-element dot product with fp32 accumulation
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float square_pair(uint32_t w, float acc) {
  const bf16x2_t v = __builtin_bit_cast(bf16x2_t, w);
  return __builtin_amdgcn_fdot2_f32_bf16(v, v, acc, false);
}

// The bit pattern of the largest magnitude of a 128 x 128 matrix, by NT threads; max_s: a word of LDS that was cleared
template <int NT>
__device__ __forceinline__ uint32_t largest_of(const float* W, uint32_t* max_s, int tid) {
  uint32_t m = 0u;
#pragma unroll
  for (int i = 0; i < 4096 / NT; ++i) {
    const u32x4 v = *reinterpret_cast<const u32x4*>(W + (i * NT + tid) * 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) m = max(m, v[e] & 0x7fffffffu);
  }
  atomicMax(max_s, m);
  __syncthreads();
  return *max_s;
}

}  // namespace tq
