// Dequantisation of codes whose centroid table is a sum of signs, on the scaled-format matrix instruction
// (tq_sign_gemm.hip: multiples of 128 from 256 on; tq_sign_128.hip: d = 128).
//
// A table of one bit is +-c, and one of two bits that is symmetric about zero is linear in the signs of its two planes,
//     c[idx] = alpha s_1 + beta s_0,   alpha = (c_2 + c_3) / 2,  beta = (c_3 - c_2) / 2,   s_p = +-1 by plane p,
// and the sketch is signs to begin with.  So the whole decoding is x~ = nu (alpha Pi^T s_1 + beta Pi^T s_0 + kappa gamma S^T z):
// products of signs with fixed matrices.  A sign is an fp4 value, and a word of bits becomes 32 of them in seven
// instructions (minus_sign_bits); an entry of a matrix is five balanced base-32 digits (25 bits of the largest entry that leads to the same output), integers
// of up to 16, which fp6 holds exactly; and v_mfma_f32_32x32x64_f8f6f4 multiplies the two at four times the rate of fp16, the
// digits' weights in its scale operand.  Five digits of one sign take 5/8 of the matrix time of two fp16 pieces, a
// two-bit centroid 10/12 of its three products, and next to nothing is left of the decoding's vector instructions.
//
// Image of a matrix W (d x d, used as W^T): [step][tile of 32 outputs][digit][64 lanes x 16 bytes, 64 lanes x 8 bytes], 32 values of
// 6 bits per lane.  With S = d / 64 steps lane (l, h) of step s holds contraction indices of group g = h S + s (so that a
// lane's words of consecutive steps lie side by side), element 8 v + i the index 32 g + 4 i + v (bit 4 i + v of the word).
// Output of lane l of tile t: d = 128: 32 t + l; else 64 (t / 2) + 2 l + t % 2 (two tiles of a wavefront make whole lines).
#pragma once
#include "tq_bf3.h"
#include "tq_h2.h"

namespace tq {

constexpr int SIGN_DIGITS = 5, SIGN_FRAG_BYTES = 64 * 24;

struct SignCoefs {
  double alpha, beta;
};
// tables the kernels take: none (bits 0), +-c, or two bits symmetric about zero with two different magnitudes
bool sign_table(int bits, const Codebook& cb, SignCoefs* c);

__host__ __device__ constexpr size_t sign_image_bytes(int d) { return (size_t)(d / 64) * (d / 32) * SIGN_DIGITS * SIGN_FRAG_BYTES; }

// the larger of two magnitudes, where NaN stays
__device__ __forceinline__ float sign_larger(float m, float mx) { return m <= mx || mx != mx ? mx : m; }

// What one unit of the last digit stands for in an output's column, from the column's largest magnitude: 16.5 32^4 units
__device__ __forceinline__ float sign_unit(float largest) {
  const float u = largest * (1.00001f / 17301504.f);
  return u > 1e-37f ? u : 1e-37f;
}

// digit j of 16 values of a column, 6 bits each
__device__ __forceinline__ void sign_digit(const float (&v)[16], float unit, int j, uint32_t (&w)[3]) {
  w[0] = w[1] = w[2] = 0u;
  const double per = 1. / (double)unit;
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    float q = (float)rint((double)v[e] * per);  // an integer below 2^24.05: exact where it matters, even above 2^24
    for (int k = 0; k < j; ++k) q = rintf(q * 0x1p-5f);
    const float up = j + 1 < SIGN_DIGITS ? rintf(q * 0x1p-5f) : 0.f;
    const int digit = (int)fminf(fmaxf(fmaf(-32.f, up, q), -16.f), 16.f);
    const uint32_t code = digit < 0 ? 32u - (uint32_t)digit : (uint32_t)digit;  // sign bit 5, magnitude 0..16
    const int at = 6 * e;
    w[at >> 5] |= code << (at & 31);
    if ((at & 31) > 26) w[(at >> 5) + 1] |= code >> (32 - (at & 31));
  }
}

typedef int v8i_t __attribute__((ext_vector_type(8)));
struct SignFrag {  // a digit's 32 values of a lane
  u32x4 a;
  uint2 b;
};
__device__ __forceinline__ v8i_t sign_operand(const SignFrag& f) {
  typedef int v4 __attribute__((ext_vector_type(4)));
  const v4 a = __builtin_bit_cast(v4, f.a), b = v4{(int)f.b.x, (int)f.b.y, 0, 0};
  return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, -1, -1);
}
// Minus the signs of 32 bits (bit set: +1) as fp4; two: 0x22222222 in a register that the compiler does not know (one v_and_or_b32 takes no two
// constants: seven instructions, twelve otherwise).  The sums are all of the other sign, which their last factor puts right.
__device__ __forceinline__ uint32_t sign_two() {
  uint32_t two = 0x22222222u;
  asm volatile("" : "+v"(two));
  return two;
}
__device__ __forceinline__ v8i_t minus_sign_bits(uint32_t w, uint32_t two) {
  typedef int v4 __attribute__((ext_vector_type(4)));
  const v4 v = {(int)(((w << 3) & 0x88888888u) | two), (int)(((w << 2) & 0x88888888u) | two), (int)(((w << 1) & 0x88888888u) | two),
                (int)((w & 0x88888888u) | two)};
  return __builtin_shufflevector(v, v, 0, 1, 2, 3, -1, -1, -1, -1);
}
// accumulator += signs x digit J, in units: 8 (fp6 holds eighths) 32^J
template <int J>
__device__ __forceinline__ floatx16 sign_mfma(const v8i_t& signs, const v8i_t& digit, const floatx16& acc) {
  constexpr int lo = 0x918C8782;  // 127 + 3 + 5 J for J = 0..3
  if constexpr (J < 4) return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(signs, digit, acc, 4, 2, 0, 127, J, lo);
  else return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(signs, digit, acc, 4, 2, 0, 127, 0, 150);
}

// d a multiple of 128 from 256 on: a tile's digits of one step in 8 KB, the units (powers of two here) behind those of step 0
constexpr int SIGN_STEP_BYTES = 8192;
__host__ __device__ constexpr size_t sign_gemm_image_bytes(int d) { return (size_t)(d / 64) * (d / 32) * SIGN_STEP_BYTES; }
bool sign_gemm_images(int d);  // images of this form are kept at this d
bool sign_gemm_serves(int bits, bool prod, int d, int64_t n);
hipError_t launch_sign_gemm_image(const float* W, int d, void* image, hipStream_t s);
hipError_t launch_sign_gemm(int bits, bool prod, const void* pi_image, const void* s_image, int d, const uint32_t* idx, const uint32_t* qjl,
                            const float* gamma, const float* norm, int64_t n, float* out, int64_t ldo, float kappa, const SignCoefs& c, hipStream_t s);

// d = 128, both in one launch: image of Pi and its units, image of S and its units
constexpr size_t SIGN128_BYTES = sign_image_bytes(128) + 128 * 4;  // of one matrix
hipError_t launch_sign128_images(const float* Pi, const float* S, void* images, hipStream_t s);
// images null: every workgroup makes its digits itself, the same ones, from Pi and S
hipError_t launch_sign128_dequant(int bits, bool prod, const uint32_t* idx, const uint32_t* qjl, const float* gamma, const float* norm,
                                  const void* images, const float* Pi, const float* S, float* out, int64_t ldo, int64_t n, float kappa,
                                  const SignCoefs& c, hipStream_t s);

}  // namespace tq
