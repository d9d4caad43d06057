// In-kernel query preparation shared by the single-kernel d = 128 scoring kernels
// (tq_score_i8_128.hip, tq_score_i8_split.hip): a workgroup of 8 (the read-out's: or 4) wavefronts rotates / sketches
// its own four queries from the transposed matrices and writes their digits.
//
//   load      wavefront w requests its thread's column of matrix w / 4 (0: Pi^T, 1: S^T), half
//             (w / 2) % 2 of k, column j = tid % 128: 64 values, to be issued before anything else
//   matvec    y_j partial sums for the four queries -> part_s[matrix][half][query][j].  The queries' coordinates lie in registers of
//             every row of 16 lanes and are broadcast by the multiplication itself.  Through scalar registers, of which they take more
//             than there are, they were three trips to memory in a row behind everything else that had been asked for: 1.4 us of
//             a read-out over 1024 keys (19.1 -> 18.3 us with its two appends; 8 x 65536 keys scored: 11.2 -> 10.9).  The matrices as
//             8 bytes per lane in half as many loads: 0.5 us slower with a sketch
//   (barrier)
//   digits    i8_digitise_terms, or what the two instances share (tq_score_i8_split.hip)
//   (barrier)
#pragma once
#include "tq_score_i8.h"

namespace tq {

// Operands of v_mfma_f32_16x16x128_f8f6f4 for masked sums at d = 128.  The mask side is fp4: of the word of a coordinate group the
// bits 4 i + {0, 1, 2} stay where they are and read as 0.5, 1 and 2, the bits 4 i + 3 are shifted down three places; dword v of a
// lane's operand has the bits 4 i + v, i = 0..7 (element 8 v + i).  The query side is fp8: a digit of coordinate c times 2, 1, 1/2 or 2
// by c % 4, so that every product is the digit itself.  A lane's 32 elements are k = 32 (lane / 16) + 0..31 of an fp4
// operand, but 16 (lane / 16) + 0..15 and 64 more of an fp8 one (found with one-hot operands): mask_slot is the byte of
// coordinate c in a digit row whose lanes read 16 bytes at 16 kq and 16 at 64 + 16 kq.
__host__ __device__ constexpr int mask_slot(int c) { return (c & ~31) + 8 * (c & 3) + ((c >> 2) & 7); }

constexpr int I8_PART_FLOATS = 2 * 2 * 4 * 128;

// max / sum over the 64 lanes: four DPP steps inside each row of 16, then the four rows
// through scalar registers
template <int CTRL>
__device__ __forceinline__ int dpp_move(int v) {
  return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xF, 0xF, false);
}
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, __int_as_float(dpp_move<0xB1>(__float_as_int(v))));   // quad_perm [1,0,3,2]
  v = fmaxf(v, __int_as_float(dpp_move<0x4E>(__float_as_int(v))));   // quad_perm [2,3,0,1]
  v = fmaxf(v, __int_as_float(dpp_move<0x141>(__float_as_int(v))));  // row_half_mirror
  v = fmaxf(v, __int_as_float(dpp_move<0x140>(__float_as_int(v))));  // row_mirror
  const float r0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0));
  const float r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 16));
  const float r2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 32));
  const float r3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 48));
  return fmaxf(fmaxf(r0, r1), fmaxf(r2, r3));
}
__device__ __forceinline__ int wave_sum(int v) {
  v += dpp_move<0xB1>(v);
  v += dpp_move<0x4E>(v);
  v += dpp_move<0x141>(v);
  v += dpp_move<0x140>(v);
  return __builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16) + __builtin_amdgcn_readlane(v, 32) +
         __builtin_amdgcn_readlane(v, 48);
}

typedef float f32x4_prep __attribute__((ext_vector_type(4), aligned(4)));  // (the queries are the caller's)

// acc[q] += sum over k = 4 I .. 4 N - 1 of w[k] * (coordinate k of vector q), which lane k / 4 of every row of 16 holds in q[q][k % 4]:
// fetched from there in one instruction with its product.  (The compiler makes two of it.  It does not look inside: s_nop is the
// distance that a register moved just before needs from its use by other lanes.)
template <int I, int N, int M>
__device__ __forceinline__ void matvec_rows(float (&acc)[4], const f32x4_prep (&q)[4], const float (&wv)[M]) {
  static_assert(4 * N <= M, "");
#define TQ_FMAC(ACC, Q, W) "\n\tv_fmac_f32_dpp %" #ACC ", %" #Q ", %" #W " row_newbcast:%24 row_mask:0xf bank_mask:0xf"
  asm("s_nop 1"
      TQ_FMAC(0, 4, 20) TQ_FMAC(1, 8, 20) TQ_FMAC(2, 12, 20) TQ_FMAC(3, 16, 20)
      TQ_FMAC(0, 5, 21) TQ_FMAC(1, 9, 21) TQ_FMAC(2, 13, 21) TQ_FMAC(3, 17, 21)
      TQ_FMAC(0, 6, 22) TQ_FMAC(1, 10, 22) TQ_FMAC(2, 14, 22) TQ_FMAC(3, 18, 22)
      TQ_FMAC(0, 7, 23) TQ_FMAC(1, 11, 23) TQ_FMAC(2, 15, 23) TQ_FMAC(3, 19, 23)
      : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3])
      : "v"(q[0][0]), "v"(q[0][1]), "v"(q[0][2]), "v"(q[0][3]), "v"(q[1][0]), "v"(q[1][1]), "v"(q[1][2]), "v"(q[1][3]), "v"(q[2][0]),
        "v"(q[2][1]), "v"(q[2][2]), "v"(q[2][3]), "v"(q[3][0]), "v"(q[3][1]), "v"(q[3][2]), "v"(q[3][3]), "v"(wv[4 * I]),
        "v"(wv[4 * I + 1]), "v"(wv[4 * I + 2]), "v"(wv[4 * I + 3]), "n"(I));
#undef TQ_FMAC
  if constexpr (I + 1 < N) matvec_rows<I + 1, N>(acc, q, wv);
}

template <bool HAVE_R, bool PROD>
struct I8Prep {
  float wv[64];
  f32x4_prep q[4];  // coordinates 4 i .. 4 i + 3 of the half of k, in lane i of every row of 16
  int mat, kh, j;
  bool work;

  __device__ __forceinline__ void load(const ScoreI8Args& a, int group, int q0, int wave, int tid) {
    load_part(a, group, q0, wave >> 2, (wave >> 1) & 1, tid);
  }
  __device__ __forceinline__ void load_part(const ScoreI8Args& a, int group, int q0, int matrix, int half, int tid) {
    mat = matrix;
    kh = half;
    j = tid & 127;
    work = mat == 0 ? HAVE_R : PROD;  // uniform
    if (work) {
      const float* WT = (mat ? a.ST : a.PiT) + (64 * kh) * 128 + j;
#pragma unroll
      for (int k = 0; k < 40; ++k) wv[k] = WT[k * 128];
      // (here: in front of the matrix they hold up what comes from a nearer cache, 11.5 us in place of 10.9, behind it the products)
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int qi = 0; qi < 4; ++qi) {
        const int64_t r = (int64_t)group * a.q_per_group + (q0 + qi < a.q_per_group ? q0 + qi : q0);
        q[qi] = *reinterpret_cast<const f32x4_prep*>(a.x + r * a.ldx + 64 * kh + 4 * (tid & 15));
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 40; k < 64; ++k) wv[k] = WT[k * 128];
    }
  }

  __device__ __forceinline__ void matvec(float* part_s) {
    if (!work) return;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    matvec_rows<0, 16>(acc, q, wv);
#pragma unroll
    for (int qi = 0; qi < 4; ++qi) part_s[((mat * 2 + kh) * 4 + qi) * 128 + j] = acc[qi];
  }
};

// Four balanced base-32 digits of the integer Q, |Q| <= 2^19, of coordinate c in the form above:
// dig_s[term][query][digit][slot] (integers up to 16 and their halves and doubles are exact in fp8, all steps here in fp32)
__device__ __forceinline__ void put_mask_digits(unsigned char* dig_s, int term, int qi, int c, float Q) {
  const float f = (c & 3) == 1 ? 1.f : (c & 3) == 2 ? 0.5f : 2.f;
  const float q1 = rintf(Q * 0x1p-5f), q2 = rintf(q1 * 0x1p-5f), q3 = rintf(q2 * 0x1p-5f);
  int w = __builtin_amdgcn_cvt_pk_fp8_f32(f * fmaf(-32.f, q1, Q), f * fmaf(-32.f, q2, q1), 0, false);
  w = __builtin_amdgcn_cvt_pk_fp8_f32(f * fmaf(-32.f, q3, q2), f * q3, w, true);
  unsigned char* o = dig_s + (term * 4 + qi) * 4 * 128 + mask_slot(c);
  o[0] = (unsigned char)w;
  o[128] = (unsigned char)(w >> 8);
  o[256] = (unsigned char)(w >> 16);
  o[384] = (unsigned char)(w >> 24);
}

__device__ __forceinline__ float wave_sum_f(float v) {
  v += __int_as_float(dpp_move<0xB1>(__float_as_int(v)));
  v += __int_as_float(dpp_move<0x4E>(__float_as_int(v)));
  v += __int_as_float(dpp_move<0x141>(__float_as_int(v)));
  v += __int_as_float(dpp_move<0x140>(__float_as_int(v)));
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0)) + __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 16)) +
         __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 32)) + __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 48));
}

// Digit images for the d = 128 single-kernel path, one per masked sum, so that all the masked sums of the
// rotated query share ONE accumulator: term t (the t-th plane subset of odd size, factor coef[m]) is the image of
// Q = round(coef[m] y 2^s), s the power of two with max |coef| max |y| 2^s <= 2^19; the sketch term (index 2^(BITS-1)) is that of S q as before.  Wavefront w takes
// (matrix w / 4, query w % 4).
//   dig_s[term][query][digit][slot]; scal_s[matrix][query][0: 2^-s, 1: matrix 0: coef[0] sum_j y_j, matrix 1:
//   2^-s sum_j Q_j]
__host__ __device__ constexpr int i8_terms(int bits, bool prod) { return (bits > 0 ? 1 << (bits - 1) : 0) + (prod ? 1 : 0); }

template <int BITS, bool PROD>
__device__ __forceinline__ void i8_digitise_terms(const ScoreI8Args& a, int q0, int wave, int lane, const float* part_s,
                                                  unsigned char* dig_s, float* scal_s) {
  constexpr int NM = (1 << BITS) - 1;
  constexpr int NTM = BITS > 0 ? 1 << (BITS - 1) : 0;
  // without a sketch both halves of the workgroup write images of the rotated query, every other one
  const int m = PROD ? wave >> 2 : 0, qi = wave & 3, part = PROD ? 0 : wave >> 2;
  if (!(m == 0 ? BITS > 0 : PROD) || (NTM == 1 && part != 0)) return;
  const bool live = q0 + qi < a.q_per_group;
  float y[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int c = lane + 64 * u;
    y[u] = live ? part_s[((m * 2 + 0) * 4 + qi) * 128 + c] + part_s[((m * 2 + 1) * 4 + qi) * 128 + c] : 0.f;
  }
  auto put = [&](int term, int u, float Q) { put_mask_digits(dig_s, term, qi, lane + 64 * u, Q); };
  float cmax = 1.f;
  if (m == 0) {
    cmax = 0.f;
#pragma unroll
    for (int v = 1; v <= NM; ++v)
      if (i8_term(v)) cmax = fmaxf(cmax, fabsf(a.coef[v]));
  }
  const float mx = wave_max(fmaxf(fabsf(y[0]), fabsf(y[1]))) * cmax;
  int e = 0;
  if (mx > 0.f) (void)frexpf(mx, &e);  // mx = f * 2^e, f in [0.5, 1): |Q| <= 2^19
  const float sc = ldexpf(1.f, 19 - e), inv = ldexpf(1.f, e - 19);
  if (m == 1) {
    const float Q0 = rintf(y[0] * sc), Q1 = rintf(y[1] * sc);
    const int tot = wave_sum((int)Q0 + (int)Q1);
    put(NTM, 0, Q0);
    put(NTM, 1, Q1);
    if (lane == 0) {
      scal_s[(4 + qi) * 4 + 0] = inv;
      scal_s[(4 + qi) * 4 + 1] = (float)tot * inv;
    }
  } else {
    int term = 0;
#pragma unroll
    for (int v = 1; v <= NM; ++v) {
      if (!i8_term(v)) continue;
      if (PROD || NTM == 1 || (term & 1) == part) {  // uniform
        put(term, 0, rintf(a.coef[v] * y[0] * sc));
        put(term, 1, rintf(a.coef[v] * y[1] * sc));
      }
      ++term;
    }
    const float ysum = wave_sum_f(y[0] + y[1]);
    if (lane == 0 && part == 0) {
      scal_s[qi * 4 + 0] = inv;
      scal_s[qi * 4 + 1] = a.coef[0] * ysum;
    }
  }
}

}  // namespace tq
