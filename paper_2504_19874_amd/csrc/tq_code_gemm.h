// Dense contractions of packed codes against the rows of a fixed operand on the fp16 matrix cores (tq_code_gemm.hip):
// dequantisation (rows of Pi^T and S^T) and the first pass of a nearest-neighbour search (rotated queries).
#pragma once
#include "tq_h2.h"

namespace tq {

// Order of the 32 coordinates of a word group along the contraction: four bytes' worth of bits at the same bit position are
// decoded together, so position 4 k + e (k = 0..7) is coordinate k + {0, 16, 8, 24}[e].
__host__ __device__ constexpr int code_position(int coord) {
  const int b = coord >> 3;
  return 4 * (coord & 7) + (b == 0 ? 0 : b == 2 ? 1 : b == 1 ? 2 : 3);
}

// A centroid table symmetric about zero as fp16 pieces by bytes: byte m of hh / hl is the high / low byte of the leading
// piece of the m-th magnitude, lh / ll those of the second piece
struct CodeTable {
  uint32_t hh[2], hl[2], lh[2], ll[2];
  float inv;  // 1 / scale of the pieces; 1 bit: the centroid itself, the operand being +-1
};
bool code_gemm_serves(int bits, const Codebook& cb);  // symmetric tables of up to 4 bits
CodeTable make_code_table(int bits, const Codebook& cb);
float code_table_error(int bits, const Codebook& cb);  // largest relative error of a leading piece (2 bits or more)

// Image of a d x d matrix's transpose in the order above: rows of two fp16 pieces, h2_image_bytes(d, d) bytes
hipError_t launch_code_image(const float* W, int d, void* image, float* w_inv, hipStream_t s);

// x~_i = nu_i (Pi^T c[idx_i] + kappa gamma_i S^T z_i) for n codes, out rows ldo floats apart (ldo and d multiples of 4)
hipError_t launch_code_dequant(int bits, bool prod, const void* pit_image, const float* pit_inv, const void* st_image, const float* st_inv,
                               int d, const uint32_t* idx, const uint32_t* qjl, const float* gamma, const float* norm, int64_t n,
                               float* out, int64_t ldo, float kappa, const Codebook& cb, hipStream_t s);

// The first pass of a search: scores of all codes from ONE piece of every factor, each within
//     eps = |nu| (e1 + kappa |gamma| e2)
// of the exact one.  sample != NULL: score - eps of codes 0, code_step, 2 code_step, ... (n of them) to sample[query][ld_sample].
// Otherwise every (score + eps, code) with score + eps >= bar[query] is appended to the query's list; count may pass cap.
// Ints between the counters of two queries: a line each.  Every workgroup adds to them, and additions to one line wait for each other on their
// way through memory (searches, us, counters side by side / so: 64 queries, k = 64, 400000 codes of 128, 3 bits, 154 / 71; 40 queries, k = 10, 300000 of 768
// 140 / 105; 300 queries 189 / 170).
constexpr int COUNT_STEP = 32;
// Bytes between the pieces of 32 coordinates of all queries and those of the next 32.  A kernel's step takes these of a block of queries: side by
// side they are whole lines on all channels of the L2; a query's coordinates side by side, they were half lines a multiple of 2 KB apart (d = 1024).
__host__ __device__ constexpr uint32_t search_step_bytes(int nq) { return (uint32_t)(nq + (nq & 1)) * 64u; }
struct CodeSearch {
  const void* r_pieces;  // [d / 32][nq][32] fp16 (search_step_bytes), the contraction's order (code_position): Pi q scaled
  const void* s_pieces;  // S q scaled
  int nq;
  const float *inv, *e1, *e2, *bar;
  int bar_step;          // floats between the bars of consecutive queries
  float s_rel;           // scale of r_pieces over that of s_pieces (the same for all queries)
  float* sample;
  int64_t ld_sample;
  float* list_u;
  int32_t* list_i;
  int32_t* count;  // [nq][COUNT_STEP], the first of each is used
  int cap;
};
hipError_t launch_code_search(int bits, bool prod, const CodeSearch& q, int d, const uint32_t* idx, const uint32_t* qjl, const float* gamma,
                              const float* norm, int64_t n, int64_t code_step, float kappa, const Codebook& cb, hipStream_t s);

}  // namespace tq
