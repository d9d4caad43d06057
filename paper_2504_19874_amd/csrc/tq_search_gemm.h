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

// Few queries (tq_search_few.hip); the number of query blocks and ranges is its own
bool search_few_serves(int M, int d, int64_t n);
hipError_t launch_search_few(int bits, bool prod, const SearchGemmArgs& a, hipStream_t s);

}  // namespace tq
