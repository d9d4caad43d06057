// Top-k of many queries over many codes without looking at every score twice (tq_search.hip).
#pragma once
#include "tq_internal.h"

namespace tq {

struct SearchArgs {
  int bits;
  bool prod;
  int nq, d, topk;        // topk 1..64
  const float *qr, *qs;   // rotated and sketched queries, [nq][d]
  const uint32_t *idx, *qjl;
  const float *gamma, *norm;
  int64_t n;
  float kappa;
  int32_t* topk_idx;
  float* topk_val;        // nullable
};

bool search_applicable(int bits, bool prod, int d, int64_t n, int nq, int topk, const Codebook& cb);
size_t search_workspace_bytes(int d, int64_t n, int64_t nq, int topk);
// The k best codes of every query whose candidates fit its list; flags[q] != 0 (device, [nq], in the workspace): those of q
// did not, its results are still to be made.  The scores returned are those of tq_score_bf3.hip, bit for bit.  The workspace
// holds the lists of as many queries as fit 512 MB; more are taken one block after the other.
hipError_t launch_search(const SearchArgs& a, const Codebook& cb, void* workspace, const int32_t** flags, hipStream_t s);

}  // namespace tq
