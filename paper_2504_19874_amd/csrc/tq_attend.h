// Shared by the attention read-out kernels (tq_attend.hip, tq_attend_128.hip).
#pragma once
#include "tq_internal.h"

namespace tq {

// Partial result of one (query, chunk of keys):  [0] m = largest logit of the chunk,
// [1] l = sum exp(logit - m), [4, 4 + d) sum exp(logit - m) nu c[idx] (rotated basis),
// [4 + d, 4 + 2 d) sum exp(logit - m) nu gamma z (sketch basis; zero for an MSE value cache).
__host__ __device__ constexpr int attend_part_stride(int d) { return 4 + 2 * d; }

struct AttendArgs {
  const float* scores;  // [n_groups * q_per_group][lds]: key scores, not yet multiplied by scale
  int64_t lds;
  const uint32_t* idx;  // value codes, n_groups * n rows
  const uint32_t* qjl;
  const float* gamma;
  const float* norm;
  float* part;          // [n_groups * q_per_group][nchunks][attend_part_stride(d)]
  int nchunks;
  int keys;             // d = 128 kernel: of a chunk, see attend128_keys
  int64_t n;            // keys per group
  int64_t group_stride; // value code rows between the first tokens of consecutive groups (>= n)
  int d;
  int q_per_group;
  float scale;
  int gs_hi;            // two instances: coordinate groups of instance hi (0: one instance); norm is [n][2] then
  // d = 128 kernel, one short chunk: the output itself, rotated back (nullptr: partial results to `part`, for launch_attend_combine)
  float* out;
  int64_t ldo;
  const float* Pi;
  const float* S;
  float kappa;
};
// the tables of the value codes (two instances: cb of instance lo); apart, since the d = 128 kernel has no use for them
struct AttendTables {
  Codebook cb;
  Codebook cb_hi;
};

// d = 128 on the integer matrix cores (tq_attend_128.hip)
// Keys of a chunk (a workgroup): 256 (four wavefronts of 64), 512 (eight of 64) or 2048 (eight of 256).
constexpr int AT_KEYS[3] = {256, 512, 2048};
// Of a value code's planes: whether chunks of 256 keys are ever taken.  The kernels for them exist for such values only.
__host__ __device__ constexpr bool attend128_takes_256(int planes) { return planes > 2; }
inline int attend128_chunks(int64_t n, int keys) { return (int)((n + keys - 1) / keys); }
// planes: of a value code, the signs of Alg. 2 or the top plane of instance hi among them
int attend128_keys(int64_t n, int n_groups, int q_per_group, int planes);
int attend128_max_chunks(int64_t n, int n_groups, int q_per_group, int planes);  // of any call with at most n keys per group
bool attend128_applicable(int d, bool prod, const Codebook& cb, const Codebook* cb_hi);
struct ScoreI8Args;
hipError_t launch_attend128(int kb, bool kprod, const ScoreI8Args* ka, bool vprod, const AttendArgs& a, const AttendTables& t, int n_groups,
                            hipStream_t s);

int attend_simple_chunks(int64_t n);
hipError_t launch_attend_values(bool prod, const AttendArgs& a, const Codebook& cb, int n_groups, hipStream_t s);
hipError_t launch_attend_combine(const float* part, int nchunks, int d, int64_t nq, const float* Pi, const float* S,
                                 float kappa, float* out, int64_t ldo, hipStream_t s);

}  // namespace tq
