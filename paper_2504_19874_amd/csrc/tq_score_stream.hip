// Scoring for a few queries per code at d > 128 (online search, logits at larger head dimensions): one pass over the
// codes, whatever d.
//
// The arithmetic is that of masked sums (the estimator of Sec. 3.2 over the bit planes of a code; tq_score_i8.h): a centroid table symmetric
// about zero has a Walsh expansion over the odd-sized subsets of the index bits, so
//     sum_j qr_j c[idx_j] = coef[0] sum_j qr_j + sum_S coef[S] M_S,   M_S = sum of qr_j over the coordinates where the XOR
//                                                                     of the plane bits in S is 1,
// and sum_j qs_j z_j = 2 M_Z - sum_j qs_j.  Every M is a contraction of query digits with 0/1 masks on
// v_mfma_i32_16x16x64_i8, exact but for the query's rounding to 21 bits.  The mask operand needs no table: a stored word
// ANDed with 0x01010101 << k is four operand bytes (bit k + 8 b in byte b, worth 2^k), and the digits on the other side
// are those of Q 2^(7 - k) (negated for k = 7, where the byte reads as -128), so that every product carries the factor 128.
//
// What bounds it: the codes have to stream from memory once (10^6 codes of 3072 coordinates, 1 + 1 bits: 776 MB) while
// the operands of the query stay on chip.  The digits of four (or eight) queries sit in LDS for the life of a workgroup;
// a wavefront takes T tiles of 16 keys and walks their rows, 64 W (BITS or 1) contiguous bytes of a key per step, the words of the next
// step on their way while those of this one are expanded.  Every operand read from LDS serves T tiles.
// (Before: 512 coordinates per launch, each launch adding to the scores of the one before.  10^6 codes, 4 queries,
// kernel time: d = 3072, 1 + 1 bits 500 us -> 182; d = 1536, 4 bits 255 -> 200, where the expansion, 8 ANDs and
// 8 matrix instructions per 4 coordinates of a lane, is what is left.  Cutting the rows over the wavefronts of a workgroup instead, digits in
// registers and the parts added through LDS, gave 190 - 202 us for the first: every line of the codes then meets several wavefronts at
// different times.)
#include <cstring>

#include "tq_score_digits.h"
#include "tq_score_i8.h"

namespace tq {
namespace {

struct StreamArgs {
  const uint4* img;   // [query][2 matrices][d / 32][digit][2] 16-byte operands
  const float* scal;  // [query][2][4]: 1 / scale, sum of the rounded coordinates
  const uint32_t* idx;
  const uint32_t* qjl;
  const float* gamma;
  const float* norm;
  float* scores;
  int64_t lds;
  int64_t n;
  int groups_d;  // d / 32
  int q_per_group;
  float kappa;
  float coef[16];
};

constexpr int kMaxDigitBytes = 144 * 1024;

template <int N>
__device__ __forceinline__ void load_words(const uint32_t* p, uint32_t (&w)[N]) {
  typedef uint32_t v2 __attribute__((ext_vector_type(2), aligned(4)));
  typedef uint32_t v3 __attribute__((ext_vector_type(3), aligned(4)));
  typedef uint32_t v4 __attribute__((ext_vector_type(4), aligned(4)));
  constexpr int N4 = N / 4 * 4;
#pragma unroll
  for (int i = 0; i < N4; i += 4) {
    const v4 v = *reinterpret_cast<const v4*>(p + i);
#pragma unroll
    for (int e = 0; e < 4; ++e) w[i + e] = v[e];
  }
  if constexpr (N - N4 == 3) {
    const v3 v = *reinterpret_cast<const v3*>(p + N4);
    w[N4] = v[0];
    w[N4 + 1] = v[1];
    w[N4 + 2] = v[2];
  }
  if constexpr (N - N4 == 2) {
    const v2 v = *reinterpret_cast<const v2*>(p + N4);
    w[N4] = v[0];
    w[N4 + 1] = v[1];
  }
  if constexpr (N - N4 == 1) w[N4] = p[N4];
}

template <int BITS, bool PROD, int QB>
struct StreamCfg {
  static constexpr int NTI = BITS > 0 ? 1 << (BITS - 1) : 0;      // masked sums of the rotated query
  static constexpr int NT = NTI + (PROD ? 1 : 0);
  static constexpr int NV = (BITS > 0 ? 1 : 0) + (PROD ? 1 : 0);  // matrices
  static constexpr int T = NT * QB <= 4 ? 4 : NT * QB <= 10 ? 2 : 1;  // tiles of 16 keys per wavefront: what the registers hold the sums of
};

// W: word groups of a key that a lane takes per step
// SHORT: one tile per wavefront at a time
template <int BITS, bool PROD, int W, int QB, bool SHORT>
__global__ __launch_bounds__(512, 2) void score_stream_kernel(const StreamArgs a) {
  using C = StreamCfg<BITS, PROD, QB>;
  constexpr int T = SHORT ? 1 : C::T, NV = C::NV, NT = C::NT;
  constexpr int NM = (1 << BITS) - 1;
  extern __shared__ __attribute__((aligned(16))) v4i dig_s[];  // [step][W][2][matrix][query block][lane]
  __shared__ float scal_s[4 * QB][4];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, kq = lane >> 4;
  const int group = blockIdx.y;
  const int q0 = blockIdx.z * (4 * QB);
  const int G = a.groups_d, steps = G / (4 * W);
  const int64_t gbase = (int64_t)group * a.n;

  // the codes of this wavefront: blocks of 16 T keys, one in every (wavefronts of the grid); lane chunk kq of a step has groups
  // 4 W step + W kq .. + W - 1
  const int64_t nblk = (a.n + 16 * T - 1) / (16 * T);
  const int waves = blockDim.x >> 6;
  const int64_t stride = (int64_t)gridDim.x * waves;
  int64_t blk = (int64_t)blockIdx.x * waves + wave;
  struct Words {
    uint32_t p[T][BITS > 0 ? W * BITS : 1], z[T][PROD ? W : 1];
  };
  auto load = [&](Words& w, int64_t b, int step) {
    const int g = (step * 4 + kq) * W;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int64_t key = (b * T + t) * 16 + col;
      const int64_t row = gbase + (key < a.n ? key : a.n - 1);  // keys past the end: not stored
      if constexpr (BITS > 0) load_words(a.idx + (row * G + g) * BITS, w.p[t]);
      if constexpr (PROD) load_words(a.qjl + row * G + g, w.z[t]);
    }
  };
  Words wa, wb;
  load(wa, blk < nblk ? blk : nblk - 1, 0);

  for (int e = tid; e < G * 2 * NV * QB * 16; e += blockDim.x) {
    const int l = e & 63, qb = (e >> 6) % QB, v = (e >> 6) / QB % NV, ws = (e >> 6) / (QB * NV);  // ws: (step * W + w) * 2 + s
    const int s = ws & 1, w = (ws >> 1) % W, step = (ws >> 1) / W;
    const int qa = q0 + 4 * qb + ((l & 15) >> 2);  // row of the operand = 4 * query + digit
    const int64_t q = (int64_t)group * a.q_per_group + (qa < a.q_per_group ? qa : a.q_per_group - 1);
    const uint4 d = a.img[((q * 2 + (BITS > 0 ? v : 1)) * G + (step * 4 + (l >> 4)) * W + w) * 8 + (l & 3) * 2 + s];
    dig_s[e] = v4i{(int)d.x, (int)d.y, (int)d.z, (int)d.w};
  }
  if (tid < 4 * QB) {
    const int64_t q = (int64_t)group * a.q_per_group + (q0 + tid < a.q_per_group ? q0 + tid : a.q_per_group - 1);
    scal_s[tid][0] = BITS > 0 ? a.scal[q * 8] : 0.f;
    scal_s[tid][1] = BITS > 0 ? a.coef[0] * a.scal[q * 8 + 1] : 0.f;
    scal_s[tid][2] = PROD ? 2.f * a.scal[q * 8 + 4] : 0.f;
    scal_s[tid][3] = PROD ? a.scal[q * 8 + 5] : 0.f;
  }
  __syncthreads();
  if (blk >= nblk) return;  // no barrier below

  // dword i of the operand of half s: bits 4 s + i + {0, 8, 16, 24} of the word where they are
  auto expand16 = [&](uint32_t w, int s) -> v4i {
    v4i b;
#pragma unroll
    for (int i = 0; i < 4; ++i) b[i] = (int)(w & (0x01010101u << (4 * s + i)));
    return b;
  };
  auto digits_sum = [&](const v4i& c) -> float { return stream_digits_sum(c[0], c[1], c[2], c[3]); };
  v4i acc[T][NT][QB];
  auto clear = [&] {
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) acc[t][j][qb] = v4i{0, 0, 0, 0};
  };
  clear();
  int step = 0;
  // one step on `cur`, the next one's words requested into `nxt`; false after the last
  auto advance = [&](const Words& cur, Words& nxt) -> bool {
    const bool last = step + 1 == steps;  // uniform
    const int64_t nblk_ = last ? blk + stride : blk;
    const int nstep = last ? 0 : step + 1;
    load(nxt, nblk_ < nblk ? nblk_ : blk, nstep);
    float nu[T], kg[T];
    if (last) {
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const int64_t key = (blk * T + t) * 16 + col;
        const int64_t row = gbase + (key < a.n ? key : a.n - 1);
        nu[t] = a.norm != nullptr ? a.norm[row] : 1.f;
        kg[t] = PROD ? a.kappa * a.gamma[row] : 0.f;
      }
    }
    const v4i* const d = dig_s + (size_t)step * (W * 2 * NV * QB * 64) + lane;
#pragma unroll
    for (int w = 0; w < W; ++w)
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        v4i A[NV][QB];
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
          for (int qb = 0; qb < QB; ++qb) A[v][qb] = d[(((w * 2 + s) * NV + v) * QB + qb) * 64];
#pragma unroll
        for (int t = 0; t < T; ++t) {
          int j = 0;
#pragma unroll
          for (int m = 1; m <= NM; ++m) {
            if (!i8_term(m)) continue;
            uint32_t x = 0u;
#pragma unroll
            for (int pl = 0; pl < BITS; ++pl)
              if (m & (1 << pl)) x ^= cur.p[t][BITS > 0 ? w * BITS + pl : 0];
            const v4i b = expand16(x, s);
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) acc[t][j][qb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A[0][qb], b, acc[t][j][qb], 0, 0, 0);
            ++j;
          }
          if constexpr (PROD) {
            const v4i b = expand16(cur.z[t][w], s);
#pragma unroll
            for (int qb = 0; qb < QB; ++qb)
              acc[t][NT - 1][qb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A[NV - 1][qb], b, acc[t][NT - 1][qb], 0, 0, 0);
          }
        }
      }
    if (last) {
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        const int qi = q0 + 4 * qb + kq;
        const float s0 = scal_s[4 * qb + kq][0], s1 = scal_s[4 * qb + kq][1], s2 = scal_s[4 * qb + kq][2], s3 = scal_s[4 * qb + kq][3];
        float* const out = a.scores + ((int64_t)group * a.q_per_group + qi) * a.lds + blk * (16 * T) + col;
#pragma unroll
        for (int t = 0; t < T; ++t) {
          float r = 0.f;
          int j = 0;
#pragma unroll
          for (int m = 1; m <= NM; ++m)
            if (i8_term(m)) r = fmaf(a.coef[m], digits_sum(acc[t][j++][qb]), r);
          float v = BITS > 0 ? fmaf(s0, r, s1) : 0.f;
          if (PROD) v = fmaf(kg[t], fmaf(s2, digits_sum(acc[t][NT - 1][qb]), -s3), v);
          if (qi < a.q_per_group && (blk * T + t) * 16 + col < a.n) out[16 * t] = nu[t] * v;
        }
      }
      clear();
    }
    blk = nblk_;
    step = nstep;
    return blk < nblk;
  };
  while (advance(wa, wb) && advance(wb, wa)) {
  }
}

template <int BITS, bool PROD, int W, int QB, bool SHORT>
hipError_t launch_t(const StreamArgs& a, int64_t gx, int qz, int threads, int n_groups, hipStream_t s) {
  static LdsLimit lds_limit;  // per instantiation: the limit is raised once per device
  if (const hipError_t e = raise_lds_limit(lds_limit, reinterpret_cast<const void*>(&score_stream_kernel<BITS, PROD, W, QB, SHORT>), kMaxDigitBytes);
      e != hipSuccess)
    return e;
  const int lds = a.groups_d * 2 * (StreamCfg<BITS, PROD, QB>::NV) * QB * 256;
  hipLaunchKernelGGL((score_stream_kernel<BITS, PROD, W, QB, SHORT>), dim3((unsigned)gx, n_groups, (unsigned)qz), dim3(threads), lds, s, a);
  return hipGetLastError();
}

template <int BITS, bool PROD, int W, int QB>
hipError_t launch_qb(const StreamArgs& a, int n_groups, hipStream_t s) {
  using C = StreamCfg<BITS, PROD, QB>;
  const int qz = (a.q_per_group + 4 * QB - 1) / (4 * QB);
  const int64_t others = (int64_t)n_groups * qz, cus = device_cu_count();
  // one workgroup per compute unit (two where registers and LDS admit them), each walking its share of the keys; a list too
  // short for that in wavefronts of one tile and workgroups of four (10^4 codes of 3072 coordinates, 2 queries, 3 + 1 bits: 20.9 us -> 16.6)
  const int64_t nwg = (a.n + 128 * C::T - 1) / (128 * C::T);
  if (nwg * others * 4 <= cus * 3) return launch_t<BITS, PROD, W, QB, true>(a, (a.n + 63) / 64, qz, 256, n_groups, s);
  const int per_cu = C::NT * QB * C::T <= 4 && a.groups_d * 2 * C::NV * QB * 256 <= 72 * 1024 ? 2 : 1;
  int64_t gx = (per_cu * cus + others - 1) / others;
  if (gx > nwg) gx = nwg;
  return launch_t<BITS, PROD, W, QB, false>(a, gx, qz, 512, n_groups, s);
}

// four queries per pass over the codes, or eight where there are more than four and their digits fit LDS
template <int BITS, bool PROD, int W>
hipError_t launch_w(const StreamArgs& a, int n_groups, hipStream_t s) {
  const bool eight = a.q_per_group > 4 && a.groups_d * 2 * StreamCfg<BITS, PROD, 2>::NV * 2 * 256 <= kMaxDigitBytes;
  return eight ? launch_qb<BITS, PROD, W, 2>(a, n_groups, s) : launch_qb<BITS, PROD, W, 1>(a, n_groups, s);
}

}  // namespace

hipError_t launch_score_stream(int bits, bool prod, const uint4* img, const float* scal, const uint32_t* idx, const uint32_t* qjl,
                               const float* gamma, const float* norm, float* scores, int64_t lds, int64_t n, int d, int n_groups,
                               int q_per_group, float kappa, const float* coef, hipStream_t stream) {
  StreamArgs a;
  a.img = img; a.scal = scal; a.idx = idx; a.qjl = qjl; a.gamma = gamma; a.norm = norm; a.scores = scores; a.lds = lds; a.n = n;
  a.groups_d = d / 32; a.q_per_group = q_per_group; a.kappa = kappa;
  std::memcpy(a.coef, coef, sizeof(a.coef));
  const int m = d / 128;
  const int w = m % 4 == 0 ? 4 : m % 3 == 0 ? 3 : m % 2 == 0 ? 2 : 1;
  if (d % 128 != 0) return hipErrorInvalidValue;
#define TQ_STREAM_W(B, P)                               \
  switch (w) {                                           \
    case 1: return launch_w<B, P, 1>(a, n_groups, stream); \
    case 2: return launch_w<B, P, 2>(a, n_groups, stream); \
    case 3: return launch_w<B, P, 3>(a, n_groups, stream); \
    default: return launch_w<B, P, 4>(a, n_groups, stream); \
  }
  switch (bits * 2 + (prod ? 1 : 0)) {
    case 1: TQ_STREAM_W(0, true)
    case 2: TQ_STREAM_W(1, false)
    case 3: TQ_STREAM_W(1, true)
    case 4: TQ_STREAM_W(2, false)
    case 5: TQ_STREAM_W(2, true)
    case 6: TQ_STREAM_W(3, false)
    case 7: TQ_STREAM_W(3, true)
    case 8: TQ_STREAM_W(4, false)
    case 9: TQ_STREAM_W(4, true)
    default: return hipErrorInvalidValue;
  }
#undef TQ_STREAM_W
}

}  // namespace tq
