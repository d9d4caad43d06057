// Scoring for a few queries per code at d > 128 (online search, logits at larger head dimensions): one pass over the
// codes, whatever d.
//
// The arithmetic is that of masked sums (the estimator of Sec. 3.2 over the bit planes of a code; tq_score_i8.h): a centroid table symmetric
// about zero has a Walsh expansion over the odd-sized subsets of the index bits, so
//     sum_j qr_j c[idx_j] = coef[0] sum_j qr_j + sum_S coef[S] M_S,   M_S = sum of qr_j over the coordinates where the XOR
//                                                                     of the plane bits in S is 1,
// and sum_j qs_j z_j = 2 M_Z - sum_j qs_j.  Every M is a contraction of query digits with masks on
// v_mfma_scale_f32_16x16x128_f8f6f4, exact but for the query's rounding to 21 bits: the digits (base 49, tq_score_digits.h) are fp6 values,
// sums stay below 2^24.  The mask operand needs no table: the bits 4 i + v of a stored word (v = 0 .. 3) are eight fp4 values where they
// are, with other bits of the nibble set so that a bit is worth 2 whatever its place (mask_operand: one instruction per eight); what the
// values without the bit come to is where the sums start.
//
// What bounds it: the codes have to stream from memory once (10^6 codes of 3072 coordinates, 1 + 1 bits: 776 MB, 129 us for a
// kernel that only reads them) while the operands of the query stay on chip.  The digits of four (or eight) queries sit in LDS for the life of a workgroup;
// a wavefront takes T tiles of 16 keys and walks their rows, 64 W (BITS or 1) contiguous bytes of a key per step, the words of the next
// step on their way while those of this one are expanded.  Every operand read from LDS serves T tiles.
// Kernel time, us, 10^6 codes, 4 queries: d = 3072, 1 + 1 bits 184 -> 145; d = 1024, 2 + 1 bits 95 -> 78; d = 1536, 4 bits 203 -> 156, of which
// the expansion takes 20.  Before: byte masks on the integer instructions (twice the ANDs, twice the matrix time), half lines per
// step (162 us for reading alone), waits for everything that was under way in every other step, scores stored block by block.
// (Cutting the rows over the wavefronts of a workgroup instead, digits in registers and the parts added through LDS, gave 190 - 202 us for the
// first: every line of the codes then meets several wavefronts at different times.)
#include <algorithm>
#include <cstring>

#include "tq_score_digits.h"
#include "tq_score_i8.h"

namespace tq {
namespace {

struct StreamArgs {
  const uint32_t* img;  // [query][2 matrices][d / 32][32]: stream_digits()
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
  int qblocks, shares;  // of queries, of keys
  int slots;  // blocks of keys whose scores a wavefront gathers in LDS
  float kappa;
  float coef[16];
};

constexpr int XCDS = 8;
constexpr int kMaxLdsBytes = 159 * 1024;  // digits and gathered scores (scal_s besides)

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ v8i digit_operand(const u32x4& lo, const u32x2& hi) {
  const u32x4 h = {hi[0], hi[1], 0u, 0u};
  return __builtin_bit_cast(v8i, __builtin_shufflevector(lo, h, 0, 1, 2, 3, 4, 5, -1, -1));
}
// 32 bits b as fp4: 4 + 2 b, 2 + 2 b, 2 b, 1 - 2 b by dword.  (The constants behind the ORs in registers that the compiler does not know: one
// v_and_or_b32 takes no two constants.)
struct MaskConst {
  uint32_t c2, c4, c6;
};
__device__ __forceinline__ v8i mask_operand(uint32_t w, const MaskConst& c) {
  const u32x4 m = {(w & 0x11111111u) | c.c6, (w & 0x22222222u) | c.c4, w & 0x44444444u, (w & 0x88888888u) | c.c2};
  return __builtin_bit_cast(v8i, __builtin_shufflevector(m, m, 0, 1, 2, 3, -1, -1, -1, -1));
}
// digits are eighths
__device__ __forceinline__ f32x4 mask_mfma(const v8i& digits, const v8i& masks, const f32x4& c) {
  return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(digits, masks, c, 2, 4, 0, 130, 0, 127);
}

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
  static constexpr int WORDS = BITS + (PROD ? 1 : 0);                 // of a key per word group
  // tiles for W word groups per step: two steps' words and the sums in 160 registers
  static constexpr int tiles(int W) {
    int t = T;
    while (t > 1 && t * (2 * W * WORDS + 4 * NT * QB) > 160) t /= 2;
    return t;
  }
  // W beyond four where it makes whole lines of what four leaves in halves (a plane or the sketch alone has 16 W bytes in a
  // step): d a multiple of 1024, or a row at once.  A line in two steps is asked for twice where 64 KB are under way per compute unit.
  static constexpr bool takes(int W) { return W <= 4 || (W == 6 ? WORDS <= 4 : W == 8 ? WORDS <= 3 && (PROD || BITS < 2) : BITS < 2 && QB == 1); }
};

// W: word groups of a key that a lane takes per step
// SHORT: one tile per wavefront at a time
template <int BITS, bool PROD, int W, int QB, bool SHORT>
__global__ __launch_bounds__(512, 2) void score_stream_kernel(const StreamArgs a) {
  using C = StreamCfg<BITS, PROD, QB>;
  constexpr int T = SHORT ? 1 : C::tiles(W), NV = C::NV, NT = C::NT;
  constexpr int NM = (1 << BITS) - 1;
  fetch_arguments<sizeof(StreamArgs)>();
  // [step][W][matrix][query block][lane]: four words of a lane's 32 digits, then two
  extern __shared__ __attribute__((aligned(16))) u32x4 dig_s[];
  __shared__ float scal_s[4 * QB][4];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, kq = lane >> 4;
  // the query blocks of one share of the keys follow each other on an XCD and share its L2
  int share = blockIdx.x, q0 = 0;
  if (a.qblocks > 1) {
    const int logical = (int)(blockIdx.x % XCDS) * (int)(gridDim.x / XCDS) + (int)(blockIdx.x / XCDS);
    share = logical / a.qblocks;
    q0 = (logical - share * a.qblocks) * (4 * QB);
    if (share >= a.shares) return;
  }
  const int group = blockIdx.y;
  const int G = a.groups_d, steps = G / (4 * W);
  const int64_t gbase = (int64_t)group * a.n;

  // the codes of this wavefront: blocks of 16 T keys, one in every (wavefronts of the grid); lane chunk kq of a step has groups
  // 4 W step + W kq .. + W - 1
  const int64_t nblk = (a.n + 16 * T - 1) / (16 * T);
  const int waves = blockDim.x >> 6;
  const int64_t stride = (int64_t)a.shares * waves;
  int64_t blk = (int64_t)share * waves + wave;
  // the digits of query qa of this workgroup, matrix v of the NV
  auto image = [&](int qa, int v) -> const uint32_t* {
    const int64_t q = (int64_t)group * a.q_per_group + (q0 + qa < a.q_per_group ? q0 + qa : a.q_per_group - 1);
    return a.img + (q * 2 + (BITS > 0 ? v : 1)) * G * 32;
  };
  struct Words {
    uint32_t p[T][BITS > 0 ? W * BITS : 1], z[T][PROD ? W : 1];
    float nu[T], ga[T];  // of a block's last step
  };
  // (codes without norms: something else with a word per row, so that the load needs no branch; chosen at its use)
  const float* const norms = a.norm != nullptr ? a.norm : PROD ? a.gamma : reinterpret_cast<const float*>(a.idx);
  auto load = [&](Words& w, int64_t b, int step) {
    const int g = (step * 4 + kq) * W;
    int64_t rows[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int64_t key = (b * T + t) * 16 + col;
      rows[t] = gbase + (key < a.n ? key : a.n - 1);  // keys past the end: not stored
    }
    // with the last words, and before them: waiting for these waits for nothing else
    if (step + 1 == steps)
#pragma unroll
      for (int t = 0; t < T; ++t) {
        w.nu[t] = norms[rows[t]];
        w.ga[t] = PROD ? a.gamma[rows[t]] : 0.f;
      }
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int64_t row = rows[t];
      if constexpr (BITS > 0) load_words(a.idx + (row * G + g) * BITS, w.p[t]);
      if constexpr (PROD) load_words(a.qjl + row * G + g, w.z[t]);
    }
  };
  Words wa, wb;
  load(wa, blk < nblk ? blk : nblk - 1, 0);

  const int operands = G * NV * QB * 16;  // lanes of all digit operands
  u32x2* const dig_hi = reinterpret_cast<u32x2*>(dig_s + operands);
  for (int e = tid; e < operands; e += blockDim.x) {
    const int l = e & 63, qb = (e >> 6) % QB, v = (e >> 6) / QB % NV, sw = (e >> 6) / (QB * NV);  // sw: step * W + w
    const int w = sw % W, step = sw / W;
    const uint32_t* const d = image(4 * qb + ((l & 15) >> 2), v) + ((step * 4 + (l >> 4)) * W + w) * 32;  // row of the operand = 4 * query + digit
    dig_s[e] = *reinterpret_cast<const u32x4*>(d + (l & 3) * 4);
    dig_hi[e] = *reinterpret_cast<const u32x2*>(d + 16 + (l & 3) * 2);
  }
  // the sums start at minus what the masks' constant parts come to (row 4 kq + r of the result: query kq, digit r)
  f32x4 start[NV][QB];
#pragma unroll
  for (int v = 0; v < NV; ++v)
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) start[v][qb] = *reinterpret_cast<const f32x4*>(image(4 * qb + kq, v) + 24);
  if (tid < 4 * QB) {
    const int64_t q = (int64_t)group * a.q_per_group + (q0 + tid < a.q_per_group ? q0 + tid : a.q_per_group - 1);
    scal_s[tid][0] = BITS > 0 ? a.scal[q * 8] : 0.f;
    scal_s[tid][1] = BITS > 0 ? a.coef[0] * a.scal[q * 8 + 1] : 0.f;
    scal_s[tid][2] = PROD ? 2.f * a.scal[q * 8 + 4] : 0.f;
    scal_s[tid][3] = PROD ? a.scal[q * 8 + 5] : 0.f;
  }
  __syncthreads();
  if (blk >= nblk) return;  // no barrier below

  MaskConst mc = {0x22222222u, 0x44444444u, 0x66666666u};
  asm volatile("" : "+v"(mc.c2), "+v"(mc.c4), "+v"(mc.c6));
  auto digits_sum = [&](const f32x4& c) -> float {
    return mask_digits_sum((int)(0.5f * c[0]), (int)(0.5f * c[1]), (int)(0.5f * c[2]), (int)(0.5f * c[3]));
  };
  f32x4 acc[T][NT][QB];
  auto clear = [&] {
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) acc[t][j][qb] = start[PROD && j == NT - 1 ? NV - 1 : 0][qb];
  };
  clear();
  int step = 0, filled = 0;
  // Finished scores wait in LDS for those of more blocks: a wavefront that stores after every block waits for its stores where
  // it waits for the next words (they are counted together), 20 us of 154 (10^6 codes of 3072, 1 + 1 bits, 4 queries).  A lane stores T keys.
  float* const out_s = reinterpret_cast<float*>(dig_hi + operands) + wave * a.slots * (QB * 64 * T);
  auto store_scores = [&](int64_t b0, int blocks) {
    typedef float vT __attribute__((ext_vector_type(T == 1 ? 2 : T), aligned(4)));
    for (int f = 0; f < blocks; ++f)
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        const int qi = q0 + 4 * qb + kq;
        if (qi >= a.q_per_group) continue;
        const float* const v = out_s + ((f * QB + qb) * 4 + kq) * (16 * T) + T * col;
        const int64_t key = (b0 + f * stride) * (16 * T) + T * col;
        float* const out = a.scores + ((int64_t)group * a.q_per_group + qi) * a.lds + key;
        if (T > 1 && key + T <= a.n) {
          *reinterpret_cast<vT*>(out) = *reinterpret_cast<const vT*>(v);
        } else {
#pragma unroll
          for (int t = 0; t < T; ++t)
            if (key + t < a.n) out[t] = v[t];
        }
      }
  };
  // one step on `cur`, the next one's words requested into `nxt`
  auto advance = [&](const Words& cur, Words& nxt) {
    const bool last = step + 1 == steps;  // uniform
    const int64_t nblk_ = last ? blk + stride : blk;
    const int nstep = last ? 0 : step + 1;
    load(nxt, nblk_ < nblk ? nblk_ : blk, nstep);
    __builtin_amdgcn_sched_barrier(0);  // all of these are asked for here (left to itself the compiler requests a word shortly before it is due)
    const int at = step * (W * NV * QB * 64) + lane;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      v8i A[NV][QB];
#pragma unroll
      for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) A[v][qb] = digit_operand(dig_s[at + ((w * NV + v) * QB + qb) * 64], dig_hi[at + ((w * NV + v) * QB + qb) * 64]);
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
          const v8i b = mask_operand(x, mc);
#pragma unroll
          for (int qb = 0; qb < QB; ++qb) acc[t][j][qb] = mask_mfma(A[0][qb], b, acc[t][j][qb]);
          ++j;
        }
        if constexpr (PROD) {
          const v8i b = mask_operand(cur.z[t][w], mc);
#pragma unroll
          for (int qb = 0; qb < QB; ++qb) acc[t][NT - 1][qb] = mask_mfma(A[NV - 1][qb], b, acc[t][NT - 1][qb]);
        }
      }
    }
    if (last) {
      // (the sums are complete here: left to itself the compiler moves the matrix instructions of a last step behind the branch around
      // a store, where the moves that put their operands together reach only some of the lanes)
#pragma unroll
      for (int t = 0; t < T; ++t)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
          for (int qb = 0; qb < QB; ++qb) asm volatile("" : "+v"(acc[t][j][qb]));
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        const float s0 = scal_s[4 * qb + kq][0], s1 = scal_s[4 * qb + kq][1], s2 = scal_s[4 * qb + kq][2], s3 = scal_s[4 * qb + kq][3];
#pragma unroll
        for (int t = 0; t < T; ++t) {
          float r = 0.f;
          int j = 0;
#pragma unroll
          for (int m = 1; m <= NM; ++m)
            if (i8_term(m)) r = fmaf(a.coef[m], digits_sum(acc[t][j++][qb]), r);
          float v = BITS > 0 ? fmaf(s0, r, s1) : 0.f;
          if (PROD) v = fmaf(a.kappa * cur.ga[t], fmaf(s2, digits_sum(acc[t][NT - 1][qb]), -s3), v);
          if (a.norm != nullptr) v *= cur.nu[t];
          if constexpr (SHORT) {
            const int qi = q0 + 4 * qb + kq;
            const int64_t key = blk * 16 + col;
            if (qi < a.q_per_group && key < a.n) a.scores[((int64_t)group * a.q_per_group + qi) * a.lds + key] = v;
          } else {
            out_s[((filled * QB + qb) * 4 + kq) * (16 * T) + 16 * t + col] = v;
          }
        }
      }
      if (!SHORT && (++filled == a.slots || nblk_ >= nblk)) {
        store_scores(blk - (filled - 1) * stride, filled);
        filled = 0;
      }
      clear();
    }
    blk = nblk_;
    step = nstep;
  };
  // (by count, two at a time: with a way out between the two the compiler takes the first one's words for still under way at the loop's
  // head, where it waits for everything before it asks for more)
  int64_t left = (nblk - blk + stride - 1) / stride * steps;
  for (; left >= 2; left -= 2) {
    advance(wa, wb);
    advance(wb, wa);
  }
  if (left > 0) advance(wa, wb);
}

template <int BITS, bool PROD, int W, int QB, bool SHORT>
hipError_t launch_t(StreamArgs a, int64_t gx, int qz, int threads, int per_cu, int n_groups, hipStream_t s) {
  static LdsLimit lds_limit;  // per instantiation: the limit is raised once per device
  if (const hipError_t e = raise_lds_limit(lds_limit, reinterpret_cast<const void*>(&score_stream_kernel<BITS, PROD, W, QB, SHORT>), kMaxLdsBytes);
      e != hipSuccess)
    return e;
  using C = StreamCfg<BITS, PROD, QB>;
  const int digits = a.groups_d * C::NV * QB * 384, slot = threads * QB * (SHORT ? 1 : C::tiles(W)) * 4;
  a.slots = SHORT ? 0 : std::max(1, std::min(8, (kMaxLdsBytes / per_cu - digits) / slot));
  const int lds = digits + a.slots * slot;
  if (lds > kMaxLdsBytes) return hipErrorInvalidValue;  // (d <= 4096 and launch_bits' choice keep it below)
  a.qblocks = qz;
  a.shares = (int)gx;
  const int64_t wgs = qz > 1 ? (gx * qz + XCDS - 1) / XCDS * XCDS : gx;
  hipLaunchKernelGGL((score_stream_kernel<BITS, PROD, W, QB, SHORT>), dim3((unsigned)wgs, n_groups), dim3(threads), lds, s, a);
  return hipGetLastError();
}

// Which grid a call takes, with QB blocks of four queries a pass and wavefronts of T tiles
struct StreamPlan {
  bool one_tile;
  int64_t gx;  // workgroups to a block of queries
  int per_cu;
  int64_t walk;  // tiles that a wavefront takes one after the other
};
StreamPlan stream_plan(const StreamArgs& a, int n_groups, int QB, int T, int NT, int NV) {
  StreamPlan p;
  const int qz = (a.q_per_group + 4 * QB - 1) / (4 * QB);
  const int64_t others = (int64_t)n_groups * qz, cus = device_cu_count();
  // one workgroup per compute unit (two where registers and LDS admit them), each walking its share of the keys; a list too
  // short for that in wavefronts of one tile and workgroups of four (10^4 codes of 3072 coordinates, 2 queries, 3 + 1 bits: 20.9 us -> 16.6), if
  // all of these are at work in one round.  Where a wavefront would have four tiles, a quarter more than that; two rounds with the digits of both
  // matrices and four queries a pass.  us, several tiles / one:
  //   two tiles, 1.04 rounds       5 queries of 3200, 4 + 1 bits, 17000 codes 51.1 / 58.7;  1.1: 3 of 3072, 2 + 1 bits, 36000 35.0 / 39.7
  //   four, 1.53 rounds            5 of 3200, 1 + 1 bits, 25000 codes 64.6 / 53.2;  3 rounds: 16 of 3072, 20000 54 / 64
  //   four, eight queries a pass   8 groups of 16 of 512, 1 + 1 bits, 5790 codes, 1.42 rounds 20.8 / 23.7;  13 of 3456, 1 bit, 11762 42.0 / 45.6
  // No more workgroups than there is room for: the last few made a second round (24 queries of 768, 2 bits, 300000 codes: 258 of them 59.9, 255 41.4).
  const int64_t nwg = (a.n + 128 * T - 1) / (128 * T);
  const int64_t short_wgs = (a.n + 63) / 64 * others, digits = a.groups_d * NV * QB * 384, held = cus * std::min<int64_t>(4, kMaxLdsBytes / digits);
  const int quarters = T < 4 ? 4 : QB == 1 && NV == 2 ? 8 : 5;
  p.one_tile = nwg * others * 4 <= cus * 3 && short_wgs * 4 <= held * quarters;
  if (p.one_tile) {
    p.gx = (a.n + 63) / 64;
    p.per_cu = 1;
    p.walk = (short_wgs + held - 1) / held;
  } else {
    p.per_cu = NT * QB * T <= 4 && digits <= 72 * 1024 ? 2 : 1;
    p.gx = std::min(nwg, std::max<int64_t>(1, p.per_cu * cus / others));
    p.walk = (nwg + p.gx - 1) / p.gx * T;
  }
  return p;
}

template <int BITS, bool PROD, int W, int QB>
hipError_t launch_w(const StreamArgs& a, int n_groups, hipStream_t s) {
  using C = StreamCfg<BITS, PROD, QB>;
  const StreamPlan p = stream_plan(a, n_groups, QB, C::tiles(W), C::NT, C::NV);
  const int qz = (a.q_per_group + 4 * QB - 1) / (4 * QB);
  return p.one_tile ? launch_t<BITS, PROD, W, QB, true>(a, p.gx, qz, 256, p.per_cu, n_groups, s)
                    : launch_t<BITS, PROD, W, QB, false>(a, p.gx, qz, 512, p.per_cu, n_groups, s);
}

// word groups per step for rows of 128 m coordinates
template <int BITS, bool PROD, int QB>
constexpr int stream_words(int m) {
  using C = StreamCfg<BITS, PROD, QB>;
  for (int w : {12, 8, 6, 4, 3, 2})
    if (C::takes(w) && (w == 6 || w == 12 ? m == w : m % w == 0)) return w;
  return 1;
}

template <int BITS, bool PROD, int QB>
hipError_t launch_qb(const StreamArgs& a, int n_groups, hipStream_t s) {
  using C = StreamCfg<BITS, PROD, QB>;
  const int words = stream_words<BITS, PROD, QB>(a.groups_d / 4);
#define TQ_STREAM_W(W)       \
  if constexpr (C::takes(W)) \
    if (words == W) return launch_w<BITS, PROD, W, QB>(a, n_groups, s);
  TQ_STREAM_W(12) TQ_STREAM_W(8) TQ_STREAM_W(6) TQ_STREAM_W(4) TQ_STREAM_W(3) TQ_STREAM_W(2)
#undef TQ_STREAM_W
  return launch_w<BITS, PROD, 1, QB>(a, n_groups, s);
}

// Four queries per pass over the codes, or eight where there are more than four and their digits fit LDS beside a block's scores.  Digits that fill it
// (two-stage codes of 3072 and 3200 coordinates) take twice as long to fetch as those of four, so there eight have to save a wavefront tiles: any where a
// tile takes long (3 + 1 bits; steps of one word group, each a trip to memory), four of them up to 2 + 1 bits, and at 4 + 1, where a wavefront has room
// for the sums of one tile instead of two, more than three of eight, or a quarter.  us, four / eight a pass:
//   3072, 1 + 1 bits   9 queries: 40000 codes 48.6 / 56.2, 400000 155 / 144;  8: 60000 41.6 / 50.5, 400000 118 / 112
//         2 + 1        16: 30000 53.7 / 61.3, 60000 69.9 / 60.0;  4 groups of 16: 8000 110 / 121, 30000 158 / 136
//         3 + 1        5: 20000 44.1 / 56.2, 40000 53.0 / 46.3, 400000 219 / 176
//         4 + 1        9: 20000 55.4 / 64.0, 30000 71.4 / 64.4, 400000 379 / 394;  16: 400000 499 / 419
//   3200, 2 + 1        5: 17000 52.6 / 63.4, 36000 65.2 / 54.3, 390000 331 / 214;  9: 36000 66.5 / 70.4
//         3 + 1        9: 40000 72.5 / 78.2;  8: 400000 398 / 273;  8 groups of 8: 20000 244 / 207
//         4 + 1        9: 36000 77.7 / 83.0, 200000 294 / 253;  5: 390000 369 / 267
template <int BITS, bool PROD>
hipError_t launch_bits(const StreamArgs& a, int n_groups, hipStream_t s) {
  using C = StreamCfg<BITS, PROD, 2>;
  const int m = a.groups_d / 4, words = stream_words<BITS, PROD, 2>(m), tiles = C::tiles(words), digits = a.groups_d * C::NV * 2 * 384;
  bool eight = a.q_per_group > 4 && digits + 512 * 2 * tiles * 4 <= kMaxLdsBytes;
  if (eight && digits > 140 * 1024) {
    using C4 = StreamCfg<BITS, PROD, 1>;
    const int64_t walk4 = stream_plan(a, n_groups, 1, C4::tiles(stream_words<BITS, PROD, 1>(m)), C4::NT, C4::NV).walk;
    const int64_t walk8 = stream_plan(a, n_groups, 2, tiles, C::NT, C::NV).walk;
    if (BITS == 4) eight = words > 1 ? 8 * walk8 < 5 * walk4 : 4 * walk8 < 3 * walk4;
    else eight = BITS == 3 || words == 1 ? walk8 < walk4 : walk8 + 4 <= walk4;
  }
  return eight ? launch_qb<BITS, PROD, 2>(a, n_groups, s) : launch_qb<BITS, PROD, 1>(a, n_groups, s);
}

}  // namespace

hipError_t launch_score_stream(int bits, bool prod, const uint4* img, const float* scal, const uint32_t* idx, const uint32_t* qjl,
                               const float* gamma, const float* norm, float* scores, int64_t lds, int64_t n, int d, int n_groups,
                               int q_per_group, float kappa, const float* coef, hipStream_t stream) {
  StreamArgs a;
  a.img = reinterpret_cast<const uint32_t*>(img); a.scal = scal; a.idx = idx; a.qjl = qjl; a.gamma = gamma; a.norm = norm; a.scores = scores; a.lds = lds; a.n = n;
  a.groups_d = d / 32; a.q_per_group = q_per_group; a.kappa = kappa;
  std::memcpy(a.coef, coef, sizeof(a.coef));
  if (d % 128 != 0) return hipErrorInvalidValue;
  switch (bits * 2 + (prod ? 1 : 0)) {
    case 1: return launch_bits<0, true>(a, n_groups, stream);
    case 2: return launch_bits<1, false>(a, n_groups, stream);
    case 3: return launch_bits<1, true>(a, n_groups, stream);
    case 4: return launch_bits<2, false>(a, n_groups, stream);
    case 5: return launch_bits<2, true>(a, n_groups, stream);
    case 6: return launch_bits<3, false>(a, n_groups, stream);
    case 7: return launch_bits<3, true>(a, n_groups, stream);
    case 8: return launch_bits<4, false>(a, n_groups, stream);
    case 9: return launch_bits<4, true>(a, n_groups, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace tq
