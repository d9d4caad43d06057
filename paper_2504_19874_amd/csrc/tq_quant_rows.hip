// Alg. 1 and Alg. 2 for a handful of long vectors (an index that grows by single embeddings), by matrix-vector products.
//
// A workgroup multiplies 8 or 16 rows of the matrix and finishes them: it has the whole vector anyway, so it takes the
// norm itself, decides its rows' coordinates and stores one or two bytes of every plane word.  Alg. 1 is one launch,
// Alg. 2 two (the sketch needs every coordinate of the residual).  Bound by latency: the launch, one round trip for the
// matrix rows and the vector together, the joining of the lanes.  One vector, d = 1536, 4 bits: the products alone 3.3 us and
// a second kernel of one workgroup
// that normalised, decided and packed 5.6; a call took 8.6 us and takes 4.3, most of it the host's (d = 3072: 18.6 -> 6.8; Alg. 2 at
// 1 + 1 bits 27.3 -> 14.9; four vectors, d = 1536, 12.0 -> 5.8 and 20.4 -> 12.7, then, asked for together on their way to LDS, 5.6 and 11.4; eight at a
// time instead 6.4 / 8.4 for eight vectors).
#include "tq_d128_tile.h"
#include "tq_score_i8_prep.h"

#include <type_traits>

namespace tq {
namespace {

struct RowsArgs {
  const float* W;
  const void* x;
  int64_t ldx;
  uint32_t* words;  // planes of the indices, or the signs
  float* norm;      // |x|: the vector's norm; gamma where x is the residual
  float* e;         // residual out [n][d], nullable
  int d, n, x_bf16, normalise;
};

// A wavefront owns R consecutive rows; its lanes share the contraction index, 4 values each.  Q = 1: the vector goes straight to
// registers, 6 steps of 256 values with everything in flight.  Q = 4 (four vectors at a time): through LDS, so that rows are
// read once for all four and vectors once for all wavefronts.  SIGN: one plane, u >= 0.
template <int BITS, bool SIGN, int Q, int R>
__global__ __launch_bounds__(256) void quant_rows_kernel(const RowsArgs a, const Codebook cb) {
  constexpr int ROWS = 4 * R;  // of a workgroup
  constexpr int U = Q == 1 ? 6 : R == 2 ? 3 : 2;
  constexpr int PL = SIGN ? 1 : BITS;
  extern __shared__ __attribute__((aligned(16))) float xs[];  // Q > 1: [Q][d]
  __shared__ unsigned char code_s[Q][ROWS];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n4 = a.d >> 2;  // float4 per row
  const int q0 = blockIdx.y * Q;
  const int j0 = blockIdx.x * ROWS + wave * R;
  const float4* const w4 = reinterpret_cast<const float4*>(a.W + (int64_t)(j0 < a.d ? j0 : 0) * a.d);
  auto load_x = [&](int64_t row, int k4) {
    if (a.x_bf16) {
      const uint2 w = reinterpret_cast<const uint2*>(reinterpret_cast<const uint16_t*>(a.x) + row * a.ldx)[k4];
      return make_float4(__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16),
                         __uint_as_float(w.y & 0xffff0000u));
    }
    return reinterpret_cast<const float4*>(reinterpret_cast<const float*>(a.x) + row * a.ldx)[k4];
  };
  const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
  float4 w[U][R], v[U];
  auto load_w = [&](int k0) {
#pragma unroll
    for (int s = 0; s < U; ++s) {
      const int k4 = k0 + 64 * s + lane;
#pragma unroll
      for (int i = 0; i < R; ++i) w[s][i] = zero;
      if (Q == 1) v[s] = zero;
      if (k4 < n4) {
#pragma unroll
        for (int i = 0; i < R; ++i) w[s][i] = w4[i * n4 + k4];
        if (Q == 1) v[s] = load_x(q0, k4);
      }
    }
  };
  load_w(0);
  if (Q > 1) {
    for (int k4 = tid; k4 < n4; k4 += 256) {  // all vectors' loads under way together
      float4 y[Q];
#pragma unroll
      for (int r = 0; r < Q; ++r) y[r] = load_x(q0 + r < a.n ? q0 + r : a.n - 1, k4);  // past the end: not stored
#pragma unroll
      for (int r = 0; r < Q; ++r) reinterpret_cast<float4*>(xs + r * a.d)[k4] = y[r];
    }
    __syncthreads();
  }
  float acc[R][Q], ss[Q];
#pragma unroll
  for (int r = 0; r < Q; ++r) {
    ss[r] = 0.f;
#pragma unroll
    for (int i = 0; i < R; ++i) acc[i][r] = 0.f;
  }
  for (int k0 = 0; k0 < n4; k0 += 64 * U) {
    if (k0 > 0) load_w(k0);
#pragma unroll
    for (int s = 0; s < U; ++s) {
      const int k4 = k0 + 64 * s + lane;
#pragma unroll
      for (int r = 0; r < Q; ++r) {
        float4 y = v[s];
        if (Q > 1) {
          y = zero;
          if (k4 < n4) y = reinterpret_cast<const float4*>(xs + r * a.d)[k4];
        }
        ss[r] = fmaf(y.x, y.x, fmaf(y.y, y.y, fmaf(y.z, y.z, fmaf(y.w, y.w, ss[r]))));
#pragma unroll
        for (int i = 0; i < R; ++i)
          acc[i][r] = fmaf(w[s][i].x, y.x, fmaf(w[s][i].y, y.y, fmaf(w[s][i].z, y.z, fmaf(w[s][i].w, y.w, acc[i][r]))));
      }
    }
  }
  // every lane has the sums; lane i Q + r finishes row i of vector r
  float y = 0.f, sq = 0.f;
#pragma unroll
  for (int r = 0; r < Q; ++r) {
    const float t = wave_sum_f(ss[r]);
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const float p = wave_sum_f(acc[i][r]);
      if (lane == i * Q + r) {
        y = p;
        sq = t;
      }
    }
  }
  const int r = lane % Q, i = lane / Q;
  const bool live = lane < R * Q && j0 < a.d && q0 + r < a.n;
  const float nu = sqrtf(sq);
  if (a.norm != nullptr && blockIdx.x == 0 && wave == 0 && lane < Q && q0 + lane < a.n) a.norm[q0 + lane] = nu;
  int code;
  if constexpr (SIGN) {
    code = y >= 0.f ? 1 : 0;
  } else {
    if (a.normalise) y *= nu > 0.f ? 1.f / nu : 0.f;  // a zero row stays zero
    code = 0;
    float c = cb.c[0];
#pragma unroll
    for (int t = 0; t < (1 << BITS) - 1; ++t) {  // on a boundary: the upper cell
      const float tj = cb.t[t], cj = cb.c[t + 1];
      const bool ge = y >= tj;
      c = ge ? cj : c;
      code += ge ? 1 : 0;
    }
    if (a.e != nullptr && live) a.e[(int64_t)(q0 + r) * a.d + j0 + i] = y - c;
  }
  if constexpr (PL > 0) {
    if (lane < R * Q) code_s[r][wave * R + i] = (unsigned char)code;
    __syncthreads();
    if (tid < Q * PL && q0 + tid / PL < a.n) {
      const int qr = tid / PL, pl = tid % PL;
      const int j = blockIdx.x * ROWS;  // d is a multiple of 32: whole bytes, whole workgroups
      uint32_t bits = 0;
#pragma unroll
      for (int b = 0; b < ROWS; ++b) bits |= (((uint32_t)code_s[qr][b] >> pl) & 1u) << b;
      unsigned char* const o = reinterpret_cast<unsigned char*>(a.words + (int64_t)(q0 + qr) * (a.d / 32) * PL + (j >> 5) * PL + pl) + ((j & 31) >> 3);
      if constexpr (ROWS == 8) *o = (unsigned char)bits;
      else *reinterpret_cast<uint16_t*>(o) = (uint16_t)bits;
    }
  }
}

template <int BITS, bool SIGN>
hipError_t launch_rows(const RowsArgs& a, const Codebook& cb, hipStream_t s) {
  auto go = [&](auto q_c, auto r_c) {
    constexpr int Q = decltype(q_c)::value, R = decltype(r_c)::value;
    hipLaunchKernelGGL((quant_rows_kernel<BITS, SIGN, Q, R>), dim3(a.d / (4 * R), (a.n + Q - 1) / Q), dim3(256),
                       Q > 1 ? (size_t)Q * a.d * sizeof(float) : 0, s, a, cb);
    return hipGetLastError();
  };
  using std::integral_constant;
  if (a.n == 1) return go(integral_constant<int, 1>{}, integral_constant<int, 2>{});
  const bool many = (int64_t)(a.d / 16) * ((a.n + 3) / 4) >= device_cu_count();
  return many ? go(integral_constant<int, 4>{}, integral_constant<int, 4>{}) : go(integral_constant<int, 4>{}, integral_constant<int, 2>{});
}

}  // namespace

hipError_t launch_quant_rows(int bits, bool bf16, const void* x, int64_t ldx, int64_t n, int d, const float* Pi, const Codebook& cb,
                             uint32_t* idx, float* norm, hipStream_t stream, const float* SPiT, float* ew, uint32_t* qjl,
                             float* gamma) {
  if (n == 0) return hipSuccess;
  if (n > 65535 || d % 32 != 0 || ldx % 4 != 0 || (size_t)4 * d * sizeof(float) > 65536) return hipErrorInvalidValue;
  RowsArgs a{Pi, x, ldx, idx, norm, ew, d, (int)n, bf16 ? 1 : 0, norm != nullptr ? 1 : 0};
  hipError_t e;
  switch (bits) {
    case 0: e = launch_rows<0, false>(a, cb, stream); break;
    case 1: e = launch_rows<1, false>(a, cb, stream); break;
    case 2: e = launch_rows<2, false>(a, cb, stream); break;
    case 3: e = launch_rows<3, false>(a, cb, stream); break;
    case 4: e = launch_rows<4, false>(a, cb, stream); break;
    default: return hipErrorInvalidValue;
  }
  if (e != hipSuccess || ew == nullptr) return e;
  const RowsArgs b{SPiT, ew, d, qjl, gamma, nullptr, d, (int)n, 0, 0};
  return launch_rows<0, true>(b, cb, stream);
}

}  // namespace tq
