// Quantisation of a few bf16 vectors at d = 128 (the tokens that a decoding step appends, a short prompt) on the fp16 matrix
// cores: the arithmetic of tq_q128_bf3.hip, two pieces of Pi against one of the vector and two by two (three products) for the
// sketch, without its prologue of 128 KB into LDS.
//
// What such a call waits for is one workgroup's chain, so the chain is short: a wavefront owns 16 coordinates of a block of 16
// vectors over the whole contraction index and keeps its slices of both matrices in registers (16 loads of 1 KB, asked for
// before anything else); the vectors are brought into the range of fp16 once per workgroup, two per wavefront, while those loads
// travel, and cross through LDS; so does the residual.  Two barriers (three for two instances, whose norms come from the
// rotated coordinates).  The fp32 instructions (tq_d128_small.hip) spend 2048 cycles of a SIMD per contraction of 16 vectors,
// these 256 and 384.  bf16 vectors, 2 + 1 bits, us a call:
// 8 vectors 6.7 -> 3.8, 4096 7.5 -> 4.5, 8192 10.4 -> 6.0, 16384 11.6 -> 8.2 (there against the large-batch kernel); 64 channels at 2 + 1
// and 64 at 1 + 1 bits, 4936 10.6 -> 6.2,
// 5.6 without the zero blocks of S Pi^T; 4 bits, 512 5.0 -> 3.6.  What is left is mostly the launch and two round trips.
// Against 64-bit arithmetic, no further off than the fp32 instructions, whose sums meet more roundings (pieces / fp32): of 7.9e8
// coordinates at 4 bits 224 / 320 on the other side of a boundary; signs at 2 + 1 bits 0.13 / 0.16 of 10^6, gamma 0.65 - 0.69e-7 / 0.73 - 0.82e-7.
//
// Where blocks leave compute units idle, a block is given to up to eight workgroups: each multiplies what the residual needs
// and finishes 16 (32, 64) coordinates of it, so that the matrix of the sketch is fetched by several units, a part each (and for
// Alg. 1, where wavefronts need nothing of each other's, Pi too).
//
// Operands of v_mfma_f32_16x16x32_f16: row / column = lane % 16, contraction index 32 step + 8 (lane / 16) + element on both
// sides; accumulator register r is coordinate 16 wave + 4 (lane / 16) + r of vector lane % 16.
#include <type_traits>

#include "tq_d128_tile.h"
#include "tq_q128.h"
#include "tq_score_i8_prep.h"

namespace tq {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

struct QuantFewArgs {
  const uint16_t* X;
  int64_t ldx;
  int64_t n;
  const float* Pi;
  const float* SPiT;
  const unsigned short* image;  // nullable, see q128_image_kernel
  uint32_t* idx;
  uint32_t* qjl;
  float* gamma;
  float* norm;
  int64_t out_first, out_step;  // vector i is written as code row out_first + i * out_step
  int normalise;
  int gs_hi;  // two instances (MIXED): coordinate groups [0, gs_hi) belong to instance hi
  Codebook cb, cb_hi;  // 64-fold
};

// A sum of matrix results, formed here and not behind a branch: this compiler leaves out the wait states between a matrix
// instruction and a use of its result on the far side of one.
__device__ __forceinline__ floatx4 settled(floatx4 v) {
  asm volatile("" : "+v"(v));
  return v;
}

constexpr int ROW_LD = 136;  // fp16 values per row in LDS: consecutive rows start 16 bytes further on in the banks

// STEPS: k-steps of 32 coordinates that the sketch of a coordinate group meets.  4, or fewer for two instances (MIXED), whose S Pi^T is
// block diagonal: as many as the larger instance has, the other instance's blocks are not fetched.
template <int BITS, bool PROD, int STEPS>
__global__ __launch_bounds__(512, 4) void q128_few_kernel(const QuantFewArgs a) {
  constexpr bool MIXED = STEPS < 4;
  if (!MIXED) fetch_arguments<sizeof(QuantFewArgs)>();
  __shared__ __attribute__((aligned(16))) unsigned short x_s[2][16 * ROW_LD];              // by parity of the block
  __shared__ __attribute__((aligned(16))) unsigned short e_s[PROD ? 2 : 1][PROD ? 16 * ROW_LD : 8];  // pieces of the residual, columns permuted
  __shared__ float nu_s[2][16], unit_s[2][16];  // norm; scaled value -> value (of the unit vector, unless MIXED)
  __shared__ float ss_s[MIXED ? 2 : 1][8][16];  // squared norms of the rotated coordinates by wavefront
  __shared__ float g2_s[2][8][16];              // squared residual norms by wavefront
  __shared__ uint32_t max_s;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, kq = lane >> 4;
  const int mt = wave >> 1;  // coordinate group of 32; this wavefront has its half wave & 1
  const int gs = MIXED ? a.gs_hi : 0;
  const bool hi = MIXED && mt < gs;  // uniform
  const int wpr = MIXED ? gs * (BITS + 1) + (4 - gs) * BITS : 4 * BITS;
  const int woff = MIXED ? (mt < gs ? mt * (BITS + 1) : gs * (BITS + 1) + (mt - gs) * BITS) : mt * BITS;
  const bool own = (wave * (int)gridDim.y >> 3) == (int)blockIdx.y;  // this workgroup finishes the wavefront's coordinates
  const bool rotates = PROD || MIXED || own;
  const int64_t blocks = (a.n + 15) / 16;

  // the two vectors that this wavefront prepares, 4 values per lane
  const int pv = 2 * wave + (lane >> 5), p4 = 4 * (lane & 31);
  auto load_x = [&](int64_t blk) {
    const int64_t i = blk * 16 + pv;
    return *reinterpret_cast<const uint2*>(a.X + (i < a.n ? i : a.n - 1) * a.ldx + p4);
  };
  uint2 raw = load_x(blockIdx.x);

  u32x4 pw[2][4], sw[2][4];  // [piece][step]; of sw the STEPS from s0 on
  const int s0 = hi ? 0 : 4 - STEPS;
  float pi_inv;
  if (a.image != nullptr) {
    pi_inv = *reinterpret_cast<const float*>(a.image + PI_ELEMS + W_ELEMS);
    const unsigned short* const row = a.image + (16 * wave + col) * 128;
#pragma unroll
    for (int m = 0; m < (PROD ? 2 : 1); ++m)
      if (m == 0 ? rotates : own)
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
          for (int s = 0; s < (m == 0 ? 4 : STEPS); ++s)
            (m == 0 ? pw : sw)[p][s] = *reinterpret_cast<const u32x4*>(row + (2 * m + p) * MAT_ELEMS + (((4 * (m == 0 ? s : s0 + s) + kq) ^ col) << 3));
  } else {
    if (tid == 0) max_s = 0u;
    __syncthreads();
    float pi_scale;
    h2_scale(largest_of<512>(a.Pi, &max_s, tid), pi_scale, pi_inv);
#pragma unroll
    for (int m = 0; m < (PROD ? 2 : 1); ++m) {
      const float* const row = (m == 0 ? a.Pi : a.SPiT) + (16 * wave + col) * 128;
      f32x4 v[4][2];
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          const int at = 32 * (m == 0 || s >= STEPS ? s : s0 + s) + 8 * kq + 4 * g;
          v[s][g] = *reinterpret_cast<const f32x4*>(row + (m == 0 ? at : q128_w_col(at)));
        }
      float sc = pi_scale;
      if (m == 1) {
        uint32_t top = 0u;
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int e = 0; e < 8; ++e) top = max(top, __float_as_uint(v[s][e >> 2][e & 3]) & 0x7fffffffu);
        top = max(top, (uint32_t)__shfl_xor((int)top, 16));
        top = max(top, (uint32_t)__shfl_xor((int)top, 32));
        float inv;
        h2_scale(top, sc, inv);
      }
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          uint32_t w1, w2;
          h2_split(sc * v[s][e >> 1][2 * (e & 1)], sc * v[s][e >> 1][2 * (e & 1) + 1], w1, w2);
          (m == 0 ? pw : sw)[0][s][e] = w1;
          (m == 0 ? pw : sw)[1][s][e] = w2;
        }
    }
  }

  // sum over the four lanes that share a vector
  auto over_vector = [](float v) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return add_across_halves(__uint_as_float(r[0]) + __uint_as_float(r[1]));
  };
  auto merge16 = [](uint32_t w) {
    const auto r = __builtin_amdgcn_permlane16_swap(w, w, false, false);
    return or_across_halves(r[0] | r[1]);
  };
  auto f16 = [](const u32x4& v) { return __builtin_bit_cast(f16x8, v); };

  int par = 0;
  for (int64_t blk = blockIdx.x; blk < blocks; blk += gridDim.x, par ^= 1) {
    // ---- the vectors as one fp16 piece each, under a power of two that brings the largest value to the top of the range ----
    {
      float ss = square_pair(raw.x, square_pair(raw.y, 0.f));
      uint32_t top = max(max(raw.x & 0x7fffu, (raw.x >> 16) & 0x7fffu), max(raw.y & 0x7fffu, (raw.y >> 16) & 0x7fffu));
      auto fold = [&](auto move) {
        ss += __int_as_float(move(__float_as_int(ss)));
        top = max(top, (uint32_t)move((int)top));
      };
      fold([](int v) { return dpp_move<0xB1>(v); });
      fold([](int v) { return dpp_move<0x4E>(v); });
      fold([](int v) { return dpp_move<0x141>(v); });
      fold([](int v) { return dpp_move<0x140>(v); });
      {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(ss), __float_as_uint(ss), false, false);
        ss = __uint_as_float(r[0]) + __uint_as_float(r[1]);
        const auto t = __builtin_amdgcn_permlane16_swap(top, top, false, false);
        top = max(t[0], t[1]);
      }
      float sc, sc_inv;
      h2_scale(top << 16, sc, sc_inv);
      // exact, or below 2^-39 of the row's largest value
      const uint32_t w0 = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(sc * __uint_as_float(raw.x << 16), sc * __uint_as_float(raw.x & 0xffff0000u)));
      const uint32_t w1 = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(sc * __uint_as_float(raw.y << 16), sc * __uint_as_float(raw.y & 0xffff0000u)));
      *reinterpret_cast<uint2*>(&x_s[par][pv * ROW_LD + p4]) = make_uint2(w0, w1);
      if ((lane & 31) == 0) {
        const float nu = sqrtf(ss);
        nu_s[par][pv] = nu;
        unit_s[par][pv] = !MIXED && a.normalise ? (nu > 0.f ? 1.f / nu : 0.f) * sc_inv : sc_inv;  // a zero row stays zero
      }
    }
    if (blk + gridDim.x < blocks) raw = load_x(blk + gridDim.x);
    __syncthreads();
    if (!rotates) continue;

    const int64_t i = blk * 16 + col;
    const bool valid = i < a.n;
    const int64_t oi = a.out_first + i * a.out_step;  // code row
    float nu = nu_s[par][col], nu_other = 1.f;
    const float unit = unit_s[par][col];
    floatx4 y = {0.f, 0.f, 0.f, 0.f}, yl = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const f16x8 xb = *reinterpret_cast<const f16x8*>(&x_s[par][col * ROW_LD + 32 * s + 8 * kq]);
      yl = __builtin_amdgcn_mfma_f32_16x16x32_f16(f16(pw[1][s]), xb, yl, 0, 0, 0);
      y = __builtin_amdgcn_mfma_f32_16x16x32_f16(f16(pw[0][s]), xb, y, 0, 0, 0);
    }
    y = settled(y + yl);
    float inv;  // accumulator -> 64 times the coordinate of the unit vector
    if (MIXED) {
      const float ss = over_vector(fmaf(y[0], y[0], y[1] * y[1]) + fmaf(y[2], y[2], y[3] * y[3]));
      if (kq == 0) ss_s[MIXED ? par : 0][wave][col] = ss;
      __syncthreads();
      float s_hi = 0.f, s_lo = 0.f;
#pragma unroll
      for (int w = 0; w < 8; ++w) {
        const float v = ss_s[MIXED ? par : 0][w][col];
        s_hi += (w >> 1) < gs ? v : 0.f;
        s_lo += (w >> 1) < gs ? 0.f : v;
      }
      const float r = sqrtf(hi ? s_hi : s_lo);
      inv = r > 0.f ? Q128_RES / r : 0.f;
      nu = r * unit * pi_inv;
      nu_other = sqrtf(hi ? s_lo : s_hi) * unit * pi_inv;
    } else {
      inv = unit * (pi_inv * Q128_RES);
    }

    // ---- the decision of Alg. 1 on four coordinates: bucket = number of boundaries not above y ----
    constexpr int NPL = BITS + (MIXED && BITS < 4 ? 1 : 0);
    uint32_t half[NPL > 0 ? NPL : 1];
    float e[4], g2 = 0.f;
    auto decide = [&](auto bits_c, const Codebook& cb) {
      constexpr int B = decltype(bits_c)::value;
      uint32_t lv[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float v = y[r] * inv;
        float yt = cb.c[0];
        lv[r] = 0u;
#pragma unroll
        for (int j = 0; j < (1 << B) - 1; ++j) {
          const float tj = cb.t[j], cj = cb.c[j + 1];  // read before the select, see quantise_tile
          const bool ge = v >= tj;
          yt = ge ? cj : yt;
          lv[r] += ge ? 1u : 0u;
        }
        e[r] = v - yt;
        g2 = fmaf(e[r], e[r], g2);
      }
#pragma unroll
      for (int pl = 0; pl < NPL; ++pl) {
        uint32_t nib = 0u;
        if (pl < B)
#pragma unroll
          for (int r = 0; r < 4; ++r) nib |= ((lv[r] >> pl) & 1u) << r;
        half[pl] = merge16(nib << (4 * kq));
      }
    };
    if (hi) decide(std::integral_constant<int, NPL>{}, a.cb_hi);
    else decide(std::integral_constant<int, BITS>{}, a.cb);
    if (valid && own) {
      // lanes of quarter kq store plane kq: 16 bits each
      if (NPL > 0) {
        uint32_t w = half[0];
#pragma unroll
        for (int pl = 1; pl < NPL; ++pl) w = kq == pl ? half[pl] : w;
        if (kq < BITS + (hi ? 1 : 0)) reinterpret_cast<uint16_t*>(a.idx + oi * wpr + woff + kq)[wave & 1] = (uint16_t)w;
      }
      if (wave == 0 && kq == 0 && a.norm != nullptr) {
        if (MIXED) {
          a.norm[2 * oi] = nu;  // wavefront 0 always belongs to instance hi
          a.norm[2 * oi + 1] = nu_other;
        } else {
          a.norm[oi] = nu;
        }
      }
    }
    if (!PROD) continue;

    g2 = over_vector(g2);
    if (kq == 0) g2_s[par][wave][col] = g2;
    {
      if constexpr (!MIXED) {
        const float room = q128_room(inv);  // the same in all wavefronts
#pragma unroll
        for (int r = 0; r < 4; ++r) e[r] *= room;
      }
      uint32_t h0, h1, l0, l1;
      h2_split(e[0], e[1], h0, l0);
      h2_split(e[2], e[3], h1, l1);
      const int at = col * ROW_LD + q128_w_col(16 * wave + 4 * kq);
      *reinterpret_cast<uint2*>(&e_s[0][at]) = make_uint2(h0, h1);
      *reinterpret_cast<uint2*>(&e_s[PROD ? 1 : 0][at]) = make_uint2(l0, l1);
    }
    __syncthreads();
    if (!own) continue;
    floatx4 u = {0.f, 0.f, 0.f, 0.f}, ul = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      const int at = col * ROW_LD + 32 * (s0 + s) + 8 * kq;
      const f16x8 eh = *reinterpret_cast<const f16x8*>(&e_s[0][at]), el = *reinterpret_cast<const f16x8*>(&e_s[PROD ? 1 : 0][at]);
      ul = __builtin_amdgcn_mfma_f32_16x16x32_f16(f16(sw[1][s]), eh, ul, 0, 0, 0);
      ul = __builtin_amdgcn_mfma_f32_16x16x32_f16(f16(sw[0][s]), el, ul, 0, 0, 0);
      u = __builtin_amdgcn_mfma_f32_16x16x32_f16(f16(sw[0][s]), eh, u, 0, 0, 0);
    }
    u = settled(u + ul);
    uint32_t nib = 0u;
#pragma unroll
    for (int r = 0; r < 4; ++r) nib |= (u[r] >= 0.f ? 1u : 0u) << r;
    const uint32_t z = merge16(nib << (4 * kq));
    if (valid && kq == 0) {
      reinterpret_cast<uint16_t*>(a.qjl + oi * 4 + mt)[wave & 1] = (uint16_t)z;
      if (wave == 0) {
        float g[2] = {0.f, 0.f};  // instance lo (or the only one), instance hi
#pragma unroll
        for (int w = 0; w < 8; ++w) g[MIXED && (w >> 1) < gs ? 1 : 0] += g2_s[par][w][col];
        if (MIXED) {
          a.gamma[2 * oi] = sqrtf(g[1]) * (1.f / Q128_RES);
          a.gamma[2 * oi + 1] = sqrtf(g[0]) * (1.f / Q128_RES);
        } else {
          a.gamma[oi] = sqrtf(g[0]) * (1.f / Q128_RES);
        }
      }
    }
  }
}

template <int BITS, bool PROD, int STEPS>
hipError_t launch_few(const QuantFewArgs& a, hipStream_t s) {
  const int64_t blocks = (a.n + 15) / 16, cu = device_cu_count();
  int share = 1;  // workgroups per block
  while (share < 8 && blocks * share * 2 <= cu) share *= 2;
  const dim3 grid((unsigned)(blocks < 2 * cu ? blocks : 2 * cu), share);
  hipLaunchKernelGGL((q128_few_kernel<BITS, PROD, STEPS>), grid, dim3(512), 0, s, a);
  return hipGetLastError();
}

template <int BITS>
hipError_t launch_bits(const QuantFewArgs& a, bool prod, hipStream_t s) {
  if (a.gs_hi > 0) {
    if constexpr (BITS < 4) {
      if (!prod) return launch_few<BITS, false, 3>(a, s);
      return a.gs_hi == 2 ? launch_few<BITS, true, 2>(a, s) : launch_few<BITS, true, 3>(a, s);
    }
    return hipErrorInvalidValue;
  }
  return prod ? launch_few<BITS, true, 4>(a, s) : launch_few<BITS, false, 4>(a, s);
}

}  // namespace

bool quant128_few_applicable(int bits, const Codebook& cb, const Codebook* cb_hi) {
  return q128_table(cb, bits) && (cb_hi == nullptr || q128_table(*cb_hi, bits + 1));
}

// rows of 128 bf16 values, 8-byte aligned with a row stride that keeps them so
hipError_t launch_quant128_few(int bits, bool prod, const void* X, int64_t ldx, int64_t n, const float* Pi, const float* SPiT, uint32_t* idx,
                               uint32_t* qjl, float* gamma, float* norm, const Codebook& cb, int gs_hi, const Codebook& cb_hi,
                               const void* image, hipStream_t s, int64_t out_first, int64_t out_step) {
  if (n <= 0) return hipSuccess;
  if (gs_hi < 0 || gs_hi > 3 || (gs_hi > 0 && (cb_hi.bits != bits + 1 || norm == nullptr)) || ldx % 4 != 0) return hipErrorInvalidValue;
  QuantFewArgs a;
  a.X = static_cast<const uint16_t*>(X); a.ldx = ldx; a.n = n; a.Pi = Pi; a.SPiT = SPiT;
  a.image = static_cast<const unsigned short*>(image);
  a.idx = idx; a.qjl = qjl; a.gamma = gamma; a.norm = norm; a.out_first = out_first; a.out_step = out_step;
  a.normalise = norm != nullptr; a.gs_hi = gs_hi; a.cb = q128_scaled(cb); a.cb_hi = q128_scaled(cb_hi);
  switch (bits) {
    case 0: return launch_bits<0>(a, prod, s);
    case 1: return launch_bits<1>(a, prod, s);
    case 2: return launch_bits<2>(a, prod, s);
    case 3: return launch_bits<3>(a, prod, s);
    case 4: return launch_bits<4>(a, prod, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace tq
