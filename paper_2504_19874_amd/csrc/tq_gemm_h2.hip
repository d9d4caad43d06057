// The quantiser's contractions at every d other than 128, on the fp16 matrix cores (tq_h2.h says how the fp32 factors
// are taken): y = Pi x with decision, packing and residual in the epilogue, then sign((S Pi^T) e).
//
// Passes.  split_rows_kernel reads the vectors once, takes norm and largest magnitude of each and writes their pieces;
// the contraction then moves both operands into LDS by direct loads and its k-loop holds nothing but LDS reads and
// matrix instructions.  Splitting inside the contraction instead costs about 25 vector instructions per k-step and
// thread for every one of the d / 256 row tiles that meet the same vectors, and vector instructions do not overlap with
// matrix instructions on this chip; the extra pass costs 8 d bytes of traffic per vector once (d = 1536: 1.9 of 13.1
// ms for 10^6 vectors).
//
// Tile.  256 rows of the matrix x 256 vectors per workgroup of eight wavefronts (2 x 4 tiles of 32 x 32 each: twelve
// 16-byte LDS reads feed 24 matrix instructions), k in steps of 32 through two buffers of 64 KB (smaller tiles, whose steps are
// shorter than a load's latency: four).  The fragments of the
// next 16 k are read while the present ones are multiplied; the one barrier of a step sits between its two halves, so
// that a step's first fragments are in registers before the step begins.  The vector is on the lane axis of the result: a lane holds 16
// coordinates of one vector per tile and the decision is lane-local.
#include "tq_bf3.h"
#include "tq_d128_tile.h"
#include "tq_h2.h"

#include <type_traits>

namespace tq {
namespace {

constexpr int XCDS = 8;

// d fp32 / bf16 values per row -> pieces.  L lanes per row (a power of two up to 64), U chunks of eight values per lane
// held in registers; rows longer than 64 * 8 * U values are read twice instead (U = 0).
template <bool BF16, bool CUT, int U>
__global__ __launch_bounds__(256) void split_rows_kernel(const void* x, int64_t ldx, int64_t n, int d, int lanes_log2, int normalise,
                                                         const float* w_inv, unsigned char* pieces, float* norm, float* fac, float* esc) {
  const int L = 1 << lanes_log2;
  const int lane = threadIdx.x & (L - 1);
  const int64_t row = (int64_t)blockIdx.x * (256 >> lanes_log2) + (threadIdx.x >> lanes_log2);
  const bool live = row < n;
  const int64_t r = live ? row : n - 1;
  const float* const xf = reinterpret_cast<const float*>(x) + (BF16 ? 0 : r * ldx);
  const uint16_t* const xh = reinterpret_cast<const uint16_t*>(x) + (BF16 ? r * ldx : 0);
  const int chunks = d >> 3;
  float v[U > 0 ? U : 1][8];
  auto load = [&](int c, float (&o)[8]) {
    if (BF16) {
      const uint2 a = *reinterpret_cast<const uint2*>(xh + c * 8), b = *reinterpret_cast<const uint2*>(xh + c * 8 + 4);
      const uint32_t w[4] = {a.x, a.y, b.x, b.y};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        o[2 * i] = __uint_as_float(w[i] << 16);
        o[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
      }
    } else {
      const float4 a = *reinterpret_cast<const float4*>(xf + c * 8), b = *reinterpret_cast<const float4*>(xf + c * 8 + 4);
      o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w; o[4] = b.x; o[5] = b.y; o[6] = b.z; o[7] = b.w;
    }
  };
  // CUT: the value's two leading bf16 pieces, 17 significant bits (see launch_h2_split)
  auto cut = [](float f) {
    const float f1 = __uint_as_float(bf16_bits(f) << 16);
    return f1 + __uint_as_float(bf16_bits(f - f1) << 16);
  };
  float ss = 0.f;
  uint32_t mx = 0;
  auto take = [&](const float (&o)[8]) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      ss = fmaf(o[i], o[i], ss);
      const uint32_t b = __float_as_uint(o[i]) & 0x7fffffffu;
      mx = mx > b ? mx : b;
    }
  };
  if constexpr (U > 0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int c = u * L + lane;
      if (c < chunks) load(c, v[u]);
      else
#pragma unroll
        for (int i = 0; i < 8; ++i) v[u][i] = 0.f;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) take(v[u]);
  } else {
    for (int c = lane; c < chunks; c += L) {
      load(c, v[0]);
      take(v[0]);
    }
  }
  // over the row's lanes, as by a butterfly over lane distances 1, 2 .. L / 2: once pairs and quads are alike, mirrored lanes hold what is to be exchanged
  auto join = [&](uint32_t sum, uint32_t o) {
    ss += __uint_as_float(sum);
    mx = mx > o ? mx : o;
  };
#define TQ_ROW_DPP(CTRL)                                                                              \
  join((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(ss), CTRL, 0xf, 0xf, true), \
       (uint32_t)__builtin_amdgcn_update_dpp(0, (int)mx, CTRL, 0xf, 0xf, true))
  TQ_ROW_DPP(0xB1);  // lane ^ 1
  TQ_ROW_DPP(0x4E);  // lane ^ 2
  if (L >= 8) TQ_ROW_DPP(0x141);   // lane ^ 7
  if (L >= 16) TQ_ROW_DPP(0x140);  // lane ^ 15
#undef TQ_ROW_DPP
  if (L >= 32) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(ss), __float_as_uint(ss), false, false);
    const auto b = __builtin_amdgcn_permlane16_swap(mx, mx, false, false);
    ss = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    mx = b[0] > b[1] ? b[0] : b[1];
  }
  if (L >= 64) {
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(ss), __float_as_uint(ss), false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(mx, mx, false, false);
    ss = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    mx = b[0] > b[1] ? b[0] : b[1];
  }
  float s, inv;
  h2_scale(mx, s, inv);
  if (live && lane == 0) {
    const float nu = sqrtf(ss);
    float f = inv;
    if (normalise) f = nu > 0.f ? (1.f / nu) * inv : 0.f;
    fac[row] = f * w_inv[0];
    if (norm != nullptr) norm[row] = nu;
    if (esc != nullptr) {
      // |residual coordinate| <= |x| + 1 (a centroid of a unit vector's coordinate is below 1)
      float se, dummy;
      h2_scale(__float_as_uint((normalise ? 1.f : nu) + 1.f), se, dummy);
      esc[row] = se;
    }
  }
  if (!live) return;
  constexpr int NP = BF16 ? 1 : 2;
  unsigned char* const dst = pieces + row * (int64_t)d * (2 * NP);
  auto store = [&](int c, const float (&o)[8]) {
    uint32_t hi[4], lo[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float f0 = CUT ? cut(o[2 * i]) : o[2 * i], f1 = CUT ? cut(o[2 * i + 1]) : o[2 * i + 1];
      h2_split(f0 * s, f1 * s, hi[i], lo[i]);
    }
    unsigned char* const q = dst + (c >> 2) * (64 * NP) + (c & 3) * 16;
    *reinterpret_cast<uint4*>(q) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
    if (!BF16) *reinterpret_cast<uint4*>(q + 64) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
  };
  if constexpr (U > 0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int c = u * L + lane;
      if (c < chunks) store(c, v[u]);
    }
  } else {
    for (int c = lane; c < chunks; c += L) {
      load(c, v[0]);
      store(c, v[0]);
    }
  }
}

// The image of a matrix: its largest magnitude (the word after the inverse scale serves as the running maximum), then
// its pieces.  Both are small beside one pass over the vectors.
__global__ void h2_zero_kernel(uint32_t* max_bits) { *max_bits = 0u; }
__global__ __launch_bounds__(256) void h2_max_kernel(const float* W, int64_t ldw, int M, int d, uint32_t* max_bits) {
  uint32_t mx = 0;
  const int per_row = d >> 2;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < (int64_t)M * per_row; e += (int64_t)gridDim.x * 256) {
    const float4 v = *reinterpret_cast<const float4*>(W + (e / per_row) * ldw + (e % per_row) * 4);
    const float f[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t b = __float_as_uint(f[i]) & 0x7fffffffu;
      mx = mx > b ? mx : b;
    }
  }
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) {
    const uint32_t o = (uint32_t)__shfl_xor((int)mx, m);
    mx = mx > o ? mx : o;
  }
  if ((threadIdx.x & 63) == 0) atomicMax(max_bits, mx);
}
__global__ __launch_bounds__(256) void h2_image_kernel(const float* W, int64_t ldw, int M, int d, const uint32_t* max_bits, float* w_inv,
                                                       unsigned char* out) {
  float s, inv;
  h2_scale(*max_bits, s, inv);
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e == 0) *w_inv = inv;
  const int chunks = d >> 3;
  if (e >= (int64_t)M * chunks) return;
  const int64_t row = e / chunks;
  const int c = (int)(e % chunks);
  const float4 a = *reinterpret_cast<const float4*>(W + row * ldw + c * 8), b = *reinterpret_cast<const float4*>(W + row * ldw + c * 8 + 4);
  uint32_t hi[4], lo[4];
  h2_split(a.x * s, a.y * s, hi[0], lo[0]);
  h2_split(a.z * s, a.w * s, hi[1], lo[1]);
  h2_split(b.x * s, b.y * s, hi[2], lo[2]);
  h2_split(b.z * s, b.w * s, hi[3], lo[3]);
  unsigned char* const q = out + row * (int64_t)d * 4 + (c >> 2) * 128 + (c & 3) * 16;
  *reinterpret_cast<uint4*>(q) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
  *reinterpret_cast<uint4*>(q + 64) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
}

template <int PL>
__device__ __forceinline__ void store_words(uint32_t* p, const uint32_t* w) {
  typedef uint32_t v2 __attribute__((ext_vector_type(2), aligned(4)));
  typedef uint32_t v3 __attribute__((ext_vector_type(3), aligned(4)));
  typedef uint32_t v4 __attribute__((ext_vector_type(4), aligned(4)));
  if constexpr (PL == 1) *p = w[0];
  else if constexpr (PL == 2) *reinterpret_cast<v2*>(p) = v2{w[0], w[1]};
  else if constexpr (PL == 3) *reinterpret_cast<v3*>(p) = v3{w[0], w[1], w[2]};
  else if constexpr (PL == 4) *reinterpret_cast<v4*>(p) = v4{w[0], w[1], w[2], w[3]};
}

struct H2Args {
  const unsigned char* W;
  const unsigned char* X;
  const float* fac;
  const float* esc;
  float* out;
  uint32_t* words;
  unsigned char* E;
  float* part;
  float* gamma;
  int64_t n;
  int d, part_tiles, tiles_m, tiles_n, per_xcd;
};

// EK 0: indices, 1: indices and residual, 2: signs, 3: the products themselves, out[vector][row].  A wavefront owns TW x UW tiles of 32 x 32, the workgroup WM x WN
// wavefronts.
template <int EK, int BITS, int NPX, int TW, int UW, int WM, int WN, int NBUF>
__global__ __launch_bounds__(WM* WN * 64, 2) void h2_kernel(const H2Args a, const Codebook cb) {
  constexpr int NW = WM * WN;
  constexpr int TM = WM * TW * 32, TN = WN * UW * 32;
  constexpr int A_BYTES = TM * 128, B_BYTES = TN * NPX * 64;
  constexpr int AL = A_BYTES / 1024 / NW, BL = B_BYTES / 1024 / NW;  // direct loads per wavefront and step
  static_assert(AL * NW * 1024 == A_BYTES && BL * NW * 1024 == B_BYTES, "whole loads");
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
  __shared__ float red[EK == 1 ? WM * TN : 1];

  const int total = a.tiles_m * a.tiles_n;
  const int logical = (int)(blockIdx.x % XCDS) * a.per_xcd + (int)(blockIdx.x / XCDS);
  if (logical >= total) return;
  const int tile_m = logical % a.tiles_m, tile_n = logical / a.tiles_m;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int l32 = lane & 31, h = lane >> 5;
  const int m0 = tile_m * TM;
  const int64_t n0 = (int64_t)tile_n * TN;
  const int n_kt = a.d >> 5;
  const int rows_m = min(TM, a.d - m0);
  const int rows_n = (int)min((int64_t)TN, a.n - n0);
  const uint32_t row_a = (uint32_t)a.d * 4u, row_b = (uint32_t)a.d * (2u * NPX);
  const unsigned char* gA = a.W + (int64_t)m0 * row_a;
  const unsigned char* gB = a.X + n0 * row_b;

  // rows past the end of an operand are clamped onto its last row: what they produce is never stored
  uint32_t va[AL], vb[BL];
  // load q of an operand's tile fills LDS lines 8 q .. 8 q + 7; its lane gives slot lane % 8 of line lane / 8
  const int l8 = lane >> 3, slot = lane & 7;
#pragma unroll
  for (int j = 0; j < AL; ++j) {
    const int r = (wave * AL + j) * 8 + l8;
    va[j] = (uint32_t)min(r, rows_m - 1) * row_a + h2_chunk<2>(r, slot) * 16;
  }
#pragma unroll
  for (int j = 0; j < BL; ++j) {
    const int line = (wave * BL + j) * 8 + l8;
    const int r = NPX == 2 ? line : 2 * line + (slot >> 2);
    vb[j] = (uint32_t)min(r, rows_n - 1) * row_b + h2_chunk<NPX>(r, slot) * 16;
  }
  const uint32_t lds0 = h2_lds_address(lds);
  int requested = 0;
  auto dma_one = [&](int buf, int j) {
    if (j < AL) h2_dma(gA, va[j < AL ? j : 0], lds0 + buf * A_BYTES + (wave * AL + j) * 1024);
    else h2_dma(gB, vb[j < AL ? 0 : j - AL], lds0 + NBUF * A_BYTES + buf * B_BYTES + (wave * BL + j - AL) * 1024);
  };
  auto dma_next = [&] {  // the last k-step is requested again and again rather than branching around the loads
    const bool more = ++requested < n_kt;
    gA += more ? 128 : 0;
    gB += more ? 64 * NPX : 0;
  };
  auto dma = [&](int buf) {
#pragma unroll
    for (int j = 0; j < AL + BL; ++j) dma_one(buf, j);
    dma_next();
  };

  // fragment addresses: [piece][k / 16] of this lane's row, tiles and buffers as immediate offsets
  const unsigned char *pa[2][2], *pb[NPX][2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
#pragma unroll
    for (int p = 0; p < 2; ++p) pa[p][s] = lds + h2_place<2>(wm * TW * 32 + l32, p * 4 + s * 2 + h);
#pragma unroll
    for (int p = 0; p < NPX; ++p) pb[p][s] = lds + NBUF * A_BYTES + h2_place<NPX>(wn * UW * 32 + l32, p * 4 + s * 2 + h);
  }
  struct Frag {
    f16x8 a[TW][2], b[UW][NPX];
  };
  constexpr int NR = 2 * TW + NPX * UW;  // fragment reads of 16 k, in the order in which the products need them
  auto read_one = [&](Frag& f, int buf, int s, int i) {
    auto ra = [&](int p, int t) { f.a[t][p] = *reinterpret_cast<const f16x8*>(pa[p][s] + buf * A_BYTES + t * 4096); };
    auto rb = [&](int p, int u) { f.b[u][p] = *reinterpret_cast<const f16x8*>(pb[p][s] + buf * B_BYTES + u * (2048 * NPX)); };
    if (i < TW) ra(1, i);
    else if (i < TW + UW) rb(0, i - TW);
    else if (i < 2 * TW + UW) ra(0, i - TW - UW);
    else if (NPX == 2) rb(NPX - 1, i - 2 * TW - UW);
  };
  auto read = [&](Frag& f, int buf, int s) {
#pragma unroll
    for (int i = 0; i < NR; ++i) read_one(f, buf, s, i);
  };
  floatx16 acc[TW][UW];
#pragma unroll
  for (int t = 0; t < TW; ++t)
#pragma unroll
    for (int u = 0; u < UW; ++u)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[t][u][r] = 0.f;
  // lo hi, hi lo, hi hi; `between(i)` after every matrix instruction is what else the wavefront has to issue, spread out
  constexpr int NPROD = NPX == 2 ? 3 : 2, NM = NPROD * TW * UW;
  auto multiply = [&](const Frag& f, auto between) {
#pragma unroll
    for (int i = 0; i < NM; ++i) {
      const int pr = i / (TW * UW), t = i / UW % TW, u = i % UW;
      const int p = pr == 0 ? 1 : 0, q = NPX == 2 && pr == 1 ? NPX - 1 : 0;
      acc[t][u] = __builtin_amdgcn_mfma_f32_32x32x16_f16(f.a[t][p], f.b[u][q], acc[t][u], 0, 0, 0);
      between(i);
    }
  };

#pragma unroll
  for (int i = 0; i < NBUF; ++i) dma(i);
  h2_wait_barrier<(NBUF - 1) * (AL + BL)>();
  Frag f0, f1;
  read(f0, 0, 0);
  // Every step is the same straight-line code (branches around the loads would make the compiler wait for more than it
  // needs), and its order is pinned: left to itself the compiler moves the reads behind their latency.
  // (the reads go into the first half of the matrix instructions: the last of them has returned when the barrier comes)
  auto from = [](int i) { return 2 * i * NR / NM < NR ? 2 * i * NR / NM : NR; };
  auto step = [&](auto buf_c) {
    constexpr int buf = decltype(buf_c)::value;
    multiply(f0, [&](int i) {
#pragma unroll
      for (int r = from(i); r < from(i + 1); ++r) read_one(f1, buf, 1, r);
      __builtin_amdgcn_sched_barrier(0);
    });
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0), so that the compiler knows the fragments have arrived
    h2_wait_barrier<(NBUF - 2) * (AL + BL)>();  // everyone has read this step; the next one has arrived
    multiply(f1, [&](int i) {
#pragma unroll
      for (int r = from(i); r < from(i + 1); ++r) read_one(f0, (buf + 1) % NBUF, 0, r);
#pragma unroll
      for (int r = i * (AL + BL) / NM; r < (i + 1) * (AL + BL) / NM; ++r) dma_one(buf, r);
      __builtin_amdgcn_sched_barrier(0);
    });
    dma_next();
  };
  int kt = 0;
  for (; kt + NBUF <= n_kt; kt += NBUF) {
    step(std::integral_constant<int, 0>{});
    step(std::integral_constant<int, 1>{});
    if constexpr (NBUF == 4) {
      step(std::integral_constant<int, 2>{});
      step(std::integral_constant<int, 3>{});
    }
  }
  if (kt < n_kt) step(std::integral_constant<int, 0>{});
  if constexpr (NBUF == 4) {
    if (kt + 1 < n_kt) step(std::integral_constant<int, 1>{});
    if (kt + 2 < n_kt) step(std::integral_constant<int, 2>{});
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // nothing of this workgroup's is under way to LDS when it ends

  // ------------------------------- epilogue -------------------------------
  constexpr int PL = EK == 2 ? 1 : EK == 3 ? 0 : BITS;
  const int words_per_row = n_kt * PL;
#pragma unroll
  for (int u = 0; u < UW; ++u) {
    const int vloc = wn * UW * 32 + u * 32 + l32;
    const int64_t i = n0 + vloc;
    const bool valid = vloc < rows_n;
    const int64_t ic = valid ? i : n0;
    float scale = 1.f, es = 1.f, g2 = 0.f;
    if (EK != 2) scale = a.fac[ic];
    if constexpr (EK == 3) {
#pragma unroll
      for (int t = 0; t < TW; ++t) {
        const int mb = m0 + (wm * TW + t) * 32;
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (valid && mb < a.d)
            *reinterpret_cast<float4*>(a.out + i * a.d + mb + 8 * k + 4 * h) =
                make_float4(acc[t][u][4 * k] * scale, acc[t][u][4 * k + 1] * scale, acc[t][u][4 * k + 2] * scale, acc[t][u][4 * k + 3] * scale);
      }
      continue;
    }
    if (EK == 1) es = a.esc[ic];
    uint32_t w[TW][4];
#pragma unroll
    for (int t = 0; t < TW; ++t) {
      __builtin_amdgcn_sched_barrier(0);  // one tile's epilogue at a time (register pressure)
      const int mb = m0 + (wm * TW + t) * 32;
      if constexpr (EK == 2) {
        uint32_t nib[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          nib[k] = 0u;
#pragma unroll
          for (int r = 3; r >= 0; --r) nib[k] = shift_in(nib[k], __builtin_amdgcn_ballot_w64(acc[t][u][4 * k + r] >= 0.f));
        }
        w[t][0] = or_across_halves((nib[0] | (nib[1] << 8) | (nib[2] << 16) | (nib[3] << 24)) << (4 * h));
      } else {
        const float g = quantise_tile_best<BITS, EK == 1>(acc[t][u], scale, cb, h, w[t]);
        if (EK == 1 && mb < a.d) {
          g2 += g;
          // a lane has rows 8 k + 4 h .. + 3 of its vector; after exchanging pairs between the half-waves half h has
          // rows 16 h .. 16 h + 15, which it stores as 16-byte runs
          uint32_t hi[4][2], lo[4][2];
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            h2_split(acc[t][u][4 * k] * es, acc[t][u][4 * k + 1] * es, hi[k][0], lo[k][0]);
            h2_split(acc[t][u][4 * k + 2] * es, acc[t][u][4 * k + 3] * es, hi[k][1], lo[k][1]);
          }
          unsigned char* const e = a.E + i * row_a + (mb >> 5) * 128 + 32 * h;
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            const auto h0 = __builtin_amdgcn_permlane32_swap(hi[k][0], hi[k + 2][0], false, false);
            const auto h1 = __builtin_amdgcn_permlane32_swap(hi[k][1], hi[k + 2][1], false, false);
            const auto l0 = __builtin_amdgcn_permlane32_swap(lo[k][0], lo[k + 2][0], false, false);
            const auto l1 = __builtin_amdgcn_permlane32_swap(lo[k][1], lo[k + 2][1], false, false);
            if (valid) {
              *reinterpret_cast<uint4*>(e + 16 * k) = make_uint4(h0[0], h1[0], h0[1], h1[1]);
              *reinterpret_cast<uint4*>(e + 64 + 16 * k) = make_uint4(l0[0], l1[0], l0[1], l1[1]);
            }
          }
        }
      }
    }
    if constexpr (PL > 0) {
      // half h stores tile h of a pair of tiles
      if constexpr (TW == 1) {
        const int mb = m0 + wm * 32;
        if (valid && h == 0 && mb < a.d) store_words<PL>(a.words + i * words_per_row + (mb >> 5) * PL, w[0]);
      } else {
#pragma unroll
        for (int t = 0; t < TW; t += 2) {
          uint32_t sel[4];
#pragma unroll
          for (int p = 0; p < PL; ++p) {
            const uint32_t w0 = w[t][p], w1 = w[t + 1][p];  // both read before the select: no array in memory
            sel[p] = h ? w1 : w0;
          }
          const int mb = m0 + (wm * TW + t + h) * 32;
          if (valid && mb < a.d) store_words<PL>(a.words + i * words_per_row + (mb >> 5) * PL, sel);
        }
      }
    }
    if constexpr (EK == 1) {
      g2 = add_across_halves(g2);
      if (h == 0) red[wm * TN + vloc] = g2;
    }
  }
  if constexpr (EK == 1) {
    __syncthreads();
    for (int c = tid; c < rows_n; c += NW * 64) {
      float v = red[c];
#pragma unroll
      for (int k = 1; k < WM; ++k) v += red[k * TN + c];
      a.part[(int64_t)tile_m * a.n + n0 + c] = v;
    }
  }
  if constexpr (EK == 2) {
    if (tile_m == 0)
      for (int c = tid; c < rows_n; c += NW * 64) {
        float v = a.part[n0 + c];
        for (int k = 1; k < a.part_tiles; ++k) v += a.part[(int64_t)k * a.n + n0 + c];
        a.gamma[n0 + c] = sqrtf(v);
      }
  }
}

// Tile by the number of workgroups it gives: the large one while it fills the chip, else smaller ones.  (A 256 x 256
// tile moves 64 KB through LDS for 384 matrix instructions, 128 x 128 half of that for a quarter.)
enum Tile { T256, T128, T64 };
Tile pick_tile(int d, int64_t n) {
  const int cu = device_cu_count();
  auto count = [&](int tm, int tn) { return (int64_t)((d + tm - 1) / tm) * ((n + tn - 1) / tn); };
  auto padded = [&](int tm) { return (double)((d + tm - 1) / tm * tm) / d; };
  if (count(256, 256) * 5 >= (int64_t)cu * 4 && padded(256) < 1.2 * padded(128)) return T256;
  if (count(128, 128) * 2 >= (int64_t)cu) return T128;
  return T64;
}

template <int EK, int BITS, int NPX, int TW, int UW, int WM, int WN, int NBUF>
hipError_t launch_tile(H2Args a, const Codebook& cb, hipStream_t s) {
  constexpr int TM = WM * TW * 32, TN = WN * UW * 32;
  constexpr int lds_bytes = NBUF * (TM * 128 + TN * NPX * 64);
  a.tiles_m = (a.d + TM - 1) / TM;
  const int64_t tiles_n = (a.n + TN - 1) / TN;
  if (tiles_n * a.tiles_m > (int64_t)1 << 30) return hipErrorInvalidValue;
  a.tiles_n = (int)tiles_n;
  const int total = a.tiles_m * a.tiles_n;
  a.per_xcd = (total + XCDS - 1) / XCDS;
  static LdsLimit lds_limit;  // per instantiation: the limit is raised once per device
  if (const hipError_t e = raise_lds_limit(lds_limit, reinterpret_cast<const void*>(&h2_kernel<EK, BITS, NPX, TW, UW, WM, WN, NBUF>), lds_bytes);
      e != hipSuccess)
    return e;
  hipLaunchKernelGGL((h2_kernel<EK, BITS, NPX, TW, UW, WM, WN, NBUF>), dim3(a.per_xcd * XCDS), dim3(WM * WN * 64), lds_bytes, s, a, cb);
  return hipGetLastError();
}

template <int EK, int BITS, int NPX>
hipError_t launch_any(const H2Args& a, const Codebook& cb, hipStream_t s) {
  switch (pick_tile(a.d, a.n)) {
    case T256: return launch_tile<EK, BITS, NPX, 2, 4, 4, 2, 2>(a, cb, s);
    case T128:  // indices only: eight wavefronts of 64 x 32 hide the decisions better than four of 64 x 64 (5 - 15 %)
      if constexpr (EK == 0) return launch_tile<EK, BITS, NPX, 2, 1, 2, 4, 4>(a, cb, s);
      else return launch_tile<EK, BITS, NPX, 2, 2, 2, 2, 4>(a, cb, s);
    default:
      // 32 vectors instead of 64 while that leaves compute units without a workgroup (a tile's bytes come through one of them), of long vectors
      // while it leaves two fifths of them and only where tiles of 64 would hold more empty places, or, beyond d = 2048, are of two pieces and all but full.  us, 64 / 32:
      //   d = 512, 4 bits     500 10.0 / 9.8
      //   d = 768, 2 + 1      300 20.6 / 19.5
      //   d = 1536, 2 + 1     130 32.1 / 29.7, 200 (168 workgroups) 32.5 / 33.6; bf16 57 26.8 / 29.4, 64 27.5 / 29.8; 2 bits, bf16 97 13.3 / 14.0
      //   d = 2048, 1 + 1     40 33.5 / 35.7, bf16 64 34.7 / 36.6
      //   d = 3072, 2 bits    64 24.3 / 21.7, 70 24.5 / 23.2, 100 (192 workgroups) 24.6 / 27.6; 1 + 1 36 46.4 / 50.9, 40 46.8 / 51.0, 64 52.4 / 49.2
      //   d = 4096, 1 + 1     bf16 33 57.6 / 66.8
      if (const int last = (int)((a.n - 1) % 64); a.d <= 1024 || last < 32 || (NPX == 2 && a.d > 2048 && last >= 56))
        if ((int64_t)((a.d + 63) / 64) * ((a.n + 31) / 32) * 5 <= (int64_t)device_cu_count() * (a.d <= 1024 ? 5 : 3))
          return launch_tile<EK, BITS, NPX, 1, 1, 2, 1, 4>(a, cb, s);
      return launch_tile<EK, BITS, NPX, 1, 1, 2, 2, 4>(a, cb, s);
  }
}

template <int EK, int NPX>
hipError_t launch_bits(int bits, const H2Args& a, const Codebook& cb, hipStream_t s) {
  switch (bits) {
    case 0:
      if constexpr (EK == 1) return launch_any<EK, 0, NPX>(a, cb, s);
      return hipErrorInvalidValue;
    case 1: return launch_any<EK, 1, NPX>(a, cb, s);
    case 2: return launch_any<EK, 2, NPX>(a, cb, s);
    case 3: return launch_any<EK, 3, NPX>(a, cb, s);
    case 4: return launch_any<EK, 4, NPX>(a, cb, s);
    default: return hipErrorInvalidValue;
  }
}

H2Args args_of(const H2Quant& q) {
  H2Args a;
  a.W = static_cast<const unsigned char*>(q.W);
  a.X = static_cast<const unsigned char*>(q.X);
  a.fac = q.fac; a.esc = q.esc; a.out = q.out; a.words = q.words;
  a.E = static_cast<unsigned char*>(q.E);
  a.part = q.part; a.gamma = q.gamma; a.n = q.n; a.d = q.d; a.part_tiles = q.part_tiles;
  a.tiles_m = a.tiles_n = a.per_xcd = 0;
  return a;
}

template <bool BF16, bool CUT>
hipError_t launch_split(const void* x, int64_t ldx, int64_t n, int d, bool normalise, const float* w_inv, void* pieces, float* norm,
                        float* fac, float* esc, hipStream_t s) {
  int lg = 2;  // d >= 32: at least four chunks of eight
  while (lg < 6 && (1 << lg) < d / 8) ++lg;
  const int rows = 256 >> lg;
  const dim3 grid((unsigned)((n + rows - 1) / rows));
  const int u = (d / 8 + (1 << lg) - 1) >> lg;
  unsigned char* const pc = static_cast<unsigned char*>(pieces);
#define TQ_SPLIT(U) hipLaunchKernelGGL((split_rows_kernel<BF16, CUT, U>), grid, dim3(256), 0, s, x, ldx, n, d, lg, normalise ? 1 : 0, w_inv, pc, norm, fac, esc)
  if (u <= 1) TQ_SPLIT(1);
  else if (u <= 2) TQ_SPLIT(2);
  else if (u <= 3) TQ_SPLIT(3);
  else if (u <= 6) TQ_SPLIT(6);
  else TQ_SPLIT(0);
#undef TQ_SPLIT
  return hipGetLastError();
}

}  // namespace

bool h2_codebook_serves(int bits, const Codebook& cb) { return bits < 3 || codebook_symmetric(cb, bits); }

size_t h2_image_bytes(int M, int d) { return (size_t)M * d * 4; }

hipError_t launch_h2_max(const float* W, int64_t ldw, int M, int d, uint32_t* max_bits, hipStream_t s) {
  hipLaunchKernelGGL(h2_zero_kernel, dim3(1), dim3(1), 0, s, max_bits);
  hipLaunchKernelGGL(h2_max_kernel, dim3(256), dim3(256), 0, s, W, ldw, M, d, max_bits);
  return hipGetLastError();
}

hipError_t launch_h2_image(const float* W, int64_t ldw, int M, int d, void* image, float* w_inv, hipStream_t s) {
  if (M <= 0 || d <= 0 || d % 32 != 0 || ldw % 4 != 0) return hipErrorInvalidValue;
  uint32_t* const max_bits = reinterpret_cast<uint32_t*>(w_inv) + 1;
  if (const hipError_t e = launch_h2_max(W, ldw, M, d, max_bits, s); e != hipSuccess) return e;
  const int64_t threads = (int64_t)M * d / 8;
  hipLaunchKernelGGL(h2_image_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, W, ldw, M, d, max_bits, w_inv,
                     static_cast<unsigned char*>(image));
  return hipGetLastError();
}

hipError_t launch_h2_split(const void* x, bool bf16, bool cut, int64_t ldx, int64_t n, int d, bool normalise, const float* w_inv, void* pieces,
                           float* norm, float* fac, float* esc, hipStream_t s) {
  if (bf16) return launch_split<true, false>(x, ldx, n, d, normalise, w_inv, pieces, norm, fac, esc, s);
  return cut ? launch_split<false, true>(x, ldx, n, d, normalise, w_inv, pieces, norm, fac, esc, s)
             : launch_split<false, false>(x, ldx, n, d, normalise, w_inv, pieces, norm, fac, esc, s);
}

int h2_part_tiles(int d, int64_t n) {
  const int tm = pick_tile(d, n) == T256 ? 256 : pick_tile(d, n) == T128 ? 128 : 64;
  return (d + tm - 1) / tm;
}

int64_t h2_full_rows(int d, int64_t rows) {
  // whole rounds of 256 x 256 tiles over the chip, so that the last round of a pass is not nearly empty
  const int64_t mt = (d + 255) / 256, cu = device_cu_count();
  const int64_t rounds = rows / 256 * mt / cu;
  return rounds > 0 ? rounds * cu / mt * 256 : rows / 256 * 256;
}

hipError_t launch_h2_quant(int bits, const H2Quant& q, const Codebook& cb, hipStream_t s) {
  const H2Args a = args_of(q);
  if (q.E != nullptr) return q.npx == 1 ? launch_bits<1, 1>(bits, a, cb, s) : launch_bits<1, 2>(bits, a, cb, s);
  return q.npx == 1 ? launch_bits<0, 1>(bits, a, cb, s) : launch_bits<0, 2>(bits, a, cb, s);
}

hipError_t launch_h2_store(const H2Quant& q, hipStream_t s) {
  const Codebook none = {};
  return launch_any<3, 0, 2>(args_of(q), none, s);
}

hipError_t launch_h2_sign(const H2Quant& q, hipStream_t s) {
  const Codebook none = {};
  return launch_any<2, 0, 2>(args_of(q), none, s);
}

}  // namespace tq
