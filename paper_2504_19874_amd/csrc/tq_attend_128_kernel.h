// Attention read-out at d = 128 (see tq_attend.hip for the decomposition): the softmax-weighted
// sum of decoded value codes on the matrix cores.
//
// A centroid table symmetric about its mean is a sum of signs, c[idx] = w0 + sum over the odd-sized plane
// subsets S of h[S] * s_S(idx), s_S = -1 / +1 as the XOR of the index bits in S is 0 / 1 (tq_score_i8.hip).  So for
// every query q and coordinate j
//     sum_i w_qi c[idx_ij] = w0 * sum_i w_qi + sum_S h[S] * sum_i w_qi s_S(idx_ij):
// sums of weights over the KEYS with signs from the code's bits.  The sign term of Alg. 2 is one more
// such sum, over the sign bits with the weights exp(logit - m) * nu_i * gamma_i (VPROD).  The weights w_qi = exp(logit - m) * nu_i
// are scaled by a power of two to 28-bit integers.  A nibble n of one, as a byte, IS the fp8 number n 2^-9 (e4m3: 0..7 are the
// subnormals, 8..15 go on evenly), so the eight base-16 digits of a weight cost two ANDs and no conversion, and a bit becomes an fp4
// operand of either sign where it stands in its word (0.5 with the bit shifted to the sign: seven instructions for 32 keys).  One
// v_mfma_scale_f32_32x32x64_f8f6f4 multiplies 32 rows (4 queries x 8 digits) with 64 keys x 32 coordinates; all sums of digits are
// exact (below 2^12 in steps of 1/2).
//
// The contraction runs over keys, but a code word holds 32 COORDINATES of one key.  Each lane
// therefore takes the words of 32 keys (one coordinate group, one plane) and transposes the
// 32 x 32 bit block in registers; the transposed words go through LDS to the lanes that need them as operands.
//
// Workgroup of WAVES (8, or 4) wavefronts = 16 WAVES TILES keys of one group, 4 queries; a wavefront owns 16 TILES consecutive
// keys (256, or 64 where 2048 keys per workgroup would leave compute units without one: attend128_keys) and takes
// up to 256 per pass (at_pass_keys: what LDS holds).  Between the scoring and the joining everything is a
// wavefront's own with long ranges; with short ones the sums are shared out by coordinate group (at_grouped), and of eight wavefronts four
// transpose (8 heads of 1024 tokens: 17.9 -> 17.2 us a step).
//
// 8 heads, 4 queries each, keys of 2 + 1 bits, values of 2, a step with its two appends: 65536 keys 29.0 -> 27.1 us, 1024 19.1 ->
// 17.3; keys and values of 4 bits, 53970 keys 61 -> 41.  Before: four base-256 digits on the integer instructions, whose byte operands
// came through a table of 64 KB in LDS, passes of 128 keys with two barriers each, and every lane fetching its own code words.  What
// bounds the 17 us after the launch: key codes until 10 (see the scoring body), then vector instructions (transposition, weights) and 2 us of matrix
// instructions, which with an fp8 operand take 64 cycles.
//
// FUSED: the logits come from the d = 128 scoring kernel run in place (tq_score_i8_128_body.h: the
// lane of (query, key) keeps its score in a register), so neither a score nor a dequantised
// value ever reaches memory.  Otherwise they are read from a score matrix computed beforehand
// (key codes the scoring body does not take).
#pragma once
#include "tq_attend.h"
#include "tq_score_i8_128_body.h"

#include <type_traits>

namespace tq {

// keys a wavefront handles per pass, its planes in words being NPL: all of its own where LDS and the 64 lanes (a block of 32 keys, a
// coordinate group and a plane each) allow it.  two: a second set of weight digits (the signs of Alg. 2, or instance hi)
__host__ __device__ constexpr int at_pass_keys(int tiles, int npl, bool two) { return tiles < 8 ? 64 : npl <= 2 && !two ? 256 : 128; }
__host__ __device__ constexpr int at_planes(int vb, bool two) { return vb + (two ? 1 : 0); }
// Short ranges: a wavefront's 64 keys are one matrix instruction per term, and what comes after it (16 sums to four) would be most of the
// work, so a wavefront takes one coordinate group for the keys of four wavefronts.  Not eight wavefronts with many planes: their registers
// leave room for one workgroup per compute unit then (8 heads of 20000 tokens, values of 4 bits: 28.5 -> 30.5 us a step).
__host__ __device__ constexpr bool at_grouped(int tiles, int waves, int npl) { return tiles < 8 && (waves == 4 || npl <= 2); }
// digits of a wavefront: [query][digit][key], a byte each; 16 more per row, so that the rows of a read are in different banks
__host__ __device__ constexpr int at_row_bytes(int pass) { return pass + 16; }
__host__ __device__ constexpr int at_wd_bytes(int pass) { return 32 * at_row_bytes(pass); }
// transposed words of a plane: [pair of blocks of 32 keys][block][coordinate]; the second block of a pair 32 words behind the first, so
// that the half-waves, which read one each, are in different halves of the banks
constexpr int AT_BLOCK_WORDS = 128 + 32, AT_PAIR_WORDS = AT_BLOCK_WORDS + 128;
__host__ __device__ constexpr int at_plane_words(int pass) { return pass / 64 * AT_PAIR_WORDS; }
constexpr int AT_FSUM_BYTES = 8 * 4 * 128 * 4;  // [wave][query][coordinate], over the digits in the end (short ranges need less)
constexpr int AT_RED_FLOATS = 3 * 8 * 4;  // [maxima | norm maxima | sums][wave][4]

// dynamic LDS: what the scoring body needs, then the digits and at last the sums; words; the reduction scratch, which like the words is
// written while other wavefronts may still be scoring
__host__ __device__ constexpr int attend128_first_bytes(int kb, int vb, bool two, bool fused, int tiles, int waves) {
  const int sets = two ? 2 : 1, wd = sets * waves * at_wd_bytes(at_pass_keys(tiles, at_planes(vb, two), two));
  const int own = wd > sets * AT_FSUM_BYTES ? wd : sets * AT_FSUM_BYTES;
  return fused && score128_lds(kb, waves) > own ? (score128_lds(kb, waves) + 15) / 16 * 16 : own;
}
__host__ __device__ constexpr int attend128_words_bytes(int vb, bool two, int tiles, int waves) {
  return waves * at_planes(vb, two) * at_plane_words(at_pass_keys(tiles, at_planes(vb, two), two)) * 4;
}
__host__ __device__ constexpr int attend128_lds(int kb, int vb, bool two, bool fused, int tiles, int waves) {
  return attend128_first_bytes(kb, vb, two, fused, tiles, waves) + attend128_words_bytes(vb, two, tiles, waves) + AT_RED_FLOATS * 4;
}

// [0]: the table's mean w0; [S]: what belongs to a plane subset of odd size, -2 h[S] (the operands are halves, and minus where the bit is set)
struct AttendCoefs {
  float c[16];
};

// max / sum over the 16 lanes of a row (lanes sharing lane / 16); every lane receives the result
__device__ __forceinline__ float row_max(float v) {
  v = fmaxf(v, __int_as_float(dpp_move<0xB1>(__float_as_int(v))));
  v = fmaxf(v, __int_as_float(dpp_move<0x4E>(__float_as_int(v))));
  v = fmaxf(v, __int_as_float(dpp_move<0x141>(__float_as_int(v))));
  v = fmaxf(v, __int_as_float(dpp_move<0x140>(__float_as_int(v))));
  return v;
}
__device__ __forceinline__ float row_sum(float v) {
  v += __int_as_float(dpp_move<0xB1>(__float_as_int(v)));
  v += __int_as_float(dpp_move<0x4E>(__float_as_int(v)));
  v += __int_as_float(dpp_move<0x141>(__float_as_int(v)));
  v += __int_as_float(dpp_move<0x140>(__float_as_int(v)));
  return v;
}

// nibble a of x[4 i + b] <-> nibble i of x[4 a + b]: four coordinates stay together
__device__ __forceinline__ void transpose_nibbles(uint32_t (&x)[32]) {
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const uint32_t a = x[k], b = x[k + 16];
    x[k + 16] = __builtin_amdgcn_perm(b, a, 0x07060302u);
    x[k] = __builtin_amdgcn_perm(b, a, 0x05040100u);
  }
#pragma unroll
  for (int k = 0; k < 32; ++k) {
    if (k & 8) continue;
    const uint32_t a = x[k], b = x[k + 8];
    x[k + 8] = __builtin_amdgcn_perm(b, a, 0x07030501u);
    x[k] = __builtin_amdgcn_perm(b, a, 0x06020400u);
  }
#pragma unroll
  for (int k = 0; k < 32; ++k) {
    if (k & 4) continue;
    const uint32_t a = x[k], b = x[k + 4];
    x[k + 4] = ((a >> 4) & 0x0F0F0F0Fu) | (b & 0xF0F0F0F0u);
    x[k] = (a & 0x0F0F0F0Fu) | ((b << 4) & 0xF0F0F0F0u);
  }
}

typedef float f32x16 __attribute__((ext_vector_type(16)));

// ka: arguments of the scoring body (FUSED only); a: value codes, partial results, and with !FUSED the score matrix
// VKIND, the kind of value code: 0 = Alg. 1; 1 = Alg. 2 (one more plane: the signs, with weights ... * gamma);
// 2 = two instances of Alg. 1 over a split of the coordinates (Sec. 4.3): groups g < a.gs_hi have VB + 1 index
// planes, the table cfh and the weights exp(.) * nu_hi, the others VB planes, cf and exp(.) * nu_lo.
// FINISH: the keys are one chunk, and the workgroup rotates its sums back itself; the joining kernel is a launch of its own, 3.5 us (8 heads, 4
// queries each, keys of 2 + 1 bits, values of 2, a step with its two appends: 100 tokens 17.9 -> 15.2 us, 512 18.2 -> 15.5).
// Short chunks of values of one plane, keys of 3 + 1 or of 4 bits: 132 or 133 registers, so that one workgroup fills a compute unit.  HELD to 128, with 8
// to 16 of them in scratch, two share it, which pays where there are more workgroups than compute units (us, as they come / held, 64 blocks of four queries over
// 2884 tokens: keys of 4 bits, values of 1 bit 21.0 / 18.6, of signs alone 22.9 / 21.0; 3 + 1 bits 20.1 / 19.0 and 21.9 / 20.6).  With one workgroup to a compute
// unit held ones are 1 to 9 % slower.  Keys of 4 + 1 bits take 151: not to be held.
__host__ __device__ constexpr bool at_may_be_held(int kb, bool kprod, int npl, int tiles, int waves, bool finish, bool fused) {
  return fused && npl == 1 && tiles < 8 && waves == 8 && !finish && (kprod ? kb == 3 : kb == 4);
}
template <int KB, bool KPROD, int VB, int VKIND, bool FUSED, int TILES, int WAVES, bool FINISH, bool HELD>
__global__ __launch_bounds__(64 * WAVES, HELD ? 4 : 1) void attend128_kernel(
    const ScoreI8Args ka, const AttendArgs a, const AttendCoefs cf, const AttendCoefs cfh) {
  constexpr bool VPROD = VKIND == 1, VSPLIT = VKIND == 2, TWO = VKIND != 0;  // TWO: a second set of weights
  fetch_arguments<sizeof(ScoreI8Args) + sizeof(AttendArgs) + 2 * sizeof(AttendCoefs)>();
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn_s[];
  constexpr int NPL = at_planes(VB, TWO);  // bit planes of a value code: index planes, then the signs of Alg. 2 / the top plane of instance hi
  constexpr int WAVE_KEYS = 16 * TILES, PASS_KEYS = at_pass_keys(TILES, NPL, TWO), PASSES = WAVE_KEYS / PASS_KEYS;
  constexpr int PT = PASS_KEYS / 16, PB = PASS_KEYS / 32, KK = PASS_KEYS / 64;  // tiles, blocks of 32 keys, k-blocks of 64 keys per pass
  constexpr int NVB = VB > 0 ? VB : 1;
  constexpr int ROW = at_row_bytes(PASS_KEYS), WD_BYTES = at_wd_bytes(PASS_KEYS), PLANE_WORDS = at_plane_words(PASS_KEYS);
  static_assert(4 * PB * NPL <= 64 && (TILES >= 8 || 16 * NPL <= 64), "a block, a group and a plane per lane");
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15;  // key within a tile
  const int kc = lane >> 4;   // query of this lane's logits
  const int l32 = lane & 31, h = lane >> 5;  // matrix instructions: row (query, digit) or column (coordinate of a group), half of the 64 keys
  const int chunk = blockIdx.x, group = blockIdx.y, q0 = blockIdx.z * 4;
  constexpr int FIRST = attend128_first_bytes(KB, VB, TWO, FUSED, TILES, WAVES);
  unsigned char* const wd = dyn_s + wave * WD_BYTES;  // digits of exp(.) nu; + WAVES WD_BYTES: of exp(.) nu gamma / nu_hi
  uint32_t* const words = reinterpret_cast<uint32_t*>(dyn_s + FIRST) + wave * (NPL * PLANE_WORDS);  // + plane * PLANE_WORDS
  float* const fsum_s = reinterpret_cast<float*>(dyn_s);  // [8][4][128], over the digits
  float* const fsumz_s = fsum_s + AT_FSUM_BYTES / 4;      // the same for the sign sums
  float* const red_s = reinterpret_cast<float*>(dyn_s + FIRST + attend128_words_bytes(VB, TWO, TILES, WAVES));  // [3][8][4]

  const int64_t gbase = (int64_t)group * a.group_stride;
  const int64_t wave_key0 = ((int64_t)chunk * WAVES + wave) * WAVE_KEYS;
  // transposing role: block kb of 32 keys, coordinate group tg, a plane.  Nibble i of the transposed word 4 a + b is to be key 8 b + i
  // (word t of the lane: key 8 (t % 4) + t / 4): eight consecutive keys, as the digits lie, make one dword of an operand, the bit of
  // the nibble being the coordinate's.
  constexpr bool GROUPED = at_grouped(TILES, WAVES, NPL), PAIRED = GROUPED && WAVES == 8;
  // Eight wavefronts of short ranges: the first four, one per SIMD and the first to have their scores, transpose for two each, four blocks of 32 keys
  constexpr int TB = PAIRED ? 4 : PB, TKEYS = 32 * TB;
  const bool transposes = !PAIRED || wave < 4;  // uniform
  const int64_t t_key0 = PAIRED ? (int64_t)chunk * (WAVES * WAVE_KEYS) + wave * TKEYS : wave_key0;
  const int kb = lane & (TB - 1), tg = (lane / TB) & 3, plane = lane / (4 * TB);

  uint32_t vw[32];
  const bool full = t_key0 + PASSES * TKEYS <= a.n;  // uniform: no key of this wavefront is past the end
  // the 16-byte pieces of the wavefront's rows, as they lie in memory; through its words' place in LDS to the lanes that transpose them
  // (lanes that fetch their own words touch every line four times: scoring ended 2 us later).  Two instances: rows are no whole pieces.
  typedef uint32_t piece __attribute__((ext_vector_type(4), aligned(4)));  // (the arrays are the caller's)
  constexpr int IP = VSPLIT ? 0 : TKEYS * VB / 64, ZP = VPROD ? TKEYS / 64 : 0;  // pieces per lane: index planes, signs
  constexpr int Z_AT = TKEYS * VB * 4 + TB * VB * 4;  // words of the index planes with 4 VB more per block of 32 keys (banks)
  piece pi[IP > 0 ? IP : 1], pz[ZP > 0 ? ZP : 1];
  auto load_codes = [&](int ps) {
    if (!transposes) return;
    if constexpr (!VSPLIT) {
      const int64_t row0 = t_key0 + ps * TKEYS, rows = a.n - row0;  // keys past the end have weight 0: the last piece again
      auto get = [&](const uint32_t* src, int per_row, int p) {
        const int64_t last = rows * per_row - 1;
        const int64_t at = full || p <= last ? p : last;
        return *reinterpret_cast<const piece*>(src + ((gbase + row0) * per_row + at) * 4);
      };
#pragma unroll
      for (int i = 0; i < IP; ++i) pi[i] = get(a.idx, VB, i * 64 + lane);
#pragma unroll
      for (int i = 0; i < ZP; ++i) pz[i] = get(a.qjl, 1, i * 64 + lane);
    } else {
      const int64_t k0 = t_key0 + ps * TKEYS + 32 * kb;
      const bool thi = tg < a.gs_hi;
      const int wpr = 4 * VB + a.gs_hi, off = (thi ? tg * (VB + 1) : a.gs_hi + tg * VB) + plane;
      const uint32_t* const src = a.idx + (gbase + (k0 < a.n ? k0 : a.n - 1)) * wpr + off;
      const int last = k0 < a.n ? (int)(a.n - 1 - k0 < 31 ? a.n - 1 - k0 : 31) : 0;
      // (asked for in the order of the keys: neighbours share a line)
#pragma unroll
      for (int k = 0; k < 32; ++k) vw[4 * (k & 7) + (k >> 3)] = plane < VB + (thi ? 1 : 0) ? src[(k < last ? k : last) * wpr] : 0u;  // no such plane: zeros
    }
  };
  uint32_t* const t_words = PAIRED ? words + (transposes ? wave : 0) * (NPL * PLANE_WORDS) : words;  // of two wavefronts: 2 wave, 2 wave + 1
  auto take_codes = [&] {
    if constexpr (!VSPLIT) {
#pragma unroll
      for (int i = 0; i < IP; ++i) {
        const int p = i * 64 + lane;
        *reinterpret_cast<u32x4*>(t_words + 4 * (p + p / (32 * NVB) * NVB)) = pi[i];
      }
#pragma unroll
      for (int i = 0; i < ZP; ++i) {
        const int p = i * 64 + lane;
        *reinterpret_cast<u32x4*>(t_words + Z_AT + 4 * (p + p / 32)) = pz[i];
      }
      const bool sign = VPROD && plane == VB;
      const int step = sign ? 4 : 4 * VB;  // words from one key's to the next key's
      const uint32_t* const src = t_words + (sign ? Z_AT + tg : tg * VB + (plane < NPL ? plane : 0)) + kb * 33 * step;
#pragma unroll
      for (int k = 0; k < 32; ++k) vw[4 * (k & 7) + (k >> 3)] = src[k * step];
    }
  };
  auto put_words = [&] {
    if (!transposes) return;
    take_codes();
    transpose_nibbles(vw);
    if (4 * TB * NPL == 64 || plane < NPL) {
      // the 16-byte pieces of a row of 32 words in an order of the lane's own: a store meets every bank equally often
      uint32_t* const row = t_words + plane * PLANE_WORDS + (kb >> 1) * (PAIRED ? NPL * PLANE_WORDS : AT_PAIR_WORDS) + (kb & 1) * AT_BLOCK_WORDS + tg * 32;
#pragma unroll
      for (int c = 0; c < 8; ++c) *reinterpret_cast<uint4*>(row + 4 * (c ^ (lane & 7))) = make_uint4(vw[4 * c], vw[4 * c + 1], vw[4 * c + 2], vw[4 * c + 3]);
    }
  };

  // value norms: lane L holds those of keys L, L + 64, ... of the wavefront
  // (and nu gamma, the factor of the sign term of Alg. 2)
  constexpr int NE = WAVE_KEYS / 64;
  float nuv[NE], ngv[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    const int64_t key = wave_key0 + 64 * e + lane;
    if (VSPLIT) {  // (nu_hi, nu_lo) per token
      nuv[e] = key < a.n ? a.norm[2 * (gbase + key) + 1] : 0.f;
      ngv[e] = key < a.n ? a.norm[2 * (gbase + key)] : 0.f;
    } else {
      nuv[e] = key < a.n ? a.norm[gbase + key] : 0.f;
      ngv[e] = VPROD && key < a.n ? nuv[e] * a.gamma[gbase + key] : 0.f;
    }
  }
  // the first pass's value codes travel while the keys are scored, where the registers allow it
  constexpr bool EARLY = !FUSED || KB + (KPROD ? 1 : 0) <= 4;
  // ---- logits: lane (kc, col) holds those of (query q0 + kc, key wave_key0 + 16 t + col), t < TILES ----
  // (kept in units of log 2, so that the weights are one v_exp_f32 each)
  float lg[TILES];
  const float scale2 = a.scale * 1.44269504088896341f;
#pragma unroll
  for (int t = 0; t < TILES; ++t) lg[t] = -INFINITY;
  if (FUSED) {
    auto sink = [&](int t, float score, bool key_live) { lg[t] = key_live ? scale2 * score : -INFINITY; };
    // (the value codes behind the first key codes and the matrices, which are due earlier)
    score128_body<KB, KPROD, TILES, WAVES>(ka, dyn_s, sink, [&] {
      if (EARLY) load_codes(0);
    });
  __builtin_amdgcn_sched_barrier(0);
  } else {
    const int64_t qrow = (int64_t)group * a.q_per_group + (q0 + kc < a.q_per_group ? q0 + kc : q0);
    const float* srow = a.scores + qrow * a.lds + wave_key0 + col;
#pragma unroll
    for (int t = 0; t < TILES; ++t)
      if (wave_key0 + 16 * t + col < a.n) lg[t] = scale2 * srow[16 * t];
  }
  if (!EARLY || !FUSED) load_codes(0);
  // FINISH: parts of ROWS rows of Pi (S) by 128 threads each, due at the end
  constexpr int ROWS = 256 / WAVES;
  float wp[FINISH ? ROWS : 1], ws[FINISH && VPROD ? ROWS : 1];
  if constexpr (FINISH) {
    const int at = (tid >> 7) * (ROWS * 128) + (tid & 127);
#pragma unroll
    for (int u = 0; u < ROWS; ++u) wp[u] = a.Pi[at + u * 128];
    if constexpr (VPROD)
#pragma unroll
      for (int u = 0; u < ROWS; ++u) ws[u] = a.S[at + u * 128];
  }
  __builtin_amdgcn_sched_barrier(0);
  put_words();  // (in front of the barrier that waits for the last wavefront's scores)

  // ---- chunk maxima: logits per query, value norm ---------------------------------------------
  {
    float v = lg[0];
#pragma unroll
    for (int t = 1; t < TILES; ++t) v = fmaxf(v, lg[t]);
    v = row_max(v);
    if (col == 0) red_s[wave * 4 + kc] = v;
    float nv = fabsf(nuv[0]), gv = fabsf(ngv[0]);
#pragma unroll
    for (int e = 1; e < NE; ++e) {
      nv = fmaxf(nv, fabsf(nuv[e]));
      gv = fmaxf(gv, fabsf(ngv[e]));
    }
    const float nm = wave_max(nv);
    if (lane == 1) red_s[32 + wave * 4] = nm;
    if (TWO) {
      const float gm = wave_max(gv);
      if (lane == 2) red_s[32 + wave * 4 + 1] = gm;
    }
  }
  __syncthreads();  // also: every wavefront is done with the scoring body's LDS
  __builtin_amdgcn_sched_barrier(0);
  float m = -INFINITY, numax = 0.f, ngmax = 0.f;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) {
    m = fmaxf(m, red_s[w * 4 + kc]);
    numax = fmaxf(numax, red_s[32 + w * 4]);
    if (TWO) ngmax = fmaxf(ngmax, red_s[32 + w * 4 + 1]);
  }
  int enu = 0, eng = 0;
  if (numax > 0.f) (void)frexpf(numax, &enu);  // numax = f * 2^enu, f in [0.5, 1)
  if (ngmax > 0.f) (void)frexpf(ngmax, &eng);
  enu = max(enu, -99), eng = max(eng, -99);  // below, the scale would not be finite: fewer than 28 bits of a weight there
  // |weights exp(logit - m) * nu * wscale| <= 2^28
#pragma unroll
  for (int e = 0; e < NE; ++e) nuv[e] *= ldexpf(1.f, 28 - enu), ngv[e] *= ldexpf(1.f, 28 - eng);
  auto rounded = [](float v) {  // to the nearest integer, in one instruction
    int i;
    asm("v_cvt_rpi_i32_f32 %0, %1" : "=v"(i) : "v"(v));
    return i;
  };

  // The eight base-16 digits of a weight (the top one with a sign), transposed among the four lanes of a quad: lane i gets digits 2 i and
  // 2 i + 1 of the quad's four keys in a word each.
  const uint32_t sel1 = lane & 1 ? 0x03070105u : 0x06020400u, sel2 = lane & 2 ? 0x03020706u : 0x05040100u;
  auto quad_transpose = [&](uint32_t w) -> uint32_t {
    w = __builtin_amdgcn_perm((uint32_t)__builtin_amdgcn_mov_dpp((int)w, 0xB1, 0xF, 0xF, true), w, sel1);
    return __builtin_amdgcn_perm((uint32_t)__builtin_amdgcn_mov_dpp((int)w, 0x4E, 0xF, 0xF, true), w, sel2);
  };
  auto put_digits = [&](unsigned char* o, int Q) {
    *reinterpret_cast<uint32_t*>(o) = quad_transpose((uint32_t)Q & 0x0F0F0F0Fu);
    *reinterpret_cast<uint32_t*>(o + 4 * ROW) = quad_transpose((uint32_t)(Q >> 4) & 0x810F0F0Fu);  // |Q| <= 2^28: the top digit is -1, 0 or 1
  };

  // the half-waves hold the digits 0, 2, 4, 6 and 1, 3, 5, 7 of the sums
  const float hf = h ? 16.f : 1.f;
  // GROUPED: wavefront w takes coordinate group w % 4 for the keys of four wavefronts, behind one barrier more
  constexpr int NG = GROUPED ? 1 : 4;  // coordinate groups of a wavefront
  float f[NG][4], fz[NG][4];           // [coordinate group][query]: coordinate 32 g + l32; VPROD: the sums of the sign term
#pragma unroll
  for (int g = 0; g < NG; ++g)
#pragma unroll
    for (int k = 0; k < 4; ++k) f[g][k] = fz[g][k] = 0.f;
  float lsum = 0.f;
  // words with coordinate 32 g + l32 for the 32 keys 64 kk + 32 h ..: see put_words
  uint32_t read_at[4];
#pragma unroll
  for (int x = 0; x < 4; ++x) read_at[x] = h * AT_BLOCK_WORDS + 4 * (((l32 >> 2) ^ h) ^ (2 * x));
  // GROUPED: in the words of wavefront kk of four
  auto read_own = [&](int kk) { return h * AT_BLOCK_WORDS + 4 * (((l32 >> 2) ^ h) ^ (2 * ((((PAIRED ? 2 * (kk & 1) : 0) + TB * (wave & 3)) & 7) / 2))); };
  // a wavefront's digits and words are its own, and LDS takes a wavefront's instructions in order
  auto wave_sync = [] {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
  };
  // 32 keys as fp4 operands +-0.5: minus where the bit is set
  uint32_t halves = 0x11111111u;  // in a register that the compiler does not know: one v_and_or_b32 takes no two constants
  asm volatile("" : "+v"(halves));
  const int to_top = 3 - (l32 & 3);
  auto signs = [halves, to_top](const u32x4& w) -> v8i {
    auto of = [halves, to_top](uint32_t v) { return (int)(((v << to_top) & 0x88888888u) | halves); };
    const v4i b = v4i{of(w[0]), of(w[1]), of(w[2]), of(w[3])};
    return __builtin_shufflevector(b, b, 0, 1, 2, 3, -1, -1, -1, -1);  // fp4: four registers
  };

#pragma unroll
  for (int ps = 0; ps < PASSES; ++ps) {
    if (ps > 0) put_words();
    if (ps + 1 < PASSES) load_codes(ps + 1);
    // weights of this lane's (query, key) pairs -> digits
#pragma unroll
    for (int tt = 0; tt < PT; ++tt) {
      const int t = PT * ps + tt;
      const float nu = __int_as_float(__builtin_amdgcn_ds_bpermute(4 * (16 * (t & 3) + col), __float_as_int(nuv[t >> 2])));
      const float p = __builtin_amdgcn_exp2f(lg[t] - m);  // 0 for keys past the end (logit -inf)
      lsum += p;
      unsigned char* const o = wd + (8 * kc + (col & 3)) * ROW + 16 * tt + (col & 12);
      put_digits(o, rounded(p * nu));
      if (TWO) {
        const float ng = __int_as_float(__builtin_amdgcn_ds_bpermute(4 * (16 * (t & 3) + col), __float_as_int(ngv[t >> 2])));
        put_digits(o + WAVES * WD_BYTES, rounded(p * ng));
      }
    }
    if constexpr (GROUPED) __syncthreads();
    else wave_sync();

  __builtin_amdgcn_sched_barrier(0);
    // an fp8 operand's 32 values of a lane are k = 16 h .. and 32 + 16 h .., an fp4 operand's k = 32 h ..
    auto digits_of = [&](const unsigned char* w, int kk) -> v8i {
      const unsigned char* const r = w + l32 * ROW + kk * 64 + 16 * h;
      const v4i lo = *reinterpret_cast<const v4i*>(r), hi = *reinterpret_cast<const v4i*>(r + 32);
      return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    // the k-blocks of this wavefront's sums: its own keys, or those of four wavefronts
    constexpr int NK = GROUPED ? 4 : KK;
    static_assert(!GROUPED || (KK == 1 && PASSES == 1), "");
    const unsigned char* const wd0 = GROUPED ? dyn_s + (wave & ~3) * WD_BYTES : wd;
    const uint32_t* const words0 = GROUPED ? words - (wave & 3) * (NPL * PLANE_WORDS) : words;
    auto digits_at = [&](const unsigned char* w, int kk) { return GROUPED ? digits_of(w + kk * WD_BYTES, 0) : digits_of(w, kk); };
    v8i aop[NK], zop[NK];
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      aop[kk] = digits_at(wd0, kk);
      if (VSPLIT) zop[kk] = digits_at(wd0 + WAVES * WD_BYTES, kk);
    }
    auto words_of = [&](int pl, int g, int kk) {
      if constexpr (GROUPED) {
        const int gw = wave & 3;
        return *reinterpret_cast<const u32x4*>(words0 + kk * (NPL * PLANE_WORDS) + pl * PLANE_WORDS + gw * 32 + read_own(kk));
      } else {
        return *reinterpret_cast<const u32x4*>(words0 + pl * PLANE_WORDS + kk * AT_PAIR_WORDS + g * 32 + read_at[((2 * kk + PB * g) & 7) / 2]);
      }
    };
    // sums of a coordinate group with these weights and signs, added to o with a factor
    auto add_sums = [&](const v8i (&wop)[NK], auto sign_of, float factor, float (&o)[4]) {
      f32x16 acc;
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
      for (int kk = 0; kk < NK; ++kk)  // (the scale 2^9 makes a digit the integer it stands for)
        acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(wop[kk], sign_of(kk), acc, 0, 4, 0, 136, 0, 127);
#pragma unroll
      for (int k = 0; k < 4; ++k)
        o[k] = fmaf(factor, fmaf(fmaf(acc[4 * k + 3], 256.f, acc[4 * k + 2]), 65536.f, fmaf(acc[4 * k + 1], 256.f, acc[4 * k])), o[k]);
    };
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      __builtin_amdgcn_sched_barrier(0);  // one group's sums at a time (registers)
      constexpr int NPI = VSPLIT ? VB + 1 : NVB;  // index planes (instance lo: the top one is all zero)
      u32x4 pw[NK][NPI];
#pragma unroll
      for (int kk = 0; kk < NK; ++kk)
#pragma unroll
        for (int pl = 0; pl < (VSPLIT ? VB + 1 : VB); ++pl) pw[kk][pl] = words_of(pl, g, kk);
      // signs of one coordinate group: plane subsets of odd size, weights and table of the group's instance
      auto terms = [&](auto planes_c, const v8i (&wop)[NK], const AttendCoefs& tab) {
        constexpr int NP = decltype(planes_c)::value;
#pragma unroll
        for (int mset = 1; mset < (1 << NP); ++mset) {
          if (!i8_term(mset)) continue;
          if (NPL > 2) __builtin_amdgcn_sched_barrier(0);  // one sum at a time
          add_sums(wop, [&](int kk) {
            u32x4 x = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
            for (int pl = 0; pl < NP; ++pl)
              if (mset & (1 << pl)) x ^= pw[kk][pl];
            return signs(x);
          }, hf * tab.c[mset], f[g]);
        }
      };
      const bool of_hi = VSPLIT && (GROUPED ? wave & 3 : g) < a.gs_hi;
      if (of_hi) terms(std::integral_constant<int, VB + 1>{}, zop, cfh);  // uniform
      else terms(std::integral_constant<int, VB>{}, aop, cf);
    }
    if constexpr (VPROD) {
#pragma unroll
      for (int kk = 0; kk < NK; ++kk) zop[kk] = digits_at(wd0 + WAVES * WD_BYTES, kk);
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        __builtin_amdgcn_sched_barrier(0);
        add_sums(zop, [&](int kk) { return signs(words_of(VB, g, kk)); }, -2.f * hf, fz[g]);
      }
    }
    if (cf.c[0] != 0.f || (VSPLIT && cfh.c[0] != 0.f)) {  // tables whose mean is not 0 (uniform; behind the sums, which it would tear apart)
      float w[4] = {0.f, 0.f, 0.f, 0.f}, wh[4] = {0.f, 0.f, 0.f, 0.f};
      add_sums(aop, [&](int) { return signs(u32x4{0u, 0u, 0u, 0u}); }, 2.f * hf * cf.c[0], w);
      if constexpr (VSPLIT) add_sums(zop, [&](int) { return signs(u32x4{0u, 0u, 0u, 0u}); }, 2.f * hf * cfh.c[0], wh);
#pragma unroll
      for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int k = 0; k < 4; ++k) f[g][k] += VSPLIT && (GROUPED ? wave & 3 : g) < a.gs_hi ? wh[k] : w[k];
    }
    wave_sync();
  }
  __builtin_amdgcn_sched_barrier(0);
  __syncthreads();  // the final sums go over the digits
  __builtin_amdgcn_sched_barrier(0);

  // ---- join the wavefronts ------------------------------------------------------------------------
  lsum = row_sum(lsum);
  if (col == 0) red_s[64 + wave * 4 + kc] = lsum;
  // the half-waves' parts of a sum together: half h then has those of queries k + 2 h
  auto join = [&](float lo, float hi) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(lo), __float_as_uint(hi), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
  };
  constexpr int PARTS = GROUPED ? WAVES / 4 : WAVES;  // sums to be added
#pragma unroll
  for (int g = 0; g < NG; ++g)
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int gw = GROUPED ? wave & 3 : g, at = ((GROUPED ? wave >> 2 : wave) * 4 + k + 2 * h) * 128 + 32 * gw + l32;
      float v = join(f[g][k], f[g][k + 2]);
      if (VSPLIT) v *= ldexpf(1.f, (gw < a.gs_hi ? eng : enu) - 28);  // each instance has its own weight scale
      fsum_s[at] = v;
      if (VPROD) fsumz_s[at] = join(fz[g][k], fz[g][k + 2]);
    }
  __syncthreads();
  constexpr int ROUNDS_Q = 8 / WAVES, QUERIES = WAVES / 2;  // 128 threads have a query's coordinates
  const int j = tid & 127, part0 = tid >> 7;
  float* const y_s = reinterpret_cast<float*>(dyn_s + FIRST);  // FINISH: [index term, sign term][query][coordinate], over the words
#pragma unroll
  for (int rq = 0; rq < ROUNDS_Q; ++rq) {
  const int qi = part0 + rq * QUERIES;
  float acc = 0.f, accz = 0.f;
#pragma unroll
  for (int w = 0; w < PARTS; ++w) {
    acc += fsum_s[(w * 4 + qi) * 128 + j];
    if (VPROD) accz += fsumz_s[(w * 4 + qi) * 128 + j];
  }
  if (!VSPLIT) acc *= ldexpf(1.f, enu - 28);
  if (VPROD) accz *= ldexpf(1.f, eng - 28);
  const int64_t row = (int64_t)group * a.q_per_group + q0 + qi;
  auto summed = [&] {
    float l = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) l += red_s[64 + w * 4 + qi];
    return l;
  };
  if constexpr (!FINISH) {
    if (q0 + qi < a.q_per_group) {
      float* o = a.part + (row * a.nchunks + chunk) * attend_part_stride(128);
      o[4 + j] = acc;
      o[4 + 128 + j] = accz;
      if (j == 0) {
        float mq = -INFINITY;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) mq = fmaxf(mq, red_s[w * 4 + qi]);
        o[0] = mq * 0.693147180559945309f;  // back to natural units
        o[1] = summed();
      }
    }
  } else {
    const float l = summed();
    static_assert(attend128_words_bytes(VB, TWO, TILES, WAVES) >= (VPROD ? 2 : 1) * 512 * 4, "LDS");
    y_s[qi * 128 + j] = acc / l;
    if (VPROD) y_s[512 + qi * 128 + j] = accz / l;
  }
  }
  if constexpr (FINISH) {
    __syncthreads();
    // (a wavefront's rows are ROWS consecutive ones: the first of four values per lane of 16, of which ROWS / 4 count)
    // Chains of 16 products as in the joining kernel; their adds cost nothing that shows (8 heads of 100 tokens 15.0 us a step either way).  Error against
    // 64 bits with equal logits, 10^-7, one chain of ROWS / chains of 16 / the joining kernel behind chunks of 2048: 256 tokens, values of 4 bits (ROWS
    // = 64) 1.61 / 1.09 / 1.22; of 2 bits (32) 1.26 / 1.06 / 1.09.
    auto rotated = [&](const float (&w)[ROWS], const float* y, float (&o)[4]) {
      f32x4_prep v[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = *reinterpret_cast<const f32x4*>(y + k * 128 + ROWS * part0 + 4 * (tid & (ROWS / 4 - 1)));
      float chain[ROWS / 16][4] = {};
      matvec_rows<0, 4>(chain[0], v, w);
      matvec_rows<4, 8>(chain[1], v, w);
      if constexpr (ROWS == 64) {
        matvec_rows<8, 12>(chain[2], v, w);
        matvec_rows<12, 16>(chain[3], v, w);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        o[k] = chain[0][k] + chain[1][k];
        if constexpr (ROWS == 64) o[k] += chain[2][k] + chain[3][k];
      }
    };
    float o[4], oz[4] = {0.f, 0.f, 0.f, 0.f};
    rotated(wp, y_s, o);
    if constexpr (VPROD) rotated(ws, y_s + 512, oz);
#pragma unroll
    for (int k = 0; k < 4; ++k) fsum_s[(part0 * 4 + k) * 128 + j] = VPROD ? fmaf(a.kappa, oz[k], o[k]) : o[k];
    __syncthreads();
#pragma unroll
    for (int rq = 0; rq < ROUNDS_Q; ++rq) {
      const int qi = part0 + rq * QUERIES;
      if (q0 + qi < a.q_per_group) {
        float r = fsum_s[qi * 128 + j];
#pragma unroll
        for (int t = 1; t < WAVES / 2; ++t) r += fsum_s[(t * 4 + qi) * 128 + j];
        a.out[((int64_t)group * a.q_per_group + q0 + qi) * a.ldo + j] = r;
      }
    }
  }
}

template <int KB, bool KPROD, int VB, int VKIND, bool FUSED, int TILES, int WAVES, bool FINISH, bool HELD>
hipError_t launch_attend128_grid(const ScoreI8Args& ka, const AttendArgs& a, const AttendCoefs& cf, const AttendCoefs& cfh, const dim3& grid,
                                 hipStream_t s) {
  constexpr int lds = attend128_lds(KB, VB, VKIND != 0, FUSED, TILES, WAVES);
  static_assert(lds <= 160 * 1024, "LDS budget");
  static LdsLimit lds_limit;  // per instantiation: the limit is raised once per device
  if (const hipError_t e = raise_lds_limit(lds_limit, reinterpret_cast<const void*>(&attend128_kernel<KB, KPROD, VB, VKIND, FUSED, TILES, WAVES, FINISH, HELD>), lds); e != hipSuccess) return e;
  hipLaunchKernelGGL((attend128_kernel<KB, KPROD, VB, VKIND, FUSED, TILES, WAVES, FINISH, HELD>), grid, dim3(64 * WAVES), lds, s, ka, a, cf, cfh);
  return hipGetLastError();
}

template <int KB, bool KPROD, int VB, int VKIND, bool FUSED, int TILES, int WAVES, bool FINISH>
hipError_t launch_attend128_tiles(const ScoreI8Args& ka, const AttendArgs& a, const AttendCoefs& cf, const AttendCoefs& cfh,
                                int n_groups, hipStream_t s) {
  const dim3 grid(a.nchunks, n_groups, (a.q_per_group + 3) / 4);
  if constexpr (at_may_be_held(KB, KPROD, at_planes(VB, VKIND != 0), TILES, WAVES, FINISH, FUSED))
    if ((int64_t)grid.x * grid.y * grid.z > device_cu_count())
      return launch_attend128_grid<KB, KPROD, VB, VKIND, FUSED, TILES, WAVES, FINISH, true>(ka, a, cf, cfh, grid, s);
  return launch_attend128_grid<KB, KPROD, VB, VKIND, FUSED, TILES, WAVES, FINISH, false>(ka, a, cf, cfh, grid, s);
}

template <int KB, bool KPROD, int VB, int VKIND, bool FUSED>
hipError_t launch_attend128_one(const ScoreI8Args& ka, const AttendArgs& a, const AttendCoefs& cf, const AttendCoefs& cfh,
                                int n_groups, hipStream_t s) {
  const bool finish = a.out != nullptr;
  if constexpr (attend128_takes_256(at_planes(VB, VKIND != 0)))
    if (a.keys == 256)
      return finish ? launch_attend128_tiles<KB, KPROD, VB, VKIND, FUSED, 4, 4, true>(ka, a, cf, cfh, n_groups, s)
                    : launch_attend128_tiles<KB, KPROD, VB, VKIND, FUSED, 4, 4, false>(ka, a, cf, cfh, n_groups, s);
  switch (a.keys) {
    case 512: return finish ? launch_attend128_tiles<KB, KPROD, VB, VKIND, FUSED, 4, 8, true>(ka, a, cf, cfh, n_groups, s)
                            : launch_attend128_tiles<KB, KPROD, VB, VKIND, FUSED, 4, 8, false>(ka, a, cf, cfh, n_groups, s);
    case 2048: return finish ? hipErrorInvalidValue : launch_attend128_tiles<KB, KPROD, VB, VKIND, FUSED, 16, 8, false>(ka, a, cf, cfh, n_groups, s);
    default: return hipErrorInvalidValue;
  }
}

// all key variants for one kind of value code; kb < 0: logits from a.scores
template <int VB, int VKIND>
hipError_t launch_attend128_vb(int kb, bool kprod, const ScoreI8Args& ka, const AttendArgs& a, const AttendCoefs& cf,
                               const AttendCoefs& cfh, int n_groups, hipStream_t s) {
  if (kb < 0) return launch_attend128_one<0, false, VB, VKIND, false>(ka, a, cf, cfh, n_groups, s);
  switch (kb * 2 + (kprod ? 1 : 0)) {
    case 1: return launch_attend128_one<0, true, VB, VKIND, true>(ka, a, cf, cfh, n_groups, s);
    case 2: return launch_attend128_one<1, false, VB, VKIND, true>(ka, a, cf, cfh, n_groups, s);
    case 3: return launch_attend128_one<1, true, VB, VKIND, true>(ka, a, cf, cfh, n_groups, s);
    case 4: return launch_attend128_one<2, false, VB, VKIND, true>(ka, a, cf, cfh, n_groups, s);
    case 5: return launch_attend128_one<2, true, VB, VKIND, true>(ka, a, cf, cfh, n_groups, s);
    case 6: return launch_attend128_one<3, false, VB, VKIND, true>(ka, a, cf, cfh, n_groups, s);
    case 7: return launch_attend128_one<3, true, VB, VKIND, true>(ka, a, cf, cfh, n_groups, s);
    case 8: return launch_attend128_one<4, false, VB, VKIND, true>(ka, a, cf, cfh, n_groups, s);
    case 9: return launch_attend128_one<4, true, VB, VKIND, true>(ka, a, cf, cfh, n_groups, s);
    default: return hipErrorInvalidValue;
  }
}

// one translation unit per kind of value code (tq_attend_128_v*.hip: MSE codes of 1..4 bits; tq_attend_128_p*.hip:
// codes of Alg. 2 with 0..2 index bits; tq_attend_128_s*.hip: two instances with 1 + 2 or 2 + 3 index bits: what fits
// LDS beside the second set of weights)
#define TQ_ATTEND128_DECL(NAME)                                                                  \
  hipError_t NAME(int kb, bool kprod, const ScoreI8Args& ka, const AttendArgs& a, const AttendCoefs& cf, \
                  const AttendCoefs& cfh, int n_groups, hipStream_t s)
TQ_ATTEND128_DECL(launch_attend128_v1);
TQ_ATTEND128_DECL(launch_attend128_v2);
TQ_ATTEND128_DECL(launch_attend128_v3);
TQ_ATTEND128_DECL(launch_attend128_v4);
TQ_ATTEND128_DECL(launch_attend128_p0);
TQ_ATTEND128_DECL(launch_attend128_p1);
TQ_ATTEND128_DECL(launch_attend128_p2);
TQ_ATTEND128_DECL(launch_attend128_s1);
TQ_ATTEND128_DECL(launch_attend128_s2);

}  // namespace tq
