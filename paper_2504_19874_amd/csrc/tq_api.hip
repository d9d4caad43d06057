// C ABI entry points: argument validation, workspace carving, kernel launches.
// No allocation, no synchronisation; everything is enqueued on the caller's
// stream.
#include <cmath>
#include <cstring>
#include <mutex>

#include "tq_attend.h"
#include "tq_code_gemm.h"
#include "tq_h2.h"
#include "tq_score_i8.h"
#include "tq_search.h"
#include "tq_sign.h"

using namespace tq;

namespace tq {
int device_cu_count() {
  static std::mutex m;
  static int count[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 256;
  std::lock_guard<std::mutex> lock(m);
  if (count[dev] == 0) {
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0) v = 256;
    count[dev] = v;
  }
  return count[dev];
}
}  // namespace tq

namespace {

constexpr int64_t kChunkRows = 65536;  // rows per pass of the quantiser at most (with a sketch the workspace holds half as many)
// Row strides of vectors (x, q) and of dequantised output: the kernels address a tile's rows with 32-bit byte
// offsets from a 64-bit tile base (up to 256 rows of ld * 4 bytes)
constexpr int64_t kMaxRowStride = int64_t(1) << 22;
// Up to here vectors take the matrix-vector route of the quantiser.  It reads every matrix once per block of four vectors, plain fp32
// multiply-adds; the contraction on the matrix cores once per tile, and reads 17 bits of an fp32 vector.  The line between them, blocks x d^2, lies
// at 4e7 elements, at 64 vectors (with a sketch 52 of 1536), and for short ones at 65536 values (half with a sketch), about where the two take
// the same time: up to there vectors keep all their bits (mean error of a rotated coordinate 0.8 - 1.2e-7 sigma; 2.0e-6 on the
// contraction, 2.4e-7 for bf16 vectors).  us, this route / the contraction:
//   Alg. 1  d = 64    1 vector 3.3 / 6.4, 256 4.7 / 7.5
//           d = 256   1 3.4 / 7.8, 256 7.8 / 8.9, 512 12.2 / 8.8
//           d = 512   128 8.3 / 10.1, 192 10.7 / 10.1
//           d = 768   64 8.5 / 11.6 (96)
//           d = 1536  64 15.6 / 15.8
//           d = 3072  16 15.7 / 22.0 (32), 32 26.7 / 22.0
//   Alg. 2  d = 256   1 6.1 / 11.3, 128 10.7 / 12.8, 192 12.7 / 12.5
//           d = 512   64 11.4 / 16.0 (96)
//           d = 1536  32 19.5 / 29.9 (48), 52 24.5 / 28.1, 56 28.2 / 28.0, 64 29.4 / 28.9; bf16 52 24.7 / 27.6, 56 29.4 / 27.0, 64 30.2 / 27.3
//           d = 2048  36 31.1 / 33.6
//           d = 3072  16 29.9 / 45.2, 32 51.3 / 49.6
bool quant_rows_serves(int64_t n, int d, bool prod) {
  if (d > 4096 || n > 256 || ((n + 3) / 4) * (int64_t)d * d > 150 * 512 * 512) return false;
  return prod ? (n <= 64 && n * d <= 52 * 1536) || n * d <= 32768 : n <= 64 || n * d <= 65536;
}

// The dequantiser's (tq_score_small.hip: both matrices in one kernel, decoding and products by vector instructions).  us, it / the kernels on the
// matrix cores:
//   4 bits      d = 64    1 code 3.1 / 5.2, 512 5.2 / 5.9, 640 6.1 / 5.9
//               d = 128   1 3.1 / 6.4, 512 5.9 / 7.3, 1024 7.8 / 7.3
//               d = 256   512 8.1 / 8.5, 640 9.1 / 8.6
//               d = 384   (3 bits) 256 8.3 / 9.9, 384 10.8 / 10.0
//               d = 512   256 9.5 / 12.6
//               d = 768   256 15.1 / 16.9
//               d = 1024  192 18.3 / 20.8, 256 22.6 / 22.1
//               d = 1536  128 26.4 / 30.4, 192 37.3 / 30.6
//               d = 3072  32 31 / 56 (48 codes), 64 58.5 / 55.8
//   3 + 1 bits  d = 384   256 12.8 / 15.0
//               d = 768   256 23.0 / 30.6
//               d = 1536  128 43.7 / 56.6, 192 63.8 / 56.8
//               d = 3072  32 94 / 108, 64 237 / 109
bool dequant_rows_serves(int64_t n, int d) { return n <= (d <= 256 ? 512 : 256) && d < 4096 && n * d <= (d <= 2048 ? 128 * 1536 : 32 * 3072); }

// Codes of a table that is a sum of signs: only a few long ones by these products, the others by digits, made in the call where they are not at
// hand, which takes ten times as long.  us and error against 64 bits (1e-7 of a coordinate's root mean square), products / digits at hand:
//   2 bits      d = 512   1 code 4.3 / 3.7, 32 4.9 / 4.2, 0.9 / 1.3
//               d = 1536  1 5.4 / 5.0, 16 9.5 / 5.3, 1.15 / 1.24 (digits made in the call 27)
//   2 + 1 bits  d = 512   1 4.4 / 5.1, 32 4.9 / 5.8, 1.1 / 1.3
//               d = 768   32 5.7 / 6.4, 1.2 / 1.2
//               d = 1024  16 5.5 / 6.7, 32 7.3 / 7.4, 1.3 / 1.1
//               d = 1536  4 6.3 / 7.7, 16 8.2 / 8.1, 32 11.0 / 9.1, 1.5 / 1.25 (digits made in the call 50)
//               d = 3072  1 13.5 / 13.2, 16 39.8 / 14.9, 1.9 / 1.5
// So products where they are the closer ones, which is without a sketch and below d = 1024, and beyond it while they take less time.
bool rows_before_digits(int64_t n, int d, int bits, bool prod, bool at_hand) {
  if (at_hand && prod && bits > 0 && d >= 1024 && n * d * d >= 32 * 1024 * 1024) return false;
  return n <= (prod ? 32 : 64) && d >= 512 && d < 4096 && (((prod ? 2 : 1) * n + 3) / 4) * (int64_t)d * d * (prod ? 2 : 1) <= 300 * 512 * 512;
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

tq_status check_params(const tq_params* p, bool need_codebook) {
  if (p == nullptr) return TQ_ERR_INVALID_ARG;
  if (p->d <= 0 || p->bits_mse < 0) return TQ_ERR_INVALID_ARG;
  if (p->d % 32 != 0 || p->bits_mse > 4 || p->d > 16384) return TQ_ERR_UNSUPPORTED;
  if (need_codebook) {
    if (p->centroids == nullptr) return TQ_ERR_INVALID_ARG;
    if (p->bits_mse > 0 && p->bounds == nullptr) return TQ_ERR_INVALID_ARG;
  }
  if (p->d_hi != 0) {
    // two instances over a split of the rotated coordinates (Sec. 4.3)
    if (p->d_hi < 0 || p->d_hi >= p->d || p->d_hi % 32 != 0 || p->bits_mse_hi < 0) return TQ_ERR_INVALID_ARG;
    if (need_codebook && (p->centroids_hi == nullptr || (p->bits_mse_hi > 0 && p->bounds_hi == nullptr)))
      return TQ_ERR_INVALID_ARG;
    // what the kernels cover: head dimension 128, one more bit for the outlier instance
    if (p->d != 128 || p->bits_mse_hi != p->bits_mse + 1 || p->bits_mse_hi > 4) return TQ_ERR_UNSUPPORTED;
  }
  return TQ_OK;
}

Codebook make_codebook_hi(const tq_params* p) {
  Codebook cb;
  std::memset(&cb, 0, sizeof(cb));
  if (p->d_hi == 0) return cb;
  cb.bits = p->bits_mse_hi;
  const int K = 1 << p->bits_mse_hi;
  for (int k = 0; k < K; ++k) cb.c[k] = p->centroids_hi[k];
  for (int k = 0; k + 1 < K; ++k) cb.t[k] = p->bounds_hi[k];
  return cb;
}

// (the bounds are left out)
Codebook make_codebook_of(int bits, const float* centroids) {
  Codebook cb;
  std::memset(&cb, 0, sizeof(cb));
  cb.bits = bits;
  for (int k = 0; k < 1 << bits; ++k) cb.c[k] = centroids[k];
  return cb;
}

Codebook make_codebook(const tq_params* p) {
  Codebook cb = make_codebook_of(p->bits_mse, p->centroids);
  for (int k = 0; k + 1 < 1 << p->bits_mse; ++k) cb.t[k] = p->bounds[k];
  return cb;
}

float kappa_of(int d) { return (float)(std::sqrt(1.5707963267948966) / (double)d); }

// TQ_FLAG_FP32_MFMA keeps every contraction of the call on the fp32 matrix instructions
bool fp32_mfma_only(const tq_params* p) { return (p->flags & TQ_FLAG_FP32_MFMA) != 0; }

// tq_params.images: [image of the d = 128 quantisation kernel][image of the d = 128 dequantisation kernel]
const void* quant_image(const tq_params* p) { return p->d == 128 ? p->images : nullptr; }
const void* dequant_image(const tq_params* p) {
  return p->d == 128 && p->images != nullptr ? static_cast<const char*>(p->images) + quant128_bf3_image_bytes() : nullptr;
}

bool sign_images(const tq_params* p) {
  constexpr uint32_t both = TQ_FLAG_DEQUANT_IMAGES | TQ_FLAG_SIGN_IMAGES;
  return p->images != nullptr && (p->flags & both) == both;
}

tq_status from_hip(hipError_t e) { return e == hipSuccess ? TQ_OK : TQ_ERR_HIP; }

// Quant_prod of fp32 vectors on the bf16 matrix cores keeps the two leading pieces of x: the rotated vector is off
// by up to 2^-17 |x| in norm (2^-18.6 in the root mean square).  The indices do not notice, but the residual norm
// gamma and the sketch signs of Alg. 2 are judged relative to gamma, which shrinks with the bit-width of the MSE
// stage (sqrt(D_mse) of Theorem 1: 1, 0.60, 0.34, 0.18, 0.097 for 0..4 bits); the error's component along the
// residual is about 2^-18.6 / sqrt(d).  Where that exceeds about 1e-6 gamma the rotation stays on fp32 MFMA
// (d = 128: the 4-bit MSE stage; 3 bits below d = 128; 2 bits at d = 32).
bool two_piece_x_serves_prod(int d, int bits_mse) {
  static const float gamma_typ[5] = {1.f, 0.60f, 0.342f, 0.183f, 0.097f};
  return gamma_typ[bits_mse] * std::sqrt((float)d) >= 2.f;
}

struct Workspace {
  char* base;
  size_t size;
  size_t used;
  void* take(size_t bytes) {
    const size_t off = round_up(used, 256);
    if (base == nullptr || off + bytes > size) return nullptr;
    used = off + bytes;
    return base + off;
  }
};

// params.images at every d other than 128: [Pi][S Pi^T] as two fp16 pieces (4 d^2 bytes each), then the inverse scales of
// the two, each followed by a word that tq_build_images uses.  With TQ_FLAG_DEQUANT_IMAGES behind those (tq_images_bytes)
// [Pi^T][S^T] in the order in which codes are decoded, [S] as it is, and the scales of these.
enum H2Image { IMG_PI = 0, IMG_SPIT = 1, IMG_CODE_PI = 2, IMG_CODE_S = 3, IMG_S = 4 };
const char* h2_images(const tq_params* p) { return p->d != 128 && aligned16(p->images) ? static_cast<const char*>(p->images) : nullptr; }
const char* h2_dequant_images(const tq_params* p) { return (p->flags & TQ_FLAG_DEQUANT_IMAGES) != 0 ? h2_images(p) : nullptr; }
const char* h2_image(const void* images, int d, int which) {
  return static_cast<const char*>(images) + (which >= 2 ? tq_images_bytes(d) : 0) + (which >= 2 ? which - 2 : which) * h2_image_bytes(d, d);
}
float* h2_image_scale(const void* images, int d, int which) {
  const char* const at = which >= 2 ? h2_image(images, d, 5) + 8 * (which - 2) : h2_image(images, d, 0) + 2 * h2_image_bytes(d, d) + 8 * which;
  return reinterpret_cast<float*>(const_cast<char*>(at));
}
// with TQ_FLAG_SIGN_IMAGES behind those, where codes are decoded as signs (tq_sign_gemm.hip): the digits of Pi^T and of S^T
char* sign_gemm_image(const void* images, int d, int which) {
  return const_cast<char*>(h2_image(images, d, 5)) + 256 + which * sign_gemm_image_bytes(d);
}
// without them: the images a call makes for itself in the workspace
size_t h2_own_images_bytes(int d, bool prod) { return kH2ImageHeader + (prod ? 2 : 1) * h2_image_bytes(d, d); }

constexpr int64_t kMatvecQueries = 64;  // up to here queries of any length are rotated by matrix-vector products
// So are short ones up to 65536 values, and at d = 128, where the alternative is gemm_kernel, 1024; with TQ_FLAG_FP32_MFMA these stay on the
// fp32 matrix instructions.  A search of 20000 codes, us, the alternative / this:
//   d = 128   70 queries 54.6 / 43.8, 1000 90.3 / 83.6 (with a sketch 115 / 99)
//   d = 256   70 53.0 / 49.8, 200 57.5 / 55.9, 400 68 / 68
//   d = 384   200 63.7 / 62.8
//   d = 768   70 75.4 / 72.0, 150 81 / 80
//   d = 3072  70 151 / 175
bool rotated_by_products(const tq_params* p, int64_t nq) {
  if (nq <= kMatvecQueries) return true;
  return !fp32_mfma_only(p) && (p->d <= 128 ? nq <= 1024 : nq * p->d <= 65536);
}

// Pi q and S q of many queries on the fp16 matrix cores, from the images of Pi and S or from ones made here.  (The error of
// a rotated coordinate is 0.62 of the fp32 instructions' at every d from 256 to 4096, 4.4e-7 against 7.0e-7 of its size at
// d = 1536; 1000 queries take 29 us against 111 there, 63 against 217 at d = 3072; an image made here 20 and 40.)
struct RotateSpace {
  int64_t rows;                         // queries per pass
  size_t pieces, fac, image[2], total;  // offsets; image: 0 where params.images holds it (then no room is taken)
  RotateSpace(const tq_params* p, int64_t nq, bool prod) {
    const size_t d = (size_t)p->d;
    rows = nq < 16384 ? nq : 16384;
    fac = round_up((size_t)rows * d * 4, 256);
    total = fac + round_up((size_t)rows * 4, 256);
    pieces = 0;  // first
    image[0] = image[1] = 0;
    const bool own[2] = {h2_images(p) == nullptr, prod && h2_dequant_images(p) == nullptr};
    for (int m = 0; m < 2; ++m)
      if (own[m]) {
        image[m] = total + kH2ImageHeader;
        total += kH2ImageHeader + round_up(h2_image_bytes(p->d, p->d), 256);
      }
  }
};

// The quantiser on the fp16 matrix cores: passes of as many vectors as the workspace holds the pieces of.  False when it
// holds too few (nothing has been launched then).
bool quantize_h2(const tq_params* p, const void* x, bool bf16, int64_t n, int64_t ldx, uint32_t* idx, uint32_t* qjl, float* gamma,
                 float* norm, bool prod, hipStream_t stream, tq_status* st) {
  const int d = p->d;
  Workspace ws{static_cast<char*>(p->workspace), p->workspace_bytes, 0};
  const char* pi_img = h2_images(p);
  const bool build = pi_img == nullptr;
  const char* s_img;
  float* w_inv;  // of the second image two floats on
  if (!build) {
    s_img = h2_image(pi_img, d, IMG_SPIT);
    w_inv = h2_image_scale(pi_img, d, IMG_PI);
  } else {  // the same bits as tq_build_images makes
    char* const own = static_cast<char*>(ws.take(h2_own_images_bytes(d, prod)));
    if (own == nullptr) return false;
    w_inv = reinterpret_cast<float*>(own);
    pi_img = own + kH2ImageHeader;
    s_img = pi_img + h2_image_bytes(d, d);
  }
  // per vector: pieces, two factors; with a sketch the residual's pieces and the partial sums of its norm
  const size_t x_bytes = (size_t)d * (bf16 ? 2 : 4);
  const size_t per_row = x_bytes + 8 + (prod ? (size_t)d * 4 + (size_t)((d + 63) / 64) * 4 : 0);
  const size_t room = ws.size > ws.used + 2048 ? ws.size - ws.used - 2048 : 0;  // alignment of the five arrays
  int64_t chunk = (int64_t)(room / per_row);
  if (chunk > kChunkRows) chunk = kChunkRows;
  if (chunk < n) {
    chunk = h2_full_rows(d, chunk);
    if (chunk < 256) return false;
  } else {
    chunk = n;
  }
  void* const xp = ws.take((size_t)chunk * x_bytes);
  float* const fac = static_cast<float*>(ws.take((size_t)chunk * 4));
  float* const esc = static_cast<float*>(ws.take((size_t)chunk * 4));
  void* const ep = prod ? ws.take((size_t)chunk * d * 4) : nullptr;
  float* const part = prod ? static_cast<float*>(ws.take((size_t)chunk * ((d + 63) / 64) * 4)) : nullptr;
  if (xp == nullptr || fac == nullptr || esc == nullptr || (prod && (ep == nullptr || part == nullptr))) return false;

  *st = TQ_ERR_HIP;
  if (build) {
    if (launch_h2_image(p->Pi, d, d, d, const_cast<char*>(pi_img), w_inv, stream) != hipSuccess) return true;
    if (prod && launch_h2_image(p->SPiT, d, d, d, const_cast<char*>(s_img), w_inv + 2, stream) != hipSuccess) return true;
  }
  const size_t esz = bf16 ? 2 : 4;
  const int words_per_row = (d / 32) * p->bits_mse;
  const Codebook cb = make_codebook(p);
  for (int64_t r0 = 0; r0 < n; r0 += chunk) {
    const int64_t rows = n - r0 < chunk ? n - r0 : chunk;
    if (launch_h2_split(static_cast<const char*>(x) + (size_t)r0 * ldx * esz, bf16, true, ldx, rows, d, norm != nullptr, w_inv, xp,
                        norm ? norm + r0 : nullptr, fac, esc, stream) != hipSuccess)
      return true;
    H2Quant a;
    std::memset(&a, 0, sizeof(a));
    a.W = pi_img; a.w_inv = w_inv; a.X = xp; a.npx = bf16 ? 1 : 2; a.d = d; a.n = rows;
    a.fac = fac; a.esc = esc; a.words = idx ? idx + r0 * words_per_row : nullptr; a.E = ep; a.part = part;
    if (launch_h2_quant(p->bits_mse, a, cb, stream) != hipSuccess) return true;
    if (prod) {
      a.W = s_img; a.X = ep; a.npx = 2; a.E = nullptr;
      a.words = qjl + r0 * (d / 32); a.part_tiles = h2_part_tiles(d, rows); a.gamma = gamma + r0;
      if (launch_h2_sign(a, stream) != hipSuccess) return true;
    }
  }
  *st = TQ_OK;
  return true;
}

tq_status quantize_common(const tq_params* p, const void* x, int32_t dtype, int64_t n, int64_t ldx,
                          uint32_t* idx, uint32_t* qjl, float* gamma, float* norm, bool prod,
                          hipStream_t stream, int64_t out_first = 0, int64_t out_step = 1, bool scattered = false) {
  tq_status st = check_params(p, true);
  if (st != TQ_OK) return st;
  if (n < 0 || ldx < p->d) return TQ_ERR_INVALID_ARG;
  if (ldx > kMaxRowStride) return TQ_ERR_UNSUPPORTED;
  if (dtype != TQ_F32 && dtype != TQ_BF16) return TQ_ERR_INVALID_ARG;
  if (n == 0) return TQ_OK;
  if (x == nullptr || p->Pi == nullptr) return TQ_ERR_INVALID_ARG;
  if (p->bits_mse > 0 && idx == nullptr) return TQ_ERR_INVALID_ARG;
  if (prod && (qjl == nullptr || gamma == nullptr || p->SPiT == nullptr)) return TQ_ERR_INVALID_ARG;
  if (ldx % 4 != 0 || !aligned16(p->Pi) || (prod && !aligned16(p->SPiT))) return TQ_ERR_UNSUPPORTED;
  if (dtype == TQ_F32 ? !aligned16(x) : (reinterpret_cast<uintptr_t>(x) & 7u) != 0)
    return TQ_ERR_UNSUPPORTED;

  const int d = p->d;
  const size_t esz = dtype == TQ_F32 ? 4 : 2;
  const int words_per_row = (d / 32) * p->bits_mse;

  const Codebook few_cb = make_codebook(p), few_cb_hi = make_codebook_hi(p);
  const bool few128_takes = d == 128 && dtype == TQ_BF16 && !fp32_mfma_only(p) &&
                            quant128_few_applicable(p->bits_mse, few_cb, p->d_hi != 0 ? &few_cb_hi : nullptr);
  if (scattered) {
    // rows scattered into a larger store (tq_append): the short-chain d = 128 kernel only
    if (d != 128 || n > kSmallQuantRows || !aligned16(x) || (ldx * esz) % 16 != 0) return TQ_ERR_UNSUPPORTED;
    if (p->d_hi != 0 && norm == nullptr) return TQ_ERR_INVALID_ARG;
    if (few128_takes)
      return from_hip(launch_quant128_few(p->bits_mse, prod, x, ldx, n, p->Pi, prod ? p->SPiT : nullptr, idx, qjl, gamma, norm, few_cb,
                                          p->d_hi / 32, few_cb_hi, quant_image(p), stream, out_first, out_step));
    return from_hip(launch_quant128_small(p->bits_mse, prod, dtype == TQ_BF16, x, ldx, n, p->Pi,
                                          prod ? p->SPiT : nullptr, idx, qjl, gamma, norm, make_codebook(p),
                                          p->d_hi / 32, p->d_hi != 0 ? make_codebook_hi(p) : make_codebook(p), stream,
                                          out_first, out_step));
  }

  // head dimension 128, a small batch of bf16 vectors
  auto few128 = [&] {
    return from_hip(launch_quant128_few(p->bits_mse, prod, x, ldx, n, p->Pi, prod ? p->SPiT : nullptr, idx, qjl, gamma, norm, few_cb,
                                        p->d_hi / 32, few_cb_hi, quant_image(p), stream));
  };
  const bool few128_serves = few128_takes && n <= kFewQuantRows && aligned16(x) && ldx % 8 == 0;

  if (p->d_hi != 0) {
    // two instances: the d = 128 kernels; both norms are always stored
    if (norm == nullptr) return TQ_ERR_INVALID_ARG;
    if (!aligned16(x) || (ldx * esz) % 16 != 0) return TQ_ERR_UNSUPPORTED;
    if (few128_serves) return few128();
    const Codebook cb_hi = make_codebook_hi(p);
    if (dtype == TQ_BF16 && n >= kBf3QuantRows && !fp32_mfma_only(p) && (!prod || aligned16(qjl)) &&
        quant128_bf3_applicable(p->bits_mse, prod, false, x, ldx, make_codebook(p), &cb_hi))
      return from_hip(launch_quant128_bf3(p->bits_mse, prod, false, x, ldx, n, p->Pi, prod ? p->SPiT : nullptr, idx, qjl, gamma,
                                          norm, make_codebook(p), p->d_hi / 32, make_codebook_hi(p), quant_image(p), stream));
    return from_hip(launch_quant128(p->bits_mse, prod, dtype == TQ_BF16, x, ldx, n, p->Pi,
                                    prod ? p->SPiT : nullptr, idx, qjl, gamma, norm, make_codebook(p),
                                    p->d_hi / 32, make_codebook_hi(p), stream));
  }

  if (few128_serves) return few128();

  // head dimension 128, a large batch of bf16 or fp32 vectors: the contractions on the 16-bit matrix cores
  if (d == 128 && n >= kBf3QuantRows && !fp32_mfma_only(p) && !(prod && dtype == TQ_F32 && !two_piece_x_serves_prod(d, p->bits_mse)) &&
      quant128_bf3_applicable(p->bits_mse, prod, dtype == TQ_F32, x, ldx, make_codebook(p), nullptr) &&
      (p->bits_mse == 0 || aligned16(idx)) && (!prod || aligned16(qjl)))
    return from_hip(launch_quant128_bf3(p->bits_mse, prod, dtype == TQ_F32, x, ldx, n, p->Pi, prod ? p->SPiT : nullptr, idx, qjl, gamma,
                                        norm, make_codebook(p), 0, make_codebook(p), quant_image(p), stream));

  // head dimension 128, a few fp32 vectors without a sketch: matrix-vector products, all bits here and there (4 bits, us, the kernel
  // below / these: 1 vector 4.8 / 3.3, 256 6.4 / 5.5, 384 6.4 / 6.6).  With a sketch they would need memory for the residual
  // between two launches, the caller's workspace, which at this d is left alone; and they took longer (1 + 1 bits, 5 vectors 7.2 / 8.6).
  if (d == 128 && dtype == TQ_F32 && !prod && n <= 256 && !fp32_mfma_only(p))
    return from_hip(launch_quant_rows(p->bits_mse, false, x, ldx, n, d, p->Pi, make_codebook(p), idx, norm, stream));

  // head dimension 128: one fused kernel, parameters resident in LDS
  if (d == 128 && aligned16(x) && (ldx * esz) % 16 == 0) {
    return from_hip(launch_quant128(p->bits_mse, prod, dtype == TQ_BF16, x, ldx, n, p->Pi,
                                    prod ? p->SPiT : nullptr, idx, qjl, gamma, norm, make_codebook(p), 0,
                                    make_codebook(p), stream));
  }

  GemmArgs a;
  std::memset(&a, 0, sizeof(a));
  a.W1 = p->Pi;
  a.ldw = d;
  a.M = d;
  a.d = d;
  a.segs = 1;
  a.ldx = ldx;
  a.normalise = norm != nullptr;
  a.kappa = kappa_of(d);
  a.cb = make_codebook(p);
  const bool pieces = !fp32_mfma_only(p);
  a.pieces = pieces && !(prod && dtype == TQ_F32 && !two_piece_x_serves_prod(d, p->bits_mse));
  // below d = 512 a large batch is bound by the passes over memory that the fp16 contraction adds (pieces of the vectors and of
  // the residual), and the contraction that splits its vectors on the fly is the faster one (2 + 1 bits, 60000 / 8000 vectors: d = 256
  // 87 against 147 us / 30 against 24; d = 384 169 against 197 / 40 against 32; d = 512 284 against 223).  It also meets all 24 bits of Pi,
  // so it stays where, without a sketch and at 3 and 4 bits, the fp16 contraction would take less time (d = 256, 4 bits, 300000 vectors 277 / 242).
  const bool h2_serves = a.pieces && (d >= 512 || n <= 16384) && h2_codebook_serves(p->bits_mse, a.cb) && (!prod || aligned16(p->SPiT));
  const NKind nk = dtype == TQ_F32 ? N_F32 : N_BF16;

  if (!prod) {
    // a handful of long vectors: a matrix-vector product per vector instead of the tiled contraction's serial k-loop
    if (quant_rows_serves(n, d, false) && !fp32_mfma_only(p))
      return from_hip(launch_quant_rows(p->bits_mse, dtype == TQ_BF16, x, ldx, n, d, p->Pi, make_codebook(p), idx, norm, stream));
    if (h2_serves && quantize_h2(p, x, dtype == TQ_BF16, n, ldx, idx, nullptr, nullptr, norm, false, stream, &st)) return st;
    a.X = x;
    a.n = n;
    a.rownorm_out = norm;
    a.words_out = idx;
    return from_hip(launch_gemm(nk, E_QUANT, p->bits_mse, a, 1, stream));
  }

  // a handful of long vectors: the matrix-vector route (see above), the sketch included, when the workspace holds the residual
  if (quant_rows_serves(n, d, true) && !fp32_mfma_only(p)) {
    Workspace ws2{static_cast<char*>(p->workspace), p->workspace_bytes, 0};
    if (float* const ew = static_cast<float*>(ws2.take((size_t)n * d * sizeof(float))); ew != nullptr)
      return from_hip(launch_quant_rows(p->bits_mse, dtype == TQ_BF16, x, ldx, n, d, p->Pi, make_codebook(p), idx, norm, stream,
                                        p->SPiT, ew, qjl, gamma));
  }

  if (h2_serves && quantize_h2(p, x, dtype == TQ_BF16, n, ldx, idx, qjl, gamma, norm, true, stream, &st)) return st;

  // prod: pass 1 writes idx and the rotated-basis residual e = y - c[idx];
  // pass 2 streams e (its row norms are gamma) against S Pi^T and packs signs.
  Workspace ws{static_cast<char*>(p->workspace), p->workspace_bytes, 0};
  int64_t chunk = n < kChunkRows ? n : kChunkRows;
  float* resid = nullptr;
  while (true) {
    resid = static_cast<float*>(ws.take((size_t)chunk * d * sizeof(float)));
    if (resid != nullptr || chunk <= 128) break;
    ws.used = 0;
    chunk = (chunk / 2 + 127) / 128 * 128;
  }
  if (resid == nullptr) return TQ_ERR_WORKSPACE;

  for (int64_t r0 = 0; r0 < n; r0 += chunk) {
    const int64_t rows = (n - r0 < chunk) ? n - r0 : chunk;
    GemmArgs a1 = a;
    a1.X = static_cast<const char*>(x) + (size_t)r0 * ldx * esz;
    a1.n = rows;
    a1.rownorm_out = norm ? norm + r0 : nullptr;
    a1.words_out = idx ? idx + r0 * words_per_row : nullptr;
    a1.resid_out = resid;
    hipError_t e = launch_gemm(nk, E_QUANT, p->bits_mse, a1, 1, stream);
    if (e != hipSuccess) return TQ_ERR_HIP;

    GemmArgs a2;
    std::memset(&a2, 0, sizeof(a2));
    a2.W1 = p->SPiT;
    a2.ldw = d;
    a2.M = d;
    a2.d = d;
    a2.segs = 1;
    a2.X = resid;
    a2.ldx = d;
    a2.n = rows;
    a2.rownorm_out = gamma + r0;
    a2.words_out = qjl + r0 * (d / 32);
    a2.pieces = pieces;  // the residual's own two pieces leave out 2^-17 of the residual: relative to gamma as it must be
    e = launch_gemm(N_F32, E_SIGN, 0, a2, 1, stream);
    if (e != hipSuccess) return TQ_ERR_HIP;
  }
  return TQ_OK;
}

// The digits of tq_dequantize (tq_sign.h) that calls with these parameters can come to multiply: of no matrix, of Pi, of Pi and S
int digit_matrices(const tq_params* p) {
  SignCoefs c;
  if (p->d_hi != 0 || p->bits_mse < 0 || p->bits_mse > 2 || (p->bits_mse == 0 && p->S == nullptr)) return 0;
  if (p->centroids != nullptr && !sign_table(p->bits_mse, make_codebook_of(p->bits_mse, p->centroids), &c)) return 0;
  return p->S != nullptr ? 2 : 1;
}

// behind tq_images_bytes(d); d = 128: digits alone
size_t dequant_images_bytes(int32_t d, int matrices) {
  if (d <= 0 || d % 32 != 0 || d > 16384) return 0;
  if (d == 128) return matrices * SIGN128_BYTES;
  return 3 * h2_image_bytes(d, d) + 256 + (sign_gemm_images(d) ? matrices * sign_gemm_image_bytes(d) : 0);
}

tq_status build_dequant_images(const tq_params* p, void* images, int matrices, void* stream) {
  if (p == nullptr || p->d <= 0) return TQ_ERR_INVALID_ARG;
  if (dequant_images_bytes(p->d, matrices) == 0) return TQ_OK;
  if (images == nullptr || p->Pi == nullptr) return TQ_ERR_INVALID_ARG;
  if (!aligned16(images)) return TQ_ERR_UNSUPPORTED;
  const hipStream_t s = static_cast<hipStream_t>(stream);
  const int d = p->d;
  if (d == 128) return from_hip(launch_sign128_images(p->Pi, p->S, static_cast<char*>(images) + tq_images_bytes(d), s));
  auto image = [&](int which) { return const_cast<char*>(h2_image(images, d, which)); };
  if (launch_code_image(p->Pi, d, image(IMG_CODE_PI), h2_image_scale(images, d, IMG_CODE_PI), s) != hipSuccess ||
      (p->S != nullptr && launch_code_image(p->S, d, image(IMG_CODE_S), h2_image_scale(images, d, IMG_CODE_S), s) != hipSuccess))
    return TQ_ERR_HIP;
  if (matrices > 0 && sign_gemm_images(d) &&
      (launch_sign_gemm_image(p->Pi, d, sign_gemm_image(images, d, 0), s) != hipSuccess ||
       (p->S != nullptr && launch_sign_gemm_image(p->S, d, sign_gemm_image(images, d, 1), s) != hipSuccess)))
    return TQ_ERR_HIP;
  // (an S that is not 16-byte aligned is refused wherever the last one is used)
  if (p->S != nullptr && aligned16(p->S) && launch_h2_image(p->S, d, d, d, image(IMG_S), h2_image_scale(images, d, IMG_S), s) != hipSuccess)
    return TQ_ERR_HIP;
  return TQ_OK;
}

}  // namespace

extern "C" {

const char* tq_status_string(tq_status s) {
  switch (s) {
    case TQ_OK: return "TQ_OK";
    case TQ_ERR_INVALID_ARG: return "TQ_ERR_INVALID_ARG";
    case TQ_ERR_UNSUPPORTED: return "TQ_ERR_UNSUPPORTED";
    case TQ_ERR_HIP: return "TQ_ERR_HIP";
    case TQ_ERR_WORKSPACE: return "TQ_ERR_WORKSPACE";
    default: return "TQ_ERR_UNKNOWN";
  }
}

size_t tq_images_bytes(int32_t d) {
  if (d == 128) return quant128_bf3_image_bytes() + dequant128_bf3_image_bytes();
  if (d <= 0 || d % 32 != 0 || d > 16384) return 0;
  return (size_t)d * d * 10;  // Pi and S Pi^T as two fp16 pieces each, and their scales
}

tq_status tq_build_images(const tq_params* p, void* images, void* stream) {
  if (p == nullptr || p->d <= 0) return TQ_ERR_INVALID_ARG;
  if (tq_images_bytes(p->d) == 0) return TQ_OK;  // no kernel at this d takes one
  if (images == nullptr || p->Pi == nullptr) return TQ_ERR_INVALID_ARG;
  if (p->d != 128) {
    // the generic quantiser: Pi, and S Pi^T when there is a sketch
    if ((p->S == nullptr) != (p->SPiT == nullptr)) return TQ_ERR_INVALID_ARG;
    if (!aligned16(images) || !aligned16(p->Pi) || (p->SPiT != nullptr && !aligned16(p->SPiT))) return TQ_ERR_UNSUPPORTED;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int d = p->d;
    if (launch_h2_image(p->Pi, d, d, d, images, h2_image_scale(images, d, IMG_PI), s) != hipSuccess) return TQ_ERR_HIP;
    if (p->SPiT != nullptr &&
        launch_h2_image(p->SPiT, d, d, d, const_cast<char*>(h2_image(images, d, IMG_SPIT)), h2_image_scale(images, d, IMG_SPIT), s) != hipSuccess)
      return TQ_ERR_HIP;
    return TQ_OK;
  }
  if (p->PiT == nullptr) return TQ_ERR_INVALID_ARG;
  if ((p->S == nullptr) != (p->ST == nullptr) || (p->S == nullptr) != (p->SPiT == nullptr)) return TQ_ERR_INVALID_ARG;
  if (!aligned16(images) || !aligned16(p->Pi) || !aligned16(p->PiT) || (p->S != nullptr && (!aligned16(p->ST) || !aligned16(p->SPiT))))
    return TQ_ERR_UNSUPPORTED;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (launch_quant128_bf3_image(p->Pi, p->SPiT, images, s) != hipSuccess) return TQ_ERR_HIP;
  if (launch_dequant128_bf3_image(p->PiT, p->ST, static_cast<char*>(images) + quant128_bf3_image_bytes(), s) != hipSuccess)
    return TQ_ERR_HIP;
  return TQ_OK;
}

size_t tq_dequant_images_bytes(int32_t d) { return dequant_images_bytes(d, 2); }
size_t tq_dequant_images_bytes_for(const tq_params* p) { return p == nullptr ? 0 : dequant_images_bytes(p->d, digit_matrices(p)); }

tq_status tq_build_dequant_images(const tq_params* p, void* images, void* stream) { return build_dequant_images(p, images, 2, stream); }
tq_status tq_build_dequant_images_for(const tq_params* p, void* images, void* stream) {
  return build_dequant_images(p, images, p == nullptr ? 0 : digit_matrices(p), stream);
}

tq_status tq_derive_params(int32_t d, const float* Pi, const float* S, float* PiT, float* ST,
                           float* SPiT, void* stream) {
  if (d <= 0 || Pi == nullptr) return TQ_ERR_INVALID_ARG;
  if (d % 32 != 0 || d > 16384) return TQ_ERR_UNSUPPORTED;
  if ((ST != nullptr || SPiT != nullptr) && S == nullptr) return TQ_ERR_INVALID_ARG;
  if (!aligned16(Pi) || (S && !aligned16(S)) || (SPiT && !aligned16(SPiT))) return TQ_ERR_UNSUPPORTED;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (PiT != nullptr && launch_transpose(d, Pi, PiT, s) != hipSuccess) return TQ_ERR_HIP;
  if (ST != nullptr && launch_transpose(d, S, ST, s) != hipSuccess) return TQ_ERR_HIP;
  if (SPiT != nullptr) {
    // row m of S Pi^T is Pi applied to row m of S: the rotate contraction with
    // the rows of S as the vectors, stored plainly
    GemmArgs a;
    std::memset(&a, 0, sizeof(a));
    a.W1 = Pi;
    a.ldw = d;
    a.M = d;
    a.d = d;
    a.segs = 1;
    a.X = S;
    a.ldx = d;
    a.n = d;
    a.out = SPiT;
    a.ldo = d;
    if (launch_gemm(N_F32, E_STORE_T, 0, a, 1, s) != hipSuccess) return TQ_ERR_HIP;
  }
  return TQ_OK;
}

size_t tq_workspace_bytes(const tq_params* p, int64_t n, int64_t nq, int32_t topk) {
  if (p == nullptr || p->d <= 0 || n < 0 || nq < 0) return 0;
  const size_t d = (size_t)p->d;
  const size_t rows = (size_t)(n < kChunkRows / 2 ? n : kChunkRows / 2);
  // the quantiser's pieces of the vectors and of the residual, two factors and the partial residual norms per vector (a handful of
  // long vectors instead keeps the fp32 residual alone)
  size_t bytes = round_up(rows * (2 * d * sizeof(float) + 8 + (d + 63) / 64 * 4), 256) + 4096;
  if (n > 0 && p->images == nullptr) bytes += round_up(h2_own_images_bytes(p->d, p->S != nullptr), 256);
  bytes += 2 * round_up((size_t)nq * d * sizeof(float), 256);      // rotated / sketched queries
  bytes += round_up(score_i8_workspace_bytes(p->d, nq), 256);      // or their digit images
  if (topk > 0) bytes += round_up((size_t)nq * (size_t)(n + 3) * sizeof(float), 256);  // scores when not returned
  // partial top-k lists of a few long rows: at most 4096 (score, index) pairs for each of at most 128 rows
  if (topk > 0) bytes += 2 * round_up((size_t)(nq < 128 ? nq : 128) * 4096 * sizeof(float), 256);
  // candidates of a search by many queries, and their rotation
  if (topk > 0 && nq > 0 && n > 0) bytes += search_workspace_bytes(p->d, n, nq, topk) + 256;
  if (!rotated_by_products(p, nq) && p->d != 128) bytes += RotateSpace(p, nq, p->S != nullptr).total + 256;
  return bytes + 256;
}

tq_status tq_quantize_mse(const tq_params* p, const void* x, int32_t dtype, int64_t n, int64_t ldx,
                          uint32_t* idx, float* norm, void* stream) {
  return quantize_common(p, x, dtype, n, ldx, idx, nullptr, nullptr, norm, false,
                         static_cast<hipStream_t>(stream));
}

tq_status tq_quantize_prod(const tq_params* p, const void* x, int32_t dtype, int64_t n, int64_t ldx,
                           uint32_t* idx, uint32_t* qjl, float* gamma, float* norm, void* stream) {
  return quantize_common(p, x, dtype, n, ldx, idx, qjl, gamma, norm, true,
                         static_cast<hipStream_t>(stream));
}

tq_status tq_append(const tq_params* p, const void* x, int32_t dtype, int64_t n, int64_t ldx, uint32_t* idx,
                    uint32_t* qjl, float* gamma, float* norm, int64_t first_row, int64_t row_step, void* stream) {
  if (first_row < 0 || row_step < 1) return TQ_ERR_INVALID_ARG;
  if (p != nullptr && p->d != 128) return TQ_ERR_UNSUPPORTED;
  if (n > kSmallQuantRows) return TQ_ERR_UNSUPPORTED;
  return quantize_common(p, x, dtype, n, ldx, idx, qjl, gamma, norm, qjl != nullptr, static_cast<hipStream_t>(stream),
                         first_row, row_step, true);
}

tq_status tq_dequantize(const tq_params* p, const uint32_t* idx, const uint32_t* qjl,
                        const float* gamma, const float* norm, int64_t n, float* x_out, int64_t ldo,
                        void* stream) {
  tq_status st = check_params(p, true);
  if (st != TQ_OK) return st;
  if (n < 0 || ldo < p->d) return TQ_ERR_INVALID_ARG;
  if (ldo > kMaxRowStride) return TQ_ERR_UNSUPPORTED;
  if (n == 0) return TQ_OK;
  const bool prod = qjl != nullptr;
  if (x_out == nullptr || p->PiT == nullptr || (p->bits_mse > 0 && idx == nullptr)) return TQ_ERR_INVALID_ARG;
  if (prod && (gamma == nullptr || p->ST == nullptr)) return TQ_ERR_INVALID_ARG;
  if (ldo % 4 != 0 || !aligned16(x_out) || !aligned16(p->PiT) || (prod && !aligned16(p->ST)))
    return TQ_ERR_UNSUPPORTED;
  if (p->d_hi != 0) {
    // two instances: d = 128 kernel only; idx rows are not 16-byte multiples there
    if (norm == nullptr || idx == nullptr || p->Pi == nullptr || (prod && p->S == nullptr)) return TQ_ERR_INVALID_ARG;
    if (!aligned16(p->Pi) || (prod && (!aligned16(p->S) || !aligned16(qjl)))) return TQ_ERR_UNSUPPORTED;
    if (n > kBf3DequantRows && !fp32_mfma_only(p) && p->PiT != nullptr && (!prod || p->ST != nullptr))
      return from_hip(launch_dequant128_bf3(p->bits_mse, prod, idx, qjl, gamma, norm, p->PiT, p->ST, x_out, ldo, n,
                                            kappa_of(p->d - p->d_hi), make_codebook(p), p->d_hi / 32, kappa_of(p->d_hi),
                                            make_codebook_hi(p), dequant_image(p), static_cast<hipStream_t>(stream)));
    return from_hip(launch_dequant128(p->bits_mse, prod, idx, qjl, gamma, norm, p->Pi, p->S, x_out, ldo, n,
                                      kappa_of(p->d - p->d_hi), make_codebook(p), p->d_hi / 32,
                                      kappa_of(p->d_hi), make_codebook_hi(p), static_cast<hipStream_t>(stream)));
  }
  // d = 128, a table that is a sum of signs: digits of Pi^T and S^T from the images, or, for few codes, made by every workgroup for
  // itself, which takes 1.2 us a matrix and no memory (us, 3 bits in all / 2 without a sketch, kernels below -> made here -> from images: 8 codes
  // 8.3 / 5.9 -> 7.2 / 4.6 -> 3.4 / 3.3, 512 9.2 / 6.8 -> 7.3 / 4.8 -> 3.3 / 3.3, 16384 11.0 / 8.2 -> 9.6 / 6.7 -> 5.9 / 4.1, 24576 11.2 / 8.3 -> 10.2 / 7.2 (1 bit
  // without a sketch: 6.9 -> 7.0); above, more workgroups would make them, and made once in a launch of their own they need memory:
  // 65536 14.1 / 11.1 that way 15.2 / 13.9, from images 11.3 / 9.0)
  SignCoefs sc;
  if (p->d == 128 && !fp32_mfma_only(p) && (p->bits_mse > 0 || prod) && sign_table(p->bits_mse, make_codebook(p), &sc)) {
    const hipStream_t s = static_cast<hipStream_t>(stream);
    const char* digits = sign_images(p) && aligned16(p->images) && (!prod || p->S != nullptr) ? static_cast<const char*>(p->images) + tq_images_bytes(128) : nullptr;
    const bool own = p->images == nullptr && n <= kSignOwnDigitRows && p->Pi != nullptr && (!prod || p->S != nullptr);
    if (digits != nullptr || own)
      return from_hip(launch_sign128_dequant(p->bits_mse, prod, idx, qjl, gamma, norm, digits, p->Pi, p->S, x_out, ldo, n, kappa_of(128), sc, s));
  }
  const bool few_rows = !fp32_mfma_only(p) && dequant_rows_serves(n, p->d);
  auto by_rows = [&] {
    return from_hip(launch_dequant_rows(p->bits_mse, prod, p->d, n, idx, qjl, gamma, norm, p->PiT, p->ST, make_codebook(p), kappa_of(p->d), x_out, ldo,
                                        static_cast<hipStream_t>(stream)));
  };
  if (p->d == 128 && few_rows) return by_rows();
  // large batches at d = 128: decoded codes straight into bf16 MFMA operands, pieces of Pi^T / S^T in LDS
  if (p->d == 128 && n > kBf3DequantRows && !fp32_mfma_only(p) && dequant128_bf3_applicable(p->bits_mse, prod, make_codebook(p), x_out, ldo))
    return from_hip(launch_dequant128_bf3(p->bits_mse, prod, idx, qjl, gamma, norm, p->PiT, p->ST, x_out, ldo, n,
                                          kappa_of(128), make_codebook(p), 0, 0.f, make_codebook(p), dequant_image(p),
                                          static_cast<hipStream_t>(stream)));
  if (p->d == 128 && p->Pi != nullptr && aligned16(p->Pi) && (!prod || (p->S != nullptr && aligned16(p->S))) &&
      aligned16(idx) && (!prod || aligned16(qjl))) {
    return from_hip(launch_dequant128(p->bits_mse, prod, idx, qjl, gamma, norm, p->Pi, p->S, x_out, ldo, n,
                                      kappa_of(p->d), make_codebook(p), 0, 0.f, make_codebook(p),
                                      static_cast<hipStream_t>(stream)));
  }
  // a few codes by matrix-vector products in fp32 (see rows_before_digits)
  const bool by_digits = !fp32_mfma_only(p) && sign_gemm_serves(p->bits_mse, prod, p->d, n) && (p->bits_mse > 0 || prod) && p->Pi != nullptr &&
                         (!prod || p->S != nullptr) && sign_table(p->bits_mse, make_codebook(p), &sc);
  const bool digits_at_hand = h2_dequant_images(p) != nullptr && sign_images(p);
  if (by_digits ? rows_before_digits(n, p->d, p->bits_mse, prod, digits_at_hand) : few_rows) return by_rows();
  // many codes of a table that is a sum of signs: digits of Pi^T and S^T, from the images or made here where the workspace holds them
  if (by_digits) {
    const hipStream_t s = static_cast<hipStream_t>(stream);
    const int d = p->d;
    const char *pi = nullptr, *si = nullptr;
    if (const char* const img = h2_dequant_images(p); img != nullptr) {
      if (sign_images(p)) pi = sign_gemm_image(img, d, 0), si = sign_gemm_image(img, d, 1);
    } else {
      Workspace ws{static_cast<char*>(p->workspace), p->workspace_bytes, 0};
      if (char* const own = static_cast<char*>(ws.take((prod ? 2 : 1) * sign_gemm_image_bytes(d))); own != nullptr) {
        pi = own, si = own + sign_gemm_image_bytes(d);
        if (launch_sign_gemm_image(p->Pi, d, own, s) != hipSuccess ||
            (prod && launch_sign_gemm_image(p->S, d, own + sign_gemm_image_bytes(d), s) != hipSuccess))
          return TQ_ERR_HIP;
      }
    }
    if (pi != nullptr)
      return from_hip(launch_sign_gemm(p->bits_mse, prod, pi, si, d, idx, qjl, gamma, norm, n, x_out, ldo, kappa_of(d), sc, s));
  }
  // many codes: fp16 pieces of Pi^T and S^T, from the images or made here where the workspace holds them
  if (!fp32_mfma_only(p) && code_gemm_serves(p->bits_mse, make_codebook(p)) && (p->bits_mse > 0 || prod) && p->Pi != nullptr && (!prod || p->S != nullptr)) {
    const hipStream_t s = static_cast<hipStream_t>(stream);
    const int d = p->d;
    const char *pit = nullptr, *sit = nullptr;
    float *pit_inv = nullptr, *sit_inv = nullptr;
    if (const char* const img = h2_dequant_images(p); img != nullptr) {
      pit = h2_image(img, d, IMG_CODE_PI), sit = h2_image(img, d, IMG_CODE_S);
      pit_inv = h2_image_scale(img, d, IMG_CODE_PI), sit_inv = h2_image_scale(img, d, IMG_CODE_S);
    } else {
      Workspace ws{static_cast<char*>(p->workspace), p->workspace_bytes, 0};
      if (char* const own = static_cast<char*>(ws.take(h2_own_images_bytes(d, prod))); own != nullptr) {
        pit = own + kH2ImageHeader, sit = h2_image(pit, d, 1);
        pit_inv = reinterpret_cast<float*>(own), sit_inv = pit_inv + 2;
        if (launch_code_image(p->Pi, d, const_cast<char*>(pit), pit_inv, s) != hipSuccess ||
            (prod && launch_code_image(p->S, d, const_cast<char*>(sit), sit_inv, s) != hipSuccess))
          return TQ_ERR_HIP;
      }
    }
    if (pit != nullptr)
      return from_hip(launch_code_dequant(p->bits_mse, prod, pit, pit_inv, sit, sit_inv, d, idx, qjl, gamma, norm, n, x_out, ldo,
                                          kappa_of(d), make_codebook(p), s));
  }
  // x~_i[k] = <e_k, DeQuant(code i)>: the scoring contraction with the rows of Pi^T (and S^T) as the queries,
  // stored one row per code; on the bf16 matrix cores where that kernel takes the codes
  if (!fp32_mfma_only(p) && score_bf3_applicable(p->bits_mse, prod, p->d, n, 1, p->d, make_codebook(p)))
    return from_hip(launch_score_bf3(p->bits_mse, prod, p->PiT, p->ST, p->d, p->d, idx, qjl, gamma, norm, n, 1, x_out, ldo,
                                     true, kappa_of(p->d), make_codebook(p), static_cast<hipStream_t>(stream)));
  GemmArgs a;
  std::memset(&a, 0, sizeof(a));
  a.W1 = p->PiT;  // x~[k] = sum_j Pi[j][k] y~[j]: rows of Pi^T against the decoded code
  a.W2 = p->ST;
  a.ldw = p->d;
  a.M = p->d;
  a.d = p->d;
  a.segs = prod ? 2 : 1;
  a.n = n;
  a.idx = idx;
  a.qjl = qjl;
  a.gamma = gamma;
  a.scale_in = norm;
  a.out = x_out;
  a.ldo = ldo;
  a.kappa = kappa_of(p->d);
  a.cb = make_codebook(p);
  return from_hip(launch_gemm(N_CODE, E_STORE_T, p->bits_mse, a, 1, static_cast<hipStream_t>(stream)));
}

}  // extern "C"

namespace {

bool rotate_h2(const tq_params* p, const float* q, int64_t ldq, int64_t nq, float* qr, float* qs, void* scratch, hipStream_t s) {
  const int d = p->d;
  const RotateSpace sp(p, nq, qs != nullptr);
  char* const base = static_cast<char*>(scratch);
  float* const fac = reinterpret_cast<float*>(base + sp.fac);
  for (int m = 0; m < (qs != nullptr ? 2 : 1); ++m) {
    const char* image;
    float* w_inv;
    if (sp.image[m] == 0) {
      image = h2_image(h2_images(p), d, m == 0 ? IMG_PI : IMG_S);
      w_inv = h2_image_scale(h2_images(p), d, m == 0 ? IMG_PI : IMG_S);
    } else {
      image = base + sp.image[m];
      w_inv = reinterpret_cast<float*>(base + sp.image[m] - kH2ImageHeader);
      if (launch_h2_image(m == 0 ? p->Pi : p->S, d, d, d, base + sp.image[m], w_inv, s) != hipSuccess) return false;
    }
    for (int64_t r0 = 0; r0 < nq; r0 += sp.rows) {
      const int64_t rows = nq - r0 < sp.rows ? nq - r0 : sp.rows;
      if (launch_h2_split(q + r0 * ldq, false, false, ldq, rows, d, false, w_inv, base + sp.pieces, nullptr, fac, nullptr, s) != hipSuccess) return false;
      H2Quant a;
      std::memset(&a, 0, sizeof(a));
      a.W = image; a.w_inv = w_inv; a.X = base + sp.pieces; a.npx = 2; a.d = d; a.n = rows; a.fac = fac; a.out = (m == 0 ? qr : qs) + r0 * d;
      if (launch_h2_store(a, s) != hipSuccess) return false;
    }
  }
  return true;
}

// How one tq_score call is carried out and what scratch memory it takes.  tq_score follows it and
// tq_score_workspace_bytes reports it, so the two cannot drift apart.
struct ScorePlan {
  enum Route { R_SPLIT_I8, R_I8, R_SMALL, R_BF3, R_GEMM } route;
  size_t img_bytes;     // digit images of the rotated queries (R_SPLIT_I8, R_I8)
  size_t q_bytes;       // one [nq][d] fp32 matrix of rotated queries (other routes; a second one for prod)
  int64_t ld_scores;    // row stride of a score matrix in scratch memory
  size_t scores_bytes;  // that matrix: only when scores == NULL and top-k is not taken inside the scoring kernel
  int ranges;           // > 0: top-k inside the scoring kernel, this many partial lists per query
  int topk_chunks;      // > 0: top-k over a score matrix of few long rows, this many chunks (partial lists) per row
  size_t part_bytes;    // one array [nq][ranges or topk_chunks][topk] (values; indices take the same again)
  bool prod;
  size_t search_bytes;  // top-k of many queries by candidates (tq_search.hip); without room for it every score is looked at
  size_t rotate_bytes;  // many queries rotated on the fp16 matrix cores; without room for it on the fp32 ones
  size_t total() const { return needed() + (ranges > 0 ? 0 : lists()) + round_up(search_bytes, 256) + round_up(rotate_bytes, 256); }
  // what the call cannot do without: the lists of a top-k over a score matrix are left out where there is no room (one workgroup per row then)
  size_t needed() const {
    const size_t a = 256;
    size_t t = round_up(img_bytes, a) + (q_bytes ? round_up(q_bytes, a) * (prod ? 2 : 1) : 0) + round_up(scores_bytes, a) + (ranges > 0 ? lists() : 0);
    return t + a;
  }
  size_t lists() const { return 2 * round_up(part_bytes, 256); }
};

ScorePlan plan_route(const tq_params* p, bool prod, int n_groups, int q_per_group, int64_t n_per_group, bool scores_given,
                     int topk, bool codes_aligned);

ScorePlan plan_score(const tq_params* p, bool prod, int n_groups, int q_per_group, int64_t n_per_group, bool scores_given,
                     int topk, bool codes_aligned) {
  ScorePlan pl = plan_route(p, prod, n_groups, q_per_group, n_per_group, scores_given, topk, codes_aligned);
  // top-k over a score matrix: a few long rows are cut into chunks so that the selection fills the chip
  if (topk > 0 && pl.ranges == 0) {
    const int64_t nq = (int64_t)n_groups * q_per_group;
    pl.topk_chunks = topk_chunks(nq, n_per_group, topk);
    if (pl.topk_chunks > 0) pl.part_bytes = (size_t)nq * pl.topk_chunks * topk * sizeof(float);
  }
  const int64_t nq = (int64_t)n_groups * q_per_group;
  if (pl.route == ScorePlan::R_BF3 && topk > 0 && !scores_given && n_groups == 1 &&
      search_applicable(p->bits_mse, prod, p->d, n_per_group, q_per_group, topk, make_codebook(p)))
    pl.search_bytes = search_workspace_bytes(p->d, n_per_group, nq, topk);
  if (pl.q_bytes > 0 && !rotated_by_products(p, nq) && p->d != 128 && !fp32_mfma_only(p)) pl.rotate_bytes = RotateSpace(p, nq, prod).total;
  return pl;
}

ScorePlan plan_route(const tq_params* p, bool prod, int n_groups, int q_per_group, int64_t n_per_group, bool scores_given,
                     int topk, bool codes_aligned) {
  ScorePlan pl;
  std::memset(&pl, 0, sizeof(pl));
  pl.prod = prod;
  const int d = p->d;
  const int64_t nq = (int64_t)n_groups * q_per_group;
  pl.ld_scores = (n_per_group + 3) / 4 * 4;
  const size_t scratch_scores = scores_given ? 0 : (size_t)nq * pl.ld_scores * sizeof(float);
  if (p->d_hi != 0) {
    pl.route = ScorePlan::R_SPLIT_I8;
    pl.img_bytes = score_i8_workspace_bytes(d, nq);
    pl.scores_bytes = scratch_scores;
    return pl;
  }
  // few queries per code; with a short code list also a few more (every block of 4 queries re-reads the
  // codes, which costs less than the launches of the contraction path while the list is short)
  // (beyond 512 coordinates up to 16 queries per group, where the dense contraction would run on tiles that are mostly
  // padding; up to 32 at d <= 1024, where the alternative is the lane-per-key kernel: 2.1-3.2 ms for 17-32 queries at
  // d = 1024 and 10^6 codes)
  if ((d <= 512 ? (q_per_group <= 32 || (q_per_group <= 64 && n_per_group <= 16384))
                : ((q_per_group <= 16 || (q_per_group <= 32 && d <= 1024)) && nq <= 64)) &&
      score_i8_applicable(p->bits_mse, d, make_codebook(p))) {
    pl.route = ScorePlan::R_I8;
    pl.img_bytes = score_i8_workspace_bytes(d, nq);
    pl.scores_bytes = scratch_scores;
    return pl;
  }
  pl.q_bytes = (size_t)nq * d * sizeof(float);
  if (q_per_group <= 32 && d % 128 == 0 && d <= 1024 && codes_aligned) {
    pl.route = ScorePlan::R_SMALL;
    pl.scores_bytes = scratch_scores;
    return pl;
  }
  if (n_per_group > 0 && !fp32_mfma_only(p) &&
      score_bf3_applicable(p->bits_mse, prod, d, n_per_group, n_groups, q_per_group, make_codebook(p))) {
    pl.route = ScorePlan::R_BF3;
    pl.ranges = topk > 0 ? score_bf3_topk_ranges(p->bits_mse, prod, n_per_group, n_groups, q_per_group, topk) : 0;
    if (pl.ranges > 0)
      pl.part_bytes = (size_t)nq * pl.ranges * topk * sizeof(float);
    else
      pl.scores_bytes = scratch_scores;
    return pl;
  }
  pl.route = ScorePlan::R_GEMM;
  pl.scores_bytes = scratch_scores;
  return pl;
}

// tq_score with the scratch memory given explicitly (the caller's workspace, or this library's static array)
tq_status score_impl(const tq_params* p, Workspace ws, const float* q, int64_t ldq, int32_t n_groups,
                     int32_t q_per_group, const uint32_t* idx, const uint32_t* qjl, const float* gamma,
                     const float* norm, int64_t n_per_group, float* scores, int64_t lds, int32_t topk,
                     int32_t* topk_idx, float* topk_val, void* stream) {
  tq_status st = check_params(p, true);
  if (st != TQ_OK) return st;
  if (n_groups < 0 || q_per_group < 0 || n_per_group < 0 || ldq < p->d || topk < 0) return TQ_ERR_INVALID_ARG;
  // groups and blocks of four queries are grid dimensions of the few-query kernels
  if (topk > 64 || n_per_group > 0x7fffffff || n_groups > 65535 || q_per_group > 4 * 65535 || ldq > kMaxRowStride)
    return TQ_ERR_UNSUPPORTED;
  const int64_t nq = (int64_t)n_groups * q_per_group;
  if (nq == 0) return TQ_OK;
  const bool prod = qjl != nullptr;
  if (q == nullptr || p->Pi == nullptr) return TQ_ERR_INVALID_ARG;
  if (n_per_group > 0 && p->bits_mse > 0 && idx == nullptr) return TQ_ERR_INVALID_ARG;
  if (prod && (gamma == nullptr || p->S == nullptr)) return TQ_ERR_INVALID_ARG;
  if (scores == nullptr && topk == 0) return TQ_ERR_INVALID_ARG;
  if (scores != nullptr && lds < n_per_group) return TQ_ERR_INVALID_ARG;
  if (topk > 0 && topk_idx == nullptr) return TQ_ERR_INVALID_ARG;
  if (ldq % 4 != 0 || !aligned16(q) || !aligned16(p->Pi) || (prod && !aligned16(p->S))) return TQ_ERR_UNSUPPORTED;
  if (p->d_hi != 0) {
    // two instances over a split of the coordinates: d = 128, the kernel written for few queries per code (every
    // block of four queries streams the group's codes once more, so many queries are served, not served fast)
    if (norm == nullptr) return TQ_ERR_INVALID_ARG;
    if (q_per_group > 4096 || !score_i8_split_applicable(p->bits_mse, make_codebook(p), make_codebook_hi(p)))
      return TQ_ERR_UNSUPPORTED;
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int d = p->d;
  const ScorePlan pl = plan_score(p, prod, n_groups, q_per_group, n_per_group, scores != nullptr, topk,
                                  aligned16(idx) && (!prod || aligned16(qjl)));

  // the scratch memory that the call cannot do without is taken before the first launch
  void* img = pl.img_bytes ? ws.take(pl.img_bytes) : nullptr;
  float* qr = pl.q_bytes ? static_cast<float*>(ws.take(pl.q_bytes)) : nullptr;
  float* qs = pl.q_bytes && prod ? static_cast<float*>(ws.take(pl.q_bytes)) : nullptr;
  int64_t ld_scores = lds;
  if (scores == nullptr && pl.scores_bytes) {
    ld_scores = pl.ld_scores;
    scores = static_cast<float*>(ws.take(pl.scores_bytes));
    if (scores == nullptr) return TQ_ERR_WORKSPACE;
  }
  auto take_lists = [&](float*& val, int32_t*& idx_of) {
    val = pl.part_bytes ? static_cast<float*>(ws.take(pl.part_bytes)) : nullptr;
    idx_of = pl.part_bytes ? static_cast<int32_t*>(ws.take(pl.part_bytes)) : nullptr;
    return val != nullptr && idx_of != nullptr;
  };
  float* part_val = nullptr;
  int32_t* part_idx = nullptr;
  if (pl.ranges > 0 && !take_lists(part_val, part_idx)) return TQ_ERR_WORKSPACE;
  if ((pl.img_bytes && img == nullptr) || (pl.q_bytes && (qr == nullptr || (prod && qs == nullptr)))) return TQ_ERR_WORKSPACE;

  if (pl.route == ScorePlan::R_SPLIT_I8) {
    if (launch_score_i8_split(p->bits_mse, prod, p->Pi, p->S, p->PiT, p->ST, q, ldq, img, idx, qjl, gamma, norm, scores, ld_scores,
                              n_per_group, n_groups, q_per_group, p->d_hi / 32, kappa_of(d - p->d_hi),
                              kappa_of(p->d_hi), make_codebook(p), make_codebook_hi(p), s) != hipSuccess)
      return TQ_ERR_HIP;
  } else if (pl.route == ScorePlan::R_I8) {
    // masked sums of fixed-point query digits on the scaled-format matrix instruction (at d = 128 one kernel; otherwise a
    // preparation kernel rotates the queries and writes their digits)
    if (launch_score_i8(p->bits_mse, prod, p->Pi, p->S, p->PiT, p->ST, q, ldq, img, idx, qjl, gamma, norm, scores, ld_scores,
                        n_per_group, d, n_groups, q_per_group, kappa_of(d), make_codebook(p), s) != hipSuccess)
      return TQ_ERR_HIP;
  } else {
    // queries into the rotated basis and the sketch basis: Pi q and S q
    void* const rot = pl.rotate_bytes > 0 ? ws.take(pl.rotate_bytes) : nullptr;
    if (rot != nullptr) {
      if (!rotate_h2(p, q, ldq, nq, qr, qs, rot, s)) return TQ_ERR_HIP;
    } else if (rotated_by_products(p, nq) && d <= 4096) {
      if (launch_matvec_rows(d, nq, p->Pi, prod ? p->S : nullptr, q, ldq, qr, qs, d, false, s) != hipSuccess)
        return TQ_ERR_HIP;
    } else {
      GemmArgs a;
      std::memset(&a, 0, sizeof(a));
      a.W1 = p->Pi;
      a.ldw = d;
      a.M = d;
      a.d = d;
      a.segs = 1;
      a.X = q;
      a.ldx = ldq;
      a.n = nq;
      a.out = qr;
      a.ldo = d;
      if (launch_gemm(N_F32, E_STORE_T, 0, a, 1, s) != hipSuccess) return TQ_ERR_HIP;
      if (prod) {
        a.W1 = p->S;
        a.out = qs;
        if (launch_gemm(N_F32, E_STORE_T, 0, a, 1, s) != hipSuccess) return TQ_ERR_HIP;
      }
    }
    if (n_per_group > 0 && pl.route == ScorePlan::R_SMALL) {
      // few queries per code: stream the codes once, lane = key
      if (launch_score_small(p->bits_mse, prod, qr, qs, idx, qjl, gamma, norm, scores, ld_scores, n_per_group,
                             d, n_groups, q_per_group, kappa_of(d), make_codebook(p), s) != hipSuccess)
        return TQ_ERR_HIP;
    } else if (pl.route == ScorePlan::R_BF3) {
      // top-k alone: candidates from one piece of every factor, scored again; what follows then only serves the queries
      // whose candidates were too many
      const int32_t* flags = nullptr;
      if (void* const space = pl.search_bytes > 0 ? ws.take(pl.search_bytes) : nullptr; space != nullptr) {
        SearchArgs sa;
        sa.bits = p->bits_mse; sa.prod = prod; sa.nq = (int)nq; sa.d = d; sa.topk = topk; sa.qr = qr; sa.qs = qs; sa.idx = idx; sa.qjl = qjl;
        sa.gamma = gamma; sa.norm = norm; sa.n = n_per_group; sa.kappa = kappa_of(d); sa.topk_idx = topk_idx; sa.topk_val = topk_val;
        if (launch_search(sa, make_codebook(p), space, &flags, s) != hipSuccess) return TQ_ERR_HIP;
      }
      // many queries per code: dense contraction on the bf16 matrix cores, every fp32 factor as two bf16 pieces;
      // with top-k wanted the kernel keeps the k best pairs of every query itself and a small kernel joins them
      if (launch_score_bf3(p->bits_mse, prod, qr, qs, q_per_group, d, idx, qjl, gamma, norm, n_per_group, n_groups, scores,
                           ld_scores, false, kappa_of(d), make_codebook(p), s, pl.ranges > 0 ? topk : 0, part_val,
                           part_idx, flags) != hipSuccess)
        return TQ_ERR_HIP;
      if (pl.ranges > 0)
        return from_hip(launch_topk_merge(part_val, part_idx, nq, pl.ranges, topk, topk_idx, topk_val, s, flags));
      if (flags != nullptr) return from_hip(launch_topk(scores, nq, n_per_group, ld_scores, topk, topk_idx, topk_val, s, 0, nullptr, nullptr, flags));
    } else if (n_per_group > 0) {
      GemmArgs a;
      std::memset(&a, 0, sizeof(a));
      a.W1 = qr;
      a.W2 = qs;
      a.ldw = d;
      a.w_group_stride = (int64_t)q_per_group * d;
      a.M = q_per_group;
      a.d = d;
      a.segs = prod ? 2 : 1;
      a.n = n_per_group;
      a.idx = idx;
      a.qjl = qjl;
      a.gamma = gamma;
      a.scale_in = norm;
      a.out = scores;
      a.ldo = ld_scores;
      a.out_group_stride = (int64_t)q_per_group * ld_scores;
      a.kappa = kappa_of(d);
      a.cb = make_codebook(p);
      if (launch_gemm(N_CODE, E_STORE_N, p->bits_mse, a, n_groups, s) != hipSuccess) return TQ_ERR_HIP;
    }
  }
  // the chunks of a top-k over a score matrix are an optimisation: without room for their lists behind everything else, one workgroup per row
  if (topk > 0 && pl.topk_chunks > 0 && take_lists(part_val, part_idx)) {
    if (launch_topk(scores, nq, n_per_group, ld_scores, topk, nullptr, nullptr, s, pl.topk_chunks, part_val, part_idx) != hipSuccess)
      return TQ_ERR_HIP;
    return from_hip(launch_topk_merge(part_val, part_idx, nq, pl.topk_chunks, topk, topk_idx, topk_val, s));
  }
  if (topk > 0) return from_hip(launch_topk(scores, nq, n_per_group, ld_scores, topk, topk_idx, topk_val, s));
  return TQ_OK;
}

// Scratch memory of tq_score_static: one copy per GPU the library runs on, held until the process ends.
constexpr size_t kStaticScratchBytes = size_t(16) << 20;
__device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices];  // device address of `scratch` on each device, once asked for

// The array's name is only a host-side handle: its address in the current device's memory has to be asked for.
tq_status static_scratch(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return TQ_ERR_HIP;
  if (dev < 0 || dev >= kMaxDevices) return TQ_ERR_UNSUPPORTED;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[dev] == nullptr) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) return TQ_ERR_HIP;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return TQ_OK;
}

}  // namespace

extern "C" {

tq_status tq_score(const tq_params* p, const float* q, int64_t ldq, int32_t n_groups,
                   int32_t q_per_group, const uint32_t* idx, const uint32_t* qjl, const float* gamma,
                   const float* norm, int64_t n_per_group, float* scores, int64_t lds, int32_t topk,
                   int32_t* topk_idx, float* topk_val, void* stream) {
  if (p == nullptr) return TQ_ERR_INVALID_ARG;
  return score_impl(p, Workspace{static_cast<char*>(p->workspace), p->workspace_bytes, 0}, q, ldq, n_groups, q_per_group,
                    idx, qjl, gamma, norm, n_per_group, scores, lds, topk, topk_idx, topk_val, stream);
}

}  // extern "C"

namespace {
// most: with everything a call makes use of; otherwise what it cannot do without
size_t score_workspace(const tq_params* p, int32_t n_groups, int32_t q_per_group, int64_t n_per_group, int32_t prod, int32_t scores_given,
                       int32_t topk, bool most) {
  if (p == nullptr || p->d <= 0 || p->bits_mse < 0 || p->bits_mse > 4 || n_groups < 0 || q_per_group < 0 || n_per_group < 0 ||
      topk < 0 || topk > 64 || p->centroids == nullptr || (p->bits_mse > 0 && p->bounds == nullptr))
    return 0;
  // codes that are not 16-byte aligned can take a route with the smaller need; report the larger
  const ScorePlan x = plan_score(p, prod != 0, n_groups, q_per_group, n_per_group, scores_given != 0, topk, true);
  const ScorePlan y = plan_score(p, prod != 0, n_groups, q_per_group, n_per_group, scores_given != 0, topk, false);
  const size_t a = most ? x.total() : x.needed(), b = most ? y.total() : y.needed();
  return a > b ? a : b;
}
}  // namespace

extern "C" {

size_t tq_score_workspace_bytes(const tq_params* p, int32_t n_groups, int32_t q_per_group, int64_t n_per_group,
                                int32_t prod, int32_t scores_given, int32_t topk) {
  return score_workspace(p, n_groups, q_per_group, n_per_group, prod, scores_given, topk, true);
}

size_t tq_score_static_scratch_bytes(void) { return kStaticScratchBytes; }

tq_status tq_score_static(const tq_params* p, const float* q, int64_t ldq, int32_t n_groups,
                          int32_t q_per_group, const uint32_t* idx, const uint32_t* qjl, const float* gamma,
                          const float* norm, int64_t n_per_group, float* scores, int64_t lds, int32_t topk,
                          int32_t* topk_idx, float* topk_val, void* stream) {
  if (p == nullptr || n_groups < 0 || q_per_group < 0 || n_per_group < 0) return TQ_ERR_INVALID_ARG;
  // the whole need of the call must fit the static array
  const size_t need = score_workspace(p, n_groups, q_per_group, n_per_group, qjl != nullptr, scores != nullptr, topk, false);
  if (need == 0) return TQ_ERR_INVALID_ARG;
  if (need > kStaticScratchBytes) return TQ_ERR_WORKSPACE;
  void* base = nullptr;
  const tq_status st = static_scratch(&base);
  if (st != TQ_OK) return st;
  return score_impl(p, Workspace{static_cast<char*>(base), kStaticScratchBytes, 0}, q, ldq, n_groups, q_per_group, idx, qjl,
                    gamma, norm, n_per_group, scores, lds, topk, topk_idx, topk_val, stream);
}

}  // extern "C"

namespace {
struct AttendPlan {
  bool fast;  // the d = 128 kernel on the integer matrix cores takes the value codes
  int nchunks, max_chunks, keys;
  int64_t ld_scores;
  size_t scores_bytes, part_bytes, score_ws_bytes;
};
AttendPlan attend_plan(const tq_params* pk, const tq_params* pv, bool v_prod, int n_groups, int q_per_group, int64_t n_per_group) {
  AttendPlan pl;
  const int64_t nq = (int64_t)n_groups * q_per_group;
  const Codebook v_hi = make_codebook_hi(pv);
  pl.fast = pv->centroids != nullptr && (pv->d_hi == 0 || pv->centroids_hi != nullptr) &&
            attend128_applicable(pv->d, v_prod, make_codebook(pv), pv->d_hi != 0 ? &v_hi : nullptr);
  const int planes = pv->bits_mse + (v_prod || pv->d_hi != 0 ? 1 : 0);
  pl.keys = attend128_keys(n_per_group, n_groups, q_per_group, planes);
  pl.nchunks = pl.fast ? attend128_chunks(n_per_group, pl.keys) : attend_simple_chunks(n_per_group);
  // what is reported covers every shorter cache too, whose chunks may be more
  pl.max_chunks = pl.fast ? attend128_max_chunks(n_per_group, n_groups, q_per_group, planes) : pl.nchunks;
  pl.ld_scores = (n_per_group + 3) / 4 * 4;
  pl.scores_bytes = round_up((size_t)nq * pl.ld_scores * sizeof(float), 256);
  pl.part_bytes = round_up((size_t)nq * pl.max_chunks * attend_part_stride(pv->d) * sizeof(float), 256);
  pl.score_ws_bytes = tq_workspace_bytes(pk, 0, nq, 0);
  return pl;
}
}  // namespace

extern "C" {

size_t tq_attend_workspace_bytes(const tq_params* pk, const tq_params* pv, int32_t n_groups, int32_t q_per_group,
                                 int64_t n_per_group) {
  if (pk == nullptr || pv == nullptr || pk->d <= 0 || pv->d <= 0 || n_groups < 0 || q_per_group < 0 || n_per_group < 0)
    return 0;
  // whichever kind of value code the call then brings
  const AttendPlan pl = attend_plan(pk, pv, true, n_groups, q_per_group, n_per_group);
  const AttendPlan pm = attend_plan(pk, pv, false, n_groups, q_per_group, n_per_group);
  return pl.scores_bytes + (pl.part_bytes > pm.part_bytes ? pl.part_bytes : pm.part_bytes) + pl.score_ws_bytes + 512;
}

tq_status tq_attend(const tq_params* pk, const tq_params* pv, const float* q, int64_t ldq, int32_t n_groups,
                    int32_t q_per_group, const uint32_t* k_idx, const uint32_t* k_qjl, const float* k_gamma,
                    const float* k_norm, const uint32_t* v_idx, const uint32_t* v_qjl, const float* v_gamma,
                    const float* v_norm, int64_t n_per_group, float scale, float* out, int64_t ldo, void* stream) {
  return tq_attend_cache(pk, pv, q, ldq, n_groups, q_per_group, k_idx, k_qjl, k_gamma, k_norm, v_idx, v_qjl, v_gamma, v_norm,
                         n_per_group, n_per_group, scale, out, ldo, stream);
}

tq_status tq_attend_cache(const tq_params* pk, const tq_params* pv, const float* q, int64_t ldq, int32_t n_groups,
                          int32_t q_per_group, const uint32_t* k_idx, const uint32_t* k_qjl, const float* k_gamma,
                          const float* k_norm, const uint32_t* v_idx, const uint32_t* v_qjl, const float* v_gamma,
                          const float* v_norm, int64_t n_per_group, int64_t group_stride, float scale, float* out,
                          int64_t ldo, void* stream) {
  tq_status st = check_params(pk, true);
  if (st != TQ_OK) return st;
  st = check_params(pv, true);
  if (st != TQ_OK) return st;
  if (n_groups < 0 || q_per_group < 0 || n_per_group < 0 || ldo < pv->d || group_stride < n_per_group) return TQ_ERR_INVALID_ARG;
  const int64_t nq = (int64_t)n_groups * q_per_group;
  if (nq == 0) return TQ_OK;
  const bool v_prod = v_qjl != nullptr;
  if (out == nullptr || pv->Pi == nullptr || (v_prod && (v_gamma == nullptr || pv->S == nullptr)))
    return TQ_ERR_INVALID_ARG;
  if (n_per_group > 0 && (v_norm == nullptr || (pv->bits_mse > 0 && v_idx == nullptr))) return TQ_ERR_INVALID_ARG;
  if (pv->d > 4096 || n_groups > 65535 || q_per_group > 4 * 65535 || ldq > kMaxRowStride || ldo > kMaxRowStride)
    return TQ_ERR_UNSUPPORTED;
  hipStream_t s = static_cast<hipStream_t>(stream);

  const AttendPlan pl = attend_plan(pk, pv, v_prod, n_groups, q_per_group, n_per_group);
  // value codes of two instances: the d = 128 kernel or nothing
  if (pv->d_hi != 0 && !pl.fast) return TQ_ERR_UNSUPPORTED;
  if (pl.nchunks > 4096) return TQ_ERR_UNSUPPORTED;  // the joining kernel keeps one factor per chunk in LDS
  Workspace ws{static_cast<char*>(pk->workspace), pk->workspace_bytes, 0};
  float* scores = static_cast<float*>(ws.take(pl.scores_bytes));
  float* part = static_cast<float*>(ws.take((size_t)nq * pl.nchunks * attend_part_stride(pv->d) * sizeof(float)));
  char* rest = static_cast<char*>(ws.take(pl.score_ws_bytes));
  if (scores == nullptr || part == nullptr || rest == nullptr) return TQ_ERR_WORKSPACE;
  if (n_per_group > 0) {
    AttendArgs a;
    a.scores = scores; a.lds = pl.ld_scores;
    a.idx = v_idx; a.qjl = v_qjl; a.gamma = v_gamma; a.norm = v_norm;
    a.part = part; a.nchunks = pl.nchunks; a.keys = pl.keys; a.n = n_per_group; a.group_stride = group_stride; a.d = pv->d; a.q_per_group = q_per_group;
    a.scale = scale; a.gs_hi = pv->d_hi / 32;
    const AttendTables tables = {make_codebook(pv), make_codebook_hi(pv)};
    // a single chunk is rotated back by the workgroup that has summed it
    const bool whole = pl.fast && pl.nchunks == 1 && pl.keys < AT_KEYS[2];
    a.out = whole ? out : nullptr; a.ldo = ldo; a.Pi = pv->Pi; a.S = v_prod ? pv->S : nullptr; a.kappa = kappa_of(pv->d);
    // keys the single-kernel d = 128 scoring path takes are scored inside the read-out kernel
    const bool k_prod = k_qjl != nullptr;
    ScoreI8Args ka;
    const bool fused = pl.fast && pk->d == 128 && pk->d_hi == 0 && q != nullptr && ldq >= 128 &&
                       score128_args(pk->bits_mse, k_prod, pk->PiT, pk->ST, q, ldq, k_idx, k_qjl, k_gamma, k_norm,
                                     n_per_group, n_groups, q_per_group, kappa_of(128), make_codebook(pk), group_stride, &ka);
    if (fused) {
      if (launch_attend128(pk->bits_mse, k_prod, &ka, v_prod, a, tables, n_groups, s) != hipSuccess) return TQ_ERR_HIP;
    } else {
      // tq_score knows densely stored groups only
      if (group_stride != n_per_group) return TQ_ERR_UNSUPPORTED;
      tq_params pk_inner = *pk;  // the scoring call carves its own needs from what is left
      pk_inner.workspace = rest;
      pk_inner.workspace_bytes = pl.score_ws_bytes;
      st = tq_score(&pk_inner, q, ldq, n_groups, q_per_group, k_idx, k_qjl, k_gamma, k_norm, n_per_group, scores,
                    pl.ld_scores, 0, nullptr, nullptr, stream);
      if (st != TQ_OK) return st;
      if ((pl.fast ? launch_attend128(0, false, nullptr, v_prod, a, tables, n_groups, s) : launch_attend_values(v_prod, a, tables.cb, n_groups, s)) !=
          hipSuccess)
        return TQ_ERR_HIP;
    }
    if (whole) return TQ_OK;
  }
  return from_hip(launch_attend_combine(part, pl.nchunks, pv->d, nq, pv->Pi, v_prod ? pv->S : nullptr,
                                        kappa_of(pv->d), out, ldo, s));
}

tq_status tq_stage_pack(const tq_params* p, const float* y, int64_t n, uint32_t* idx, void* stream) {
  tq_status st = check_params(p, true);
  if (st != TQ_OK) return st;
  if (p->d_hi != 0) return TQ_ERR_UNSUPPORTED;  // the stand-alone stages know one instance only
  if (n < 0) return TQ_ERR_INVALID_ARG;
  if (n == 0 || p->bits_mse == 0) return TQ_OK;
  if (y == nullptr || idx == nullptr) return TQ_ERR_INVALID_ARG;
  return from_hip(launch_stage_pack(make_codebook(p), p->d, y, n, idx, static_cast<hipStream_t>(stream)));
}

tq_status tq_stage_sign_pack(int32_t d, const float* u, int64_t n, uint32_t* qjl, void* stream) {
  if (d <= 0 || n < 0) return TQ_ERR_INVALID_ARG;
  if (d % 32 != 0) return TQ_ERR_UNSUPPORTED;
  if (n == 0) return TQ_OK;
  if (u == nullptr || qjl == nullptr) return TQ_ERR_INVALID_ARG;
  return from_hip(launch_stage_sign_pack(d, u, n, qjl, static_cast<hipStream_t>(stream)));
}

tq_status tq_stage_unpack(const tq_params* p, const uint32_t* idx, int64_t n, float* y_tilde,
                          void* stream) {
  tq_status st = check_params(p, true);
  if (st != TQ_OK) return st;
  if (p->d_hi != 0) return TQ_ERR_UNSUPPORTED;  // the stand-alone stages know one instance only
  if (n < 0) return TQ_ERR_INVALID_ARG;
  if (n == 0) return TQ_OK;
  if (y_tilde == nullptr || (p->bits_mse > 0 && idx == nullptr)) return TQ_ERR_INVALID_ARG;
  return from_hip(launch_stage_unpack(make_codebook(p), p->d, idx, n, y_tilde, static_cast<hipStream_t>(stream)));
}

}  // extern "C"
