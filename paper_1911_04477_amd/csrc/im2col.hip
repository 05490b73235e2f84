// Packed im2col (section 2.1 im2col applied to the encoded input of section 3.1).
//
// Small inputs in one launch (im2col_band_kernel), others in two streaming passes, both HBM-bound:
//   1. encode_nchw_kernel (encode.hip): fp32 NCHW -> packed NHWC, ceil(C/64) words per
//      pixel.  The fp32 image is read exactly once.
//   2. im2col_gather_kernel (here): every output pixel's kH*kW taps are whole-word
//      copies out of the packed image (which is 32x smaller than the fp32 one and
//      stays in L2), or the "+1" pad word for taps outside the image: zero-padding
//      before the sign makes every real channel of such a tap +1, i.e. bit 1.
// A 1x1 / pad-0 convolution has no patch expansion: pass 1 writes the patch matrix
// directly, sampling the strided pixels.
#include <algorithm>

#include "common.h"

namespace bnn {

bool encode_nchw_supported(int N, int C, int H, int W, int OHp, int OWp);
bnn_status launch_encode_nchw(const float *x, int N, int C, int H, int W, int OHp, int OWp, int sH, int sW,
                              uint64_t *out, hipStream_t s);

struct GatherParams {
  int C, H, W, OH, OW, kH, kW, sH, sW, pH, pW, Cw;
  FastDiv divRow;   // pieces per patch row
  FastDiv divTap;   // pieces per tap
  FastDiv divKW, divOW, divOH;
  uint32_t total;   // pieces (unused by the band kernel)
};

// words of a tap that lies outside the image
__device__ __forceinline__ uint64_t pad_word(int C, int cw) {
  const int left = C - cw * 64;
  return left >= 64 ? ~0ull : (left <= 0 ? 0ull : ((1ull << left) - 1ull));
}

template <int PIECE>  // words per thread: 2 (16-byte copies) or 1
__global__ __launch_bounds__(256) void im2col_gather_kernel(const uint64_t *__restrict__ img,
                                                            uint64_t *__restrict__ cols, GatherParams g) {
  const uint32_t o = blockIdx.x * 256u + threadIdx.x;
  if (o >= g.total) return;
  const uint32_t p = fdiv(o, g.divRow);
  const uint32_t r = o - p * g.divRow.d;
  const uint32_t tap = fdiv(r, g.divTap);
  const uint32_t q = r - tap * g.divTap.d;
  const uint32_t kh = fdiv(tap, g.divKW);
  const uint32_t kw = tap - kh * g.kW;
  const uint32_t t = fdiv(p, g.divOW);
  const uint32_t ow = p - t * g.OW;
  const uint32_t n = fdiv(t, g.divOH);
  const uint32_t oh = t - n * g.OH;
  const int ih = (int)(oh * g.sH + kh) - g.pH;
  const int iw = (int)(ow * g.sW + kw) - g.pW;
  const bool inside = ih >= 0 && ih < g.H && iw >= 0 && iw < g.W;
  if (PIECE == 2) {
    uint4 v;
    if (inside) {
      v = *reinterpret_cast<const uint4 *>(img + (((size_t)n * g.H + ih) * g.W + iw) * g.Cw + 2 * q);
    } else {
      const uint64_t w0 = pad_word(g.C, 2 * q), w1 = pad_word(g.C, 2 * q + 1);
      v.x = (uint32_t)w0; v.y = (uint32_t)(w0 >> 32); v.z = (uint32_t)w1; v.w = (uint32_t)(w1 >> 32);
    }
    reinterpret_cast<uint4 *>(cols)[o] = v;
  } else {
    uint64_t v;
    if (inside) v = img[(((size_t)n * g.H + ih) * g.W + iw) * g.Cw + q];
    else v = pad_word(g.C, q);
    cols[o] = v;
  }
}

struct BandParams {
  GatherParams g;
  int R, nb;        // output rows per band, bands per image
  FastDiv divNb, divG;
};

// Both passes in one launch for small inputs (band_rows): a workgroup encodes the image rows that a band of R output rows
// needs into LDS (half words, one granule of 32 channels per wave and step, 32 plane-strided loads in flight per
// lane) and emits the band's patch rows from there.  Saves a launch and the packed image's round trip; the bands
// read their halo rows again, and a workgroup does not read while it writes.  16 waves per workgroup keep as many
// loads in flight on a compute unit as the two-pass encode does.  Two passes -> this: 128 x 128 x 32 x 32, 3x3
// 19.1 -> 15.7 us (86 MB moved, 5.5 TB/s); 256 x 512 x 8 x 8 12.7 -> 7.5; 250 x 3 x 32 x 32 21.4 -> 9.5; one
// 64 x 8 x 8 image 5.0 -> 3.0.
constexpr int BAND_T = 1024;
template <int PIECE>
__global__ __launch_bounds__(BAND_T) void im2col_band_kernel(const float *__restrict__ x, uint64_t *__restrict__ cols,
                                                             BandParams b) {
  extern __shared__ uint32_t s_half[];  // [pixels of the band's image rows][2 * Cw + 1]
  const GatherParams &g = b.g;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = (int)fdiv(blockIdx.x, b.divNb), band = (int)blockIdx.x - n * b.nb;
  const int oh0 = band * b.R, oh1 = min(oh0 + b.R, g.OH);
  const int ih0 = max(0, oh0 * g.sH - g.pH), ih1 = min(g.H, (oh1 - 1) * g.sH - g.pH + (int)g.kH);
  const int npix = max(0, ih1 - ih0) * g.W;  // consecutive in every channel plane; 0: the band sees padding only
  const size_t plane = (size_t)g.H * g.W;
  const float *xb = x + ((size_t)n * g.C * plane + (size_t)ih0 * g.W);
  const int G = 2 * g.Cw, rs = G + 1;
  const int tasks = ((npix + 63) >> 6) * G;
  for (int t = wave; t < tasks; t += BAND_T / 64) {
    const int pg = (int)fdiv((uint32_t)t, b.divG), gr = t - pg * G;
    const int pix = pg * 64 + lane;
    const float *xp = xb + min(pix, npix - 1);
    const int c0 = gr * 32, left = g.C - c0;  // real channels in this granule
    uint32_t acc = 0;
    if (left >= 32) {
      float v[32];
#pragma unroll
      for (int j = 0; j < 32; ++j) v[j] = __builtin_nontemporal_load(xp + (size_t)(c0 + j) * plane);
#pragma unroll
      for (int j = 0; j < 32; ++j) acc |= (uint32_t)sign_bit(v[j]) << j;
    } else {
      for (int j0 = 0; j0 < left; j0 += 4) {
        float v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)  // channels past C re-read the last channel and are masked out
          v[j] = __builtin_nontemporal_load(xp + (size_t)(c0 + min(j0 + j, left - 1)) * plane);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc |= (uint32_t)(sign_bit(v[j]) && j0 + j < left) << (j0 + j);
      }
    }
    if (pix < npix) s_half[pix * rs + gr] = acc;
  }
  __syncthreads();
  const uint32_t total = (uint32_t)((oh1 - oh0) * g.OW) * g.divRow.d;
  char *out = reinterpret_cast<char *>(cols) + ((size_t)n * g.OH + oh0) * g.OW * g.divRow.d * (8 * PIECE);
  for (uint32_t o = threadIdx.x; o < total; o += BAND_T) {
    const uint32_t p = fdiv(o, g.divRow);
    const uint32_t r = o - p * g.divRow.d;
    const uint32_t tap = fdiv(r, g.divTap);
    const uint32_t q = r - tap * g.divTap.d;
    const uint32_t kh = fdiv(tap, g.divKW);
    const uint32_t kw = tap - kh * g.kW;
    const uint32_t ohl = fdiv(p, g.divOW);
    const uint32_t ow = p - ohl * g.OW;
    const int ih = (int)((oh0 + ohl) * g.sH + kh) - g.pH;
    const int iw = (int)(ow * g.sW + kw) - g.pW;
    uint32_t w[2 * PIECE];
    if (ih >= 0 && ih < g.H && iw >= 0 && iw < g.W) {
      const uint32_t *src = &s_half[((ih - ih0) * g.W + iw) * rs + 2 * PIECE * q];
#pragma unroll
      for (int i = 0; i < 2 * PIECE; ++i) w[i] = src[i];
    } else {
#pragma unroll
      for (int i = 0; i < PIECE; ++i) {
        const uint64_t pad = pad_word(g.C, PIECE * q + i);
        w[2 * i] = (uint32_t)pad;
        w[2 * i + 1] = (uint32_t)(pad >> 32);
      }
    }
    if constexpr (PIECE == 2) reinterpret_cast<uint4 *>(out)[o] = make_uint4(w[0], w[1], w[2], w[3]);
    else reinterpret_cast<uint2 *>(out)[o] = make_uint2(w[0], w[1]);
  }
}

static bool conv_geometry_ok(int N, int C, int H, int W, int kH, int kW, int sH, int sW, int pH, int pW) {
  return N >= 0 && C > 0 && H > 0 && W > 0 && kH > 0 && kW > 0 && sH > 0 && sW > 0 && pH >= 0 && pW >= 0 &&
         bnn_conv_out_dim(H, kH, sH, pH) > 0 && bnn_conv_out_dim(W, kW, sW, pW) > 0;
}

static inline size_t round256(size_t b) { return (b + 255) & ~(size_t)255; }

static inline bool is_pointwise(int kH, int kW, int pH, int pW) { return kH == 1 && kW == 1 && pH == 0 && pW == 0; }

// Output rows per band for im2col_band_kernel, or 0 where encode + gather is the better form.  The smallest bands
// that give every compute unit at most one workgroup: a second one per unit re-reads more halo rows than its overlap
// returns (128 x 128 x 32 x 32, 3x3: 15.7 us with one per unit, 19.6 with two, 19.6 in two passes).  Not taken
//   * where a workgroup reads over 384 KB: two passes overlap reading and writing across workgroups (262 KB each:
//     15.7 us against 19.6; 524 KB, 256 x 128 x 32 x 32: 34.8 against 34.1; 64 x 256 x 56 x 56: 65 against 48);
//   * where over 48 KB of that are halo rows (32 KB: 4.8 against 5.8 us; 115 KB, 8 x 256 x 56 x 56: 13.7 against 10.3);
//   * where units stay idle, unless the call is short anyway (up to 64 KB per workgroup; one 128 x 32 x 32 image:
//     4.2 against 5.3);
//   * where a workgroup emits much more than its share of the chip: the gather spreads the patches over every unit
//     whatever the bands are.  A workgroup emits BAND_T pieces per 0.4 us; the form gives way where these rounds, and
//     the reading where units are idle (16 KB per round), exceed the share by more than 7 + 2/5 of it (one row of 4096
//     pixels, 101 taps: 404 rounds, 153 against 6.3 us; 32 rows of 226 pixels of 64 channels, 101 taps: 13 rounds,
//     8.1 against 6.0; one 3 x 224 x 224 image, 7x7: 6 rounds, 7.0 against 9.0; 215 rows of 250 pixels, 251 taps: 62
//     rounds, a share of 52, 29.7 against 33.2).  Of 500 random calls that the other lines pass, 449 are taken, 4 of
//     them 6 to 18 % slower in this form, and 3 are left that it would have made faster.
static int band_rows(int N, int C, int H, int W, int kH, int sH, int OH, int OW, int64_t Cw, int64_t per_row) {
  const int cu = device_cu_count();
  if (N > cu) return 0;
  const int R = (OH + cu / N - 1) / (cu / N);
  const int64_t rows = std::min<int64_t>((int64_t)(R - 1) * sH + kH, H), row_bytes = (int64_t)W * C * 4;
  const int64_t lds = rows * W * (2 * Cw + 1) * 4;
  if (lds > 64 * 1024) return 0;
  const int64_t wgs = (int64_t)N * ((OH + R - 1) / R);
  if (rows * row_bytes > 384 * 1024 || (rows - (int64_t)R * sH) * row_bytes > 48 * 1024) return 0;
  const bool idle = wgs * 8 < (int64_t)cu * 7;
  if (idle && rows * row_bytes > 64 * 1024) return 0;
  const int64_t rounds = ((int64_t)R * OW * per_row + BAND_T - 1) / BAND_T;
  const int64_t share = (int64_t)N * OH * OW * per_row / ((int64_t)cu * BAND_T);
  const int64_t reading = idle ? rows * row_bytes / (16 * 1024) : 0;
  return 5 * (rounds + reading) <= 5 * 7 + 7 * share ? R : 0;
}

// Shared by bnn_im2col_packed and bnn_conv2d; arguments already validated.
bnn_status run_im2col(const float *x, int N, int C, int H, int W, int kH, int kW, int sH, int sW, int pH, int pW,
                      uint64_t *cols, void *workspace, hipStream_t s) {
  const int OH = (int)bnn_conv_out_dim(H, kH, sH, pH), OW = (int)bnn_conv_out_dim(W, kW, sW, pW);
  if (is_pointwise(kH, kW, pH, pW)) return launch_encode_nchw(x, N, C, H, W, OH, OW, sH, sW, cols, s);
  const int Cw = (int)bnn_packed_words(C);
  const int piece = (Cw % 2 == 0) ? 2 : 1;
  const int64_t per_tap = Cw / piece;
  const int64_t per_row = per_tap * kH * kW;
  const int64_t total = (int64_t)N * OH * OW * per_row;
  if (total > 0x7fffffffLL) return BNN_ERR_UNSUPPORTED;
  GatherParams g;
  g.C = C; g.H = H; g.W = W; g.OH = OH; g.OW = OW; g.kH = kH; g.kW = kW; g.sH = sH; g.sW = sW; g.pH = pH; g.pW = pW;
  g.Cw = Cw;
  g.divRow = FastDiv((uint32_t)per_row);
  g.divTap = FastDiv((uint32_t)per_tap);
  g.divKW = FastDiv((uint32_t)kW);
  g.divOW = FastDiv((uint32_t)OW);
  g.divOH = FastDiv((uint32_t)OH);
  g.total = (uint32_t)total;
  if (!encode_nchw_supported(N, C, H, W, H, W)) return BNN_ERR_UNSUPPORTED;
  if (const int R = band_rows(N, C, H, W, kH, sH, OH, OW, Cw, per_row)) {
    BandParams b;
    b.g = g;
    b.R = R;
    b.nb = (OH + R - 1) / R;
    b.divNb = FastDiv((uint32_t)b.nb);
    b.divG = FastDiv((uint32_t)(2 * Cw));
    const unsigned nblk = (unsigned)(N * b.nb);
    const size_t lds = (size_t)std::min<int64_t>((int64_t)(R - 1) * sH + kH, H) * W * (2 * Cw + 1) * 4;
    ProfScope ps(KID_IM2COL_BAND, s);
    if (piece == 2)
      hipLaunchKernelGGL(im2col_band_kernel<2>, dim3(nblk), dim3(BAND_T), lds, s, x, cols, b);
    else
      hipLaunchKernelGGL(im2col_band_kernel<1>, dim3(nblk), dim3(BAND_T), lds, s, x, cols, b);
    return launch_status();
  }
  uint64_t *img = reinterpret_cast<uint64_t *>(workspace);
  bnn_status st = launch_encode_nchw(x, N, C, H, W, H, W, 1, 1, img, s);
  if (st != BNN_OK) return st;
  const unsigned blocks = (unsigned)((total + 255) / 256);
  {
    ProfScope ps(KID_IM2COL_GATHER, s);
    if (piece == 2)
      hipLaunchKernelGGL(im2col_gather_kernel<2>, dim3(blocks), dim3(256), 0, s, img, cols, g);
    else
      hipLaunchKernelGGL(im2col_gather_kernel<1>, dim3(blocks), dim3(256), 0, s, img, cols, g);
  }
  return launch_status();
}

bnn_status check_conv_geometry(int N, int C, int H, int W, int kH, int kW, int sH, int sW, int pH, int pW) {
  if (!conv_geometry_ok(N, C, H, W, kH, kW, sH, sW, pH, pW)) return BNN_ERR_SHAPE;
  const int64_t OH = bnn_conv_out_dim(H, kH, sH, pH), OW = bnn_conv_out_dim(W, kW, sW, pW);
  const int64_t Cw = bnn_packed_words(C);
  if ((int64_t)N * C * H * W > 0x7fffffffLL * 4 || (int64_t)N * H * W > 0x7fffffffLL ||
      (int64_t)N * OH * OW * kH * kW * Cw > 0x7fffffffLL || (int64_t)kH * kW > 0x7fff)
    return BNN_ERR_UNSUPPORTED;
  return BNN_OK;
}

}  // namespace bnn

using namespace bnn;

extern "C" size_t bnn_im2col_workspace_bytes(int N, int C, int H, int W, int kH, int kW, int sH, int sW, int pH,
                                             int pW) {
  if (!conv_geometry_ok(N, C, H, W, kH, kW, sH, sW, pH, pW)) return 0;
  if (is_pointwise(kH, kW, pH, pW)) return 0;
  return round256((size_t)N * H * W * (size_t)bnn_packed_words(C) * 8);
}

extern "C" size_t bnn_conv2d_workspace_bytes(int N, int C, int H, int W, int kH, int kW, int sH, int sW, int pH,
                                             int pW) {
  if (!conv_geometry_ok(N, C, H, W, kH, kW, sH, sW, pH, pW)) return 0;
  // the packed image the implicit GEMM gathers from: the whole input, or, for a 1x1 / pad-0
  // convolution, only the pixels its strides sample
  if (is_pointwise(kH, kW, pH, pW)) {
    const size_t OH = (size_t)bnn_conv_out_dim(H, kH, sH, pH), OW = (size_t)bnn_conv_out_dim(W, kW, sW, pW);
    return round256((size_t)N * OH * OW * (size_t)bnn_packed_words(C) * 8);
  }
  return round256((size_t)N * H * W * (size_t)bnn_packed_words(C) * 8);
}

extern "C" bnn_status bnn_im2col_packed(const float *x, int N, int C, int H, int W, int kH, int kW, int sH, int sW,
                                        int pH, int pW, uint64_t *cols, void *workspace, size_t workspace_bytes,
                                        void *stream) {
  bnn_status st = check_conv_geometry(N, C, H, W, kH, kW, sH, sW, pH, pW);
  if (st != BNN_OK) return st;
  if (N == 0) return BNN_OK;
  const size_t need = bnn_im2col_workspace_bytes(N, C, H, W, kH, kW, sH, sW, pH, pW);
  if (!x || !cols || (need > 0 && !workspace)) return BNN_ERR_NULL;
  if (!aligned16(x) || !aligned16(cols) || (need > 0 && !aligned16(workspace))) return BNN_ERR_ALIGN;
  if (workspace_bytes < need) return BNN_ERR_WORKSPACE;
  return run_im2col(x, N, C, H, W, kH, kW, sH, sW, pH, pW, cols, workspace, (hipStream_t)stream);
}
