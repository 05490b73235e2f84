// Binarized convolution drivers: the forward graph of Figure 3 of the paper (encode the
// input, pre-encoded weight, Xnor-Bitcount, reshape to the output feature map).
//  * The reshape (col2im of section 2.1) costs nothing: the GEMM store writes each
//    accumulator straight to its NCHW position.
//  * The patch matrix of im2col is never materialised: the GEMM gathers its B tiles from
//    the packed NHWC image (implicit GEMM).
//  * bnn_conv2d_packed keeps activations packed between layers: packed NHWC in, and with
//    the binarizing epilogue packed NHWC out (2x2 max-pool, affine map and sign fused into
//    the GEMM store), so a stack of binarized layers moves 1 bit per activation.
//  * bnn_conv2d_f32_sign is the real-valued first layer producing that packed format.
#include <mutex>

#include "common.h"
#include "bnn_testing.h"
#include "conv_first.h"

namespace bnn {

bnn_status launch_encode_nchw(const float *x, int N, int C, int H, int W, int OHp, int OWp, int sH, int sW,
                              uint64_t *out, hipStream_t s);

static void fill_geom(ConvGeom &g, const uint64_t *act, int N, int C, int H, int W, int kH, int kW, int sH, int sW, int pH,
                      int pW, int pool) {
  g.act = act;
  g.Nimg = N; g.C = C; g.H = H; g.W = W;
  g.Cw = (int)bnn_packed_words(C);
  g.OH = (int)bnn_conv_out_dim(H, kH, sH, pH);
  g.OW = (int)bnn_conv_out_dim(W, kW, sW, pW);
  g.kH = kH; g.kW = kW; g.sH = sH; g.sW = sW; g.pH = pH; g.pW = pW;
  g.pool = pool;
  g.divCw = FastDiv((uint32_t)g.Cw);
  g.divKW = FastDiv((uint32_t)kW);
  g.divOW = FastDiv((uint32_t)(pool ? g.OW / 2 : g.OW));
  g.divOH = FastDiv((uint32_t)(pool ? g.OH / 2 : g.OH));
}

// The GEMM of a convolution over a packed NHWC image; arguments validated by the callers.
static GemmParams conv_gemm(const uint64_t *act, const uint64_t *w_packed, int N, int C, int H, int W, int D, int kH,
                            int kW, int sH, int sW, int pH, int pW, int pool, int32_t *out_i32,
                            float *out_f32, uint64_t *out_packed, const float *scale, const float *bias) {
  const int64_t OH = bnn_conv_out_dim(H, kH, sH, pH), OW = bnn_conv_out_dim(W, kW, sW, pW);
  const int64_t Kw = bnn_conv_kwords(C, kH, kW);
  const int64_t cols = pool ? 4 * ((int64_t)N * (OH / 2) * (OW / 2)) : (int64_t)N * OH * OW;
  GemmParams p = {};
  p.A = reinterpret_cast<const uint32_t *>(w_packed);
  p.B = nullptr;
  p.lda32 = 2 * Kw;
  p.ldb = Kw;
  p.M = D;
  p.N = (int)cols;
  p.Kbits = (int)(Kw * 64);  // pad bits are 0 in both operands: they cancel in the exclusive-or
  p.Kformula = C * kH * kW;
  p.Kd = (int)(Kw * 2);
  p.Kw64 = (int)Kw;
  p.b_vec16 = 0;
  p.C = out_i32;
  p.Y = out_f32;
  p.ldc = p.ldy = OH * OW;
  p.scale = scale;
  p.bias = bias;
  p.axis = BNN_CH_ROW;
  p.OHW = (uint32_t)(OH * OW);
  p.divOHW = FastDiv((uint32_t)(OH * OW));
  p.img_stride = (int64_t)D * OH * OW;
  fill_geom(p.g, act, N, C, H, W, kH, kW, sH, sW, pH, pW, pool);
  p.outp = out_packed;
  p.cw_out = (int)bnn_packed_words(D);
  return p;
}

static bnn_status conv_from_packed(const uint64_t *act, const uint64_t *w_packed, int N, int C, int H, int W, int D,
                                   int kH, int kW, int sH, int sW, int pH, int pW, int pool, int32_t *out_i32,
                                   float *out_f32, uint64_t *out_packed, const float *scale, const float *bias,
                                   hipStream_t s, const GemmTune &tune) {
  GemmParams p = conv_gemm(act, w_packed, N, C, H, W, D, kH, kW, sH, sW, pH, pW, pool, out_i32, out_f32, out_packed,
                           scale, bias);
  return run_gemm(p, 1, out_packed ? 1 : 0, s, tune);
}

static bnn_status conv_limits(int N, int C, int H, int W, int D, int kH, int kW, int sH, int sW, int pH, int pW) {
  const int64_t OH = bnn_conv_out_dim(H, kH, sH, pH), OW = bnn_conv_out_dim(W, kW, sW, pW);
  const int64_t P = (int64_t)N * OH * OW;
  const int64_t Kw = bnn_conv_kwords(C, kH, kW);
  // column count, 32-bit byte offsets into the filter bank, output elements, pixels, and the
  // reduction length in bits (an int in the kernel's parameters)
  if (P > 0x7ffffff0LL / 4 || (int64_t)D * 8 * Kw > 0xffffffffLL || (int64_t)D * P > 0x7fffffffLL * 8 ||
      (int64_t)N * H * W > 0x7fffffffLL || Kw * 64 > 0x7fffffffLL)
    return BNN_ERR_UNSUPPORTED;
  return BNN_OK;
}

// ---- real-valued first layer with binarized, packed output ----------------------------------
// One thread per output pixel.  The input patch (K = C*kH*kW <= 32 taps) sits in registers.
// The filter bank, scale and bias are wave-uniform, so they are read through the constant
// address space with scalar loads and enter v_fma as the scalar operand (an LDS copy would
// make the CU's single LDS pipe the bottleneck: four SIMDs reading 7 x 16 bytes per channel).
// Every output channel is the sequential fma chain over (c, kh, kw), then fma(scale, acc,
// bias); only its sign is kept, 64 channels per stored word.
constexpr int F32S_KMAX = 32;
#define BNN_CONST_AS __attribute__((address_space(4)))
typedef const float BNN_CONST_AS *cf32_ptr;

template <int KT>  // KT = K when known at compile time (27 for 3x3x3), else 0
__global__ __launch_bounds__(256) void conv2d_f32_sign_kernel(const float *__restrict__ x, const float *w_, int C,
                                                              int H, int W, int D, int kH, int kW, int sH, int sW,
                                                              int pH, int pW, int OH, int OW, const float *scale_,
                                                              const float *bias_, uint64_t *__restrict__ outp,
                                                              int cw_out, FastDiv divOW, FastDiv divOH,
                                                              uint32_t total_pix, int K_rt) {
  const int K = KT > 0 ? KT : K_rt;
  const cf32_ptr w = (cf32_ptr)(uintptr_t)w_;
  const cf32_ptr scale = (cf32_ptr)(uintptr_t)scale_;
  const cf32_ptr bias = (cf32_ptr)(uintptr_t)bias_;
  const uint32_t p = blockIdx.x * 256u + threadIdx.x;
  if (p >= total_pix) return;
  const uint32_t t = fdiv(p, divOW);
  const uint32_t ow = p - t * OW;
  const uint32_t n = fdiv(t, divOH);
  const uint32_t oh = t - n * OH;
  const int ih0 = (int)(oh * sH) - pH, iw0 = (int)(ow * sW) - pW;
  const float *xn = x + (size_t)n * C * H * W;
  const int taps = kH * kW;
  constexpr int KU = KT > 0 ? KT : F32S_KMAX;
  float xv[KU];
#pragma unroll
  for (int k = 0; k < KU; ++k) {
    float v = 0.0f;
    if (k < K) {
      const int c = k / taps, r = k - c * taps;
      const int kh = r / kW, kw = r - kh * kW;
      const int ih = ih0 + kh, iw = iw0 + kw;
      if (ih >= 0 && ih < H && iw >= 0 && iw < W) v = xn[((size_t)c * H + ih) * W + iw];
    }
    xv[k] = v;
  }
  for (int d0 = 0; d0 < D; d0 += 64) {
    uint32_t lo = 0, hi = 0;
    const int dn = D - d0 < 64 ? D - d0 : 64;
#pragma unroll 4
    for (int dd = 0; dd < dn; ++dd) {
      const cf32_ptr wr = w + (size_t)(d0 + dd) * K;
      float acc = 0.0f;
#pragma unroll
      for (int k = 0; k < KU; ++k)
        if (k < K) acc = fmaf(xv[k], wr[k], acc);
      const uint32_t bit = fmaf(scale[d0 + dd], acc, bias[d0 + dd]) >= 0.0f ? 1u : 0u;
      if (dd < 32) lo |= bit << dd; else hi |= bit << (dd - 32);
    }
    outp[(size_t)p * cw_out + (d0 >> 6)] = ((uint64_t)hi << 32) | lo;
  }
}

// ---- the 3x3x3 layer (K = 27) on the fp32 matrix cores: conv_first.h --------------------------
// Packed-sign output for few pixels, and for images beyond the 32-bit offsets of conv_first_sign.hip, which takes the others.  NG:
// groups of 32 channels per workgroup.  Few pixels: one, since the chains of a group are 27 dependent instructions of 64 clocks
// (batch 1 of the 32 x 32, 128-channel layer: four groups 8.6 us, one 4.3).  Very large images: four, which share a patch's loads (256
// images of 32 x 32 22.5 us, one 27.3) and keep blockIdx.y small.  On this chip the fp32 matrix instructions and the vector ALU do
// not run side by side (vector instructions placed between the matrix instructions of a chain lengthen it by their full
// issue time, measured), so the loop is the plain sequence loads, chain, sign step, store.
template <int NG>
__global__ __launch_bounds__(256, 4) void conv2d_f32_k27_mfma_sign_kernel(
    const float *__restrict__ x, const float *__restrict__ w, int H, int W, int D, int sH, int sW, int pH, int pW,
    int OH, int OW, const float *__restrict__ scale, const float *__restrict__ bias, uint64_t *__restrict__ outp,
    int cw_out, FastDiv divOW, FastDiv divOH, uint32_t total_pix, uint32_t ngroups, int groups_per_wave) {
  __shared__ float sTap[27 * C1M_RS(NG)];
  __shared__ __attribute__((aligned(16))) float sSc[32 * NG];
  __shared__ __attribute__((aligned(16))) float sBi[32 * NG];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int half = lane >> 5, l32 = lane & 31;
  const int ch0 = 32 * NG * (int)blockIdx.y;
  const uint32_t g_first = ((uint32_t)blockIdx.x * 4u + (uint32_t)wave) * (uint32_t)groups_per_wave;
  const uint32_t g_end = min(g_first + (uint32_t)groups_per_wave, ngroups);
  const int nch = min(32 * NG, D - ch0);  // >= 1 by the grid
  // the first patch is requested before the filters are staged, so the two latencies overlap
  // (a wave without pixel groups loads pixel 0's and discards it)
  C1mFilters<NG> filters;
  filters.request(w, scale, bias, ch0, nch, true);
  float xv[27];
  uint32_t inside;
  c1m_issue_patch(x, g_first * 64u + (uint32_t)lane, total_pix, H, W, sH, sW, pH, pW, OH, OW, divOW, divOH, xv, inside);
  filters.stage(sTap, sSc, sBi, nch, true);
  __syncthreads();  // the only barrier: from here on the waves run independently

  for (uint32_t grp = g_first; grp < g_end; ++grp) {  // wave-uniform bounds
    const uint32_t p = grp * 64u + (uint32_t)lane;
    if (grp != g_first)
      c1m_issue_patch(x, p, total_pix, H, W, sH, sW, pH, pW, OH, OW, divOW, divOH, xv, inside);
#pragma unroll
    for (int k = 0; k < 27; ++k) xv[k] = ((inside >> (k % 9)) & 1u) ? xv[k] : 0.0f;
    uint32_t gw[NG];
#pragma unroll
    for (int c = 0; c < NG; ++c) gw[c] = 0u;
#pragma unroll
    for (int c = 0; c < NG; ++c) {
      if (32 * c >= nch) break;  // workgroup-uniform: groups past the last channel keep zero bits
      gw[c] = c1m_sign_bits(c1m_chain<NG>(sTap + 32 * c + l32, xv), sSc, sBi, c, half);
    }
    if (p < total_pix) {  // 32-channel half words; the last group also writes the half that holds no channel
      uint32_t *o = reinterpret_cast<uint32_t *>(outp + (size_t)p * cw_out);
#pragma unroll
      for (int c = 0; c < NG; ++c) {
        const int h0 = NG * (int)blockIdx.y + c;
        if (32 * c >= nch) break;
        o[h0] = gw[c];
        if (32 * (h0 + 1) >= D && h0 + 1 < 2 * cw_out) o[h0 + 1] = 0u;
      }
    }
  }
}

// fp32 NCHW output (the map itself, with the affine map if has_affine), same chains, no pipelining.
template <int NG>
__global__ __launch_bounds__(256) void conv2d_f32_k27_mfma_kernel(const float *__restrict__ x,
                                                                  const float *__restrict__ w, int H, int W, int D,
                                                                  int sH, int sW, int pH, int pW, int OH, int OW,
                                                                  const float *__restrict__ scale,
                                                                  const float *__restrict__ bias, FastDiv divOW,
                                                                  FastDiv divOH, uint32_t total_pix, uint32_t ngroups,
                                                                  int groups_per_wave, float *__restrict__ outf,
                                                                  int has_affine) {
  __shared__ float sTap[27 * C1M_RS(NG)];
  __shared__ float sSc[32 * NG], sBi[32 * NG];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int half = lane >> 5, l32 = lane & 31;
  const int ch0 = 32 * NG * (int)blockIdx.y;
  const int nch = min(32 * NG, D - ch0);  // >= 1 by the grid
  const uint32_t g_first = ((uint32_t)blockIdx.x * 4u + (uint32_t)wave) * (uint32_t)groups_per_wave;
  // One channel group: the first patch is requested before the filters are staged, as in the kernel above.  Four: 14 filter values a
  // thread beside it cost more than they hide (8 x 512 x 224 x 224 213 us, 220).
  constexpr bool AHEAD = NG == 1;
  C1mFilters<NG> filters;
  filters.request(w, scale, bias, ch0, nch, has_affine != 0);
  float xv[27];
  uint32_t inside;
  if (AHEAD)
    c1m_issue_patch(x, g_first * 64u + (uint32_t)lane, total_pix, H, W, sH, sW, pH, pW, OH, OW, divOW, divOH, xv, inside);
  filters.stage(sTap, sSc, sBi, nch, has_affine != 0);
  __syncthreads();  // the only barrier

  const size_t ohw = (size_t)OH * OW;
  for (int gi = 0; gi < groups_per_wave; ++gi) {
    const uint32_t grp = g_first + (uint32_t)gi;
    if (grp >= ngroups) break;  // wave-uniform
    if (!AHEAD || gi > 0)
      c1m_issue_patch(x, grp * 64u + (uint32_t)lane, total_pix, H, W, sH, sW, pH, pW, OH, OW, divOW, divOH, xv, inside);
#pragma unroll
    for (int k = 0; k < 27; ++k) xv[k] = ((inside >> (k % 9)) & 1u) ? xv[k] : 0.0f;
    // NCHW offsets of (image, channel 0, pixel) for the two pixels this lane holds results of
    size_t obase[2];
    bool ov[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const uint32_t q = grp * 64u + 32u * (uint32_t)b + (uint32_t)l32;
      ov[b] = q < total_pix;
      const uint32_t qc = ov[b] ? q : 0u;
      const uint32_t qn = fdiv(fdiv(qc, divOW), divOH);
      obase[b] = (size_t)qn * D * ohw + ((size_t)qc - (size_t)qn * ohw);
    }
#pragma unroll 1
    for (int g = 0; g < NG; ++g) {
      if (32 * g >= nch) break;  // workgroup-uniform
      const c1m_v32f acc = c1m_chain<NG>(sTap + 32 * g + l32, xv);
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int rr = 0; rr < 16; ++rr) {
          const int chl = 32 * g + 8 * (rr >> 2) + 4 * half + (rr & 3);
          if (chl < nch && ov[b]) {
            const float a = acc[16 * b + rr];
            outf[obase[b] + (size_t)(ch0 + chl) * ohw] = has_affine ? fmaf(sSc[chl], a, sBi[chl]) : a;
          }
        }
    }
  }
}

// Launch shape of the matrix-core first layer: one wave per `*gpw` groups of 64 pixels (enough
// groups per wave to amortise the filter staging, enough waves to give every SIMD four).
static dim3 c1m_grid(int64_t total_pix, int D, int ng, int *gpw, int64_t wave_slots = 4096) {
  const int64_t ngroups = (total_pix + 63) / 64;
  int64_t g = ngroups / wave_slots;
  g = g < 1 ? 1 : (g > 8 ? 8 : g);
  *gpw = (int)g;
  const int64_t waves = (ngroups + g - 1) / g;
  return dim3((unsigned)((waves + 3) / 4), (unsigned)((D + 32 * ng - 1) / (32 * ng)));
}

// Chains for the signs of more than a few pixels: four channel groups per workgroup from more than 24 pairs of 64 pixels and 32
// channels a unit on, or 12 if a SIMD gets more than four waves per 128 channels (32 x 32 maps, 128 channels: batch 63 9.2 us, one group
// 8.4; batch 128 13.5 against 14.0; batch 63, 512 channels 21.9, 26.6).
static bool first_chains_by_four(int64_t total_pix, int D, int64_t cu) {
  const int64_t groups = (total_pix + 63) / 64, q = groups * (((int64_t)D + 31) / 32);
  return q > 24 * cu || (q > 12 * cu && groups > 4 * cu);
}

// Filter bank of a fully-connected layer whose input is a flattened NCHW map [C, H, W],
// re-ordered to the packed NHWC bit order (h, w, c) of the activations: a common
// permutation of the reduction axis leaves the result unchanged.
__global__ __launch_bounds__(256) void pack_fc_weight_nhwc_kernel(const float *__restrict__ w, int C, int HW, int Cw,
                                                                  uint64_t *__restrict__ out, int64_t total_words) {
  const int lane = threadIdx.x & 63;
  const int64_t g = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (g >= total_words) return;
  const int cw = (int)(g % Cw);
  const int hw = (int)((g / Cw) % HW);
  const int64_t n = g / ((int64_t)Cw * HW);
  const int c = cw * 64 + lane;
  float v = -1.0f;
  if (c < C) v = w[(n * C + c) * HW + hw];
  const uint64_t m = __ballot(v >= 0.0f);
  if (lane == 0) out[g] = m;
}

}  // namespace bnn

using namespace bnn;

static bnn_status conv2d_impl(const float *x, const uint64_t *w_packed, int N, int C, int H, int W, int D, int kH,
                              int kW, int sH, int sW, int pH, int pW, int32_t *out_i32, float *out_f32,
                              const float *scale, const float *bias, void *workspace, size_t workspace_bytes,
                              void *stream, const GemmTune &tune) {
  bnn_status st = check_conv_geometry(N, C, H, W, kH, kW, sH, sW, pH, pW);
  if (st != BNN_OK) return st;
  if (D < 0) return BNN_ERR_SHAPE;
  if (N == 0 || D == 0) return BNN_OK;
  if (!x || !w_packed || !workspace || (!out_i32 && !out_f32)) return BNN_ERR_NULL;
  if (out_f32 && (!scale || !bias)) return BNN_ERR_NULL;
  if (!aligned16(x) || !aligned16(w_packed) || !aligned16(workspace) || (out_i32 && !aligned16(out_i32)) ||
      (out_f32 && !aligned16(out_f32)))
    return BNN_ERR_ALIGN;
  const size_t need = bnn_conv2d_workspace_bytes(N, C, H, W, kH, kW, sH, sW, pH, pW);
  if (workspace_bytes < need) return BNN_ERR_WORKSPACE;
  st = conv_limits(N, C, H, W, D, kH, kW, sH, sW, pH, pW);
  if (st != BNN_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  uint64_t *img = reinterpret_cast<uint64_t *>(workspace);
  if (kH == 1 && kW == 1 && pH == 0 && pW == 0) {
    // no patch expansion: encode and multiply only the sampled pixels
    GemmParams p = conv_gemm(nullptr, w_packed, N, C, H, W, D, 1, 1, sH, sW, 0, 0, 0, out_i32, out_f32, nullptr, scale, bias);
    if (tune.cfg < 0 && pointwise_applicable(p)) return launch_conv_pointwise(p, x, img, s);
    // the same in two launches: a stride-1 1x1 problem on the encoded pixels
    const int OH = (int)bnn_conv_out_dim(H, 1, sH, 0), OW = (int)bnn_conv_out_dim(W, 1, sW, 0);
    st = launch_encode_nchw(x, N, C, H, W, OH, OW, sH, sW, img, s);
    if (st != BNN_OK) return st;
    return conv_from_packed(img, w_packed, N, C, OH, OW, D, 1, 1, 1, 1, 0, 0, 0, out_i32, out_f32, nullptr, scale,
                            bias, s, tune);
  }
  if (tune.cfg < 0 ? tune.lean != 0 : tune.cfg == 40 || tune.cfg == 41) {
    GemmParams p = conv_gemm(nullptr, w_packed, N, C, H, W, D, kH, kW, sH, sW, pH, pW, 0, out_i32, out_f32, nullptr, scale, bias);
    p.n_cu = device_cu_count();
    const int shape = conv_image_shape(p, tune.cfg < 0 ? -1 : tune.cfg - 40);
    if (shape >= 0) return launch_conv_image(p, x, img, shape, s);
  }
  st = launch_encode_nchw(x, N, C, H, W, H, W, 1, 1, img, s);
  if (st != BNN_OK) return st;
  return conv_from_packed(img, w_packed, N, C, H, W, D, kH, kW, sH, sW, pH, pW, 0, out_i32, out_f32, nullptr, scale,
                          bias, s, tune);
}

extern "C" bnn_status bnn_conv2d(const float *x, const uint64_t *w_packed, int N, int C, int H, int W, int D, int kH,
                                 int kW, int sH, int sW, int pH, int pW, int32_t *out_i32, float *out_f32,
                                 const float *scale, const float *bias, void *workspace, size_t workspace_bytes,
                                 void *stream) {
  return conv2d_impl(x, w_packed, N, C, H, W, D, kH, kW, sH, sW, pH, pW, out_i32, out_f32, scale, bias, workspace,
                     workspace_bytes, stream, GemmTune());
}

// ---- bnn_conv2d for callers that cannot allocate ---------------------------------------------
// The packed image goes to a fixed array in device memory instead of a caller workspace.  Every
// GPU the library runs on holds its own copy of the array (at its own address) until the process
// ends.  In host code the array's name is only a handle: its device address is looked up once per
// device, with that device current, and from then on only that address is used.
static __device__ __align__(256) unsigned char scratch[BNN_CONV2D_NOALLOC_MAX_BYTES];

namespace {
constexpr int NOALLOC_MAX_DEVICES = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[NOALLOC_MAX_DEVICES] = {nullptr};

// Device address of `scratch` on the current device, or nullptr on failure.
void *scratch_address() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= NOALLOC_MAX_DEVICES) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void *ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) {
      (void)hipGetLastError();
      return nullptr;
    }
    g_scratch_ptr[dev] = ptr;
  }
  return g_scratch_ptr[dev];
}
}  // namespace

extern "C" size_t bnn_conv2d_noalloc_max_bytes(void) { return BNN_CONV2D_NOALLOC_MAX_BYTES; }

extern "C" bnn_status bnn_conv2d_noalloc(const float *x, const uint64_t *w_packed, int N, int C, int H, int W, int D,
                                         int kH, int kW, int sH, int sW, int pH, int pW, int32_t *out_i32,
                                         float *out_f32, const float *scale, const float *bias, void *stream) {
  // the size check comes first and needs no device: a request over the limit never reaches HIP
  bnn_status st = check_conv_geometry(N, C, H, W, kH, kW, sH, sW, pH, pW);
  if (st != BNN_OK) return st;
  if (D < 0) return BNN_ERR_SHAPE;
  if (N == 0 || D == 0) return BNN_OK;
  const size_t need = bnn_conv2d_workspace_bytes(N, C, H, W, kH, kW, sH, sW, pH, pW);
  if (need > BNN_CONV2D_NOALLOC_MAX_BYTES) return BNN_ERR_WORKSPACE;
  if (!x || !w_packed || (!out_i32 && !out_f32)) return BNN_ERR_NULL;
  if (out_f32 && (!scale || !bias)) return BNN_ERR_NULL;
  if (!aligned16(x) || !aligned16(w_packed) || (out_i32 && !aligned16(out_i32)) || (out_f32 && !aligned16(out_f32)))
    return BNN_ERR_ALIGN;
  void *ptr = scratch_address();
  if (!ptr) return BNN_ERR_HIP;
  return conv2d_impl(x, w_packed, N, C, H, W, D, kH, kW, sH, sW, pH, pW, out_i32, out_f32, scale, bias, ptr,
                     BNN_CONV2D_NOALLOC_MAX_BYTES, stream, GemmTune());
}

// Declared in bnn_testing.h.
extern "C" bnn_status bnn_testing_conv2d(const float *x, const uint64_t *w_packed, int N, int C, int H, int W, int D,
                                         int kH, int kW, int sH, int sW, int pH, int pW, int32_t *out_i32,
                                         float *out_f32, const float *scale, const float *bias, void *workspace,
                                         size_t workspace_bytes, int cfg, int lean, void *stream) {
  GemmTune tune;
  tune.cfg = cfg;
  tune.lean = lean;
  return conv2d_impl(x, w_packed, N, C, H, W, D, kH, kW, sH, sW, pH, pW, out_i32, out_f32, scale, bias, workspace,
                     workspace_bytes, stream, tune);
}

static bnn_status conv2d_packed_impl(const uint64_t *x_packed, const uint64_t *w_packed, int N, int C, int H, int W,
                                     int D, int kH, int kW, int sH, int sW, int pH, int pW, int pool,
                                     int32_t *out_i32, float *out_f32, uint64_t *out_packed, const float *scale,
                                     const float *bias, void *stream, const GemmTune &tune) {
  bnn_status st = check_conv_geometry(N, C, H, W, kH, kW, sH, sW, pH, pW);
  if (st != BNN_OK) return st;
  if (D < 0 || (pool != 0 && pool != 2)) return BNN_ERR_SHAPE;
  const int64_t OH = bnn_conv_out_dim(H, kH, sH, pH), OW = bnn_conv_out_dim(W, kW, sW, pW);
  if (pool == 2 && ((OH & 1) || (OW & 1))) return BNN_ERR_SHAPE;
  if (N == 0 || D == 0) return BNN_OK;
  if (!x_packed || !w_packed || (!out_i32 && !out_f32 && !out_packed)) return BNN_ERR_NULL;
  if ((out_f32 || out_packed) && (!scale || !bias)) return BNN_ERR_NULL;
  if (out_packed && (out_i32 || out_f32)) return BNN_ERR_UNSUPPORTED;  // one kind of output per call
  if (pool == 2 && !out_packed) return BNN_ERR_UNSUPPORTED;            // pooling lives in the packed epilogue
  if (!aligned16(x_packed) || !aligned16(w_packed) || (out_i32 && !aligned16(out_i32)) ||
      (out_f32 && !aligned16(out_f32)) || (out_packed && !aligned16(out_packed)))
    return BNN_ERR_ALIGN;
  st = conv_limits(N, C, H, W, D, kH, kW, sH, sW, pH, pW);
  if (st != BNN_OK) return st;
  return conv_from_packed(x_packed, w_packed, N, C, H, W, D, kH, kW, sH, sW, pH, pW, pool, out_i32, out_f32,
                          out_packed, scale, bias, (hipStream_t)stream, tune);
}

extern "C" bnn_status bnn_conv2d_packed(const uint64_t *x_packed, const uint64_t *w_packed, int N, int C, int H, int W,
                                        int D, int kH, int kW, int sH, int sW, int pH, int pW, int pool,
                                        int32_t *out_i32, float *out_f32, uint64_t *out_packed, const float *scale,
                                        const float *bias, void *stream) {
  return conv2d_packed_impl(x_packed, w_packed, N, C, H, W, D, kH, kW, sH, sW, pH, pW, pool, out_i32, out_f32,
                            out_packed, scale, bias, stream, GemmTune());
}

// Declared in bnn_testing.h.
extern "C" bnn_status bnn_testing_conv2d_packed(const uint64_t *x_packed, const uint64_t *w_packed, int N, int C,
                                                int H, int W, int D, int kH, int kW, int sH, int sW, int pH, int pW,
                                                int pool, int32_t *out_i32, float *out_f32, uint64_t *out_packed,
                                                const float *scale, const float *bias, int cfg, int lean,
                                                void *stream) {
  GemmTune tune;
  tune.cfg = cfg;
  tune.lean = lean;
  return conv2d_packed_impl(x_packed, w_packed, N, C, H, W, D, kH, kW, sH, sW, pH, pW, pool, out_i32, out_f32,
                            out_packed, scale, bias, stream, tune);
}

// Declared in bnn_testing.h.
extern "C" int bnn_testing_conv_region(int N, int C, int H, int W, int kH, int kW, int sH, int sW, int pH, int pW,
                                       int pool, int columns, int64_t *region) {
  if (check_conv_geometry(N, C, H, W, kH, kW, sH, sW, pH, pW) != BNN_OK || N == 0 || !region || columns <= 0 ||
      (pool != 0 && pool != 2))
    return -1;
  if (pool && ((bnn_conv_out_dim(H, kH, sH, pH) & 1) || (bnn_conv_out_dim(W, kW, sW, pW) & 1))) return -1;
  GemmParams p = {};
  fill_geom(p.g, nullptr, N, C, H, W, kH, kW, sH, sW, pH, pW, pool);
  p.Kw64 = (int)bnn_conv_kwords(C, kH, kW);
  int64_t rows = 0;
  if (!halo_region(p, columns, pool != 0, rows)) return 0;
  const int64_t v[BNN_TESTING_REGION_VALUES] = {rows, p.halo.Wp, p.halo.plane, p.halo.bytes};
  for (int i = 0; i < BNN_TESTING_REGION_VALUES; ++i) region[i] = v[i];
  return 1;
}

// Declared in bnn_testing.h.
extern "C" int bnn_testing_conv_word(int N, int C, int H, int W, int D, int kH, int kW, int sH, int sW, int pH, int pW, int pool,
                                     int packed, int units) {
  if (check_conv_geometry(N, C, H, W, kH, kW, sH, sW, pH, pW) != BNN_OK || N == 0 || D <= 0 || units <= 0 ||
      (pool != 0 && pool != 2) || (pool && packed != 1) || packed < 0 || packed > 2)
    return -1;
  if (pool && ((bnn_conv_out_dim(H, kH, sH, pH) & 1) || (bnn_conv_out_dim(W, kW, sW, pW) & 1))) return -1;
  if (conv_limits(N, C, H, W, D, kH, kW, sH, sW, pH, pW) != BNN_OK) return -1;
  const uintptr_t i32 = packed == 1 ? 0 : 4096, f32 = packed == 2 ? 4096 : 0;  // not read
  GemmParams p = conv_gemm(nullptr, nullptr, N, C, H, W, D, kH, kW, sH, sW, pH, pW, pool, reinterpret_cast<int32_t *>(i32),
                           reinterpret_cast<float *>(f32), nullptr, nullptr, nullptr);
  p.n_cu = units;
  return !conv_word_applicable(p, 1) ? 0 : conv_word_faster(p, packed == 1) ? 2 : 1;
}

// Declared in bnn_testing.h.
extern "C" int bnn_testing_conv_word_nontemporal(int N, int C, int H, int W, int D, int kH, int kW, int sH, int sW, int pH, int pW) {
  if (check_conv_geometry(N, C, H, W, kH, kW, sH, sW, pH, pW) != BNN_OK || N == 0 || D <= 0 ||
      conv_limits(N, C, H, W, D, kH, kW, sH, sW, pH, pW) != BNN_OK)
    return -1;
  const GemmParams p = conv_gemm(nullptr, nullptr, N, C, H, W, D, kH, kW, sH, sW, pH, pW, 0, reinterpret_cast<int32_t *>((uintptr_t)4096),
                                 nullptr, nullptr, nullptr, nullptr);
  return !conv_word_applicable(p, 1) ? -1 : nontemporal_maps(p, 1, true) ? 1 : 0;
}

// Declared in bnn_testing.h.
extern "C" int bnn_testing_conv_image(int N, int C, int H, int W, int D, int kH, int kW, int sH, int sW, int pH, int pW,
                                      int units, int shape, int pixel, int64_t *rows) {
  if (check_conv_geometry(N, C, H, W, kH, kW, sH, sW, pH, pW) != BNN_OK || N == 0 || D <= 0 || units <= 0 || !rows || shape > 1 ||
      conv_limits(N, C, H, W, D, kH, kW, sH, sW, pH, pW) != BNN_OK)
    return -1;
  GemmParams p = conv_gemm(nullptr, nullptr, N, C, H, W, D, kH, kW, sH, sW, pH, pW, 0, nullptr, nullptr, nullptr, nullptr, nullptr);
  p.n_cu = units;
  if (pixel < 0 || pixel >= p.N) return -1;
  const int r = conv_image_shape(p, shape);
  if (r >= 0) conv_image_rows(p, pixel, rows);
  return r;
}

// Declared in bnn_testing.h.
extern "C" int bnn_testing_first_sign(int N, int H, int W, int D, int sH, int sW, int pH, int pW, int units) {
  if (check_conv_geometry(N, 3, H, W, 3, 3, sH, sW, pH, pW) != BNN_OK || N == 0 || D <= 0 || units <= 0) return -1;
  const int shape = first_sign_f16(N, H, W, D, sH, sW, pH, pW, units);
  const int64_t total = (int64_t)N * bnn_conv_out_dim(H, 3, sH, pH) * bnn_conv_out_dim(W, 3, sW, pW);
  return shape >= 0 ? 2 + shape : first_chains_by_four(total, D, units) ? 1 : 0;
}

extern "C" bnn_status bnn_conv2d_f32_sign(const float *x, const float *w, int N, int C, int H, int W, int D, int kH,
                                          int kW, int sH, int sW, int pH, int pW, const float *scale,
                                          const float *bias, uint64_t *out_packed, void *stream) {
  bnn_status st = check_conv_geometry(N, C, H, W, kH, kW, sH, sW, pH, pW);
  if (st != BNN_OK) return st;
  if (D < 0) return BNN_ERR_SHAPE;
  if (N == 0 || D == 0) return BNN_OK;
  if (!x || !w || !scale || !bias || !out_packed) return BNN_ERR_NULL;
  if (!aligned16(x) || !aligned16(w) || !aligned16(out_packed)) return BNN_ERR_ALIGN;
  const int64_t K = (int64_t)C * kH * kW;
  if (K > F32S_KMAX) return BNN_ERR_UNSUPPORTED;
  const int64_t OH = bnn_conv_out_dim(H, kH, sH, pH), OW = bnn_conv_out_dim(W, kW, sW, pW);
  const int64_t total = (int64_t)N * OH * OW;
  if (total > 0x7fffffffLL) return BNN_ERR_UNSUPPORTED;
  hipStream_t s = (hipStream_t)stream;
  {
    ProfScope ps(KID_CONV_F32_SIGN, s);
    const dim3 block(256);
    if (K == 27 && C == 3 && kH == 3 && kW == 3) {
      const int shape = first_sign_f16(N, H, W, D, sH, sW, pH, pW, device_cu_count());
      if (shape >= 0) return launch_first_sign_f16(x, w, N, H, W, D, sH, sW, pH, pW, scale, bias, out_packed, shape, s);
      const bool four = first_chains_by_four(total, D, device_cu_count());
      int gpw;
      const dim3 grid = c1m_grid(total, D, four ? 4 : 1, &gpw);
      hipLaunchKernelGGL((four ? conv2d_f32_k27_mfma_sign_kernel<4> : conv2d_f32_k27_mfma_sign_kernel<1>), grid, block, 0, s, x, w, H,
                         W, D, sH, sW, pH, pW, (int)OH, (int)OW, scale, bias, out_packed, (int)bnn_packed_words(D),
                         FastDiv((uint32_t)OW), FastDiv((uint32_t)OH), (uint32_t)total, (uint32_t)((total + 63) / 64), gpw);
    } else {
      const dim3 grid((unsigned)((total + 255) / 256));
      hipLaunchKernelGGL(conv2d_f32_sign_kernel<0>, grid, block, 0, s, x, w, C, H, W, D, kH, kW, sH, sW, pH, pW,
                         (int)OH, (int)OW, scale, bias, out_packed, (int)bnn_packed_words(D), FastDiv((uint32_t)OW),
                         FastDiv((uint32_t)OH), (uint32_t)total, (int)K);
    }
  }
  return launch_status();
}

namespace bnn {
// 3x3x3 real-valued convolution with fp32 NCHW output on the kernel above (arguments validated by
// the caller; scale and bias both given or both null).
bnn_status launch_conv2d_f32_k27(const float *x, const float *w, int N, int H, int W, int D, int sH, int sW, int pH,
                                 int pW, const float *scale, const float *bias, float *out, hipStream_t s) {
  const int64_t OH = bnn_conv_out_dim(H, 3, sH, pH), OW = bnn_conv_out_dim(W, 3, sW, pW);
  const int64_t total = (int64_t)N * OH * OW;
  // One channel group per workgroup: the stores of the map hide the repeated loads (32 x 32 maps, 128 channels: batch 1
  // 17.6 -> 6.0 us, batch 64 20.6 -> 13.2, batch 256 45.8 -> 38.8; 32 x 128 x 224 x 224 255 -> 219), but not those of many
  // groups into a large map, which take four (256 x 384 x 32 x 32 132 -> 102 us, 8 x 512 x 224 x 224 237 -> 210, 128 x 1024 x
  // 56 x 56 474 -> 403; 16 x 256 x 224 x 224 217 against 229, 4 x 384 x 224 x 224 80 against 81).
  const bool four = D > 256 && total * D * 4 > 350000000;
  int gpw;
  const dim3 grid = c1m_grid(total, D, four ? 4 : 1, &gpw, four ? 2048 : 4096), block(256);
  const FastDiv dOW((uint32_t)OW), dOH((uint32_t)OH);
  const uint32_t ngroups = (uint32_t)((total + 63) / 64);
  if (four)
    hipLaunchKernelGGL(conv2d_f32_k27_mfma_kernel<4>, grid, block, 0, s, x, w, H, W, D, sH, sW, pH, pW, (int)OH, (int)OW,
                       scale, bias, dOW, dOH, (uint32_t)total, ngroups, gpw, out, scale ? 1 : 0);
  else
    hipLaunchKernelGGL(conv2d_f32_k27_mfma_kernel<1>, grid, block, 0, s, x, w, H, W, D, sH, sW, pH, pW, (int)OH, (int)OW,
                       scale, bias, dOW, dOH, (uint32_t)total, ngroups, gpw, out, scale ? 1 : 0);
  return launch_status();
}
}  // namespace bnn

extern "C" bnn_status bnn_pack_fc_weight_nhwc(const float *w, int64_t Nout, int C, int H, int W, uint64_t *w_packed,
                                              void *stream) {
  if (Nout < 0 || C <= 0 || H <= 0 || W <= 0) return BNN_ERR_SHAPE;
  if (Nout == 0) return BNN_OK;
  if (!w || !w_packed) return BNN_ERR_NULL;
  if (!aligned16(w) || !aligned16(w_packed)) return BNN_ERR_ALIGN;
  const int64_t Cw = bnn_packed_words(C);
  const int64_t HW = (int64_t)H * W;
  if (HW > 0x7fffffffLL || Nout * C * HW > 0x7fffffffLL * 64) return BNN_ERR_UNSUPPORTED;
  const int64_t total = Nout * HW * Cw;
  const int64_t blocks = (total + 3) / 4;
  if (blocks > 0x7fffffffLL) return BNN_ERR_UNSUPPORTED;
  hipStream_t s = (hipStream_t)stream;
  {
    ProfScope ps(KID_PACK_CONV_WEIGHT, s);
    hipLaunchKernelGGL(pack_fc_weight_nhwc_kernel, dim3((unsigned)blocks), dim3(256), 0, s, w, C, (int)HW, (int)Cw,
                       w_packed, total);
  }
  return launch_status();
}
