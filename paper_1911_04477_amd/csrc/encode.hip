// Sign-encode kernels (section 3.1 of the paper: value -1 <-> bit 0, +1 <-> bit 1).
//
// All three kernels are pure streaming: 4 bytes read and 1/8 byte written per
// element, so they are bound by HBM bandwidth.  Layout decisions:
//   * row-major matrices: lanes run along K, one v_cmp per 64 elements yields the
//     64-bit word directly (the wave-wide compare mask IS the packed word);
//     a wave covers 16 consecutive words so that 16 independent 256-byte loads are
//     in flight per wave and the 16 words leave in one contiguous 128-byte store.
//     The fp32 input is read exactly once, with non-temporal loads (5.44 -> 5.76 TB/s).
//   * NCHW images: the packing axis (channel) is strided by H*W floats, so lanes
//     run along pixels (coalesced 256-byte loads per channel) and every lane
//     shift-ORs 32 channels at a time; the four waves of a workgroup share the
//     channel axis of 64 pixels and assemble the packed NHWC words through LDS.
#include "common.h"

namespace bnn {

constexpr int ENC_BLOCK = 256;

// Where a word lies is uniform over the wave: addresses are running sums on the scalar unit and one offset per lane, the only
// division is by a constant of the launch.  Bound: the launch up to about 10 MB, then memory.  In a graph, against 64-bit
// divisions (one of them per lane) and an address and bounds per lane for every load: 16 x 256 3.35 -> 1.95 us, 256 x 4096 3.4 ->
// 2.45, 5000 x 1024 6.2 -> 2.9, 20000 x 4096 (328 MB) 60.5 -> 50.3, 32000 x 4000 94 -> 86.
constexpr int ENC_WORDS_PER_WAVE = 16;
__global__ __launch_bounds__(ENC_BLOCK) void encode_rows_kernel(const float *__restrict__ src, int64_t src_ld,
                                                                 uint64_t *__restrict__ dst, int64_t dst_ld, FastDiv divKw,
                                                                 uint32_t tail,  // values of a row's last word
                                                                 uint32_t total_words) {
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t g0 = (blockIdx.x * (ENC_BLOCK / 64) + wave) * ENC_WORDS_PER_WAVE;  // < 2^30
  if (g0 >= total_words) return;
  const uint32_t Kw = divKw.d, count = total_words - g0;  // words of this wave, if less than 16
  const uint32_t row = fdiv(g0, divKw);
  uint32_t w = g0 - row * Kw;
  const float *p = src + (int64_t)row * src_ld + (int64_t)w * 64;
  const int64_t gap = src_ld - (int64_t)Kw * 64;

  // All 16 loads are issued back to back, unconditionally; conditional ones would each wait for the previous one.  Read once:
  // non-temporal, out of the caches.
  float v[ENC_WORDS_PER_WAVE];
  uint64_t mine = 0;
  constexpr uint32_t LAST = ENC_WORDS_PER_WAVE - 1;
  if (count > LAST && (w + LAST < Kw || (gap == 0 && tail == 64u))) {
    // words of one row, or of rows without a gap between them: one address, and only the last word may be a partial one
    const uint32_t left = w + LAST == Kw - 1u ? tail : 64u;
#pragma unroll
    for (uint32_t u = 0; u < LAST; ++u) v[u] = __builtin_nontemporal_load(p + lane + 64u * u);
    v[LAST] = __builtin_nontemporal_load(p + min(lane, left - 1u) + 64u * LAST);
#pragma unroll
    for (uint32_t u = 0; u <= LAST; ++u) {
      const uint64_t m = __ballot(sign_bit(v[u])) & (u == LAST && left < 64u ? (1ull << left) - 1ull : ~0ull);
      if (lane == u) mine = m;
    }
  } else {
    // a lane past the end of a row re-reads its last value, words past the last one re-read the first value, both masked out
    uint32_t real[ENC_WORDS_PER_WAVE];  // values of the word, uniform
#pragma unroll
    for (uint32_t u = 0; u < ENC_WORDS_PER_WAVE; ++u) {
      const bool last = w + 1u == Kw, any = u < count;
      real[u] = !any ? 0u : last ? tail : 64u;
      v[u] = __builtin_nontemporal_load((any ? p : src) + min(lane, max(real[u], 1u) - 1u));
      p += last ? gap + 64 : 64;
      w = last ? 0u : w + 1u;
    }
#pragma unroll
    for (uint32_t u = 0; u < ENC_WORDS_PER_WAVE; ++u) {
      const uint64_t m = __ballot(sign_bit(v[u])) & (real[u] < 64u ? (1ull << real[u]) - 1ull : ~0ull);
      if (lane == u) mine = m;
    }
  }

  if (lane < ENC_WORDS_PER_WAVE && lane < count) {
    const uint32_t g = g0 + lane;
    int64_t o = g;
    if (dst_ld != (int64_t)Kw) {  // uniform
      const uint32_t r = fdiv(g, divKw);
      o = (int64_t)r * dst_ld + (g - r * Kw);
    }
    dst[o] = mine;
  }
}

// Filter bank [D,C,kH,kW] -> packed [D, kH*kW*Cw] in (kh, kw, c) order.  Tiny data
// (a few hundred KB at most), one wave per output word.
__global__ __launch_bounds__(256) void pack_conv_weight_kernel(const float *__restrict__ w, int D, int C,
                                                               int taps, int Cw,
                                                               uint64_t *__restrict__ out,
                                                               int64_t total_words) {
  const int lane = threadIdx.x & 63;
  const int64_t g = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (g >= total_words) return;
  const int cw = (int)(g % Cw);
  const int tap = (int)((g / Cw) % taps);
  const int64_t d = g / ((int64_t)Cw * taps);
  const int c = cw * 64 + lane;
  float v = -1.0f;
  if (c < C) v = w[(d * C + c) * taps + tap];
  const uint64_t m = __ballot(sign_bit(v));
  if (lane == 0) out[g] = m;
}

// NCHW fp32 -> packed pixels [N*OHp*OWp, Cw].  Output pixel (n, oh, ow) samples input
// pixel (oh*sH, ow*sW); with sH = sW = 1 and OHp = H, OWp = W this is the packed NHWC
// image, with the strides of a 1x1 / pad-0 convolution it is the patch matrix itself.
//
// A workgroup owns 64 consecutive output pixels (one per lane).  The channel axis is cut
// into granules of 32 channels (one half word) dealt round-robin to the workgroup's four
// waves, so four times as many waves stream as there are pixel groups and each lane has
// 32 independent plane-strided loads in flight per granule.  The half words meet in LDS
// and leave as one contiguous run of 64 * Cw words.  (A variant with four pixels per lane
// and 16-byte loads measured no faster, from cache or from HBM, and was dropped.)
constexpr int ENCN_PIX = 64;
__global__ __launch_bounds__(256) void encode_nchw_kernel(const float *__restrict__ x, int C, int H, int W,
                                                          int OHp, int OWp, int sH, int sW, FastDiv divOW,
                                                          FastDiv divOH, uint64_t *__restrict__ out,
                                                          uint32_t total_pix, int Cw) {
  extern __shared__ uint32_t s_half[];  // [64 pixels][2*Cw + 1]
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t p0 = blockIdx.x * (uint32_t)ENCN_PIX;
  const uint32_t p = p0 + lane;
  const uint32_t pc = p < total_pix ? p : total_pix - 1;  // lanes past the end re-read the last pixel
  const uint32_t t = fdiv(pc, divOW);
  const uint32_t ow = pc - t * OWp;
  const uint32_t n = fdiv(t, divOH);
  const uint32_t oh = t - n * OHp;
  const size_t plane = (size_t)H * W;
  // Address = wave-uniform 64-bit base (first image of the workgroup, channel plane) + a
  // 32-bit per-lane byte offset: one VGPR of address per lane instead of one pair per load.
  // The host checks that the offset (the images a workgroup can span) fits.
  const uint32_t n0 = fdiv(fdiv(p0 < total_pix ? p0 : total_pix - 1, divOW), divOH);
  const uint32_t off =
      (uint32_t)(((size_t)(n - n0) * C * plane + (size_t)(oh * sH) * W + (size_t)ow * sW) * sizeof(float));
  const char *xb = reinterpret_cast<const char *>(x + (size_t)n0 * C * plane);
#define BNN_ENC_LD(c) \
  __builtin_nontemporal_load(reinterpret_cast<const float *>(xb + (size_t)(c) * plane * sizeof(float) + off))
  const int G = 2 * Cw;  // granules, the last ones possibly partial or empty
  const int rs = G + 1;
  for (int g = wave; g < G; g += 4) {
    const int c0 = g * 32;
    const int left = C - c0;  // real channels in this granule
    uint32_t acc = 0;
    if (left >= 32) {
      float v[32];
#pragma unroll
      for (int j = 0; j < 32; ++j) v[j] = BNN_ENC_LD(c0 + j);
#pragma unroll
      for (int j = 0; j < 32; ++j) acc |= (uint32_t)sign_bit(v[j]) << j;
    } else if (left > 0) {
      // channels past C re-read the last channel and are masked out
      float v[32];
#pragma unroll
      for (int j = 0; j < 32; ++j) v[j] = BNN_ENC_LD(c0 + (j < left ? j : left - 1));
#pragma unroll
      for (int j = 0; j < 32; ++j) acc |= (uint32_t)sign_bit(v[j]) << j;
      acc &= (1u << left) - 1u;
    }
    s_half[lane * rs + g] = acc;
  }
#undef BNN_ENC_LD
  __syncthreads();
  // 64 * Cw words, contiguous in global memory from pixel p0
  const uint32_t nwords = (uint32_t)ENCN_PIX * (uint32_t)Cw;
  const uint64_t limit = (uint64_t)total_pix * (uint64_t)Cw;
  uint64_t *o = out + (size_t)p0 * Cw;
  for (uint32_t j = threadIdx.x; j < nwords; j += 256u) {
    if ((uint64_t)p0 * Cw + j >= limit) break;
    const uint32_t pix = j / (uint32_t)Cw, cw = j - pix * (uint32_t)Cw;
    const uint32_t lo = s_half[pix * rs + 2 * cw], hi = s_half[pix * rs + 2 * cw + 1];
    o[j] = ((uint64_t)hi << 32) | lo;
  }
}

// The same encode for a column stride above 1 (the sampled pixels of a strided 1x1 / pad-0
// convolution).  A wave's load then uses only every sW-th float of the sectors it touches, rows
// between the sampled ones are skipped, and what bounds the kernel is how many independent
// requests are in flight rather than bytes: a read-only kernel over the same addresses tops out
// at 60 % of the streaming rate.  So every wave works alone on 64 pixels x ONE granule of 16
// channels (16 loads in flight per lane), keeps its 16 sign bits per pixel and writes them
// straight to its quarter of the pixel's word: no LDS, no barrier, four times as many waves.
// The partial-word stores meet in the L2; the packed output is 1/32 of the input.  (Measured on
// the 64 x 200 x 56 x 56 input with stride 2: 19.4 us against 24.1 us for the kernel above;
// for stride 1 the kernel above is the faster one at every size tried.)
constexpr int ENCS_GR = 16;
__global__ __launch_bounds__(256) void encode_nchw_sampled_kernel(const float *__restrict__ x, int C, int H, int W,
                                                                  int OHp, int OWp, int sH, int sW, FastDiv divOW,
                                                                  FastDiv divOH, uint16_t *__restrict__ out,
                                                                  uint32_t total_pix, int Cw) {
  const uint32_t p = blockIdx.x * 256u + threadIdx.x;
  const int g = blockIdx.y;  // granule: channels [16 g, 16 g + 16)
  const uint32_t pc = p < total_pix ? p : total_pix - 1;  // lanes past the end re-read the last pixel
  const uint32_t t = fdiv(pc, divOW);
  const uint32_t ow = pc - t * OWp;
  const uint32_t n = fdiv(t, divOH);
  const uint32_t oh = t - n * OHp;
  const size_t plane = (size_t)H * W;
  const float *xp = x + (size_t)n * C * plane + (size_t)(oh * sH) * W + (size_t)ow * sW;
  const int c0 = g * ENCS_GR;
  const int left = C - c0;  // real channels in this granule; <= 0 for the padding granules of the last word
  uint32_t acc = 0;
  if (left > 0) {
    float v[ENCS_GR];
#pragma unroll
    for (int j = 0; j < ENCS_GR; ++j)  // channels past C re-read the last channel and are masked out
      v[j] = __builtin_nontemporal_load(xp + (size_t)(c0 + (j < left ? j : left - 1)) * plane);
#pragma unroll
    for (int j = 0; j < ENCS_GR; ++j) acc |= (uint32_t)sign_bit(v[j]) << j;
    if (left < ENCS_GR) acc &= (1u << left) - 1u;
  }
  if (p < total_pix) out[(size_t)p * (4 * Cw) + g] = (uint16_t)acc;
}

}  // namespace bnn

using namespace bnn;

extern "C" bnn_status bnn_encode(const float *src, int64_t rows, int64_t K, int64_t src_ld, uint64_t *dst,
                                 int64_t dst_ld, void *stream) {
  if (rows < 0) return BNN_ERR_SHAPE;
  if (K <= 0) return BNN_ERR_SHAPE;
  const int64_t Kw = bnn_packed_words(K);
  if (src_ld < K || dst_ld < Kw) return BNN_ERR_STRIDE;
  if (rows == 0) return BNN_OK;
  if (!src || !dst) return BNN_ERR_NULL;
  if (!aligned16(src) || !aligned16(dst)) return BNN_ERR_ALIGN;
  if (rows > (INT64_MAX / 4) / src_ld) return BNN_ERR_UNSUPPORTED;
  constexpr int64_t per_block = (ENC_BLOCK / 64) * ENC_WORDS_PER_WAVE, most = (1LL << 30) - per_block;
  if (Kw > most) return BNN_ERR_UNSUPPORTED;  // a row of 2^36 values: 256 GB
  hipStream_t s = (hipStream_t)stream;
  {
    ProfScope ps(KID_ENCODE_ROWS, s);
    // words are numbered in 31 bits, the threads of a launch in 32
    for (int64_t r = 0; r < rows;) {
      const int64_t n = rows - r < most / Kw ? rows - r : most / Kw, total = n * Kw;
      hipLaunchKernelGGL(encode_rows_kernel, dim3((unsigned)((total + per_block - 1) / per_block)), dim3(ENC_BLOCK), 0, s,
                         src + r * src_ld, src_ld, dst + r * dst_ld, dst_ld, FastDiv((uint32_t)Kw), (uint32_t)(K - 64 * (Kw - 1)),
                         (uint32_t)total);
      r += n;
    }
  }
  return launch_status();
}

extern "C" bnn_status bnn_pack_conv_weight(const float *w, int D, int C, int kH, int kW, uint64_t *w_packed,
                                           void *stream) {
  if (D < 0 || C <= 0 || kH <= 0 || kW <= 0) return BNN_ERR_SHAPE;
  if (D == 0) return BNN_OK;
  if (!w || !w_packed) return BNN_ERR_NULL;
  if (!aligned16(w) || !aligned16(w_packed)) return BNN_ERR_ALIGN;
  const int64_t taps = (int64_t)kH * kW;
  const int64_t Cw = bnn_packed_words(C);
  if (taps > 0x7fff || (int64_t)D * C * taps > 0x7fffffffLL) return BNN_ERR_UNSUPPORTED;
  const int64_t total = (int64_t)D * taps * Cw;
  const int64_t blocks = (total + 3) / 4;
  if (blocks > 0x7fffffffLL) return BNN_ERR_UNSUPPORTED;
  hipStream_t s = (hipStream_t)stream;
  {
    ProfScope ps(KID_PACK_CONV_WEIGHT, s);
    hipLaunchKernelGGL(pack_conv_weight_kernel, dim3((unsigned)blocks), dim3(256), 0, s, w, D, C, (int)taps,
                       (int)Cw, w_packed, total);
  }
  return launch_status();
}

namespace bnn {
// Sizes that launch_encode_nchw takes.
bool encode_nchw_supported(int N, int C, int H, int W, int OHp, int OWp) {
  if ((int64_t)N * OHp * OWp > 0x7fffffffLL) return false;
  if ((int64_t)ENCN_PIX * (2 * bnn_packed_words(C) + 1) * (int64_t)sizeof(uint32_t) > 64 * 1024) return false;  // C > 8128
  // 32-bit per-lane byte offsets: a workgroup's 64 pixels span at most `span` images past its first
  const int64_t span = (ENCN_PIX + (int64_t)OHp * OWp - 1) / ((int64_t)OHp * OWp);
  return (span + 1) * (int64_t)C * H * W * 4 <= 0x7fffffffLL;
}

// Host launcher used by the im2col / conv drivers.  Arguments are validated by the caller.
bnn_status launch_encode_nchw(const float *x, int N, int C, int H, int W, int OHp, int OWp, int sH, int sW,
                              uint64_t *out, hipStream_t s) {
  const int64_t total = (int64_t)N * OHp * OWp;
  if (total == 0) return BNN_OK;
  if (!encode_nchw_supported(N, C, H, W, OHp, OWp)) return BNN_ERR_UNSUPPORTED;
  const int Cw = (int)bnn_packed_words(C);
  const unsigned blocks = (unsigned)((total + ENCN_PIX - 1) / ENCN_PIX);
  const size_t lds = (size_t)ENCN_PIX * (2 * Cw + 1) * sizeof(uint32_t);
  FastDiv dOW((uint32_t)OWp), dOH((uint32_t)OHp);
  ProfScope ps(KID_ENCODE_NCHW, s);
  if (sW > 1 && 4 * Cw <= 65535) {
    const dim3 grid((unsigned)((total + 255) / 256), (unsigned)(4 * Cw));
    hipLaunchKernelGGL(encode_nchw_sampled_kernel, grid, dim3(256), 0, s, x, C, H, W, OHp, OWp, sH, sW, dOW, dOH,
                       reinterpret_cast<uint16_t *>(out), (uint32_t)total, Cw);
    return launch_status();
  }
  hipLaunchKernelGGL(encode_nchw_kernel, dim3(blocks), dim3(256), lds, s, x, C, H, W, OHp, OWp, sH, sW, dOW, dOH, out,
                     (uint32_t)total, Cw);
  return launch_status();
}
}  // namespace bnn
