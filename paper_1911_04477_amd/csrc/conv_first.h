// The real-valued 3x3x3 first layer: the fused multiply-add chains of its outputs on the fp32 matrix cores, shared by the
// kernels that need them for every output (conv.hip) and for the few whose sign is in doubt (conv_first_sign.hip).
#pragma once
#include "common.h"

namespace bnn {

// ---- the 3x3x3 layer (K = 27) on the fp32 matrix cores --------------------------------------
// V_MFMA_F32_32X32X1_2B_F32 multiplies a 32 x 1 column by a 1 x 32 row and adds the 32 x 32
// product to its accumulator, for two independent blocks at once; one reduction step at a time,
// each output element goes through exactly the fused multiply-add chain over (c, kh, kw) that
// the general kernel above runs (checked bit for bit against fmaf chains, denormals, infinities
// and signed zeros included), at twice the rate of unpacked vector multiply-adds.
//   rows (operand A)    : 32 output channels; lanes l and l + 32 hold the same filter tap
//   columns (operand B) : the wave's 64 pixels, block 0 = pixels 0..31, block 1 = pixels 32..63;
//                         lane l supplies the patch value of pixel l
//   accumulators        : register r of block b, lane l = channel 8*(r/4) + 4*(l/32) + r%4 of
//                         pixel 32*b + l%32
// A workgroup of four waves stages the filter taps of 32 * NG channels in LDS ([tap][channel], odd row stride), then each
// wave walks over its pixel groups: 27 clamped loads per lane, 27 matrix instructions per channel group, and the affine map +
// sign on the vector unit.  With few pixels NG = 1: more waves for chains of 27 dependent instructions of 64 clocks.
constexpr int C1M_RS(int NG) { return 32 * NG + 1; }  // LDS row stride of the tap-major filter tile
typedef float c1m_v32f __attribute__((ext_vector_type(32)));

__device__ __forceinline__ uint32_t c1m_spread_nibbles(uint32_t m) {
  // nibble q of a 16-bit mask -> bits 8q .. 8q+3
  return (m & 0xFu) | ((m & 0xF0u) << 4) | ((m & 0xF00u) << 8) | ((m & 0xF000u) << 12);
}

// The filter taps of channels ch0 .. ch0 + 32 * NG - 1, staged tap-major in LDS (read [channel][tap]
// contiguously; channels past D are zero), and their scale / bias (past D, or without an affine
// map: fma(0, acc, -1) < 0, so such bits are 0).  Every load is issued before the first is waited for: a loop over them, with a
// condition around each, was four memory round trips one after the other (signs of one 32 x 32
// image, 128 channels 4.15 -> 3.7 us).  With one channel group they are requested ahead of the first patch and staged behind it: loads
// return in order, so that the wait for these leaves the patch in flight.  (The patch first: the slow ones among its loads, which
// the chain of matrix instructions hides, delayed the staging; fp32 maps of 70 images of 32 x 16 by stride 2 6.85 us, 6.2 so.)
template <int NG>
struct C1mFilters {
  static constexpr int ALL = 27 * 32 * NG, PER = (ALL + 255) / 256;
  float v[PER], sc, bi;
  __device__ __forceinline__ void request(const float *__restrict__ w, const float *__restrict__ scale,
                                          const float *__restrict__ bias, int ch0, int nch, bool affine) {
    const int tid = threadIdx.x;
    const float *const wc = w + (size_t)ch0 * 27;
#pragma unroll
    for (int i = 0; i < PER; ++i) v[i] = wc[min(tid + 256 * i, 27 * nch - 1)];
    // no condition around the loads: a wait for older ones could not tell how many follow
    const int ch = affine ? ch0 + min(tid, nch - 1) : 0;
    sc = (affine ? scale : w)[ch];
    bi = (affine ? bias : w)[ch];
  }
  __device__ __forceinline__ void stage(float *sTap, float *sSc, float *sBi, int nch, bool affine) const {
    const int tid = threadIdx.x;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int idx = tid + 256 * i, ch = idx / 27, k = idx - 27 * ch;
      if (i + 1 < PER || idx < ALL) sTap[k * C1M_RS(NG) + ch] = idx < 27 * nch ? v[i] : 0.0f;
    }
    if (tid < 32 * NG) {
      sSc[tid] = affine && tid < nch ? sc : 0.0f;
      sBi[tid] = affine && tid < nch ? bi : -1.0f;
    }
  }
};

// Issue the 27 loads of pixel p's patch: every tap unconditionally from a clamped (always
// readable) position; bit r of `inside` says whether tap (r / 3, r % 3) lies in the image.
__device__ __forceinline__ void c1m_issue_patch(const float *__restrict__ x, uint32_t p, uint32_t total_pix, int H,
                                                int W, int sH, int sW, int pH, int pW, int OH, int OW, FastDiv divOW,
                                                FastDiv divOH, float (&raw)[27], uint32_t &inside) {
  const bool pv = p < total_pix;
  const uint32_t pc = pv ? p : 0u;
  const uint32_t t = fdiv(pc, divOW);
  const uint32_t ow = pc - t * OW;
  const uint32_t n = fdiv(t, divOH);
  const uint32_t oh = t - n * OH;
  const int ih0 = (int)(oh * sH) - pH, iw0 = (int)(ow * sW) - pW;
  const float *xn = x + (size_t)n * 3 * H * W;
  uint32_t rok = 0, cok = 0;
  int roff[3], coff[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const int ih = ih0 + j, iw = iw0 + j;
    rok |= (uint32_t)(pv && ih >= 0 && ih < H) << j;
    cok |= (uint32_t)(iw >= 0 && iw < W) << j;
    roff[j] = (ih < 0 ? 0 : (ih >= H ? H - 1 : ih)) * W;
    coff[j] = iw < 0 ? 0 : (iw >= W ? W - 1 : iw);
  }
  inside = 0;
#pragma unroll
  for (int r = 0; r < 9; ++r) inside |= (((rok >> (r / 3)) & (cok >> (r % 3))) & 1u) << r;
#pragma unroll
  for (int k = 0; k < 27; ++k) {
    const int c = k / 9, r = k % 9;
    raw[k] = xn[(size_t)c * H * W + roff[r / 3] + coff[r % 3]];
  }
}

// 27 dependent matrix instructions: channel group g (32 channels) x this wave's 64 pixels.
template <int NG>
__device__ __forceinline__ c1m_v32f c1m_chain(const float *wg, const float (&xv)[27]) {
  c1m_v32f acc;
#pragma unroll
  for (int r = 0; r < 32; ++r) acc[r] = 0.0f;
#pragma unroll
  for (int k = 0; k < 27; ++k) acc = __builtin_amdgcn_mfma_f32_32x32x1f32(wg[k * C1M_RS(NG)], xv[k], acc, 0, 0, 0);
  return acc;
}

// Affine map and sign of one channel group's accumulators -> the 32 channel bits of this
// lane's own pixel.  Lanes l and l + 32 hold the two channel halves of a pixel: l < 32 keeps
// its block-0 bits and receives the partner's, l >= 32 likewise with block 1.
__device__ __forceinline__ uint32_t c1m_sign_bits(const c1m_v32f &acc, const float *sSc, const float *sBi, int g,
                                                  int half) {
  // rows descend: every sign is shifted in with one add-with-carry, m = 2 * m + (y >= 0)
  uint32_t m[2] = {0u, 0u};
#pragma unroll
  for (int q = 3; q >= 0; --q) {
    const float4 sc = *reinterpret_cast<const float4 *>(sSc + 32 * g + 8 * q + 4 * half);
    const float4 bi = *reinterpret_cast<const float4 *>(sBi + 32 * g + 8 * q + 4 * half);
    const float scv[4] = {sc.x, sc.y, sc.z, sc.w}, biv[4] = {bi.x, bi.y, bi.z, bi.w};
#pragma unroll
    for (int e = 3; e >= 0; e -= 2) {
      const int rr = 4 * q + e;
      const float y[4] = {fmaf(scv[e], acc[rr], biv[e]), fmaf(scv[e], acc[16 + rr], biv[e]),
                          fmaf(scv[e - 1], acc[rr - 1], biv[e - 1]), fmaf(scv[e - 1], acc[15 + rr], biv[e - 1])};
      shift_in_signs<2>(m, y);
    }
  }
  const uint32_t own = half ? m[1] : m[0];
  const uint32_t got = (uint32_t)__shfl_xor((int)(half ? m[0] : m[1]), 32);
  const uint32_t lo = half ? got : own, hi = half ? own : got;  // channels 8q+0..3 / 8q+4..7
  return c1m_spread_nibbles(lo) | (c1m_spread_nibbles(hi) << 4);
}

}  // namespace bnn
