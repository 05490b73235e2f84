// Signs of the real-valued 3x3x3 first layer from half-precision products, each proved or computed exactly.
//
// The layer's contract is a chain of 27 fp32 fused multiply-adds per output, then the affine map; only its sign is kept.
// The chain costs a fp32 matrix instruction of 64 clocks per step (conv_first.h), 11.9 us for 256 images of 32 x 32 and 128
// channels, and the sign step beside it does not overlap.  A sign needs less: with every factor split into two halves of
// fp16 (v = hi + lo + e, |e| <= 2^-22 |v|, or 2^-25 where lo is subnormal, which matrix instructions keep), the products hi hi + hi lo
// + lo hi are exact and their fp32 sum y' differs from the chain's y by less than E = 2^-17 |x'| |w'| (2-norms; w' the filter times
// its scale, with the bias as a 28th weight; x' the patch, with a 1 there):
//   2^-18    32 additions of the two hi hi instructions, each off by at most an ulp (2^-23) of a partial sum, rounded or cut
//            off, in any order; hi lo and lo hi come first, when the partial sums are 2^-10 of that
//   2^-19.2  28 rounded operations of the chain and the affine map, 2^-24 each
//   2^-20.4  the products left out: lo lo, e w', x' e
//   2^-20.6  their part where lo is subnormal: 28 values of 2^-25 against |x'| >= 1/4 (2^-22.6 against 1)
//   2^-23    rounding of scale * weight and of the normalization below
// (7.1e-6 in all against 7.6e-6; largest seen in 10^7 sums of six distributions: 3.1e-7).  Where |y'| > E, y has the sign of y'.
// For the others, about one of 30,000 outputs of normal inputs, the chain itself decides: a pixel with doubt in a group of 32
// channels is computed for all 32 in lanes, tap by tap.  So every bit is the chain's.  fp16 instructions run 16 times as fast as
// fp32 ones, take 16 of K, and overlap with the vector ALU.  256 x 3 x 32 x 32 -> 128 channels 20.2 -> 9.9 us.
//
// A positive factor per channel changes no sign: filters are normalized to |w'| = 16, so that E depends on the pixel only.
//
// What could leave whole areas in doubt, and what is done once more than EXACT_MAX of a wave's 64 pixels are (256 images as above, every
// pixel such a one; by chains alone 20.5 us; without any of this, 31 to 34):
//   patches of zeros     the bias decides (12 us; so in areas of an image; without a bias nothing else would)
//   patches with a NaN   the sum is one (12 us)
//   beyond fp16, or small beside no bias at all (then the 1 is left out of |x'|)  scaled by a power of two (13 to 14 us)
//   filters of zeros without a bias  +1, by a bias of 1 (no doubt)
//   anything else        the group as in conv.hip (extreme filters, infinities, sums that are 0: 23.7 us)
#include <algorithm>
#include <cmath>

#include "common.h"
#include "conv_first.h"
#include "fp4_tile.h"

namespace bnn {

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// A pixel exactly takes about 1400 clocks, a group by chains 27 * 64 and its loads.  256 images of normal values (128 with an infinity in
// every 1009 values) 11.8 us (14.9) for 1, 11.3 (14.0) for 2, 11.3 (15.5) for 3, 11.2 (21.8) for 6.
constexpr int EXACT_MAX = 2;
constexpr int GIVE_UP = 8;  // what leaves so many pixels of a group in doubt does so in the next: all others by chains
constexpr float SIZE_LEAST = 0x1p-4f, SIZE_MOST = 0x1p30f;  // of |x|^2, as it is

// The order of the 28 factors: half h (lanes l / 32) of slots 0 .. 15, of which an instruction takes eight.  Slots 0 .. 8 are
// the taps (c, 0, kw) of half 0 and (c, 2, kw) of half 1, slots 9 .. 11 (c, 1, 0) and (c, 1, 2), slots 12 .. 14 (c, 1, 1) of half 0,
// and half 1 has the bias in slot 12: a lane's patch is read at 5 offsets from three planes.  The filter's eight of
// instruction k and half h, a byte each; 27: the bias, 28: nothing.
__device__ __forceinline__ void first_slot_taps(int h, int k, uint32_t (&taps)[2]) {
  const uint32_t a0 = k ? 0x150c0314u : 0x09020100u, a1 = k ? 0x1c160d04u : 0x13120b0au;
  const uint32_t b0 = k ? 0x170e051au : 0x0f080706u, b1 = k ? 0x1c1c1c1bu : 0x19181110u;
  taps[0] = h ? b0 : a0;
  taps[1] = h ? b1 : a1;
}

// minus: -1, unknown to the optimizer, which would make a conversion and a subtraction of each multiply-add.
__device__ __forceinline__ void split_f16(float a, float b, float minus, f16x2 &hi, f16x2 &lo) {
  hi = __builtin_convertvector(f32x2{a, b}, f16x2);
  lo.x = (_Float16)fmaf((float)hi.x, minus, a);  // one mixed-precision instruction
  lo.y = (_Float16)fmaf((float)hi.y, minus, b);
}

struct FirstGeom {
  int H, W, sH, sW, pH, pW, OH, OW;
  FastDiv divOW, divOH;
  uint32_t total_pix;
};

// T threads; blockIdx.y: 32 * NG channels.
template <int T, int NG>
__global__ __launch_bounds__(T, T == 256 ? 5 : 4) void conv2d_f32_k27_f16_sign_kernel(const float *__restrict__ x,
                                                                       const float *__restrict__ w, FirstGeom g, int D,
                                                                       const float *__restrict__ scale,
                                                                       const float *__restrict__ bias,
                                                                       uint64_t *__restrict__ outp, int cw_out,
                                                                       uint32_t ngroups, int groups_per_wave) {
  constexpr int CH = 32 * NG, RS = C1M_RS(NG);
  __shared__ float sTap[29 * RS];
  __shared__ __attribute__((aligned(16))) float sSc[CH];
  __shared__ __attribute__((aligned(16))) float sBi[CH];
  __shared__ __attribute__((aligned(16))) f16x8 sA[2][2][2][CH];  // hi / lo, instruction, half
  __shared__ uint32_t sFlag[CH / 16];  // of 16 channels: 1 one that the bound does not cover, 2 one with a factor of the bias' slot
  asm volatile("" ::"s"(x), "s"(w), "s"(scale), "s"(bias), "s"(outp), "s"(cw_out), "s"(ngroups));  // requested together
  float minus = -1.0f;
  asm("" : "+s"(minus));
  const int tid = threadIdx.x;
  const int lane = tid & 63, half = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ch0 = CH * (int)blockIdx.y, nch = min(CH, D - ch0);  // >= 1 by the grid
  const uint32_t g_first = ((uint32_t)blockIdx.x * (uint32_t)(T / 64) + (uint32_t)wave) * (uint32_t)groups_per_wave;
  const uint32_t g_end = min(g_first + (uint32_t)groups_per_wave, ngroups);

  // Rows of an instruction's result: register r of half h is row 8 (r / 4) + 4 h + r % 4, given to channel 16 h + r.
  const int row_channel = 16 * ((l32 >> 2) & 1) + 4 * (l32 >> 3) + (l32 & 3);

  // This lane's 15 taps of the pixels 32 b + l % 32, b = 0, 1, of a group of 64: every load from a readable place.  A lane
  // decodes its own pixel 32 half + l % 32; v_permlane32_swap(q, r) then gives the lower lanes q of both blocks' pixels and
  // the upper ones r.
  float v[2][15];
  uint32_t ok[2];  // bits kw: row of slots 0 .. 8; bit 3: slots 9 .. 11; bit 4: slots 12 .. 14
  const uint32_t hw4 = (uint32_t)(g.H * g.W) * 4u, w4 = (uint32_t)g.W * 4u;
  auto issue = [&](uint32_t grp) {
    const uint32_t p = min(grp * 64u + (uint32_t)lane, g.total_pix - 1u);
    const uint32_t t = fdiv_sel(p, g.divOW), ow = p - t * (uint32_t)g.OW;
    const uint32_t n = fdiv_sel(t, g.divOH), oh = t - n * (uint32_t)g.OH;
    const int ih0 = (int)(oh * (uint32_t)g.sH) - g.pH, iw0 = (int)(ow * (uint32_t)g.sW) - g.pW;
    // from the first pixel's image on, uniform: the host keeps what 64 pixels span below 4 GiB
    const uint32_t n0 = fdiv_sel(fdiv_sel(min(grp * 64u, g.total_pix - 1u), g.divOW), g.divOH);
    const uint32_t img = (n - n0) * 3u * hw4;
    uint32_t row[3], col[3], rok[3], cok = 0u;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int ih = min(max(ih0 + k, 0), g.H - 1), iw = min(max(iw0 + k, 0), g.W - 1);
      row[k] = img + (uint32_t)ih * w4;
      col[k] = (uint32_t)iw * 4u;
      rok[k] = ih == ih0 + k ? ~0u : 0u;
      cok |= iw == iw0 + k ? 1u << k : 0u;
    }
    // half 0: (c, 1, 0) and (c, 1, 1); half 1: (c, 1, 2) and nothing
    const auto oks = __builtin_amdgcn_permlane32_swap((rok[0] & cok) | (rok[1] & (cok << 3 & 0x18u)),
                                                      (rok[2] & cok) | (rok[1] & (cok << 1 & 8u)), false, false);
    const auto rowa = __builtin_amdgcn_permlane32_swap(row[0], row[2], false, false);
    const auto rowm = __builtin_amdgcn_permlane32_swap(row[1], row[1], false, false);
    const auto col0 = __builtin_amdgcn_permlane32_swap(col[0], col[0], false, false);
    const auto col1 = __builtin_amdgcn_permlane32_swap(col[1], col[1], false, false);
    const auto col2 = __builtin_amdgcn_permlane32_swap(col[2], col[2], false, false);
    const auto side = __builtin_amdgcn_permlane32_swap(col[0], col[2], false, false);
    const char *const xb = reinterpret_cast<const char *>(x) + (size_t)n0 * 3u * hw4;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      ok[b] = oks[b];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const char *const plane = xb + (size_t)c * hw4;
        v[b][3 * c] = *reinterpret_cast<const float *>(plane + (rowa[b] + col0[b]));
        v[b][3 * c + 1] = *reinterpret_cast<const float *>(plane + (rowa[b] + col1[b]));
        v[b][3 * c + 2] = *reinterpret_cast<const float *>(plane + (rowa[b] + col2[b]));
        v[b][9 + c] = *reinterpret_cast<const float *>(plane + (rowm[b] + side[b]));
        v[b][12 + c] = *reinterpret_cast<const float *>(plane + (rowm[b] + col1[b]));
      }
    }
  };
  // Filters: four threads per channel, eight slots each.  Loaded by every lane from a readable place.
  constexpr int ITEMS = CH * 4;  // whole waves
  float r8[8], fsc, fbi;
  uint32_t taps[2];
  auto load_filters = [&](int i) {
    const uint32_t from = (uint32_t)(ch0 + min(i >> 2, nch - 1));
    first_slot_taps((i >> 1) & 1, i & 1, taps);
#pragma unroll
    for (int e = 0; e < 8; ++e) r8[e] = w[from * 27u + min(taps[e >> 2] >> (8 * (e & 3)) & 255u, 26u)];  // host: below 2^30
    fsc = scale[from];
    fbi = bias[from];
  };
  auto sum_of_four = [](float v) {  // over the lanes of a channel
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, true));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, true));
    return v;
  };
  auto stage_filters = [&](int i) {
    asm volatile("" : "+v"(fsc), "+v"(fbi));  // not loaded under a condition below, which would wait for all loads in flight
    const int ch = i >> 2;  // past the last channel: the last one again, whose bits are left out
    float r[8], sum = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint32_t tap = taps[e >> 2] >> (8 * (e & 3)) & 255u;
      r[e] = tap < 27u ? r8[e] : 0.0f;
      sTap[tap * RS + ch] = r[e];  // rows 27 and 28 are not read
      sum += fabsf(r[e]);          // NaN stays
    }
    sum = sum_of_four(sum);
    // neither a scale nor a filter, and no bias: fma(scale, 0, 0) >= 0
    const float b28 = (fsc == 0.0f || sum == 0.0f) && fbi == 0.0f ? 1.0f : fbi;
    float u[8], n2 = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint32_t tap = taps[e >> 2] >> (8 * (e & 3)) & 255u;
      u[e] = tap == 27u ? b28 : fsc * r[e];
      n2 = fmaf(u[e], u[e], n2);
    }
    n2 = sum_of_four(n2);
    // where the bound does not hold: zeros, so that y' = 0 and every pixel is in doubt
    const bool fine = n2 >= 0x1p-80f && n2 <= 0x1p60f && sum + fabsf(fsc) <= 0x1p30f;
    const float f = 16.0f * __builtin_amdgcn_rsqf(n2);
    f16x8 hi, lo;
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      f16x2 a, b;
      split_f16(fine ? u[e] * f : 0.0f, fine ? u[e + 1] * f : 0.0f, minus, a, b);
      hi[e] = a.x;
      hi[e + 1] = a.y;
      lo[e] = b.x;
      lo[e + 1] = b.y;
    }
    sA[0][i & 1][(i >> 1) & 1][ch] = hi;
    sA[1][i & 1][(i >> 1) & 1][ch] = lo;
    if ((i & 3) == 0) {
      sSc[ch] = fsc;
      sBi[ch] = fbi;
    }
    const uint32_t flag = (__ballot(!fine) != 0ull ? 1u : 0u) | (__ballot(b28 != 0.0f) != 0ull ? 2u : 0u);
    if (lane == 0) sFlag[i >> 6] = flag;
  };
  // requested before anything is computed: the latencies overlap
  if (tid < ITEMS) load_filters(tid);  // whole waves
  issue(min(g_first, ngroups - 1u));
  if (tid < ITEMS) stage_filters(tid);
#pragma unroll 1
  for (int i = tid + T; i < ITEMS; i += T) {
    load_filters(i);
    stage_filters(i);
  }

  // Group c of channels of pixel p (uniform), exactly: lane l the chain of channel 32 c + l % 32, bits in channel order.
  auto exact_pixel = [&](uint32_t p, int c) {
    int lane = tid & 63;
    asm volatile("" : "+v"(lane));  // computed here, not ahead of every loop
    const int l32 = lane & 31;
    const uint32_t t = fdiv_sel(p, g.divOW), ow = p - t * (uint32_t)g.OW;
    const uint32_t n = fdiv_sel(t, g.divOH), oh = t - n * (uint32_t)g.OH;
    const int k = min(lane, 26), ci = k / 9, kh = (k - 9 * ci) / 3, kw = k - 9 * ci - 3 * kh;
    const int ih = (int)(oh * (uint32_t)g.sH) - g.pH + kh, iw = (int)(ow * (uint32_t)g.sW) - g.pW + kw;
    const bool in = ih >= 0 && ih < g.H && iw >= 0 && iw < g.W;
    float xv = 0.0f;
    if (in) xv = x[((size_t)n * 3 + (size_t)ci) * (size_t)(g.H * g.W) + (size_t)ih * (size_t)g.W + (size_t)iw];
    float acc = 0.0f;
#pragma unroll
    for (int j = 0; j < 27; ++j)
      acc = fmaf(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(xv), j)), sTap[j * RS + 32 * c + l32], acc);
    return (uint32_t)__ballot(fmaf(sSc[32 * c + l32], acc, sBi[32 * c + l32]) >= 0.0f);
  };
  f16x8 bh[2][2], bl[2][2];  // pixel block, instruction
  float size[2];             // |x'|^2
  auto mask_patch = [&](int b, float (&u)[16]) {
    uint32_t mask[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) mask[k] = (uint32_t)((int)(ok[b] << (31 - k)) >> 31);
#pragma unroll
    for (int s = 0; s < 15; ++s)
      u[s] = __int_as_float((int)((uint32_t)__float_as_int(v[b][s]) & mask[s < 9 ? s % 3 : (s < 12 ? 3 : 4)]));
    u[15] = 0.0f;
  };
  auto split_block = [&](int b, float (&u)[16], uint32_t one) {
    u[12] = __int_as_float((int)((uint32_t)__float_as_int(u[12]) | one));  // half 1: the bias' factor
    float n2 = 0.0f;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        f16x2 a, l;
        split_f16(u[8 * kk + e], u[8 * kk + e + 1], minus, a, l);
        bh[b][kk][e] = a.x;
        bh[b][kk][e + 1] = a.y;
        bl[b][kk][e] = l.x;
        bl[b][kk][e + 1] = l.y;
        n2 = __builtin_amdgcn_fdot2(a, a, n2, false);  // 2^-10 off: E has the room
      }
    const auto both = __builtin_amdgcn_permlane32_swap((uint32_t)__float_as_int(n2), (uint32_t)__float_as_int(n2), false, false);
    size[b] = __int_as_float((int)both[0]) + __int_as_float((int)both[1]);  // patches that fp16 does not hold: infinity or NaN
  };
  auto split_patch = [&]() {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      float u[16];
      mask_patch(b, u);
      split_block(b, u, half ? 0x3f800000u : 0u);
    }
  };
  // Patches of no ordinary size once more, from the start.  Scaled by a power of two, which changes no sign, where fp16 does not
  // hold them, or without a bias where they are below 1/4 (e would count); those of zeros and those with a NaN are told apart.
  auto scale_patch = [&](uint32_t grp, bool biased, uint64_t &zeros, uint64_t &nans) {  // by pixel
    asm volatile("" : "+s"(grp));  // computed here, not ahead of every loop
    issue(grp);
    uint64_t z[2], n[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      float u[16];
      mask_patch(b, u);
      uint32_t top = 0u;  // ordered as the magnitudes are, infinity and NaN last
#pragma unroll
      for (int s = 0; s < 15; ++s) top = max(top, (uint32_t)__float_as_int(u[s]) & 0x7fffffffu);
      top = max(top, (uint32_t)__shfl_xor((int)top, 32));
      z[b] = __ballot(top == 0u);
      n[b] = __ballot(top > 0x7f800000u);
      const int e = (int)(top >> 23) - 127;
      const bool scaled = !(size[b] < SIZE_MOST) || (!biased && size[b] < 1.0f + SIZE_LEAST);
      const bool in_range = e >= -48 && e <= 60;  // neither chains of filters that are fine nor their doubt over- or underflow
      const float f = scaled && in_range ? __int_as_float((127 - e) << 23) : 1.0f;
#pragma unroll
      for (int s = 0; s < 15; ++s) u[s] *= f;
      split_block(b, u, half ? (uint32_t)__float_as_int(biased ? f : 1.0f) : 0u);
      if (scaled && !in_range && top != 0u) size[b] = INFINITY;  // in doubt
    }
    zeros = (z[0] & 0xffffffffull) | z[1] << 32;
    nans = (n[0] & 0xffffffffull) | n[1] << 32;
  };
  split_patch();
  __syncthreads();  // the only barrier: from here on the waves run independently
  uint32_t grp = g_first;  // wave-uniform
  if (grp >= g_end) return;
  const uint32_t flag = sFlag[lane % (CH / 16)];
  const uint32_t bad = (uint32_t)__ballot((flag & 1u) != 0u);  // two bits a group: a filter that the bound does not cover
  const bool biased = __ballot((flag & 2u) != 0u) != 0ull;
  const float beside = biased ? 0.0f : 1.0f, size_floor = biased ? 1.0f : SIZE_LEAST;  // below it E covers smaller ones
  const int groups = (nch + 31) >> 5;
  while (true) {
    const uint32_t p = grp * 64u + (uint32_t)lane;
    uint32_t gw[NG];
#pragma unroll
    for (int c = 0; c < NG; ++c) gw[c] = 0u;
    uint32_t by_chains = 0u;
    bool scaled = false;
    uint64_t zeros = 0ull, nans = 0ull;
    float doubt[2];  // E
    auto set_doubt = [&]() {
#pragma unroll
      for (int b = 0; b < 2; ++b) doubt[b] = 0x1p-13f * __builtin_amdgcn_sqrtf(fmaxf(size[b] - beside, size_floor));  // 16 * 2^-17 |x'|
    };
    set_doubt();
    int c = 0;
#pragma unroll 1
    while (c < groups) {  // workgroup-uniform: groups past the last channel keep zero bits
      int next = c + 1;
      const int ch = 32 * c + row_channel;
      const f16x8 ah0 = sA[0][0][half][ch], ah1 = sA[0][1][half][ch], al0 = sA[1][0][half][ch], al1 = sA[1][1][half][ch];
      v16f acc[2];
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[b][r] = 0.0f;
#define BNN_STEP(A, B)                                                                    \
  acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(A, B(0), acc[0], 0, 0, 0);              \
  acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(A, B(1), acc[1], 0, 0, 0);
#define BNN_H0(b) bh[b][0]
#define BNN_H1(b) bh[b][1]
#define BNN_L0(b) bl[b][0]
#define BNN_L1(b) bl[b][1]
      BNN_STEP(al0, BNN_H0)
      BNN_STEP(al1, BNN_H1)
      BNN_STEP(ah0, BNN_L0)
      BNN_STEP(ah1, BNN_L1)
      BNN_STEP(ah0, BNN_H0)
      BNN_STEP(ah1, BNN_H1)
#undef BNN_STEP
#undef BNN_H0
#undef BNN_H1
#undef BNN_L0
#undef BNN_L1
      // sign bits, last row first, and the smallest |y'| of this lane's 16 channels of either pixel
      asm volatile("s_nop 15\n\ts_nop 15" : "+v"(acc[0]), "+v"(acc[1]));  // before written-out reads, as in settle()
      uint32_t m[2] = {0u, 0u};
      float least[2] = {INFINITY, INFINITY};
#pragma unroll
      for (int r = 14; r >= 0; r -= 2)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          m[b] = __builtin_amdgcn_alignbit(m[b], (uint32_t)__float_as_int(acc[b][r + 1]), 31);
          m[b] = __builtin_amdgcn_alignbit(m[b], (uint32_t)__float_as_int(acc[b][r]), 31);
          asm("v_min3_f32 %0, %0, |%1|, |%2|" : "+v"(least[b]) : "v"(acc[b][r]), "v"(acc[b][r + 1]));
        }
      // lanes l and l + 32 hold the channel halves of the same pixels: the lower lanes assemble block 0, the upper ones 1
      const auto h = __builtin_amdgcn_permlane32_swap(m[0], m[1], false, false);
      uint32_t word = ~(h[0] | h[1] << 16);
      const uint64_t d0 = __ballot(!(least[0] > doubt[0])), d1 = __ballot(!(least[1] > doubt[1]));
      if (__builtin_expect((d0 | d1) != 0ull, 0)) {
        auto by_pixel = [](uint64_t b0, uint64_t b1) {
          return (uint64_t)((uint32_t)b0 | (uint32_t)(b0 >> 32)) | (uint64_t)((uint32_t)b1 | (uint32_t)(b1 >> 32)) << 32;
        };
        uint64_t d = by_pixel(d0, d1);
        int lane = tid & 63;
        asm volatile("" : "+v"(lane));  // as above
        const uint32_t left = g.total_pix - grp * 64u;
        if (left < 64u) d &= (1ull << left) - 1ull;
        if (__builtin_expect(__popcll(d) > EXACT_MAX, 0)) {
          const bool known = (bad >> (2 * c) & 3u) == 0u;
          if (known && !scaled) {
            auto ordinary = [&](float e) { return e > 0x1p-13f * (biased ? 1.0f : 0.25f) && e < 0x1p2f; };  // by the sizes' limits
            if ((d & by_pixel(__ballot(!ordinary(doubt[0])), __ballot(!ordinary(doubt[1])))) != 0ull) {
              scaled = true;
              scale_patch(grp, biased, zeros, nans);
              set_doubt();
              next = c;  // this group once more
              if (__popcll(by_pixel(__ballot(!(doubt[0] < INFINITY)), __ballot(!(doubt[1] < INFINITY))) & ~nans) > EXACT_MAX) {
                by_chains |= (1u << groups) - (1u << c);
                next = groups;
              }
              d = 0ull;
            }
          }
          if (__popcll(d) > EXACT_MAX && known) {
            // a NaN makes the sum one, and its sign bit 0; zeros leave the bias
            const uint32_t zero_word = (uint32_t)__ballot(sBi[32 * c + (lane & 31)] >= 0.0f);
            word = d & (zeros | nans) & 1ull << lane ? (zeros & 1ull << lane ? zero_word : 0u) : word;
            d &= ~(zeros | nans);
          }
          if (__popcll(d) > EXACT_MAX) {
            by_chains |= 1u << c;
            if (known && __popcll(d) > GIVE_UP) {  // the groups that follow too
              by_chains |= (1u << groups) - (1u << c);
              next = groups;
            }
            d = 0ull;
          }
        }
        while (d != 0ull) {
          const int l = __builtin_ctzll(d);
          d &= d - 1ull;
          const uint32_t exact = exact_pixel(grp * 64u + (uint32_t)l, c);
          word = lane == l ? exact : word;
        }
      }
#pragma unroll
      for (int k = 0; k < NG; ++k) gw[k] = c == k ? word : gw[k];
      c = next;
    }
    if (__builtin_expect(by_chains != 0u, 0)) {  // as conv2d_f32_k27_mfma_sign_kernel computes them; here, where the halves of the patches are not held
      int own = (int)p, h = half, l = l32;
      asm volatile("" : "+v"(own), "+v"(h), "+v"(l));  // as above
      float xv[27];
      uint32_t inside;
      c1m_issue_patch(x, (uint32_t)own, g.total_pix, g.H, g.W, g.sH, g.sW, g.pH, g.pW, g.OH, g.OW, g.divOW, g.divOH, xv, inside);
#pragma unroll
      for (int k = 0; k < 27; ++k) xv[k] = ((inside >> (k % 9)) & 1u) ? xv[k] : 0.0f;
#pragma unroll 1
      for (int c = 0; c < NG; ++c)
        if (by_chains >> c & 1u) {
          const uint32_t word = c1m_sign_bits(c1m_chain<NG>(sTap + 32 * c + l, xv), sSc, sBi, c, h);
#pragma unroll
          for (int k = 0; k < NG; ++k) gw[k] = c == k ? word : gw[k];
        }
    }
#pragma unroll
    for (int k = 0; k < NG; ++k)  // the last group's channels past the last
      if (32 * k < nch && 32 * k + 32 > nch) gw[k] &= (1u << (nch - 32 * k)) - 1u;
    if (p < g.total_pix) {
      if constexpr (NG == 4) {
        const int word0 = 2 * (int)blockIdx.y;
        uint64_t *o = outp + (size_t)p * cw_out + word0;
        o[0] = ((uint64_t)gw[1] << 32) | gw[0];
        if (word0 + 1 < cw_out) o[1] = ((uint64_t)gw[3] << 32) | gw[2];
      } else {
        static_assert(NG == 2, "whole words");
        outp[(size_t)p * cw_out + blockIdx.y] = ((uint64_t)gw[1] << 32) | gw[0];
      }
    }
    if (++grp >= g_end) return;
    issue(grp);
    split_patch();
  }
}

// -1: does not apply.  By q, pairs of 64 pixels and 32 channels per compute unit:
//   up to 8, two waves a SIMD, the chains alone, a workgroup per pair and four, are 5 % faster and the same whatever the values (128
//   channels of 32 x 32: 17 images 4.9 us against 5.3, 32 5.0, 5.3; 64 channels: 38 images 4.75, 5.5); their third wave makes it
//   6.3 at once (33 images 6.3, 5.75; 48 6.35 to 6.55, 6.55; 64 channels, 97 images 7.1, 6.7), and only areas of zeros without a
//   bias stay faster (48 images of them 7.9 here);
//   up to 27 workgroups of four waves and 64 channels, which spread best (128 channels: 64 images 6.4 against 7.9 by eight
//   waves and 128 channels, 96 7.5, 8.0, 128 8.8, 7.8; 256 channels: 48 images 7.5, 8.6, 64 9.1, 8.7);
//   beyond, workgroups of 16 waves, one to a unit, split the filters least often (256 images, 128 channels 9.9 us; eight
//   waves 11.4), but those of eight, two to a unit, where the last round would be half empty (192 images, 256 channels
//   17.3 against 15.6; 96 images, 512 channels 17.1, 15.6).
// The chains for every output (the kernel before this one): 64 images 7.9, 128 12.6, 192 16.5, 256 20.2, 768 53.1 (23.7 here).
static int first_sign_shape(int64_t groups, int D, int64_t cu) {
  const int64_t q = groups * (((int64_t)D + 31) / 32);
  if (q <= 8 * cu) return -1;
  if (q <= 27 * cu) return 0;
  const int64_t halves = (groups * (((int64_t)D + 127) / 128) + 8 * cu - 1) / (8 * cu);
  return halves % 2 == 1 && halves <= 5 ? 1 : 2;
}

int first_sign_f16(int N, int H, int W, int D, int sH, int sW, int pH, int pW, int units) {
  const int64_t OH = bnn_conv_out_dim(H, 3, sH, pH), OW = bnn_conv_out_dim(W, 3, sW, pW);
  // 32-bit offsets: a wave's 64 pixels from their first image on, the filters
  const double span = (63.0 / ((double)OH * (double)OW) + 2.0) * 12.0 * (double)H * (double)W;
  return span < 4294967296.0 && D < (1 << 25) ? first_sign_shape((N * OH * OW + 63) / 64, D, units) : -1;
}

bnn_status launch_first_sign_f16(const float *x, const float *w, int N, int H, int W, int D, int sH, int sW, int pH, int pW,
                                 const float *scale, const float *bias, uint64_t *out, int shape, hipStream_t s) {
  FirstGeom g;
  g.H = H; g.W = W; g.sH = sH; g.sW = sW; g.pH = pH; g.pW = pW;
  g.OH = (int)bnn_conv_out_dim(H, 3, sH, pH);
  g.OW = (int)bnn_conv_out_dim(W, 3, sW, pW);
  g.divOW = FastDiv((uint32_t)g.OW);
  g.divOH = FastDiv((uint32_t)g.OH);
  g.total_pix = (uint32_t)((int64_t)N * g.OH * g.OW);
  const uint32_t ngroups = (g.total_pix + 63u) / 64u;
  const int cw = (int)bnn_packed_words(D);
  auto go = [&](auto kernel, int T, int ng) {
    const int64_t waves = T / 64, blocks = (ngroups + waves - 1) / waves;
    // several groups a wave once there are 16 waves a unit
    const int64_t slots = 16 * (int64_t)device_cu_count() / waves, gpw = std::max<int64_t>(1, std::min<int64_t>(blocks / slots, 8));
    const dim3 grid((unsigned)((ngroups + waves * gpw - 1) / (waves * gpw)), (unsigned)((D + 32 * ng - 1) / (32 * ng)));
    hipLaunchKernelGGL(kernel, grid, dim3((unsigned)T), 0, s, x, w, g, D, scale, bias, out, cw, ngroups, (int)gpw);
  };
  switch (shape) {
    case 0: go(conv2d_f32_k27_f16_sign_kernel<256, 2>, 256, 2); break;
    case 1: go(conv2d_f32_k27_f16_sign_kernel<512, 4>, 512, 4); break;
    case 2: go(conv2d_f32_k27_f16_sign_kernel<1024, 4>, 1024, 4); break;
    default: return BNN_ERR_UNSUPPORTED;
  }
  return launch_status();
}

}  // namespace bnn
