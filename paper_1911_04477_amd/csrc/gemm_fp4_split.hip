// Xnor-Bitcount GEMM (section 3.2) and implicit-GEMM convolution on the matrix cores for few outputs: the
// reduction axis split over the waves of a workgroup.
//
// A fully-connected layer at serving batch, or a convolution over a handful of images, has too few 128 x 128
// tiles to occupy the chip, and a tile walked by one workgroup lasts as long as its reduction is long.  Here a
// tile is 32 x 32 or 64 x 64 outputs, KS waves take contiguous ranges of the reduction in chunks of 256 bits, and
// every wave reads its operands straight from memory in fragment order (lane l: row l % 32, 128-bit half l / 32 of
// the chunk): no LDS staging, no barrier before the end.  Two chunks are in flight per wave.  The partial sums meet in
// LDS once, as integers or, maps of 64 x 64 tiles, as the accumulators' fp32; waves 0 .. 3 each finish the accumulator quad q = wave
// (rows 8q + 4 * (l / 32) + 0..3 of every block).
//
// Bound: latency (launch, one memory round trip for the operands, one exchange through LDS).
//
// A convolution from an fp32 image that small (SG_IMAGE) is one launch: the tile encodes the input rows that it reads into LDS
// and takes its columns from there, and the first row of tiles writes the packed image out.  In a launch of its own the encode is
// 2.3 us and a gap of about as much, for 0.3 us of loads.  One 256 x 16 x 16 image to 256 channels, 3 x 3: 7.3 -> 5.4 us in a
// graph; the addresses of the 32 planes of a granule as a running sum, not as products: 5.7 -> 5.4.
#include <algorithm>
#include <numeric>
#include <type_traits>

#include "common.h"
#include "fp4_tile.h"

namespace bnn {

enum : int { SG_EXPL16 = 0, SG_EXPL8 = 1, SG_CONV = 2, SG_IMAGE = 3 };

// SG_IMAGE: the fp32 image of a convolution, encoded by the tile that reads it.
struct ImageParams : GemmParams {
  const float *x;   // [Nimg, C, H, W]
  uint64_t *img;    // its packed pixels leave there: bnn_conv2d's workspace receives them
  FastDiv divHW;
  uint32_t HW;
};

// fdiv_sel, for the host too.
__host__ __device__ inline uint32_t image_div(uint32_t n, const FastDiv &f) {
#if defined(__HIP_DEVICE_COMPILE__)
  return fdiv_sel(n, f);
#else
  return n / f.d;
#endif
}

// Input rows, of the rows of all images one after the other, that the output pixels n0 .. n0 + cols - 1 read (taps outside an
// image moved to its first or last row), and the rows up to where the next tile's begin, so that the tiles of an image read all
// of it.
__host__ __device__ inline void image_rows(const ConvGeom &g, uint32_t n0, uint32_t cols, uint32_t total, int &r0, int &r1) {
  const uint32_t end = n0 + cols;
  const uint32_t t0 = image_div(n0, g.divOW), t1 = image_div((end < total ? end : total) - 1u, g.divOW);
  const int i0 = (int)image_div(t0, g.divOH), i1 = (int)image_div(t1, g.divOH);
  const int a = ((int)t0 - i0 * g.OH) * g.sH - g.pH, b = ((int)t1 - i1 * g.OH) * g.sH - g.pH + g.kH - 1;
  r0 = i0 * g.H + (a < 0 ? 0 : a < g.H ? a : g.H - 1);
  r1 = i1 * g.H + (b < 0 ? 0 : b < g.H ? b : g.H - 1);
  if (end >= total) {
    r1 = g.Nimg * g.H - 1;
  } else {
    const uint32_t t2 = image_div(end, g.divOW);
    const int i2 = (int)image_div(t2, g.divOH);
    const int c = ((int)t2 - i2 * g.OH) * g.sH - g.pH;
    const int next = i2 * g.H + (c < 0 ? 0 : c < g.H ? c : g.H - 1) - 1;
    r1 = r1 > next ? r1 : next;
  }
}

template <int WT, int KS, int GM, int EMODE, class Params = GemmParams>
__global__ __launch_bounds__(64 * KS, 2) void xnor_gemm_fp4_split_kernel(Params p) {
  constexpr int B32 = 32 * WT;  // rows and columns of the tile
  constexpr bool IMAGE = GM == SG_IMAGE, CONV = GM == SG_CONV || IMAGE, SIGN = EMODE != 0;
  extern __shared__ __attribute__((aligned(16))) uint32_t sImg[];  // IMAGE: [pixel][2 * Cw]
  __shared__ __attribute__((aligned(16))) int4 sPart[KS * WT * WT * 4 * 64];
  __shared__ __attribute__((aligned(16))) uint8_t sO[SIGN ? B32 * WT * 4 : 16];  // sign bytes [column][row group of 8]
  const int tid = threadIdx.x;
  const int lane = tid & 63, half = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ni = (int)fdiv_sel(blockIdx.x, p.divTilesM), mi = (int)(blockIdx.x - (uint32_t)ni * (uint32_t)p.tilesM);
  const int m0 = mi * B32, n0 = ni * B32;
  const ConvGeom &g = p.g;

  // ---- this lane's rows and columns: column block j, lane l = tile column WT * l + j ---------------------
  const char *arow[WT], *brow[WT];
  int bih[WT], biw[WT], bpx[WT];
  int r0 = 0, r1 = 0;
  if constexpr (IMAGE) image_rows(g, (uint32_t)n0, (uint32_t)B32, (uint32_t)p.N, r0, r1);  // uniform
#pragma unroll
  for (int i = 0; i < WT; ++i)
    arow[i] = reinterpret_cast<const char *>(p.A) + (size_t)min(m0 + 32 * i + l32, p.M - 1) * (size_t)p.lda32 * 4u;
#pragma unroll
  for (int j = 0; j < WT; ++j) {
    const int n = min(n0 + WT * l32 + j, p.N - 1);  // columns past N recompute column N - 1
    if constexpr (CONV) {
      uint32_t img, oh, ow;
      column_pixel(g, (uint32_t)n, g.pool != 0, img, oh, ow);
      if constexpr (IMAGE) bpx[j] = ((int)img * g.H - r0) * g.W;  // of the region
      else brow[j] = reinterpret_cast<const char *>(g.act + (size_t)img * (size_t)g.H * (size_t)g.W * (size_t)g.Cw);
      bih[j] = (int)oh * g.sH - g.pH;
      biw[j] = (int)ow * g.sW - g.pW;
    } else {
      brow[j] = reinterpret_cast<const char *>(p.B) + (size_t)n * (size_t)p.ldb * 8u;
    }
  }

  // The columns' affine constants, requested before the operands: after them, a wait for the first operands could not
  // tell how many loads follow.  (Requested when they are used: a memory round trip, 256 x 4096 x 4096 8.1 -> 7.0 us; 6.3 with
  // the branches of the exchange and the stores taken once.)
  float csc[WT], cbi[WT];
#pragma unroll
  for (int j = 0; j < WT; ++j) csc[j] = cbi[j] = 0.0f;
  if (!SIGN && p.Y && p.axis == BNN_CH_COL) {  // uniform
#pragma unroll
    for (int j = 0; j < WT; ++j) {
      const int n = min(n0 + WT * l32 + j, p.N - 1);
      csc[j] = p.scale[n];
      cbi[j] = p.bias[n];
    }
  }

  // ---- operands of one chunk: words 4c + 2 * half and the next; past the row's end the last word again, masked later
  const bool a16 = GM == SG_EXPL16 || (CONV && p.b_vec16);
  const bool cw_even = CONV && (g.Cw & 1) == 0;
  const uint64_t part = (g.C & 63) ? (1ull << (g.C & 63)) - 1ull : ~0ull;  // real channels of a tap's last word
  // IMAGE: a tap's pixel in LDS, of taps outside the image the nearest one inside (not used)
  auto tap_pixel = [&](int j, int ih, int iw) {
    return bpx[j] + min(max(ih, 0), g.H - 1) * g.W + min(max(iw, 0), g.W - 1);
  };
  auto load_rows = [&](int c, u32x4 (&a)[WT]) {
    const int w = 4 * c + 2 * half;
    const uint32_t wo = (uint32_t)max(min(w, p.Kw64 - 2), 0) * 8u;
    if (a16) {
      const uint32_t o = (uint32_t)min(w, p.Kw64 - 2) * 8u;
#pragma unroll
      for (int i = 0; i < WT; ++i) a[i] = *reinterpret_cast<const u32x4 *>(arow[i] + o);
    } else {
      load_pieces_any<WT>(a, p.Kw64 > 1, [&](int i) { return arow[i] + wo; });
    }
  };
  auto load_columns = [&](int c, u32x4 (&b)[WT]) {
    const int w = 4 * c + 2 * half;
    if constexpr (GM == SG_EXPL16) {
      const uint32_t o = (uint32_t)min(w, p.Kw64 - 2) * 8u;
#pragma unroll
      for (int j = 0; j < WT; ++j) b[j] = *reinterpret_cast<const u32x4 *>(brow[j] + o);
    } else if constexpr (GM == SG_EXPL8) {
      const uint32_t wo = (uint32_t)max(min(w, p.Kw64 - 2), 0) * 8u;
      load_pieces_any<WT>(b, p.Kw64 > 1, [&](int j) { return brow[j] + wo; });
    } else if (cw_even) {  // both words belong to one tap
      const uint32_t ww = (uint32_t)min(w, p.Kw64 - 2);
      const uint32_t tap = fdiv_sel(ww, g.divCw), cw = ww - tap * (uint32_t)g.Cw;
      const uint32_t kh = fdiv_sel(tap, g.divKW), kw = tap - kh * (uint32_t)g.kW;
      const uint64_t pad = cw + 2u == (uint32_t)g.Cw ? part : ~0ull;
#pragma unroll
      for (int j = 0; j < WT; ++j) {
        const int ih = bih[j] + (int)kh, iw = biw[j] + (int)kw;
        u32x4 v = {0xffffffffu, 0xffffffffu, (uint32_t)pad, (uint32_t)(pad >> 32)};
        const bool inside = ih >= 0 && ih < g.H && iw >= 0 && iw < g.W;
        if constexpr (IMAGE) {
          const u32x4 t = *reinterpret_cast<const u32x4 *>(sImg + 2 * (tap_pixel(j, ih, iw) * g.Cw + (int)cw));
          v = inside ? t : v;
        } else if (inside)
          v = *reinterpret_cast<const u32x4 *>(brow[j] + (((size_t)ih * (size_t)g.W + (size_t)iw) * (size_t)g.Cw + cw) * 8u);
        b[j] = v;
      }
    } else {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t ww = (uint32_t)min(w + h, p.Kw64 - 1);
        const uint32_t tap = fdiv_sel(ww, g.divCw), cw = ww - tap * (uint32_t)g.Cw;
        const uint32_t kh = fdiv_sel(tap, g.divKW), kw = tap - kh * (uint32_t)g.kW;
        const uint64_t pad = cw + 1u == (uint32_t)g.Cw ? part : ~0ull;  // taps outside the image: +1 in every channel
#pragma unroll
        for (int j = 0; j < WT; ++j) {
          const int ih = bih[j] + (int)kh, iw = biw[j] + (int)kw;
          u32x2 v = {(uint32_t)pad, (uint32_t)(pad >> 32)};
          const bool inside = ih >= 0 && ih < g.H && iw >= 0 && iw < g.W;
          if constexpr (IMAGE) {
            const u32x2 t = *reinterpret_cast<const u32x2 *>(sImg + 2 * (tap_pixel(j, ih, iw) * g.Cw + (int)cw));
            v = inside ? t : v;
          } else if (inside)
            v = *reinterpret_cast<const u32x2 *>(brow[j] + (((size_t)ih * (size_t)g.W + (size_t)iw) * (size_t)g.Cw + cw) * 8u);
          if (h == 0) b[j].lo = v;
          else b[j].hi = v;
        }
      }
    }
  };
  auto load_chunk = [&](int c, u32x4 (&a)[WT], u32x4 (&b)[WT]) {
    load_rows(c, a);
    load_columns(c, b);
  };
  auto mask_chunk = [&](int c, u32x4 (&a)[WT], u32x4 (&b)[WT]) {  // bits past the end of the row become 0 in both operands
    u32x4 m;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const int left = (int)((uint32_t)p.Kbits - (uint32_t)(8 * c + 4 * half + d) * 32u);  // any row length
      m[d] = left >= 32 ? 0xffffffffu : (left <= 0 ? 0u : (1u << left) - 1u);
    }
    const bool shifted = 4 * c + 2 * half == p.Kw64 - 1 && p.Kw64 > 1;  // a row's odd last word, read as the second
#pragma unroll
    for (int i = 0; i < WT; ++i) {
      if (!a16 && shifted) a[i].lo = a[i].hi;
      if (GM == SG_EXPL8 && shifted) b[i].lo = b[i].hi;
      a[i] &= m;
      b[i] &= m;
    }
  };

  Fp4Acc<WT, WT> acc;
  acc.init(0.0f);
  // the operands of a dword are expanded beside the products of the dword before it
  auto multiply_chunk = [&](const u32x4 (&a)[WT], const u32x4 (&b)[WT]) {
    v8i ea[WT], eb[WT];
#pragma unroll
    for (int i = 0; i < WT; ++i) {
      ea[i] = expand_e2m1<true>(a[i][0]);
      eb[i] = expand_e2m1<true>(b[i][0]);
    }
#pragma unroll
    for (int d = 1; d < 4; ++d) {
      uint32_t xa[WT], xb[WT];
      v8i na[WT], nb[WT];
#pragma unroll
      for (int i = 0; i < WT; ++i) {
        xa[i] = a[i][d];
        xb[i] = b[i][d];
      }
      multiply_and_expand<SignCodes, WT, WT>(acc, ea, eb, xa, xb, na, nb, [](int) {});
#pragma unroll
      for (int i = 0; i < WT; ++i) {
        ea[i] = na[i];
        eb[i] = nb[i];
      }
    }
    // by columns: two matrix instructions stand between the last fragment's expansion and the one that reads it
#pragma unroll
    for (int j = 0; j < WT; ++j)
#pragma unroll
      for (int i = 0; i < WT; ++i) {
        acc.v[i][j] = mfma_e2m1(ea[i], eb[j], acc.v[i][j]);
        asm volatile("" : "+v"(acc.v[i][j]));
      }
  };

  const int nc = (p.Kw64 + 3) >> 2;
  const int per = (nc + KS - 1) / KS;
  const int cb = min(wave * per, nc), ce = min(cb + per, nc);
  // 64 x 64 explicit tiles leave the loop between its chunks, which keeps their accumulators where they are (256 x 4096 x 4096
  // 7.2 -> 6.8 us in turn on one card, 7.2 on another; 512 x 2048 x 4608 7.5 -> 7.1); the others are up to 3 % faster with a condition around the second chunk.
  constexpr bool LEAVE = WT == 2 && !CONV;
  u32x4 a0[WT], b0[WT], a1[WT], b1[WT], ab[2][WT], bb[2][WT];
  if constexpr (LEAVE) {
#pragma unroll
    for (int u = 0; u < 2; ++u)
      if (cb + u < ce) load_chunk(cb + u, ab[u], bb[u]);
  } else if constexpr (IMAGE) {
    if (cb < ce) load_rows(cb, a0);
    if (cb + 1 < ce) load_rows(cb + 1, a1);
  } else {
    if (cb < ce) load_chunk(cb, a0, b0);
    if (cb + 1 < ce) load_chunk(cb + 1, a1, b1);
  }
  // the finishing waves' affine constants of the rows travel with the operands
  const int mq = m0 + 8 * (wave & 3) + 4 * half;  // first of this lane's rows in row block 0
  const bool row_affine = SIGN || (p.Y && p.axis == BNN_CH_ROW);
  float sc[WT][4], bi[WT][4];
#pragma unroll
  for (int i = 0; i < WT; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int m = mq + 32 * i + e;
      const bool on = row_affine && wave < 4 && m < p.M;
      sc[i][e] = on ? p.scale[m] : 0.0f;  // rows past M: sign bit 0
      bi[i][e] = on ? p.bias[m] : -1.0f;
    }
  if constexpr (IMAGE) {
    // ---- the region's pixels -> sImg: a wave 64 pixels x 32 channels at a time -------------------------------
    const int npx = (r1 - r0 + 1) * g.W, np = (npx + 63) >> 6, dw = 2 * g.Cw;
    const uint32_t px0 = (uint32_t)r0 * (uint32_t)g.W, i0 = fdiv_sel(px0, p.divHW);
    const float *const base = p.x + (size_t)i0 * (size_t)g.C * (size_t)p.HW;  // the host: 32 bits reach the region's images
    int gr = 0, chunk = wave;  // granule of 32 channels, chunk of 64 pixels
    for (;; chunk += KS) {
      while (chunk >= np && gr < dw) {
        chunk -= np;
        ++gr;
      }
      if (gr >= dw) break;
      const int px = 64 * chunk + lane;
      const uint32_t q = px0 + (uint32_t)min(px, npx - 1), qi = fdiv_sel(q, p.divHW);
      const uint32_t off = ((qi - i0) * (uint32_t)g.C - qi) * p.HW + q;
      const int left = g.C - 32 * gr;
      const float *plane = base + (size_t)(32 * gr) * p.HW;
      uint32_t bits = 0u;
      auto take = [&](auto count, auto whole) {
        constexpr int N = decltype(count)::value;
        float v[N];
#pragma unroll
        for (int k = 0; k < N; ++k) {
          v[k] = plane[off];
          if (decltype(whole)::value || k < left - 1) plane += p.HW;  // channels past C: the last one once more, masked
        }
#pragma unroll
        for (int k = 0; k < N; ++k) bits |= (uint32_t)sign_bit(v[k]) << k;
      };
      if (left >= 32) take(std::integral_constant<int, 32>(), std::true_type());
      else if (left > 8) take(std::integral_constant<int, 32>(), std::false_type());
      else if (left > 0) take(std::integral_constant<int, 8>(), std::false_type());
      if (left < 32) bits &= left > 0 ? (1u << left) - 1u : 0u;
      if (px < npx) sImg[px * dw + gr] = bits;
    }
    __syncthreads();
    if (mi == 0) {
      uint64_t *const o = p.img + (size_t)px0 * (size_t)g.Cw;
      for (int k = tid; k < npx * g.Cw; k += 64 * KS) o[k] = reinterpret_cast<const uint64_t *>(sImg)[k];
    }
    if (cb < ce) load_columns(cb, b0);
    if (cb + 1 < ce) load_columns(cb + 1, b1);
  }
  // Partial sums -> LDS [wave][block][quad][lane].  64 x 64 tiles of maps leave them as the accumulators hold them while the padded row
  // has at most 2^24 values: sums are exact then (64 conversions a wave less).  Else as integers, and a wave whose range
  // is longer than FLUSH chunks adds up its own slots.
  constexpr int FLUSH = 1 << 15;
  const bool as_int = WT == 1 || SIGN || nc > (1 << 16);
  bool flushed = false;
  auto flush = [&]() {
#pragma unroll
    for (int i = 0; i < WT; ++i)
#pragma unroll
      for (int j = 0; j < WT; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const v16f &v = acc.v[i][j];
          int4 *d = &sPart[((wave * WT * WT + i * WT + j) * 4 + q) * 64 + lane];
          int4 t = make_int4((int)v[4 * q], (int)v[4 * q + 1], (int)v[4 * q + 2], (int)v[4 * q + 3]);
          if (flushed) {
            const int4 o = *d;
            t = make_int4(t.x + o.x, t.y + o.y, t.z + o.z, t.w + o.w);
          }
          *d = t;
        }
  };
#pragma unroll 1
  for (int c = cb; c < ce; c += 2) {
    if constexpr (LEAVE) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (u > 0 && c + u >= ce) break;  // uniform
        if (c + u == nc - 1) mask_chunk(c + u, ab[u], bb[u]);
        u32x4 ta[WT], tb[WT];
#pragma unroll
        for (int i = 0; i < WT; ++i) {
          ta[i] = ab[u][i];
          tb[i] = bb[u][i];
        }
        if (c + u + 2 < ce) load_chunk(c + u + 2, ab[u], bb[u]);
        multiply_chunk(ta, tb);
      }
    } else {
      if (c == nc - 1) mask_chunk(c, a0, b0);
      u32x4 ta[WT], tb[WT];
#pragma unroll
      for (int i = 0; i < WT; ++i) {
        ta[i] = a0[i];
        tb[i] = b0[i];
      }
      if (c + 2 < ce) load_chunk(c + 2, a0, b0);
      multiply_chunk(ta, tb);
      if (c + 1 < ce) {
        if (c + 1 == nc - 1) mask_chunk(c + 1, a1, b1);
#pragma unroll
        for (int i = 0; i < WT; ++i) {
          ta[i] = a1[i];
          tb[i] = b1[i];
        }
        if (c + 3 < ce) load_chunk(c + 3, a1, b1);
        multiply_chunk(ta, tb);
      }
    }
    if (((c - cb + 2) & (FLUSH - 1)) == 0) {
      flush();
      flushed = true;
      acc.init(0.0f);
    }
  }
  if (as_int) {  // uniform
    flush();
  } else {
#pragma unroll
    for (int i = 0; i < WT; ++i)
#pragma unroll
      for (int j = 0; j < WT; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const v16f &v = acc.v[i][j];
          reinterpret_cast<float4 *>(sPart)[((wave * WT * WT + i * WT + j) * 4 + q) * 64 + lane] =
              make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
        }
  }
  __syncthreads();

  // ---- wave q < 4 sums quad q ----------------------------------------------------------------------------------
  // the rows' padding, 0 bits in both operands, counted +1 each
  const int corr = (int)((uint32_t)p.Kformula - (uint32_t)nc * 256u);
  int s[WT][WT][4];
  if (wave < 4) {  // wave-uniform
    auto sum = [&](auto first, auto four) {
      using V4 = decltype(four);
#pragma unroll
      for (int i = 0; i < WT; ++i)
#pragma unroll
        for (int j = 0; j < WT; ++j) {
          V4 t = {first, first, first, first};
#pragma unroll
          for (int k = 0; k < KS; ++k) {
            const V4 v = reinterpret_cast<const V4 *>(sPart)[((k * WT * WT + i * WT + j) * 4 + wave) * 64 + lane];
            t.x += v.x;
            t.y += v.y;
            t.z += v.z;
            t.w += v.w;
          }
          s[i][j][0] = (int)t.x;
          s[i][j][1] = (int)t.y;
          s[i][j][2] = (int)t.z;
          s[i][j][3] = (int)t.w;
        }
    };
    // one branch around all: inside, it kept the reads of a block behind the sums of the one before
    if (as_int) sum(corr, int4());
    else sum((float)corr, float4());
  }

  if constexpr (!SIGN) {
    if (wave >= 4 || m0 + 8 * wave >= p.M) return;  // uniform
    const int n = n0 + WT * l32;
    if (n >= p.N) return;
    // Columns past N hold column N - 1 once more and go there; rows past M (of partial tiles) don't: with few rows, they would
    // all write the same line (1 x 1024 x 8192 3.75 us, 4.1).
    int64_t off[WT];
#pragma unroll
    for (int j = 0; j < WT; ++j) {
      const int c = min(n + j, p.N - 1);
      off[j] = c;
      if (p.img_stride != 0) {  // NCHW planes
        const uint32_t img = fdiv_sel((uint32_t)c, p.divOHW);
        off[j] = (int64_t)img * p.img_stride + ((uint32_t)c - img * p.OHW);
      }
    }
    const bool full = m0 + B32 <= p.M;
    auto store = [&](auto *base, int64_t ld, auto value) {
      using V = typename std::remove_pointer<decltype(base)>::type;
      typedef V vec __attribute__((ext_vector_type(WT)));
      V *ptr[WT];
#pragma unroll
      for (int j = 0; j < WT; ++j) ptr[j] = base + off[j] + (int64_t)mq * ld;
      auto rows = [&](auto whole, auto pairs) {
#pragma unroll
        for (int i = 0; i < WT; ++i) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if (!decltype(whole)::value && mq + 32 * i + e >= p.M) continue;
            const int64_t row = (int64_t)(32 * i + e) * ld;  // uniform
            if constexpr (decltype(pairs)::value) {
              vec v;
#pragma unroll
              for (int j = 0; j < WT; ++j) v[j] = value(i, j, e);
              *reinterpret_cast<vec *>(ptr[0] + row) = v;
            } else {
#pragma unroll
              for (int j = 0; j < WT; ++j) ptr[j][row] = value(i, j, e);
            }
          }
        }
      };
      // both uniform, and branched on once: around each store they cost 8 rows by two branches
      const std::true_type yes;
      const std::false_type no;
      if constexpr (WT == 1) rows(no, no);  // no second copy of its few stores
      else if (p.pairs) full ? rows(yes, yes) : rows(no, yes);
      else full ? rows(yes, no) : rows(no, no);
    };
    if (p.C) store(p.C, p.ldc, [&](int i, int j, int e) { return s[i][j][e]; });
    if (row_affine) store(p.Y, p.ldy, [&](int i, int j, int e) { return fmaf(sc[i][e], (float)s[i][j][e], bi[i][e]); });
    else if (p.Y) store(p.Y, p.ldy, [&](int i, int j, int e) { return fmaf(csc[j], (float)s[i][j][e], cbi[j]); });
  } else {
    // four sign bits per column and row block; lanes l and l + 32 hold the two nibbles of a byte.  The members of a
    // pooling window are consecutive columns: WT in this lane, the others in its neighbours.
    if (wave < 4) {
#pragma unroll
      for (int i = 0; i < WT; ++i)
#pragma unroll
        for (int j = 0; j < WT; ++j) {
          uint32_t nib = 0u;
#pragma unroll
          for (int e = 3; e >= 0; --e) {
            int m = s[i][j][e];
            if constexpr (EMODE == 2) {
              if constexpr (WT == 2) m = max(s[i][0][e], s[i][1][e]);
              else m = max(m, __builtin_amdgcn_mov_dpp(m, 0xB1, 0xF, 0xF, true));        // lane ^ 1
              m = max(m, __builtin_amdgcn_mov_dpp(m, WT == 2 ? 0xB1 : 0x4E, 0xF, 0xF, true));  // lane ^ 1 / lane ^ 2
            }
            nib = 2u * nib + (fmaf(sc[i][e], (float)m, bi[i][e]) >= 0.0f ? 1u : 0u);
          }
          const uint32_t other = (uint32_t)__shfl_xor((int)nib, 32);
          if (half == 0) sO[(WT * l32 + j) * (4 * WT) + 4 * i + wave] = (uint8_t)(nib | (other << 4));
        }
    }
    __syncthreads();
    // one thread per output pixel and 32 channels
    const int npix = EMODE == 2 ? B32 / 4 : B32;
    if (tid < npix * WT) {
      const int px = tid / WT, i = tid % WT;
      const uint32_t w = *reinterpret_cast<const uint32_t *>(&sO[(EMODE == 2 ? 4 * px : px) * (4 * WT) + 4 * i]);
      const int64_t gp = (int64_t)(EMODE == 2 ? n0 >> 2 : n0) + px;
      const int64_t limit = EMODE == 2 ? (int64_t)(p.N >> 2) : (int64_t)p.N;
      const int w32 = mi * WT + i;  // 32-channel half word
      if (gp < limit && w32 < 2 * p.cw_out) {
        uint32_t *o = reinterpret_cast<uint32_t *>(p.outp) + gp * p.cw_out * 2;
        o[w32] = w;
        // an odd number of 32-channel tiles: the last word's upper half holds no channel
        if (WT == 1 && mi == p.tilesM - 1 && (p.tilesM & 1)) o[w32 + 1] = 0u;
      }
    }
  }
}

template <int WT>
static bnn_status split_tiles(GemmParams &p) {
  p.tilesM = (p.M + 32 * WT - 1) / (32 * WT);
  const int64_t tn = ((int64_t)p.N + 32 * WT - 1) / (32 * WT);
  const int64_t blocks = p.tilesM * tn;
  if (blocks > 0x7fffffffLL) return BNN_ERR_UNSUPPORTED;
  p.tilesN = (int)tn;
  p.divTilesM = FastDiv((uint32_t)p.tilesM);
  p.pairs = p.N % 2 == 0 && (!p.C || p.ldc % 2 == 0) && (!p.Y || p.ldy % 2 == 0) &&
            (p.img_stride == 0 || (p.OHW % 2 == 0 && p.img_stride % 2 == 0));
  return BNN_OK;
}

template <int WT, int KS>
static bnn_status launch_split(GemmParams &p, int bmode, int emode, hipStream_t s) {
  const bnn_status st = split_tiles<WT>(p);
  if (st != BNN_OK) return st;
  const dim3 grid((unsigned)p.tilesM * (unsigned)p.tilesN), block(64 * KS);
  ProfScope ps(KID_XNOR_GEMM_FP4_SPLIT, s);
  if (bmode == 0) {
    const bool v16 = p.Kw64 % 2 == 0 && p.lda32 % 4 == 0 && p.ldb % 2 == 0;
    if (v16) hipLaunchKernelGGL((xnor_gemm_fp4_split_kernel<WT, KS, SG_EXPL16, 0>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((xnor_gemm_fp4_split_kernel<WT, KS, SG_EXPL8, 0>), grid, block, 0, s, p);
    return launch_status();
  }
  p.b_vec16 = p.Kw64 % 2 == 0 && p.lda32 % 4 == 0;
  if (emode == 0) hipLaunchKernelGGL((xnor_gemm_fp4_split_kernel<WT, KS, SG_CONV, 0>), grid, block, 0, s, p);
  else if (p.g.pool) hipLaunchKernelGGL((xnor_gemm_fp4_split_kernel<WT, KS, SG_CONV, 2>), grid, block, 0, s, p);
  else hipLaunchKernelGGL((xnor_gemm_fp4_split_kernel<WT, KS, SG_CONV, 1>), grid, block, 0, s, p);
  return launch_status();
}

// By t, tiles of 32 x 32 outputs per compute unit.  Up to 2 latency is all there is: 32 x 32 tiles, K split 8 ways up to 1
// (1 x 1024 x 8192 3.7 us, 4 ways 4.0; a 3 x 3 layer of 512 channels, 6 images of 4 x 4, 4.9 against 5.0), then 4 (3 x 3 of 320
// channels at t = 1.1 5.4 against 6.1, 1024 x 485 x 2560 4.5 against 4.7; 64 x 64 tiles 7.4 and 5.9, staged ones 11 and 8), but
// for the longest gathers (5 x 5 of 512 channels, t = 1.8 11.1 against 10.8), which are shorter where a pixel has an odd number of
// words and is gathered word by word (5 x 5 of 320 channels, t = 1.4 9.5 against 8.9).
// Beyond, a 32 x 32 tile reads twice the operands of a 64 x 64 one for its outputs (32 lines for every load instruction,
// about 1.1 us for each workgroup that a unit gets at K = 4096) and a 64 x 64 one pays a larger exchange (1.2 us),
// so it depends on t times the words of a row:
//   up to 4, where a unit has one 64 x 64 tile: below 240 words 32 x 32 (300 x 2164 x 4096 6.5 against 7.0; 512 x 1551 x 2304 5.2
//            against 6.0), above 64 x 64 (256 x 4096 x 4096 6.8 against 7.5, 512 x 1124 x 9216 9.0 against 9.9); convolutions
//            only up to t = 3, the third workgroup (3 x 3 of 512 channels 7.7 against 8.5; 5 x 5 of 100 channels, t = 3.2 7.1
//            against 6.6), and their 64 x 64 tiles take 8 ways, which share the gather (1024 channels of 8 x 8, t = 3.4: 10.4 against
//            10.9), signs of an odd number of words a pixel from 200 words (3 x 3 of 704 channels, t = 2.2 10.2 against 9.3); short
//            rows 32 x 32 (3 x 3 of 128 channels, t = 3.3 5.3 against 5.4);
//   up to 8, where it has two: 32 x 32 below 320 words up to 6 (512 x 2380 x 4096 8.7 against 9.7; 64 x 20268 x 2304 6.5 against
//            7.8), for convolutions up to 5 (3 x 3 of 256 channels of 7 x 7, t = 4.5 7.3 against 8.9, t = 5.9 7.8 against 7.4),
//            unless of an odd number of words a pixel, gathered word by word; short ones up to 5.5 (t = 5.4 7.2 against 8.0);
//   short rows beyond that: 64 x 64 for convolutions of small maps, whose regions staged tiles copy with most lanes idle (192
//            channels of 4 x 4, t = 5.8 8.2 against 10.6 on 128 x 128; 64 of 8 x 8, t = 7.8 5.9 against 6.5; but 100 of 56 x
//            56, t = 6.1 8.8 against 7.9), as long as a unit holds its tiles, two of them (96 channels are two tiles high: 100 of 10
//            x 10, t = 6.6 9.1 against 7.0; signs of the smallest maps then take 32 x 32: 128 of 2 x 2 9.3, 7.7, staged 11.4), and not
//            for fp32 maps from 64 pixels on, whose stores staged tiles overlap (128 of 10 x 10, t = 7.1 9.0 against 8.6, of 16
//            x 16 8.8, 8.0), from 36 on without a stride and with few words (64 of 7 x 7, t = 6.1 8.8 against 8.1, 192 of 7 x 7 9.4, 10.1);
//            else 128 x 128 (100 x 14516 x 512 5.2 against 6.3);
//   one row or one column of tiles, up to 8: 32 x 32, a larger tile has nothing to use twice and computes rows for nothing
//            (4 x 40000 x 1024: 4.1 us, 64 x 64 split 6.7, 64 x 256 staged 5.4; 4 x 40000 x 4096 6.6, 10.2, 10.4; 32 x 65536 x
//            4096 12.3, 16.0, 12.5; 40000 x 10 x 2048 5.0, 9.4, 15.7), above 6 from 16 words (4 x 65536 x 1024 5.2 against 5.6,
//            x 300 4.7 against 4.5).
// From 8 on staged tiles reuse their operands better.  -1: does not apply.
static int split_shape(const GemmParams &p, int bmode) {
  const int64_t t = (((int64_t)p.M + 31) / 32) * (((int64_t)p.N + 31) / 32), cu = p.n_cu;
  const int64_t words = t * p.Kw64 / cu;  // of the tiles of a unit
  const bool conv = bmode != 0, single = p.M <= 32 || p.N <= 32, short_rows = p.Kw64 <= 32;
  const bool odd = conv && (p.g.Cw & 1), signs = p.outp != nullptr;
  if (t <= cu || (t <= 2 * cu && conv && p.Kw64 > (odd ? 110 : 160))) return 1;
  if (t <= 2 * cu) return 0;
  if (single && (t <= 6 * cu || (t <= 8 * cu && p.Kw64 >= 16))) return 0;
  if (short_rows && 2 * t <= 11 * cu) return 0;
  if (t <= 4 * cu) {
    if (words <= (odd && signs ? 200 : 240) && (!conv || t <= 3 * cu)) return 0;
    return conv ? 3 : 2;
  }
  if (t <= 8 * cu) {
    if (short_rows) {
      if (!conv || p.Kw64 < 9 || !halo_lanes_idle(p.g)) return -1;
      const int64_t pixels = (int64_t)p.g.OH * p.g.OW;
      if ((((int64_t)p.M + 63) / 64) * (((int64_t)p.N + 63) / 64) > 2 * cu) return signs && pixels <= 32 ? 0 : -1;
      return p.Y && pixels >= (p.g.sH * p.g.sW == 1 && p.Kw64 <= 18 ? 36 : 64) ? -1 : 2;
    }
    if (words <= 320 && (conv ? !odd && t <= 5 * cu : t <= 6 * cu)) return 0;
    return 2;
  }
  // rows beyond the exact range of the other kernel's accumulators
  return p.Kw64 >= (1 << 18) - 2 ? 2 : -1;
}

bool fp4_split_applicable(const GemmParams &p, int bmode) { return split_shape(p, bmode) >= 0; }

bnn_status launch_gemm_fp4_split(GemmParams &p, int bmode, int emode, hipStream_t s, int shape) {
  switch (shape < 0 ? split_shape(p, bmode) : shape) {
    case 0: return launch_split<1, 4>(p, bmode, emode, s);
    case 1: return launch_split<1, 8>(p, bmode, emode, s);
    case 2: return launch_split<2, 4>(p, bmode, emode, s);
    case 3: return launch_split<2, 8>(p, bmode, emode, s);
    default: return BNN_ERR_UNSUPPORTED;
  }
}

// ---- convolution from the fp32 image in one launch ---------------------------------------------------------
// Most input rows of a tile of 32 output pixels, which begins at a multiple of 32.  In one image its ends are as far apart as
// its first and last output row by the stride and a window, and moving them into the image brings them no further apart; an
// image's end between them counts the whole image, less as much as the last one's end lies above the first one's begin there,
// but for what moving them into the image takes from that.  Linear between the numbers of images a tile may touch: the largest
// is at an end.
static int64_t image_rows_most(const ConvGeom &g) {
  const int64_t OW = g.OW, OH = g.OH, H = g.H, start = OW - std::gcd((int64_t)32, OW);  // last column that a tile may begin in
  auto most = [&](int64_t pixels, int64_t window) {
    const int64_t d = std::min<int64_t>((start + pixels - 1) / OW, (int64_t)g.Nimg * OH - 1);  // output rows apart
    const int64_t moved = std::max<int64_t>(0, g.pH - (window - 1)) + std::max<int64_t>(0, (OH - 1) * g.sH - g.pH - (H - 1));
    int64_t rows = 0;
    for (const int64_t i : {d / OH, (d + OH - 1) / OH}) {
      const int64_t apart = (d - i * OH) * g.sH + window - 1;
      rows = std::max(rows, i * H + (apart < 0 ? std::min<int64_t>(0, apart + moved) : apart) + 1);
    }
    return rows;
  };
  // to where the next tile's begin; the last tile's: to the image's end
  const int64_t rows = std::max(most(32, g.kH), most(33, 1)) + g.sH - 1;
  return std::min<int64_t>(rows, (int64_t)g.Nimg * H);
}

bool encode_nchw_supported(int N, int C, int H, int W, int OHp, int OWp);

static int64_t image_pixels(const GemmParams &p) { return image_rows_most(p.g) * p.g.W; }

// By t, tiles of 32 x 32 outputs per compute unit, and b, the fp32 values in KB that a tile encodes: a launch and the gap before it
// are gone (about 2.5 us in a graph, 4 in a stream), and every row of tiles encodes its columns' pixels again, on its own, at
// about 50 KB a microsecond.  In graphs, two launches against one:
//   t up to 1, 8 ways: b 32 (128 x 16 x 16 to 256, 3 x 3) 6.4, 4.6 us; 65 (256 x 16 x 16 to 256) 7.3, 5.4; 131 (512 x 8 x 8 to 512) 9.5,
//     7.2; 136 (3 x 256 x 13 x 19 to 35, 5 x 5) 10.3, 8.4; 123 (3 x 128 x 6 x 40 to 256, 5 x 5, t = 0.7) 7.4, 6.6; but 172 (128 x 39 x
//     48 to 256, 5 x 5 by 2) 7.3, 7.45; 287 (5 x 256 x 7 x 40 to 64, 5 x 5) 10.1, 11.9;
//   t up to 2, 4 ways: b 12 (28 x 64 x 8 x 6 to 256) 6.9, 5.5; 32 (8 x 128 x 16 x 16 to 256) 7.4, 5.8; 65 (8 x 256 x 16 x 16 to 256) 8.6, 7.3; but
//     123 (8 x 99 x 25 x 52 to 64, 5 x 5) 9.3, 13.8; 184 (2 x 256 x 12 x 45 to 256, t = 1.06) 8.3, 10.5;
//   t up to 3, the same up to 24: 21 (57 x 64 x 6 x 14 to 256, t = 2.7) 7.7, 6.6; but 54 (34 x 64 x 62 x 18 to 64 by 2, t = 2.3) 9.3, 9.3;
//   beyond, two launches: t = 3.5, b 43 8.8, 9.8; t = 4, 49 8.3, 9.5; t = 16, 65 15.5, 30.7.
// shape >= 0: that one where the kernel can take the problem.
int conv_image_shape(const GemmParams &p, int shape) {
  const ConvGeom &g = p.g;
  if (!encode_nchw_supported(g.Nimg, g.C, g.H, g.W, g.H, g.W)) return -1;  // what the encode refuses stays refused
  const int64_t px = image_pixels(p), hw = (int64_t)g.H * g.W;
  // LDS; 32-bit offsets over the images of a region
  if (px * g.Cw * 8 > 24576 || (px / hw + 2) * hw * g.C >= (1LL << 30)) return -1;
  if (shape >= 0) return shape;
  const int64_t t = (((int64_t)p.M + 31) / 32) * (((int64_t)p.N + 31) / 32), bytes = 4 * px * g.C;
  const int64_t cu = p.n_cu, kb = 1024;
  if (t <= cu) return bytes <= 160 * kb ? 1 : -1;
  return (t <= 2 * cu && bytes <= 80 * kb) || (t <= 3 * cu && bytes <= 24 * kb) ? 0 : -1;
}

void conv_image_rows(const GemmParams &p, int pixel, int64_t *rows) {
  int r0, r1;
  image_rows(p.g, (uint32_t)pixel, 32u, (uint32_t)p.N, r0, r1);
  rows[0] = r0;
  rows[1] = r1;
  rows[2] = image_rows_most(p.g);
}

template <int KS>
static bnn_status launch_image(ImageParams &p, hipStream_t s) {
  const bnn_status st = split_tiles<1>(p);
  if (st != BNN_OK) return st;
  p.b_vec16 = p.Kw64 % 2 == 0 && p.lda32 % 4 == 0;
  const dim3 grid((unsigned)p.tilesM * (unsigned)p.tilesN), block(64 * KS);
  ProfScope ps(KID_XNOR_GEMM_FP4_SPLIT, s);
  hipLaunchKernelGGL((xnor_gemm_fp4_split_kernel<1, KS, SG_IMAGE, 0, ImageParams>), grid, block,
                     (size_t)(image_pixels(p) * p.g.Cw * 8), s, p);
  return launch_status();
}

bnn_status launch_conv_image(const GemmParams &p, const float *x, uint64_t *img, int shape, hipStream_t s) {
  ImageParams q;
  static_cast<GemmParams &>(q) = p;
  q.x = x;
  q.img = img;
  q.HW = (uint32_t)p.g.H * (uint32_t)p.g.W;
  q.divHW = FastDiv(q.HW);
  return shape == 0 ? launch_image<4>(q, s) : launch_image<8>(q, s);
}

}  // namespace bnn
