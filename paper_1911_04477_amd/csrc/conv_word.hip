// Binarized convolution of an image of few words per pixel (at most 256 channels, 1 x 1 and 3 x 3) on the matrix cores, taps
// straight from memory to operand fragments.
//
// xnor_gemm_fp4_kernel copies a tile's input region to LDS, tabulates where every column's pixel and every word of a patch
// lie, and stages the filters in a ring with a barrier per stage: 3 to 6 thousand clocks before its first matrix
// instruction, beside 1152 clocks of them per wave for 9 words.  Here a lane loads the words of its own pixel under every
// tap (contiguous over a wave; the taps of several pixels meet in the L1), a lane exchange turns the word of 64 pixels into
// the fragments of two column blocks (a matrix instruction takes half a word of 32 pixels from either half of the wave), and
// that is all a column needs.  The filters' codes are expanded once per workgroup into LDS, in fragment order, so that a wave
// expands the columns only: 14 vector instructions beside the four matrix instructions of a word, against 28.  One barrier.
// A wave owns 64 channels x 64 pixels (two row blocks of 64 per wave, which halve the columns' expansions: 0.6 to 1.0 times as
// fast, half the waves).  Bound: latency below about one workgroup a unit (4.0 us of 9 words, 4.5 of 18, 9.5 of 36), then the
// matrix loop.  3 x 3, against the tiles of xnor_gemm_fp4_kernel, per launch: 32 x 64 x 57 x 55 -> 64 packed 7.3 -> 4.9 us;
// 256 x 64 x 32 x 32 -> 64 10.9 -> 7.2; 64 x 64 x 56 x 56 -> 256 27.9 -> 17.6; 256 x 128 x 16 x 16 -> 256 12.0 -> 9.8;
// 128 x 128 x 32 x 32 -> 128 int32 17.1 -> 16.5; 64 x 256 x 56 x 56 -> 256 fp32 68.8 -> 64.6; 1 x 1 of 64, 128, 256
// channels: 64 x 56 x 56 -> 256, 128, 256 packed 21.5 -> 9.5, 12.1 -> 6.2, 23.1 -> 12.5.
#include "common.h"
#include "fp4_tile.h"

namespace bnn {

enum : int { CW_SIGN = 3, CW_POOL = 4 };  // below: map stores MS_NT, MS_VEC, MS_ONE

template <int KH, int KW, int CW, int T, int EMODE>
__global__ __launch_bounds__(T, T > 256 ? 4 : 2) void conv_word_kernel(GemmParams p) {
  constexpr int TAPS = KH * KW, WORDS = TAPS * CW, BM = 64, BN = T;
  constexpr bool MAPS = EMODE < CW_SIGN, POOL = EMODE == CW_POOL;
  constexpr bool DEALT = EMODE != MS_ONE && EMODE != CW_SIGN;  // a lane's two columns are consecutive
  __shared__ __attribute__((aligned(16))) u32x4 sA[WORDS + WORDS % 2][2][2][32];  // word, row block, half, row
  __shared__ __attribute__((aligned(16))) float sSc[BM];
  __shared__ __attribute__((aligned(16))) float sBi[BM];
  const int tid = threadIdx.x;
  const int lane = tid & 63, half = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const ConvGeom &g = p.g;
  // row tiles of one column tile are neighbours, and each XCD gets a contiguous run
  const uint32_t nwg = gridDim.x;
  uint32_t bid = blockIdx.x;
  {
    const uint32_t q = nwg >> 3, r = nwg & 7u, xcd = bid & 7u, i = bid >> 3;
    bid = xcd * q + min(xcd, r) + i;
  }
  const int ni = (int)fdiv_sel(bid, p.divTilesM), mi = (int)(bid - (uint32_t)ni * (uint32_t)p.tilesM);
  const int m0 = mi * BM, n0 = ni * BN + 64 * wave;

  // ---- filters: T / 64 threads to a row of the tile, as many dwords apart ------------------------------------
  constexpr int DW = 2 * WORDS, TR = T / BM, PER = (DW + TR - 1) / TR;
  const int wrow = tid / TR, wq = tid % TR;
  uint32_t wa[PER];
  {
    const uint32_t *const row = p.A + (size_t)(uint32_t)min(m0 + wrow, p.M - 1) * (size_t)p.lda32;
#pragma unroll
    for (int i = 0; i < PER; ++i) wa[i] = row[min(wq + TR * i, DW - 1)];
  }
  const bool affine = !MAPS || (p.Y && p.axis == BNN_CH_ROW);  // uniform
  float fsc, fbi;
  {  // no condition around the loads: a wait for older ones could not tell how many follow
    const float *const ps = affine ? p.scale : reinterpret_cast<const float *>(p.A);
    const float *const pb = affine ? p.bias : reinterpret_cast<const float *>(p.A);
    const int r = affine ? min(m0 + (tid & 63), p.M - 1) : 0;
    fsc = ps[r];
    fbi = pb[r];
  }

  // ---- this lane's pixel, of column block `half`: its word under every tap, from a readable place ---------------
  constexpr uint32_t PX = 8u * CW;  // bytes of a pixel
  const uint32_t wpx = (uint32_t)g.W * PX, ipx = (uint32_t)g.H * wpx;
  uint32_t img0, oh0, ow0, img, oh, ow;
  column_pixel(g, (uint32_t)min(n0, p.N - 1), POOL, img0, oh0, ow0);  // uniform
  column_pixel(g, (uint32_t)min(n0 + (DEALT ? 2 * l32 + half : lane), p.N - 1), POOL, img, oh, ow);
  const char *const base = reinterpret_cast<const char *>(g.act) + (size_t)img0 * (size_t)ipx;
  uint32_t row[KH], col[KW], rmask[KH], cmask[KW];
  {
    const int ih0 = (int)oh * g.sH - g.pH, iw0 = (int)ow * g.sW - g.pW;
#pragma unroll
    for (int k = 0; k < KH; ++k) {
      const int ih = min(max(ih0 + k, 0), g.H - 1);
      rmask[k] = ih == ih0 + k ? ~0u : 0u;
      row[k] = (img - img0) * ipx + (uint32_t)ih * wpx;  // host: 64 pixels span less than 4 GiB
    }
#pragma unroll
    for (int k = 0; k < KW; ++k) {
      const int iw = min(max(iw0 + k, 0), g.W - 1);
      cmask[k] = iw == iw0 + k ? ~0u : 0u;
      col[k] = (uint32_t)iw * PX;
    }
  }
  constexpr int DEPTH[] = {9, 6, 4, 3}, RING = TAPS < DEPTH[CW - 1] ? TAPS : DEPTH[CW - 1];  // taps in flight
  u32x2 raw[RING][CW];
  auto load_tap = [&](int t) {
    const char *const px = base + (row[t / KW] + col[t % KW]);
    u32x2 *const r = raw[t % RING];
    if constexpr (CW % 2 == 0) {
#pragma unroll
      for (int w = 0; w < CW; w += 2) {
        const u32x4 v = reinterpret_cast<const u32x4 *>(px)[w / 2];
        r[w] = v.lo;
        r[w + 1] = v.hi;
      }
    } else {
#pragma unroll
      for (int w = 0; w < CW; ++w) r[w] = reinterpret_cast<const u32x2 *>(px)[w];
    }
  };
#pragma unroll
  for (int t = 0; t < RING; ++t) load_tap(t);

  // ---- filter codes, affine constants -> LDS ---------------------------------------------------------------
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int d = wq + TR * i;
    const v8i c = expand_e2m1<false>(wa[i]);
    // an odd number of words: the last dwords once more, to a place that is not read
    if (DW % TR == 0 || TR <= 4 || d < DW)
      sA[d >> 1][wrow >> 5][d & 1][wrow & 31] = u32x4{(uint32_t)c[0], (uint32_t)c[1], (uint32_t)c[2], (uint32_t)c[3]};
  }
  if (tid < BM) {  // rows past M: sign bit 0; maps: such rows are row M - 1
    const bool on = affine && (MAPS || m0 + tid < p.M);
    sSc[tid] = on ? fsc : 0.0f;
    sBi[tid] = on ? fbi : -1.0f;
  }
  // the values past a tap's channels are 0 bits in both operands and count +1 each
  Fp4Acc<2, 2> acc;
  acc.init(-(float)(64 * WORDS - p.Kformula));
  __syncthreads();

  // ---- taps: two row blocks x two column blocks, the next tap's columns expanded beside them -------------------
  // The lower lanes hold pixels of block 0, the upper ones of block 1; exchanged, the lower halves of both blocks' words and
  // the upper ones.  Outside the image: +1 in every real channel.
  const uint64_t word = (g.C & 63) ? (1ull << (g.C & 63)) - 1ull : ~0ull;
  const uint32_t plo = (uint32_t)word, phi = (uint32_t)(word >> 32);
  auto fragments = [&](int t, uint32_t (&x)[2]) {
    const int tap = t / CW, kh = tap / KW, kw = tap % KW;
    const bool last = t % CW == CW - 1;
    const uint32_t m = rmask[kh] & cmask[kw], lo = last ? plo : ~0u, hi = last ? phi : ~0u;
    const u32x2 r = raw[tap % RING][t % CW];
    const auto w = __builtin_amdgcn_permlane32_swap((r.x & m) | (lo & ~m), (r.y & m) | (hi & ~m), false, false);
    x[0] = w[0];
    x[1] = w[1];
  };
  u32x4 a[2], na[2];
  v8i eb[2], nb[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) a[i] = sA[0][i][half][l32];
  uint32_t x[2];
  fragments(0, x);
#pragma unroll
  for (int j = 0; j < 2; ++j) eb[j] = expand_e2m1<true>(x[j]);
#pragma unroll
  for (int t = 0; t < WORDS; ++t) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int i = k / 2, j = k % 2;
      v16f &c = acc.v[i][j];
      c = mfma_e2m1(v8i{(int)a[i].x, (int)a[i].y, (int)a[i].z, (int)a[i].w, 0, 0, 0, 0}, eb[j], c);
      asm volatile("" : "+v"(c));  // emits nothing; keeps the order, as in multiply_and_expand
      if (t + 1 < WORDS) {
        if (k < 2) na[k] = sA[t + 1][k][half][l32];
        if (k == 0) {
          fragments(t + 1, x);
          nb[0] = expand_e2m1<false>(x[0]);
        }
        if (k == 2) nb[1] = expand_e2m1<false>(x[1]);
        // a tap's last word has been taken: its place is free
        if (k == 3 && (t + 2) % CW == 0 && (t + 1) / CW + RING < TAPS) load_tap((t + 1) / CW + RING);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (t + 1 < WORDS) {
#pragma unroll
      for (int i = 0; i < 2; ++i) a[i] = na[i];
#pragma unroll
      for (int j = 0; j < 2; ++j) eb[j] = nb[j];
    }
  }
  settle(acc);
  if constexpr (MAPS) store_maps<2, 2, EMODE>(p, acc, m0, n0, lane, sSc, sBi);
  else if constexpr (POOL) store_signs_pooled<2, 2>(p, acc, m0, n0, lane, sSc, sBi);
  else store_signs<2, 2, false>(p, acc, m0, n0, lane, sSc, sBi);
}

template <int KH, int KW, int CW>
static bnn_status launch_word(GemmParams &p, int emode, hipStream_t s) {
  // more waves where the filters' codes let few workgroups onto a unit
  constexpr int T = KH * KW * CW > 18 ? 512 : 256;
  p.tilesM = (p.M + 63) / 64;
  const int64_t tn = ((int64_t)p.N + T - 1) / T, blocks = p.tilesM * tn;
  if (blocks > 0x7fffffffLL) return BNN_ERR_UNSUPPORTED;
  p.tilesN = (int)tn;
  p.divTilesM = FastDiv((uint32_t)p.tilesM);
  const dim3 grid((unsigned)blocks), block(T);
  ProfScope ps(KID_XNOR_GEMM_FP4, s);  // a form of it
  if (emode == 1) {
    if (p.g.pool) hipLaunchKernelGGL((conv_word_kernel<KH, KW, CW, T, CW_POOL>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((conv_word_kernel<KH, KW, CW, T, CW_SIGN>), grid, block, 0, s, p);
  } else if (!p.colperm) {
    hipLaunchKernelGGL((conv_word_kernel<KH, KW, CW, T, MS_ONE>), grid, block, 0, s, p);
  } else if (p.nt_store) {
    hipLaunchKernelGGL((conv_word_kernel<KH, KW, CW, T, MS_NT>), grid, block, 0, s, p);
  } else {
    hipLaunchKernelGGL((conv_word_kernel<KH, KW, CW, T, MS_VEC>), grid, block, 0, s, p);
  }
  return launch_status();
}

bool conv_word_applicable(const GemmParams &p, int bmode) {
  const ConvGeom &g = p.g;
  if (bmode != 1 || g.Cw > 4 || g.kH != g.kW || (g.kH != 1 && g.kH != 3)) return false;
  const double span = (63.0 / ((double)g.OH * (double)g.OW) + 2.0) * 8.0 * (double)g.Cw * (double)g.H * (double)g.W;
  return span < 4294967296.0;
}

// By t, tiles of 32 x 32 outputs per compute unit, and u, tiles of 64 x 256, against the kernels that take the call otherwise (u's, the
// other's time first).  Both maps of a call are twice the epilogue, and more than three rows of tiles (192 channels) load and
// expand a column as often: maps then need more work.
// 1 x 1: signs and one word always (1 x 15 x 18 x 29 3.3 -> 3.0 us; maps by stride 2 5.9 -> 4.1, 7.6 -> 4.7; a pointwise map without a
//   stride is an explicit GEMM and does not get here); maps of more words to at most 32 channels or, in whole rows of tiles, 160 pixels
//   (256 x 60 pixels to 64 3.3, 2.9; 45 pixels to 52 3.15, 3.4), else of two and three words from t = 1.6 (D = 256, t = 1.2 3.45, 3.9; 1.8
//   3.55, 3.5), up to 128 channels 0.9 (0.3 3.3, 3.4; 1.25 3.65, 3.45), of four from 2 (256 x 7 x 14 x 9 to 128, t = 0.12 3.15, 3.7; 1.1
//   3.5, 4.05; 2.1 3.9, 3.7), of small images to many channels 3 (18 pixels, t = 2.0 3.8, 4.3; 9 pixels 4.0, 5.4; 24, t = 4.2 5.2, 4.0).
// 3 x 3, by words of a pixel:
//   1: signs from t = 1.8, up to 64 channels 2 (1.9 3.8 against 3.95, 2.06 4.15, 3.8; 6.2 5.4, 3.8; 31 8.7, 5.8), maps, whose split tiles
//      have a shorter epilogue, from 2.5 (2.0 4.0 against 4.4, 2.5 4.5, 4.6, 2.7 4.9, 4.5, 13 7.7, 5.4, 95 22.7, 20.5), both of more than
//      32 channels from 3.2 (2.7 9.0 against 9.6, 3.6 9.8, 9.55; 12 channels, 3.2 8.7, 8.2), any to more than 192 from 4 (3.1 4.5 against
//      4.8, 4.2 5.2, 4.7; both 2.75 8.5, 10.3, 4.6 9.7, 8.7 to 9.9);
//   2: signs from t = 3 (2.2 4.4 against 4.5, 2.85 4.4, 4.65, 3.3 4.8, 4.6, 5.7 6.1, 4.6, 64 12.0, 9.8), maps from 4 (3.7 5.2 against 5.6,
//      4.4 6.4, 6.2, 6.9 8.0, 6.2, 115 32.1, 29.6);
// (up to three words: maps so small that a region's lanes idle stay on the split-K tiles where those take them, from 5.5 to 8
// tiles a unit, which their tests state: 216 x 128 x 6 x 8 -> 166 7.6 us against 5.4);
//   3: from u = 0.75 (0.56 7.8 against 8.0 and 9.9, 7.9; 0.67 8.5, 8.2; 0.98 9.7, 8.9; 2.3 14.7, 12.4; 14 50.5, 42.0), maps not
//      with a second workgroup of 512 pixels on less than half of the units (u 2.08 16.6, 17.9; 2.4 17.2, 18.3; 2.9 17.7, 17.7; 3.05
//      19.5, 16.9);
//   4: its codes let one workgroup of 512 pixels run beside another, so it is whole rounds of them, two a unit: from u = 1 (0.95
//      8.8 against 9.6, 1.04 11.6, 9.5) up to one a unit (1.98 12.0, 9.9; 2.2 14.9, 15.3; 2.6 15.3, 15.4; maps 1.97 16.1, 15.1; 259 of them,
//      33 on the 32 units of an XCD, 17.0, 18.2; 2.2 17.5, 19.7; 2.6 19.2, 20.3), and from one and a half on (3.03 18.5, 15.5; 3.06
//      23.2, 19.7; 4.7 23.4, 21.8; 7.9 31.7, 29.5; 12 65.9, 60.4), but maps not with the first eighth of a third (4.1 24.4, 25.7; 4.3
//      28.6, 29.4; 4.4 23.7, 25.8; 4.65 27.0, 26.4);
//   3 and 4: both maps not from 1.7 workgroups of 512 pixels a unit on, where their stores are the time (1.6 39.0, 36.8; 1.9 43.6,
//      46.1; 3.1 60.9, 66.4; 4.2 78.5, 87.0), unless the other kernel's go past the caches in pieces of lines (102, 87).
bool conv_word_faster(const GemmParams &p, int emode) {
  const ConvGeom &g = p.g;
  const int64_t cu = p.n_cu;
  const int64_t tiles = (((int64_t)p.M + 31) / 32) * (((int64_t)p.N + 31) / 32);
  const int64_t wide = (((int64_t)p.M + 63) / 64) * (((int64_t)p.N + 255) / 256);
  const int64_t groups = (((int64_t)p.M + 63) / 64) * (((int64_t)p.N + 511) / 512);
  const bool signs = emode != 0, both = p.C && p.Y, tall = p.M > 192;
  if (g.kH == 1) {
    if (signs || g.Cw == 1 || p.M <= 32 || (p.M >= 64 && p.N <= 160)) return true;
    if (tall && (int64_t)g.OH * g.OW < 64) return tiles > 3 * cu;
    return 10 * tiles > (g.Cw == 4 ? 20 : p.M > 128 ? 16 : 9) * cu;
  }
  if (g.Cw < 4 && 2 * tiles > 11 * cu && fp4_split_applicable(p, 1)) return false;
  if (g.Cw > 2 && both && 10 * groups > 17 * cu &&
      !(map_columns_by_four(p) && nontemporal_maps(p, 1) && !nontemporal_maps(p, 1, true)))
    return false;
  switch (g.Cw) {
    case 1:
      if (signs) return p.M <= 64 ? tiles >= 2 * cu : 5 * tiles > 9 * cu;
      return tall ? tiles > 4 * cu : both && p.M > 32 ? 5 * tiles > 16 * cu : 2 * tiles > 5 * cu;
    case 2: return tiles > (signs ? 3 : 4) * cu;
    case 3: return 4 * wide > 3 * cu && (signs || groups <= cu || 2 * groups > 3 * cu);
    default: return wide > cu && (groups <= cu || 2 * groups > 3 * cu) && (signs || groups <= 2 * cu || 4 * groups > 9 * cu);
  }
}

bnn_status launch_conv_word(GemmParams &p, int emode, hipStream_t s) {
  switch (p.g.kH * 10 + p.g.Cw) {
    case 11: return launch_word<1, 1, 1>(p, emode, s);
    case 12: return launch_word<1, 1, 2>(p, emode, s);
    case 13: return launch_word<1, 1, 3>(p, emode, s);
    case 14: return launch_word<1, 1, 4>(p, emode, s);
    case 31: return launch_word<3, 3, 1>(p, emode, s);
    case 32: return launch_word<3, 3, 2>(p, emode, s);
    case 33: return launch_word<3, 3, 3>(p, emode, s);
    case 34: return launch_word<3, 3, 4>(p, emode, s);
    default: return BNN_ERR_UNSUPPORTED;
  }
}

}  // namespace bnn
