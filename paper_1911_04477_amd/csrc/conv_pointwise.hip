// Pointwise (1x1, no padding) binarized convolution from an fp32 image in one launch: a workgroup encodes 64 output
// pixels (sampled by the strides) into LDS and multiplies all output channels with them there.
//
// Bound by memory: 4 bytes read per input value used (whole 128-byte lines where a stride skips columns), 4 or 8
// written per output; the multiplication is a few thousand clocks a workgroup.  Encoding in a launch of its own reads
// while nothing is written, and the multiplication after it writes while nothing is read; here some workgroups of a
// unit read while others write, the packed image is not read back, and there is one launch instead of two.
#include <algorithm>

#include "common.h"
#include "fp4_tile.h"

namespace bnn {

struct PointwiseParams {
  GemmParams p;  // A, M, N, Kw64, lda32, Kformula, outputs; p.g: the image's geometry (act unused)
  const float *x;
  uint64_t *img; // the sampled pixels' words leave there too: bnn_conv2d's workspace receives the packed image
  int rs;        // dwords between two pixels' rows in LDS
  int chunks;    // of 256 bits of a row
  int ytiles;    // workgroups that share a pixel tile's output channels
};

// NC: groups of 64 pixels per workgroup; its waves take NC of them times 4 / NC groups of rows.
template <int WTM, int NC, int MS>
__global__ __launch_bounds__(256, 3) void conv_pointwise_kernel(PointwiseParams q) {
  extern __shared__ __attribute__((aligned(16))) uint32_t sB[];  // [64 * NC pixels][rs]
  __shared__ __attribute__((aligned(16))) float sSc[4 / NC * 32 * WTM], sBi[4 / NC * 32 * WTM];
  const GemmParams &p = q.p;
  const ConvGeom &g = p.g;
  const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  // neighbouring pixel tiles on one XCD: they share lines of the image and of the maps
  uint32_t bid = blockIdx.x;
  {
    const uint32_t per = gridDim.x >> 3, r = gridDim.x & 7u, xcd = bid & 7u, i = bid >> 3;
    bid = xcd * per + min(xcd, r) + i;
  }
  const int n0 = (int)bid * 64 * NC;

  // ---- encode: lane = pixel, the waves of a pixel group share its granules of 32 channels (see encode_nchw_kernel) ----
  {
    const int group = wave % NC;
    const uint32_t pix = (uint32_t)min(n0 + 64 * group + lane, p.N - 1);
    const uint32_t t = fdiv(pix, g.divOW), n = fdiv(t, g.divOH);
    const uint32_t ow = pix - t * (uint32_t)g.OW, oh = t - n * (uint32_t)g.OH;
    const size_t plane = (size_t)g.H * g.W;
    const float *xp = q.x + (size_t)n * g.C * plane + (size_t)(oh * g.sH) * g.W + (size_t)ow * g.sW;
    uint32_t *const row = sB + (64 * group + lane) * q.rs;
    const int G = 8 * q.chunks;  // granules of the row, the last ones partial or empty
    for (int gr = wave / NC; gr < G; gr += 4 / NC) {
      const int c0 = gr * 32, left = g.C - c0;
      uint32_t acc = 0u;
      // channels past C re-read the last one and are masked out
      if (left > 8) {
        float v[32];
#pragma unroll
        for (int j = 0; j < 32; ++j) v[j] = __builtin_nontemporal_load(xp + (size_t)(c0 + min(j, left - 1)) * plane);
#pragma unroll
        for (int j = 0; j < 32; ++j) acc |= (uint32_t)sign_bit(v[j]) << j;
      } else if (left > 0) {
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = __builtin_nontemporal_load(xp + (size_t)(c0 + min(j, left - 1)) * plane);
#pragma unroll
        for (int j = 0; j < 8; ++j) acc |= (uint32_t)sign_bit(v[j]) << j;
      }
      if (left < 32) acc &= left > 0 ? (1u << left) - 1u : 0u;
      row[gr] = acc;
    }
  }

  __syncthreads();  // the pixels' bits are there
  if (blockIdx.y == 0) {
    // The packed image, whole lines.  64 x 200 x 56 x 56 by stride 2: 33.5 us without it, 33.75 with; 240 random layers 0.7 % on
    // average, to 6 % (behind the multiplication 1.0 and 1.8 %, half words straight from the encoding lanes 2.5 %).
    const uint32_t Cw = (uint32_t)g.Cw, words = (uint32_t)min(64 * NC, p.N - n0) * Cw;
    uint64_t *const out = q.img + (size_t)n0 * Cw;
    for (uint32_t j = threadIdx.x; j < words; j += 256u) {
      const uint32_t pix = fdiv_sel(j, g.divCw), cw = j - pix * Cw;
      out[j] = *reinterpret_cast<const uint64_t *>(sB + pix * (uint32_t)q.rs + 2u * cw);
    }
  }

  // ---- multiply: a wave 32 * WTM channels x 64 pixels at a time ------------------------------------------
  constexpr int BM = 4 / NC * 32 * WTM;
  const int wr = wave / NC, nw = n0 + 64 * (wave % NC);
  const bool a16 = p.b_vec16 != 0;  // uniform: rows of A may be read with 16-byte loads
  const bool affine = p.Y != nullptr;
  for (int m_tile = (int)blockIdx.y * BM; m_tile < p.M; m_tile += q.ytiles * BM) {
    if (affine && threadIdx.x < BM) {
      const int m = min(m_tile + (int)threadIdx.x, p.M - 1);
      sSc[threadIdx.x] = p.scale[m];
      sBi[threadIdx.x] = p.bias[m];
    }
    const int m0 = m_tile + 32 * WTM * wr;
    Fp4Acc<WTM, 2> acc;
    acc.init(-(float)(q.chunks * 256 - p.Kformula));
    if (m0 < p.M) {  // wave-uniform
      const char *arow[WTM];
#pragma unroll
      for (int i = 0; i < WTM; ++i)
        arow[i] = reinterpret_cast<const char *>(p.A) + (size_t)min(m0 + 32 * i + l32, p.M - 1) * (size_t)p.lda32 * 4u;
      const uint32_t *brow[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) brow[j] = sB + (nw - n0 + (MS == MS_ONE ? 32 * j + l32 : 2 * l32 + j)) * q.rs + 4 * half;
      for (int c = 0; c < q.chunks; ++c) {
        const int w = 4 * c + 2 * half;  // this half's two words
        u32x4 a[WTM], b[2];
        if (a16) {
#pragma unroll
          for (int i = 0; i < WTM; ++i) a[i] = *reinterpret_cast<const u32x4 *>(arow[i] + (size_t)min(w, p.Kw64 - 2) * 8u);
        } else {
#pragma unroll
          for (int i = 0; i < WTM; ++i) {
            a[i].lo = *reinterpret_cast<const u32x2 *>(arow[i] + (size_t)min(w, p.Kw64 - 1) * 8u);
            a[i].hi = *reinterpret_cast<const u32x2 *>(arow[i] + (size_t)min(w + 1, p.Kw64 - 1) * 8u);
          }
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) b[j] = *reinterpret_cast<const u32x4 *>(brow[j] + 8 * c);
        // words past the row's end are 0 in both operands
        const uint32_t k0 = w < p.Kw64 ? ~0u : 0u, k1 = w + 1 < p.Kw64 ? ~0u : 0u;
#pragma unroll
        for (int i = 0; i < WTM; ++i) a[i] &= u32x4{k0, k0, k1, k1};
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          v8i ea[WTM], eb[2];
#pragma unroll
          for (int j = 0; j < 2; ++j) eb[j] = expand_e2m1<true>(b[j][d]);
#pragma unroll
          for (int i = 0; i < WTM; ++i) ea[i] = expand_e2m1<true>(a[i][d]);
#pragma unroll
          for (int i = 0; i < WTM; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc.v[i][j] = mfma_e2m1(ea[i], eb[j], acc.v[i][j]);
        }
      }
    }
    __syncthreads();  // the constants are there
    store_maps<WTM, 2, MS>(p, acc, m0, nw, lane, sSc + 32 * WTM * wr, sBi + 32 * WTM * wr);
    if (m_tile + q.ytiles * BM < p.M) __syncthreads();  // the constants have been read
  }
}

template <int WTM, int NC>
static void launch_pointwise(const PointwiseParams &q, dim3 grid, size_t lds, hipStream_t s) {
  if (!q.p.colperm) hipLaunchKernelGGL((conv_pointwise_kernel<WTM, NC, MS_ONE>), grid, dim3(256), lds, s, q);
  else if (q.p.nt_store) hipLaunchKernelGGL((conv_pointwise_kernel<WTM, NC, MS_NT>), grid, dim3(256), lds, s, q);
  else hipLaunchKernelGGL((conv_pointwise_kernel<WTM, NC, MS_VEC>), grid, dim3(256), lds, s, q);
}

bool encode_nchw_supported(int N, int C, int H, int W, int OHp, int OWp);

static int64_t pixel_tiles(const GemmParams &p, int nc) { return ((int64_t)p.N + 64 * nc - 1) / (64 * nc); }

// Where one launch is the faster form (96 shapes of 10 MB and less to 380 MB, graph replays): by 1.04 to 1.3 times in
// general (64 x 200 x 56 x 56, stride 2, to 256 channels fp32 36.5 -> 33.2 us; 64 x 256 x 56 x 56 to 64 50.2 -> 44.3; 128 x
// 256 x 28 x 28, stride 2, to 512 40.0 -> 32.4), 1.2 to 2 where a launch counts or waves idle in the encode (one 256 x 56 x 56
// image 8.4 -> 4.6, 256 x 3 x 32 x 32 20.1 -> 9.3).  Two launches
//   * for 33 to 64 channels into twice as many and more from 150 MB on: little is read, and the stores of whole rows of
//     tiles go out better (64 to 256, 261 MB: 51.1 against 49.4; to 128, 260 MB: 48.8, 47.5; 100 MB 18.9, 21.6);
//   * for many channels of few pixels, where the GEMM splits the reduction (2 x 1536 x 14 x 14 to 256: 15.7 against 13.8;
//     1 x 2048 x 7 x 7 19.2, 16.5; 4 x 1024 x 14 x 14 to 512 12.7, 13.1).
bool pointwise_applicable(const GemmParams &p) {
  const ConvGeom &g = p.g;
  if (!encode_nchw_supported(g.Nimg, g.C, g.H, g.W, g.OH, g.OW)) return false;  // what the encode refuses stays refused
  if (g.C > 2048 || (g.C >= 1024 && pixel_tiles(p, 1) * 128 < g.C)) return false;
  const int64_t bytes = 4 * (int64_t)p.N * (g.C + (int64_t)p.M * ((p.C ? 1 : 0) + (p.Y ? 1 : 0)));
  return !(g.C > 32 && g.C <= 64 && p.M >= 2 * g.C && bytes >= 150000000);
}

// p: the GEMM of the sampled pixels (as for run_gemm, maps only); p.g: the image as it is, OH x OW sampled by sH, sW;
// img: receives their words.
bnn_status launch_conv_pointwise(GemmParams &p, const float *x, uint64_t *img, hipStream_t s) {
  PointwiseParams q;
  p.colperm = map_columns_by_four(p) ? 1 : 0;
  p.nt_store = nontemporal_maps(p, 1) ? 1 : 0;
  p.b_vec16 = p.Kw64 % 2 == 0 && p.lda32 % 4 == 0;
  q.p = p;
  q.x = x;
  q.img = img;
  q.chunks = (p.Kw64 + 3) / 4;
  q.rs = 8 * q.chunks + 4;  // rows of 16-byte pieces, on distinct banks
  const int64_t cu = device_cu_count();
  // up to 64 channels one pixel group leaves waves without a granule: two, while every unit gets two workgroups (200 x 8 x
  // 30 x 30 9.9 -> 7.9 us, 256 x 3 x 32 x 32 13.6 -> 9.3)
  const int nc = p.g.C <= 64 && pixel_tiles(p, 2) >= 2 * cu ? 2 : 1;
  const int64_t tiles = pixel_tiles(p, nc);
  const bool wide = p.M > 128 / nc && tiles >= cu;
  const int64_t bm = (wide ? 256 : 128) / nc;
  // few pixel tiles: several workgroups encode the same one and share its output channels
  q.ytiles = (int)std::max<int64_t>(1, std::min<int64_t>((p.M + bm - 1) / bm, cu / tiles));
  const size_t lds = (size_t)64 * nc * q.rs * 4;
  const dim3 grid((unsigned)tiles, (unsigned)q.ytiles);
  ProfScope ps(KID_CONV_POINTWISE, s);
  if (nc == 2) wide ? launch_pointwise<2, 2>(q, grid, lds, s) : launch_pointwise<1, 2>(q, grid, lds, s);
  else wide ? launch_pointwise<2, 1>(q, grid, lds, s) : launch_pointwise<1, 1>(q, grid, lds, s);
  return launch_status();
}

}  // namespace bnn
