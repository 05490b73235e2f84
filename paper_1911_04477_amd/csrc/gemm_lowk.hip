// Xnor-Bitcount GEMM (section 3.2) for short reduction axes on the matrix cores: explicit rows of at most four 64-bit
// words (K <= 256), int32 / fp32 output.
//
// One chunk of 256 bits is the whole reduction, so there is nothing to stage or to pipeline: a wave reads the rows of its
// columns once, expands them once (the operands of all four steps stay in registers), and takes a block of rows, one load of
// 16 bytes per row, four expansions, the products, and the store of the block; or several blocks, where there would be more
// workgroups than a launch may have.  No LDS but for the affine constants, no barrier, and 150 bytes of arguments (the host
// copies them for every launch).
// Without the loop over blocks the kernel takes 42 registers instead of 168, and small calls 0.4 us less (64 x 64 x 256 2.7 ->
// 2.3); but its stores then come from eight waves a SIMD instead of three, and beyond the caches that costs more (4096 x 30001 x
// 250 94 -> 162 us, 4096 x 30000 x 250 86 -> 113; with LDS held back so that three fit, 95 and 110).
// Bound by the launch for small calls and by the store of the result for large ones.
#include <algorithm>

#include "common.h"
#include "fp4_tile.h"

namespace bnn {

struct ShortParams {
  const char *A, *B;
  int64_t lda, ldb;  // bytes
  int M, N, Kbits, Kformula, words;
  int rounds;        // blocks of rows that a wave walks over
  int abreast;       // the four waves of a workgroup stand side by side, not one above the other
  int runs;          // an XCD gets a contiguous run of workgroups
  int axis;
  int32_t *C;
  float *Y;
  int64_t ldc, ldy, img_stride;
  const float *scale, *bias;
  uint32_t OHW;
  FastDiv divOHW, divTilesN;
};

template <int WTM, int WTN, int MS, bool V16>
__global__ __launch_bounds__(256, 3) void xnor_gemm_lowk_kernel(ShortParams p) {
  constexpr int BM = 32 * WTM, BN = 32 * WTN;  // rows and columns of a wave's block
  __shared__ __attribute__((aligned(16))) float sSc[4][BM], sBi[4][BM];
  const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  uint32_t bid = blockIdx.x;
  if (p.runs) {
    const uint32_t per = gridDim.x >> 3, r = gridDim.x & 7u, xcd = bid & 7u, i = bid >> 3;
    bid = xcd * per + min(xcd, r) + i;
  }
  const uint32_t mi = fdiv_sel(bid, p.divTilesN);
  const uint32_t ni = bid - mi * p.divTilesN.d;
  const int n0 = (int)(p.abreast ? 4 * ni + wave : ni) * BN;
  const int mstep = p.abreast ? BM : 4 * BM;
  int m0 = (int)mi * p.rounds * mstep + (p.abreast ? 0 : wave * BM);
  if (m0 >= p.M || n0 >= p.N) return;  // wave-uniform; the kernel has no barrier

  // this half's two words of a row; past the row's end whatever is there, masked
  const int w0 = V16 ? min(2 * half, p.words - 2) : min(2 * half, p.words - 1), w1 = min(2 * half + 1, p.words - 1);
  auto load = [&](const char *row) {
    u32x4 v;
    if constexpr (V16) {
      v = *reinterpret_cast<const u32x4 *>(row + w0 * 8);
    } else {
      v.lo = *reinterpret_cast<const u32x2 *>(row + w0 * 8);
      v.hi = *reinterpret_cast<const u32x2 *>(row + w1 * 8);
    }
    return v;
  };
  u32x4 mask;  // bits past K become 0 in both operands: +1 * +1, subtracted by the starting value
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const int left = p.Kbits - 32 * (4 * half + d);
    mask[d] = left >= 32 ? ~0u : (left <= 0 ? 0u : (1u << left) - 1u);
  }
  u32x4 a[WTM], b[WTN];
#pragma unroll
  for (int j = 0; j < WTN; ++j) {
    const int n = min(n0 + (MS == MS_ONE ? 32 * j + l32 : WTN * l32 + j), p.N - 1);
    b[j] = load(p.B + (size_t)n * (size_t)p.ldb);
  }
  auto load_rows = [&](int m) {
#pragma unroll
    for (int i = 0; i < WTM; ++i) a[i] = load(p.A + (size_t)min(m + 32 * i + l32, p.M - 1) * (size_t)p.lda);
  };
  load_rows(m0);
  const bool affine = p.Y && p.axis == BNN_CH_ROW;  // uniform
  v8i eb[4][WTN];
#pragma unroll
  for (int j = 0; j < WTN; ++j) b[j] &= mask;
#pragma unroll
  for (int d = 0; d < 4; ++d)
#pragma unroll
    for (int j = 0; j < WTN; ++j) eb[d][j] = expand_e2m1<true>(b[j][d]);
  const float start = -(float)(256 - p.Kformula);
  for (int r = 0;;) {
    if (affine && lane < BM) {  // the wave's own rows: LDS keeps a wave's order
      sSc[wave][lane] = p.scale[min(m0 + lane, p.M - 1)];
      sBi[wave][lane] = p.bias[min(m0 + lane, p.M - 1)];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // the compiler keeps the order, too
    Fp4Acc<WTM, WTN> acc;
    acc.init(start);
    u32x4 x[WTM];
#pragma unroll
    for (int i = 0; i < WTM; ++i) x[i] = a[i] & mask;
    const int next = m0 + mstep;
    const bool more = ++r < p.rounds && next < p.M;  // wave-uniform
    if (more) load_rows(next);
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      v8i ea[WTM];
#pragma unroll
      for (int i = 0; i < WTM; ++i) ea[i] = expand_e2m1<true>(x[i][d]);
#pragma unroll
      for (int i = 0; i < WTM; ++i)
#pragma unroll
        for (int j = 0; j < WTN; ++j) acc.v[i][j] = mfma_e2m1(ea[i], eb[d][j], acc.v[i][j]);
    }
    store_maps<WTM, WTN, MS>(p, acc, m0, n0, lane, sSc[wave], sBi[wave]);
    if (!more) break;
    m0 = next;
  }
}

// Whether the short-row kernel can run the problem described by p (explicit B).
bool lowk_applicable(const GemmParams &p) { return p.Kw64 <= 4; }

// What a launch looks like: F_64 blocks of 64 x 64 instead of 32 x 32; F_ABREAST a workgroup's waves side by side instead of
// one above the other; F_RUNS contiguous runs of workgroups on an XCD.  -1: another kernel is at least as fast.
// Measured over 27 sizes in every form, rows of one and four words, and 300 random sizes against the vector-ALU
// kernel that took rows of two and four words before (16-byte stores, 32 rows per wave) and the other matrix-core
// kernels (us; "before"):
//   rows that start at whole or half lines: side by side, a workgroup writes 512 or 1024 bytes of a row together.  64 x 64
//     blocks up to 150 MB (256 x 50176 x 250 14.4 -> 11.7, 4096 x 8192 x 250 30.7 -> 24.3, 600 x 30000 x 250 20.5 -> 15.8),
//     32 x 32 from there on for whole lines, and beyond the last-level cache for both (256 x 200704 x 250 46.6 -> 36.7;
//     4096 x 30000 x 250 107 -> 88; 800 x 120016 x 250 84 -> 66; but 2801 x 18768, 210 MB, half lines 40.8 against 36.8);
//     with 49 to 64 rows from 80 MB on (64 x 400000 x 250 25.0 -> 20.0, 64 x 64 blocks 21.3), with fewer never (17 x 3148928 x
//     128 70 against 45, 41 x 2200448 x 64 94, 70);
//   rows that start elsewhere: side by side and in runs, neighbours share lines (130 x 60004 x 240 15.2 -> 11.0, 700 x 30004 x
//     240 30.4 -> 18.2, 3000 x 8004 x 240 31.2 -> 18.9, 2856 x 25828 x 240 94 -> 54; without runs 11.6, 19.1, 21.3, 57);
//     staged tiles where the second row of blocks would be half empty (83 x 31124 x 98 5.9 against 6.8) and for rows of one
//     and three words, which had them before (642 x 39884 x 170 20.9 against 22.3; others equal);
//     staged tiles also for 17 to 32 rows, half a block (32 x 948728 x 128 37.7 against 43.4, 30 x 5801148 x 78 225, 270) from 32 MB on (21 x 472760 x 66
//     12.6, 13.8; but 19 x 325160 x 200 11.4 against 9.6);
//   columns that are no multiple of 4: the staged tiles and the split kernel are equal or faster (256 x 50177 x 50 13.5
//     against 14.2), except beyond the cache, where rows share lines and it counts which workgroups of an XCD run together
//     (70 sizes of 256 to 700 MB): from 257 to 2100 rows 32 x 32 side by side in runs from 275 MB on (987 x 140757 x 64 107, staged
//     140, one above the other 170; 1689 x 52870 x 256 76, 92, 84; but 541 x 119587 x 64, 258 MB, 52 against 44 staged); more rows one
//     above the other in runs (4096 x 30001 x 250 95, staged 161), staged below 300 MB, or 330 MB with few columns (15380 x 4763 x
//     100 55 against 71; 200000 x 401 x 128 73 against 109); fewer rows staged (36 x 3408733 x 53 152 against 237 one above the
//     other, 165 x 852363 x 256 157, 199; 256 x 332765 x 100
//     87, 119; but 260 x 347289 x 200 93, 74);
//   small calls: 32 x 32 blocks up to two of 64 x 64 per unit (64 x 64 x 256 4.6 -> 3.0, 256 x 1000 x 200 5.3 -> 3.3); rows of
//     one and three words have the split kernel up to 300 of them, equal within 5 % either way.
enum : int { F_64 = 1, F_ABREAST = 2, F_RUNS = 4 };
static int lowk_rule(const GemmParams &p) {
  const int64_t t64 = (((int64_t)p.M + 63) / 64) * (((int64_t)p.N + 63) / 64), cu = p.n_cu;
  const int64_t out = (int64_t)p.M * p.N * 4 * ((p.C ? 1 : 0) + (p.Y ? 1 : 0));
  const bool beyond = out > 256000000, odd_words = p.Kw64 % 2 != 0;
  if (!map_columns_by_four(p)) {
    if (p.M <= 256 || out < 275000000) return -1;
    if (p.M <= 2100) return F_RUNS | F_ABREAST;
    return p.N >= 2000 && out >= (p.N >= 14000 ? 300000000 : 330000000) ? F_RUNS : -1;
  }
  if (odd_words && t64 < 300) return -1;
  if (t64 <= 2 * cu) return p.N >= p.M ? F_ABREAST : 0;
  if (!map_rows_start_every(p, 16))
    return odd_words || (p.M > 64 && p.M <= 96) || (p.M > 16 && p.M <= 32 && out >= 32000000) ? -1 : F_RUNS | F_ABREAST | F_64;
  if (p.M <= 48) return F_ABREAST | F_64;
  if (beyond) return F_ABREAST;
  return map_rows_start_every(p, 32) && out >= (p.M > 64 ? 150000000 : 80000000) ? F_ABREAST : F_ABREAST | F_64;
}

bool lowk_faster(const GemmParams &p) { return lowk_rule(p) >= 0; }

template <int WTM, int WTN, bool V16>
static void launch_forms(const ShortParams &q, const GemmParams &p, dim3 grid, hipStream_t s) {
  const dim3 block(256);
  if (!p.colperm && WTN > 1) hipLaunchKernelGGL((xnor_gemm_lowk_kernel<WTM, WTN, MS_ONE, V16>), grid, block, 0, s, q);
  else if (p.nt_store) hipLaunchKernelGGL((xnor_gemm_lowk_kernel<WTM, WTN, MS_NT, V16>), grid, block, 0, s, q);
  else hipLaunchKernelGGL((xnor_gemm_lowk_kernel<WTM, WTN, MS_VEC, V16>), grid, block, 0, s, q);
}

// form: as of lowk_rule; -1: the rule's.  rounds: blocks of rows per wave at least.
bnn_status launch_lowk(GemmParams &p, int form, hipStream_t s, int rounds) {
  p.colperm = map_columns_by_four(p) ? 1 : 0;
  p.nt_store = nontemporal_maps(p, 0) ? 1 : 0;
  if (form < 0) form = std::max(lowk_rule(p), 0);
  ShortParams q;
  q.A = reinterpret_cast<const char *>(p.A);
  q.B = reinterpret_cast<const char *>(p.B);
  q.lda = p.lda32 * 4;
  q.ldb = p.ldb * 8;
  q.M = p.M; q.N = p.N; q.Kbits = p.Kbits; q.Kformula = p.Kformula; q.words = p.Kw64;
  q.axis = p.axis;
  q.C = p.C; q.Y = p.Y; q.ldc = p.ldc; q.ldy = p.ldy; q.img_stride = p.img_stride;
  q.scale = p.scale; q.bias = p.bias;
  q.OHW = p.OHW; q.divOHW = p.divOHW;
  // a launch is limited to 2^32 threads: the widest workgroups for more columns than that, several rounds for more rows
  constexpr int64_t MAX_BLOCKS = 0xffffff;
  int64_t tilesM, tilesN;
  auto tiles = [&]() {
    const int b32 = form & F_64 ? 64 : 32, bn = form & F_ABREAST ? 4 * b32 : b32, bm = form & F_ABREAST ? b32 : 4 * b32;
    tilesN = ((int64_t)p.N + bn - 1) / bn;
    tilesM = ((int64_t)p.M + bm - 1) / bm;
    return tilesM * tilesN;
  };
  if (tiles() > MAX_BLOCKS) {
    form |= F_64 | F_ABREAST;
    tiles();
  }
  const int64_t rows = MAX_BLOCKS / tilesN;  // of workgroups; N is below 2^31: at least one
  q.rounds = (int)std::max<int64_t>(rounds, (tilesM + rows - 1) / rows);
  tilesM = (tilesM + q.rounds - 1) / q.rounds;
  q.abreast = form & F_ABREAST ? 1 : 0;
  q.runs = form & F_RUNS ? 1 : 0;
  q.divTilesN = FastDiv((uint32_t)tilesN);
  const bool v16 = p.Kw64 % 2 == 0 && p.lda32 % 4 == 0 && p.ldb % 2 == 0;
  const dim3 grid((unsigned)(tilesM * tilesN));
  ProfScope ps(KID_XNOR_GEMM_LOWK, s);
  if (!(form & F_64)) v16 ? launch_forms<1, 1, true>(q, p, grid, s) : launch_forms<1, 1, false>(q, p, grid, s);
  else v16 ? launch_forms<2, 2, true>(q, p, grid, s) : launch_forms<2, 2, false>(q, p, grid, s);
  return launch_status();
}

}  // namespace bnn
