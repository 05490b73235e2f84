// Xnor-Bitcount GEMM (section 3.2 of the paper) for gfx950, in the exclusive-or form
//     C[m,n] = K - 2 * sum_w popcount(A[m,w] ^ B[n,w]).
//
// This file holds the vector-ALU form of the GEMM and the rule that picks a kernel for a call (run_gemm).  No call
// without a forced configuration runs the vector-ALU form any more: of the sizes that the short-row kernels
// (gemm_lowk.hip, gemm_fewrows.hip) leave, the matrix-core kernels (gemm_fp4.hip, gemm_fp4_split.hip) were faster at all that were
// compared (1 to 4096 rows, 1 to 400000 columns, 128 to 9216 bits, layers of 8 to 512 channels), but for up to 8 rows
// of 40000 to 50000 columns and at most 512 bits, where a former one-wave form of the vector ALU took 3.4 to 3.6 us
// against 3.6 to 4.4.  It stays as the yardstick that computes the method literally and as the second implementation
// that tests compare with.
//
// CDNA4 has no 1-bit matrix instruction; on the vector ALU the contraction costs
// two lane-instructions per 32 bit-MACs per output (v_xor_b32, then v_bcnt_u32_b32
// which adds its popcount into the accumulator).  The kernel is built so that the
// inner loop is almost nothing else:
//   * lanes of a wave run along N (64 consecutive columns per register column);
//     every lane keeps 8 x TN int32 accumulators;
//   * the 8 rows of A a wave works on are the same for all of its lanes, so A is
//     fetched with SCALAR loads into SGPRs and enters v_xor as the scalar operand:
//     no LDS traffic, no VGPRs and no VALU instructions are spent on A;
//   * the block's B tile (BN columns x 8 dwords) is staged once per K-chunk through
//     double-buffered LDS, row-per-column with a 4-dword pad so that both the 16-byte
//     staging writes and the 16-byte per-lane reads are bank-conflict free; the next
//     chunk's global loads are issued before the current chunk is computed and first
//     touched after it;
//   * B is either an explicit K-contiguous matrix or (implicit GEMM) gathered on the
//     fly from a packed NHWC image: column = output pixel, row word = tap word, pad
//     taps replaced by the "+1" word -- no patch matrix is ever written.  The gather has
//     a general form (BMODE 1) and a lean one (BMODE 2) that keeps every division and all
//     geometry out of the chunk loop: a per-slot tap-validity mask and 32-bit base offset,
//     and a per-workgroup LDS table of tap offsets;
//   * K tails: two leftover words run a half chunk; one or three re-read the final 8
//     dwords of the rows (a window that overlaps the previous chunk) with the overlap and
//     the bits past K zeroed in both operands (A in SGPRs with scalar moves, B in the
//     staging), so they run the same instruction sequence as a full chunk; rows shorter
//     than four words go one dword at a time;
//   * everything a chunk needs besides the math is kept off the vector ALU and out of
//     long-lived SGPRs (row offsets are recomputed by scalar adds per chunk), because the
//     kernel is VALU-bound and SGPR spills are VALU instructions (v_readlane);
//   * the store does K - 2*acc and then either writes int32 / fma(scale, acc, bias) fp32
//     (row-major or scattered to NCHW; 256 contiguous bytes per wave store, or, on the
//     256-column tiles when N and the strides are multiples of 4, 1 KB: the tile's columns are
//     then dealt to the LDS rows so that a lane's four columns are consecutive), or -- the
//     binarizing epilogue -- takes the 2x2 max (optional), applies the fma, keeps only the
//     sign and writes packed NHWC words for the next layer (32x fewer output bytes).
// Workgroup ids are remapped so that tiles sharing a B tile run on the same XCD
// (one L2 per XCD; hardware deals consecutive ids round-robin over the 8 XCDs).
#include "common.h"
#include "bnn_testing.h"
#include "gemm_rows.inc"

namespace bnn {

using u32x4 = uint32_t __attribute__((ext_vector_type(4)));
using u32x8 = uint32_t __attribute__((ext_vector_type(8)));
// A is only ever read by the kernel.  Reading it through the constant address space lets
// the compiler use scalar (SMEM) loads for wave-uniform addresses.
#define BNN_CONST_AS __attribute__((address_space(4)))
typedef const uint32_t BNN_CONST_AS *cu32_ptr;

// acc += popcount(x) as ONE instruction.  Written as asm because the optimizer otherwise
// re-associates a chain of popcount-adds into v_bcnt(x, 0) plus separate three-operand adds.
__device__ __forceinline__ int popc_acc(uint32_t x, int acc) {
  asm("v_bcnt_u32_b32 %0, %1, %0" : "+v"(acc) : "v"(x));
  return acc;
}

// The K axis is consumed in chunks of KC = 8 dwords (256 bits); a wave owns TM = 8 rows.
constexpr int KC = 8;
constexpr int TM = 8;
// lean implicit gather: chunks per row the per-workgroup tap table holds, and its flag bits
constexpr int LEAN_MAX_STAGES = 512;
constexpr uint32_t LEAN_LIVE = 1u, LEAN_TAP_END = 2u;

template <int TN, int WM, int WN>
struct GemmCfg {
  static constexpr int BM = TM * WM;
  static constexpr int BN = 64 * TN * WN;
  static constexpr int THREADS = 64 * WM * WN;
  static constexpr int RS = KC + 4;                      // LDS row stride in dwords
  static constexpr int TILE = BN * RS;                   // dwords per LDS buffer
  static constexpr int PIECES = BN * (KC / 4);           // 16-byte pieces per chunk
  static constexpr int PPT = (PIECES + THREADS - 1) / THREADS;
  static_assert(PIECES % THREADS == 0 || PIECES < THREADS, "staging must divide evenly");
};

// words of a tap that lies outside the image: every real channel is +1 (bit 1)
__device__ __forceinline__ uint64_t pad_word64(int C, int cw) {
  const int left = C - cw * 64;
  return left >= 64 ? ~0ull : (left <= 0 ? 0ull : ((1ull << left) - 1ull));
}

// Column n of an implicit GEMM -> output pixel.  Without pooling the columns are the
// output pixels in NHWC order.  With 2x2 pooling a tile of 256 columns holds 64 pooling
// windows: column 256*t + 64*j + l is member j (row-major in the 2x2 window) of window
// 64*t + l, so that the four members of a window are the four register columns of one lane.
__device__ __forceinline__ void decode_col(const ConvGeom &g, uint32_t n, uint32_t &img, int &oh, int &ow) {
  if (g.pool == 0) {
    const uint32_t t = fdiv(n, g.divOW);
    ow = (int)(n - t * g.OW);
    img = fdiv(t, g.divOH);
    oh = (int)(t - img * g.OH);
  } else {
    const uint32_t j = (n >> 6) & 3u;
    const uint32_t wdx = (n >> 8) * 64u + (n & 63u);
    const uint32_t PW = g.OW >> 1, PH = g.OH >> 1;
    const uint32_t t = fdiv(wdx, g.divOW);
    const uint32_t wx = wdx - t * PW;
    img = fdiv(t, g.divOH);
    const uint32_t wy = t - img * PH;
    oh = (int)(2 * wy + (j >> 1));
    ow = (int)(2 * wx + (j & 1));
  }
}

// Store of an 8 x TN accumulator tile: K - 2*acc as int32 and / or fma(scale, acc, bias) as
// fp32, row-major or scattered to NCHW.  The store-only parameters are read from the
// kernel-argument segment through a pointer the optimizer cannot see through, so that they
// occupy no SGPRs (or spill slots) during the main loop.
template <int TN>
__device__ __forceinline__ void store_tile(const int (&acc)[TM][TN], int m0, int nbase) {
  const GemmParams BNN_CONST_AS *kp = (const GemmParams BNN_CONST_AS *)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(kp));
  const int M = kp->M, N = kp->N, Kformula = kp->Kformula;
  const float *const scale = kp->scale, *const bias = kp->bias;
  const int axis = kp->axis;
  int32_t *const Cp = kp->C;
  float *const Yp = kp->Y;
  const int64_t ldc = kp->ldc, ldy = kp->ldy, img_stride = kp->img_stride;
  const uint32_t OHW = kp->OHW;
  // Non-temporal stores when every 256-byte piece a wave stores covers whole 128-byte lines (measured
  // 1 % faster then); ordinary stores otherwise, so that pieces that share a line meet in the L2
  // instead of each going to memory as a partial line (49.6 -> 40.7 us on a 31 x 33 map).
  const bool nt = kp->nt_store != 0;
  FastDiv divOHW;
  divOHW.d = kp->divOHW.d; divOHW.mul = kp->divOHW.mul; divOHW.shift = kp->divOHW.shift;
  // per-row affine constants once per tile (wave-uniform: scalar loads; rows past M re-read row M - 1)
  typedef const float BNN_CONST_AS *cf32_ptr;
  const cf32_ptr cscale = (cf32_ptr)(uintptr_t)scale, cbias = (cf32_ptr)(uintptr_t)bias;
  float scr[TM], bir[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    scr[i] = 1.0f;
    bir[i] = 0.0f;
  }
  if (Yp && axis == BNN_CH_ROW) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int mi = min(m0 + i, M - 1);
      scr[i] = cscale[mi];
      bir[i] = cbias[mi];
    }
  }
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int n = nbase + j * 64;
    if (n >= N) continue;
    const uint32_t img = fdiv((uint32_t)n, divOHW);
    const uint32_t pix = (uint32_t)n - img * OHW;
    const int64_t coff = (int64_t)img * img_stride + pix + (int64_t)m0 * ldc;
    const int64_t yoff = (int64_t)img * img_stride + pix + (int64_t)m0 * ldy;
    int32_t *cp = Cp ? Cp + coff : nullptr;
    float *yp = Yp ? Yp + yoff : nullptr;
    float sc = 1.0f, bi = 0.0f;
    if (Yp && axis == BNN_CH_COL) {
      sc = scale[n];
      bi = bias[n];
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      if (m0 + i < M) {
        const int v = Kformula - 2 * acc[i][j];
        if (cp) {
          if (nt) __builtin_nontemporal_store(v, cp);
          else *cp = v;
        }
        if (yp) {
          const float s1 = axis == BNN_CH_ROW ? scr[i] : sc, b1 = axis == BNN_CH_ROW ? bir[i] : bi;
          const float y = fmaf(s1, (float)v, b1);
          if (nt) __builtin_nontemporal_store(y, yp);
          else *yp = y;
        }
      }
      if (cp) cp += ldc;
      if (yp) yp += ldy;
    }
  }
}

// The same store for a column-permuted tile (GemmParams::colperm): the lane's four accumulators of a
// row are four consecutive columns, first column nfirst (a multiple of 4), stored with one 16-byte
// store per row.  The host sets colperm only where N, the leading dimensions and the columns per
// image are multiples of 4, so the four columns are all inside or all outside the matrix, lie in one
// image and start on a 16-byte boundary.
__device__ __forceinline__ void store_tile_x4(const int (&acc)[TM][4], int m0, int nfirst) {
  using i32x4 = int __attribute__((ext_vector_type(4)));
  using f32x4 = float __attribute__((ext_vector_type(4)));
  const GemmParams BNN_CONST_AS *kp = (const GemmParams BNN_CONST_AS *)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(kp));
  const int M = kp->M, N = kp->N, Kformula = kp->Kformula;
  if (nfirst >= N) return;
  const float *const scale = kp->scale, *const bias = kp->bias;
  const int axis = kp->axis;
  int32_t *const Cp = kp->C;
  float *const Yp = kp->Y;
  const int64_t ldc = kp->ldc, ldy = kp->ldy, img_stride = kp->img_stride;
  const uint32_t OHW = kp->OHW;
  const bool nt = kp->nt_store != 0;
  FastDiv divOHW;
  divOHW.d = kp->divOHW.d; divOHW.mul = kp->divOHW.mul; divOHW.shift = kp->divOHW.shift;
  typedef const float BNN_CONST_AS *cf32_ptr;
  const cf32_ptr cscale = (cf32_ptr)(uintptr_t)scale, cbias = (cf32_ptr)(uintptr_t)bias;
  float scr[TM], bir[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    scr[i] = 1.0f;
    bir[i] = 0.0f;
  }
  if (Yp && axis == BNN_CH_ROW) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int mi = min(m0 + i, M - 1);
      scr[i] = cscale[mi];
      bir[i] = cbias[mi];
    }
  }
  f32x4 csc = {1.f, 1.f, 1.f, 1.f}, cbi = {0.f, 0.f, 0.f, 0.f};
  if (Yp && axis == BNN_CH_COL) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {  // scale / bias carry no alignment requirement
      csc[j] = scale[nfirst + j];
      cbi[j] = bias[nfirst + j];
    }
  }
  const uint32_t img = fdiv((uint32_t)nfirst, divOHW);
  const uint32_t pix = (uint32_t)nfirst - img * OHW;
  int32_t *cp = Cp ? Cp + ((int64_t)img * img_stride + pix + (int64_t)m0 * ldc) : nullptr;
  float *yp = Yp ? Yp + ((int64_t)img * img_stride + pix + (int64_t)m0 * ldy) : nullptr;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    if (m0 + i < M) {
      i32x4 v;
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = Kformula - 2 * acc[i][j];
      if (cp) {
        if (nt) __builtin_nontemporal_store(v, reinterpret_cast<i32x4 *>(cp));
        else *reinterpret_cast<i32x4 *>(cp) = v;
      }
      if (yp) {
        f32x4 y;
#pragma unroll
        for (int j = 0; j < 4; ++j)
          y[j] = axis == BNN_CH_ROW ? fmaf(scr[i], (float)v[j], bir[i]) : fmaf(csc[j], (float)v[j], cbi[j]);
        if (nt) __builtin_nontemporal_store(y, reinterpret_cast<f32x4 *>(yp));
        else *reinterpret_cast<f32x4 *>(yp) = y;
      }
    }
    if (cp) cp += ldc;
    if (yp) yp += ldy;
  }
}

template <int TN, int WM, int WN, int MINW, int BMODE, int EMODE, int YIELD>
__global__ __launch_bounds__(64 * WM * WN, MINW) void xnor_gemm_kernel(GemmParams p) {
  using Cfg = GemmCfg<TN, WM, WN>;
  constexpr int RS = Cfg::RS;
  constexpr int PPT = Cfg::PPT;
  constexpr int QPR = KC / 4;  // 16-byte pieces per row
  static_assert(EMODE == 0 || ((WM == 8 || WM == 4) && WN == 1 && (TN == 4 || TN == 2)),
                "packed epilogue needs 64- or 32-row tiles");
  __shared__ __attribute__((aligned(16))) uint32_t sB[2 * Cfg::TILE];
  __shared__ uint2 sTab[BMODE == 2 ? 2 * LEAN_MAX_STAGES : 1];

  __builtin_amdgcn_s_setprio(3);  // prologue and epilogue are short and latency-bound: let them through
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % WM;
  const int wn = wave / WM;

  // XCD-aware tile order: ids that land on one XCD get consecutive tiles.
  const uint32_t nb = gridDim.x, bid = blockIdx.x;
  const uint32_t xcd = bid & 7u, loc = bid >> 3;
  const uint32_t base = nb >> 3, rem = nb & 7u;
  const uint32_t tile = xcd * base + (xcd < rem ? xcd : rem) + loc;
  const int mi = (int)(tile % (uint32_t)p.tilesM);
  const int ni = (int)(tile / (uint32_t)p.tilesM);
  const int m0 = mi * Cfg::BM + wm * TM;
  const int n0 = ni * Cfg::BN;
  // Tile column held by LDS row `row` of the B tile: the row itself, or (column-permuted tiles, see
  // GemmParams::colperm) 4 * (row % 64) + row / 64.
  const bool colperm = EMODE == 0 && TN == 4 && WN == 1 && p.colperm != 0;
  auto tile_col = [&](int row) { return colperm ? ((row & 63) << 2) + (row >> 6) : row; };

  // Byte offsets of this wave's TM rows: first row + i * row bytes, clamped to the last row of A
  // (rows past M recompute row M-1 and are not stored).  Three SGPRs; the eight offsets are
  // recomputed on the scalar unit every chunk instead of living in (spilled) registers.
  // 32-bit: the host checks that M * lda32 * 4 < 2^32.
  const uint32_t arow_bytes = (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)p.lda32 * 4u));
  const uint32_t aoff_max = (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(p.M - 1) * (uint32_t)p.lda32 * 4u));
  uint32_t aoff_first;
  {
    const int mf = m0 < p.M ? m0 : p.M - 1;
    aoff_first = (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)mf * (uint32_t)p.lda32 * 4u));
  }
  // Re-defining the first offset through an empty asm inside the loop keeps the compiler from
  // hoisting the eight derived offsets out of it.
#define BNN_AOFF(i) min(aoff_cur + (uint32_t)(i) * arow_bytes, aoff_max)
  // 64-bit base of A in an SGPR pair (readfirstlane returns a signed int: each half is cast
  // to unsigned before widening).
  const uint32_t Abase_lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(uintptr_t)p.A);
  const uint32_t Abase_hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uintptr_t)p.A >> 32));
  const uint64_t Abase0 = ((uint64_t)Abase_hi << 32) | (uint64_t)Abase_lo;
  const cu32_ptr Ac = (cu32_ptr)(uintptr_t)p.A;

  // Zeroed through an opaque statement: a plain "= 0" is re-materialised by the compiler on
  // every path into the loop (the accumulators were cleared twice per tile).
  int acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) asm volatile("v_mov_b32 %0, 0" : "=v"(acc[i][j]));

  // K bookkeeping (all wave-uniform).  Full chunks cover words [0, 4*nfull).  Two words left
  // over are done by a half chunk; one or three by a last "window" chunk over words
  // [Kw64-4, Kw64) when the row has at least 4 words; else one dword at a time.
  const int nfull = p.Kbits / (32 * KC);
  const int rem_bits = p.Kbits - nfull * 32 * KC;
  const int r_words = p.Kw64 - 4 * nfull;                           // words past the full chunks: 0..3
  const bool half = r_words == 2;                                   // finished by one half chunk (4 dwords)
  const bool window = BMODE != 2 && rem_bits > 0 && !half && p.Kw64 >= 4;  // finished by an overlapping chunk
  const bool slow_tail = BMODE != 2 && rem_bits > 0 && !half && !window;   // rows of 1 or 3 words only
  const int nstages = nfull + (rem_bits > 0 ? 1 : 0);
  const int last_w = p.Kw64 - 1;
  const int tail_bits = p.Kbits & 63;
  const uint64_t tail_mask = tail_bits ? ((1ull << tail_bits) - 1ull) : ~0ull;
  // first word of stage s: 4*s for full chunks (and for the slow tail), Kw64-4 for the window
  auto stage_word0 = [&](int s) { return (s == nfull && window) ? p.Kw64 - 4 : 4 * s; };

  // ---- staging: global -> registers -> LDS (double-buffered) -----------------------
  // Per-slot constants of the implicit-GEMM gather (one output pixel per slot).
  int s_ih0[PPT], s_iw0[PPT];
  uint32_t s_pix0[PPT];
  bool s_ok[PPT];
  if constexpr (BMODE == 1) {
#pragma unroll
    for (int t = 0; t < PPT; ++t) {
      const int idx = t * Cfg::THREADS + tid;
      const int row = idx / QPR;
      const uint32_t n = (uint32_t)(n0 + tile_col(row));
      // pooled ordering: a column is real iff its window exists (N = 4 * windows, but the
      // columns of the last tile's missing windows are interleaved with real ones)
      const uint32_t wdx = (n >> 8) * 64u + (n & 63u);
      s_ok[t] = idx < Cfg::PIECES && (p.g.pool ? wdx < (uint32_t)(p.N >> 2) : n < (uint32_t)p.N);
      uint32_t img = 0;
      int oh = 0, ow = 0;
      if (s_ok[t]) decode_col(p.g, n, img, oh, ow);
      s_ih0[t] = oh * p.g.sH - p.g.pH;
      s_iw0[t] = ow * p.g.sW - p.g.pW;
      s_pix0[t] = img * (uint32_t)(p.g.H * p.g.W);
    }
  }
  // Lean gather (BMODE 2: even Cw, at most 32 taps, image under 4 GiB, at most LEAN_MAX_STAGES
  // chunks).  Per slot: the byte offset of the pixel under tap (0, 0) (may be "negative": 32-bit
  // wrap-around arithmetic, only used for taps inside the image) and one validity bit per tap.
  // Per (chunk, 16-byte piece): an LDS table entry {byte offset of the tap word | flags, tap bit},
  // built once per workgroup, so the loop holds no division, no geometry and no scalar state for
  // the gather: a chunk costs a lane one LDS read, one and, one compare, one add, one select.
  uint32_t f_base[PPT], f_vmask[PPT];
  bool f_valid[PPT];
  const int my_piece = tid & 1;  // a thread always stages the same piece of a chunk
  if constexpr (BMODE == 2) {
    static_assert(QPR == 2, "two pieces per chunk");
#pragma unroll
    for (int t = 0; t < PPT; ++t) {
      const int idx = t * Cfg::THREADS + tid;
      const int row = idx / QPR;
      const uint32_t n = (uint32_t)(n0 + tile_col(row));
      const uint32_t wdx = (n >> 8) * 64u + (n & 63u);
      const bool ok = idx < Cfg::PIECES && (p.g.pool ? wdx < (uint32_t)(p.N >> 2) : n < (uint32_t)p.N);
      uint32_t img = 0;
      int oh = 0, ow = 0;
      if (ok) decode_col(p.g, n, img, oh, ow);
      const int ih0 = oh * p.g.sH - p.g.pH, iw0 = ow * p.g.sW - p.g.pW;
      uint32_t colbits = 0, vm = 0;
#pragma unroll 1
      for (int kw = 0; kw < p.g.kW; ++kw) colbits |= (uint32_t)(iw0 + kw >= 0 && iw0 + kw < p.g.W) << kw;
#pragma unroll 1
      for (int kh = 0; kh < p.g.kH; ++kh)
        if (ih0 + kh >= 0 && ih0 + kh < p.g.H) vm |= colbits << (kh * p.g.kW);
      f_vmask[t] = ok ? vm : 0u;  // columns past N read nothing but pad words and are not stored
      f_base[t] = (uint32_t)((((int64_t)img * p.g.H + ih0) * p.g.W + iw0) * p.g.Cw * 8);
      f_valid[t] = false;
    }
    // entry e = 2 * chunk + piece: words w = 2 e, 2 e + 1 of the row (same tap: Cw is even)
    const int n_entries = 2 * nstages;
    for (int e = tid; e < n_entries; e += Cfg::THREADS) {
      const uint32_t w = 2u * (uint32_t)e;
      const uint32_t tap = fdiv(w, p.g.divCw);
      const uint32_t cw = w - tap * (uint32_t)p.g.Cw;
      const uint32_t kh = fdiv(tap, p.g.divKW);
      const uint32_t kw = tap - kh * (uint32_t)p.g.kW;
      const bool live = (int)w <= last_w;  // words past K: no tap, pad word 0
      uint32_t lo = ((kh * (uint32_t)p.g.W + kw) * (uint32_t)p.g.Cw + cw) * 8u;  // multiple of 16
      if (live) lo |= LEAN_LIVE;
      if ((int)cw + 2 == p.g.Cw) lo |= LEAN_TAP_END;
      sTab[e] = make_uint2(lo, live ? (1u << tap) : 0u);
    }
    __syncthreads();
  }
  // One word of an implicit B row: tap = w / Cw, channel word = w % Cw.
  auto gather_word = [&](int t, int w) -> uint64_t {
    const uint32_t tap = fdiv((uint32_t)w, p.g.divCw);
    const int cw = w - (int)tap * p.g.Cw;
    const uint32_t kh = fdiv(tap, p.g.divKW);
    const int kw = (int)(tap - kh * p.g.kW);
    const int ih = s_ih0[t] + (int)kh, iw = s_iw0[t] + kw;
    if (ih >= 0 && ih < p.g.H && iw >= 0 && iw < p.g.W)
      return p.g.act[((size_t)s_pix0[t] + (size_t)(ih * p.g.W + iw)) * p.g.Cw + cw];
    return pad_word64(p.g.C, cw);
  };

  // stage_load only ISSUES the global loads (raw words stay in registers, nothing uses them
  // until stage_store a whole chunk of compute later), so their latency is never waited on.
  u32x4 stage[PPT];
  uint32_t staged_flags = 0;  // lean gather: flags of the table entry the last stage_load used
  auto stage_load = [&](int s) {
    const int wbase = stage_word0(s);
    if constexpr (BMODE == 2) {
      // (both words are used unconditionally, the flags by stage_store: one 8-byte LDS read; when
      // only the offset depended on it the compiler fetched it behind a branch, for valid taps only)
      const uint2 ent = sTab[2 * s + my_piece];
      staged_flags = ent.x;  // stage_store(s) selects the pad word by the same entry
      const uint32_t my_off = ent.x & ~15u;
      const char *base = reinterpret_cast<const char *>(p.g.act);
#pragma unroll
      for (int t = 0; t < PPT; ++t) {
        const bool valid = (f_vmask[t] & ent.y) != 0u;
        const uint32_t off = valid ? f_base[t] + my_off : 0u;  // taps outside: any readable address
        f_valid[t] = valid;
        stage[t] = *reinterpret_cast<const u32x4 *>(base + off);
      }
      return;
    }
    int tap_cw[2] = {0, 0}, tap_kh[2] = {0, 0}, tap_kw[2] = {0, 0};
    if constexpr (BMODE == 1) {
#pragma unroll
      for (int qq = 0; qq < 2; ++qq) {
        const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane(wbase + 2 * qq);
        const uint32_t tap = fdiv(w, p.g.divCw);
        tap_cw[qq] = (int)(w - tap * (uint32_t)p.g.Cw);
        const uint32_t kh = fdiv(tap, p.g.divKW);
        tap_kh[qq] = (int)kh;
        tap_kw[qq] = (int)(tap - kh * (uint32_t)p.g.kW);
      }
    }
#pragma unroll
    for (int t = 0; t < PPT; ++t) {
      const int idx = t * Cfg::THREADS + tid;
      const int row = idx / QPR, q = idx % QPR;
      const int w0 = wbase + 2 * q;
      u32x4 v = {0u, 0u, 0u, 0u};
      if constexpr (BMODE == 0) {
        const int n = n0 + tile_col(row);
        if (idx < Cfg::PIECES && n < p.N && w0 <= last_w) {
          const uint64_t *src = p.B + (int64_t)n * p.ldb + w0;
          if (p.b_vec16 && !(wbase & 1) && w0 + 1 <= last_w) {
            v = *reinterpret_cast<const u32x4 *>(src);
          } else {
            const uint2 lo = *reinterpret_cast<const uint2 *>(src);
            v.x = lo.x; v.y = lo.y;
            if (w0 + 1 <= last_w) {
              const uint2 hi = *reinterpret_cast<const uint2 *>(src + 1);
              v.z = hi.x; v.w = hi.y;
            }
          }
        }
      } else {
        if (s_ok[t] && w0 <= last_w) {
          if (!(p.g.Cw & 1) && !(wbase & 1)) {
            // both words of the piece belong to one tap: one 16-byte load.  The tap of each of
            // the two pieces of a chunk is wave-uniform (decoded once per chunk on the scalar
            // unit, see tap_* below); a lane only selects by its piece index q.
            const int cw = q ? tap_cw[1] : tap_cw[0];
            const int ih = s_ih0[t] + (q ? tap_kh[1] : tap_kh[0]);
            const int iw = s_iw0[t] + (q ? tap_kw[1] : tap_kw[0]);
            if (ih >= 0 && ih < p.g.H && iw >= 0 && iw < p.g.W) {
              v = *reinterpret_cast<const u32x4 *>(
                  p.g.act + ((size_t)s_pix0[t] + (size_t)(ih * p.g.W + iw)) * p.g.Cw + cw);
            } else {
              const uint64_t x0 = pad_word64(p.g.C, cw), x1 = pad_word64(p.g.C, cw + 1);
              v.x = (uint32_t)x0; v.y = (uint32_t)(x0 >> 32); v.z = (uint32_t)x1; v.w = (uint32_t)(x1 >> 32);
            }
          } else {
            const uint64_t x0 = gather_word(t, w0);
            const uint64_t x1 = w0 + 1 <= last_w ? gather_word(t, w0 + 1) : 0ull;
            v.x = (uint32_t)x0; v.y = (uint32_t)(x0 >> 32); v.z = (uint32_t)x1; v.w = (uint32_t)(x1 >> 32);
          }
        }
      }
      stage[t] = v;
    }
  };
  // Zeroes the words a window chunk shares with the full chunks before it, masks the bits
  // past K in the row's last word, then writes the pieces to LDS buffer buf.
  auto stage_store = [&](int buf, int s) {
    const int wbase = stage_word0(s);
    if constexpr (BMODE == 2) {
      // pad words: all ones, except the last word of a tap (low C % 64 bits) and words past K (0);
      // rows hold whole words, so there is no tail mask
      const uint32_t fl = staged_flags;
      const uint64_t last = pad_word64(p.g.C, p.g.Cw - 1);
      const uint32_t a1 = (fl & LEAN_LIVE) ? 0xffffffffu : 0u;
      const bool te = (fl & LEAN_TAP_END) != 0u;
      const u32x4 padv = {a1, a1, te ? (uint32_t)last & a1 : a1, te ? (uint32_t)(last >> 32) & a1 : a1};
#pragma unroll
      for (int t = 0; t < PPT; ++t) {
        const int idx = t * Cfg::THREADS + tid;
        const int row = idx / QPR, q = idx % QPR;
        const u32x4 v = f_valid[t] ? stage[t] : padv;
        if (idx < Cfg::PIECES) *reinterpret_cast<u32x4 *>(&sB[buf * Cfg::TILE + row * RS + q * 4]) = v;
      }
      return;
    }
    const int wdone = (s == nfull && window) ? 4 * nfull : 0;  // words below this are already counted
    const uint32_t tm_lo = (uint32_t)tail_mask, tm_hi = (uint32_t)(tail_mask >> 32);
#pragma unroll
    for (int t = 0; t < PPT; ++t) {
      const int idx = t * Cfg::THREADS + tid;
      const int row = idx / QPR, q = idx % QPR;
      const int w0 = wbase + 2 * q;
      u32x4 v = stage[t];
      if (w0 == last_w) { v.x &= tm_lo; v.y &= tm_hi; }
      if (w0 + 1 == last_w) { v.z &= tm_lo; v.w &= tm_hi; }
      if (w0 < wdone) { v.x = 0u; v.y = 0u; }
      if (w0 + 1 < wdone) { v.z = 0u; v.w = 0u; }
      if (idx < Cfg::PIECES) *reinterpret_cast<u32x4 *>(&sB[buf * Cfg::TILE + row * RS + q * 4]) = v;
    }
  };

  const int lane_row = (wn * 64 * TN + lane) * RS;

  if (nstages > 0) {
    stage_load(0);
    stage_store(0, 0);
  }
  __syncthreads();

  // ---- chunks ----------------------------------------------------------------------------
  // Per chunk: the wave's 8 rows of A arrive with 8 scalar loads of 8 dwords (64 SGPRs),
  // issued together with the LDS reads of B; one wait; then 2 * 8 * TN * 8 xor / popcount
  // instructions and nothing else.  Loads, wait and the per-row compute statements are
  // volatile inline asm, so their order in the instruction stream is the order written
  // here; the wait names every loaded SGPR as in/out operand, which orders all uses after
  // it.  The latency of one wave's loads is covered by the other waves on the SIMD.
  const int nfast = nfull + (window ? 1 : 0);
  // Wave priority.  The instruction arbiter prefers older waves, so of the workgroups resident
  // on a compute unit the oldest runs at nearly full speed, the others in its gaps, and they
  // finish one after the other; the last one then runs alone, at an occupancy where neither its
  // latencies nor the yield slots of its pairs are filled.  The workgroups of the last resident
  // set (ids >= prio_from) therefore lower their priority as they advance through K: whoever is
  // behind gets the issue slots, and they finish within an eighth of K of each other.  Earlier
  // workgroups keep one priority and free their slot as early as before.
  const bool paced = (int)blockIdx.x >= p.prio_from;
  // Prologue and store run at priority 3 (set at kernel entry and before the store): they are
  // short and latency-bound, and a new workgroup that gets through its prologue quickly is one
  // more set of waves with work to issue.  The K loop runs below that: at 2 for the earlier
  // workgroups, stepping down from 2 for the paced ones (from 3 when every workgroup of the
  // launch is paced, so that the steps at 1/2, 3/4 and 7/8 of K all exist).
  const int prio_top = p.prio_from == 0 ? 3 : 2;
  int prio_cur = prio_top;
  if (prio_top == 2) __builtin_amdgcn_s_setprio(2);
  for (int c = 0; c < nfast; ++c) {
    if (paced) {
      const int steps = (2 * c < nstages) ? 0 : (4 * c < 3 * nstages) ? 1 : (8 * c < 7 * nstages) ? 2 : 3;
      const int lvl = max(prio_top - steps, 0);  // wave-uniform
      if (lvl != prio_cur) {
        prio_cur = lvl;
        if (lvl == 2) __builtin_amdgcn_s_setprio(2);
        else if (lvl == 1) __builtin_amdgcn_s_setprio(1);
        else __builtin_amdgcn_s_setprio(0);
      }
    }
    const int buf = c & 1;
    const bool more = c + 1 < nstages;
    if (more) stage_load(c + 1);
    const uint32_t *sBl = &sB[buf * Cfg::TILE + lane_row];
    const bool is_window = c == nfull;  // only possible for the last iteration
    const uint64_t Abase = Abase0 + (uint64_t)(uint32_t)stage_word0(c) * 8u;
    u32x8 a[TM];
    u32x8 b[TN];
    uint32_t aoff_cur = aoff_first;
    asm volatile("" : "+s"(aoff_cur));
#pragma unroll
    for (int i = 0; i < TM; ++i)
      asm volatile("s_load_dwordx8 %0, %1, %2" : "=s"(a[i]) : "s"(Abase), "s"(BNN_AOFF(i)));
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      b[j].lo = *reinterpret_cast<const u32x4 *>(&sBl[j * 64 * RS]);
      b[j].hi = *reinterpret_cast<const u32x4 *>(&sBl[j * 64 * RS + 4]);
    }
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+s"(a[0]), "+s"(a[1]), "+s"(a[2]), "+s"(a[3]), "+s"(a[4]), "+s"(a[5]), "+s"(a[6]), "+s"(a[7]));
    if (is_window) {
      // dwords already counted by the full chunks, and the bits past K, leave A as zeros
      int dw_done = 2 * (4 * nfull - (p.Kw64 - 4));
      asm volatile("" : "+s"(dw_done));  // the eight compares below stay here, not in registers across the loop
      const uint32_t m6 = (uint32_t)tail_mask, m7 = (uint32_t)(tail_mask >> 32);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int d = 0; d < 8; ++d)
          if (d < dw_done) a[i][d] = 0u;
        a[i][6] &= m6;
        a[i][7] &= m7;
      }
    }
    uint32_t t0, t1;
#define BNN_BV(j, d) b[j][d]
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      if constexpr (YIELD) {
        if constexpr (TN == 8) BNN_GEMM_ROW_8(acc[i], a[i], BNN_BV, t0, t1);
        else if constexpr (TN == 4) BNN_GEMM_ROW_4(acc[i], a[i], BNN_BV, t0, t1);
        else if constexpr (TN == 2) BNN_GEMM_ROW_2(acc[i], a[i], BNN_BV, t0, t1);
        else BNN_GEMM_ROW_1(acc[i], a[i], BNN_BV, t0, t1);
      } else {
        if constexpr (TN == 8) BNN_GEMM_ROW_8_NY(acc[i], a[i], BNN_BV, t0, t1);
        else if constexpr (TN == 4) BNN_GEMM_ROW_4_NY(acc[i], a[i], BNN_BV, t0, t1);
        else if constexpr (TN == 2) BNN_GEMM_ROW_2_NY(acc[i], a[i], BNN_BV, t0, t1);
        else BNN_GEMM_ROW_1_NY(acc[i], a[i], BNN_BV, t0, t1);
      }
    }
#undef BNN_BV
    if (more) {
      stage_store(buf ^ 1, c + 1);  // that buffer was last read in chunk c-1, before the previous barrier
      __syncthreads();
    }
  }

  // ---- half chunk: the last two words of rows of 4*n + 2 words -------------------------------
  if (half) {
    const uint32_t *sBl = &sB[(nfull & 1) * Cfg::TILE + lane_row];
    const uint64_t Abase = Abase0 + (uint64_t)(uint32_t)(4 * nfull) * 8u;
    u32x4 a[TM];
    u32x4 b[TN];
    uint32_t aoff_cur = aoff_first;
    asm volatile("" : "+s"(aoff_cur));
#pragma unroll
    for (int i = 0; i < TM; ++i)
      asm volatile("s_load_dwordx4 %0, %1, %2" : "=s"(a[i]) : "s"(Abase), "s"(BNN_AOFF(i)));
#pragma unroll
    for (int j = 0; j < TN; ++j) b[j] = *reinterpret_cast<const u32x4 *>(&sBl[j * 64 * RS]);
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+s"(a[0]), "+s"(a[1]), "+s"(a[2]), "+s"(a[3]), "+s"(a[4]), "+s"(a[5]), "+s"(a[6]), "+s"(a[7]));
    const uint32_t m2 = (uint32_t)tail_mask, m3 = (uint32_t)(tail_mask >> 32);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      a[i][2] &= m2;
      a[i][3] &= m3;
    }
    uint32_t t0, t1;
#define BNN_BV(j, d) b[j][d]
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      if constexpr (YIELD) {
        if constexpr (TN == 8) BNN_GEMM_HALF_8(acc[i], a[i], BNN_BV, t0, t1);
        else if constexpr (TN == 4) BNN_GEMM_HALF_4(acc[i], a[i], BNN_BV, t0, t1);
        else if constexpr (TN == 2) BNN_GEMM_HALF_2(acc[i], a[i], BNN_BV, t0, t1);
        else BNN_GEMM_HALF_1(acc[i], a[i], BNN_BV, t0, t1);
      } else {
        if constexpr (TN == 8) BNN_GEMM_HALF_8_NY(acc[i], a[i], BNN_BV, t0, t1);
        else if constexpr (TN == 4) BNN_GEMM_HALF_4_NY(acc[i], a[i], BNN_BV, t0, t1);
        else if constexpr (TN == 2) BNN_GEMM_HALF_2_NY(acc[i], a[i], BNN_BV, t0, t1);
        else BNN_GEMM_HALF_1_NY(acc[i], a[i], BNN_BV, t0, t1);
      }
    }
#undef BNN_BV
  }

  // ---- rows of one or three words (K < 193): one dword at a time ----------------------------
  // B is already masked / zero-filled by the staging; A is masked here.
  if (slow_tail) {
    const uint32_t *sBl = &sB[(nfull & 1) * Cfg::TILE + lane_row];
    const int kd0 = nfull * KC;
    const int tb32 = p.Kbits & 31;
#pragma unroll 1
    for (int kd = kd0; kd < p.Kd; ++kd) {
      const uint32_t amask = (kd == p.Kd - 1 && tb32) ? ((1u << tb32) - 1u) : 0xffffffffu;
      uint32_t b[TN];
#pragma unroll
      for (int j = 0; j < TN; ++j) b[j] = sBl[j * 64 * RS + (kd - kd0)];
      uint32_t aoff_cur = aoff_first;
      asm volatile("" : "+s"(aoff_cur));
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const uint32_t a = Ac[(BNN_AOFF(i) >> 2) + kd] & amask;
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = popc_acc(a ^ b[j], acc[i][j]);
      }
    }
  }

  // ---- store ------------------------------------------------------------------------
  __builtin_amdgcn_s_setprio(3);
  if constexpr (EMODE == 0) {
    if constexpr (TN == 4 && WN == 1) {
      if (colperm) store_tile_x4(acc, m0, n0 + 4 * lane);
      else store_tile<TN>(acc, m0, n0 + lane);
    } else {
      store_tile<TN>(acc, m0, n0 + wn * 64 * TN + lane);
    }
  } else {
    // Binarizing epilogue.  Row m is output channel m; the workgroup's 8 * WM rows are one
    // 64-bit channel word (WM = 8), or one 32-bit half of it (WM = 4), of every pixel in its
    // tile.  Each lane turns its 8 channels into a byte per output pixel, the waves' bytes
    // meet in LDS, and one thread per pixel writes the assembled (half) word.
    const GemmParams BNN_CONST_AS *kp = (const GemmParams BNN_CONST_AS *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(kp));
    const int M = kp->M, N = kp->N, Kformula = kp->Kformula;
    const float *const scale = kp->scale, *const bias = kp->bias;
    const int pool = kp->g.pool;
    uint64_t *const outp = kp->outp;
    const int cw_out = kp->cw_out;
    uint32_t bytes[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) bytes[j] = 0u;
    // The affine constants of the wave's 8 rows: wave-uniform, read through the constant address
    // space (scalar loads), all 16 requested before the first is used, rows past M re-reading row
    // M - 1.  (Loaded row by row inside the loop below they were 16 dependent vector loads, each
    // waited for: eight memory round trips at the end of every tile, during which the wave held
    // its slot without issuing.)
    typedef const float BNN_CONST_AS *cf32_ptr;
    const cf32_ptr cscale = (cf32_ptr)(uintptr_t)scale, cbias = (cf32_ptr)(uintptr_t)bias;
    float scr[TM], bir[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int mc = min(m0 + i, M - 1);
      scr[i] = cscale[mc];
      bir[i] = cbias[mc];
    }
    // Rows run from the last to the first so that each sign is shifted in with one add-with-carry
    // (byte = 2 * byte + bit).  K - 2*acc decreases in acc: the 2x2 max is K - 2*min(acc).
    auto sign_arg = [&](int i, int a) {
      const bool row_ok = m0 + i < M;  // rows past M give bit 0
      return fmaf(row_ok ? scr[i] : 0.0f, (float)(Kformula - 2 * a), row_ok ? bir[i] : -1.0f);
    };
    static_assert(TM % 4 == 0, "four signs at a time");
    if (pool) {
#pragma unroll
      for (int i = TM - 1; i >= 0; i -= 4) {
        float y[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          int a = acc[i - k][0];
#pragma unroll
          for (int j = 1; j < TN; ++j) a = min(a, acc[i - k][j]);
          y[k] = sign_arg(i - k, a);
        }
        uint32_t b[1] = {bytes[0]};
        shift_in_signs<1>(b, y);
        bytes[0] = b[0];
      }
    } else {
      constexpr int ROWS = 4 / TN;
#pragma unroll
      for (int i = TM - 1; i >= 0; i -= ROWS) {
        float y[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) y[k] = sign_arg(i - k / TN, acc[i - k / TN][k % TN]);
        shift_in_signs<TN>(bytes, y);
      }
    }
    __syncthreads();  // every wave is done reading the B tiles: LDS is reused for the output bytes
    uint8_t *sO = reinterpret_cast<uint8_t *>(sB);
    if (pool) {
      sO[lane * WM + wm] = (uint8_t)bytes[0];
    } else {
#pragma unroll
      for (int j = 0; j < TN; ++j) sO[(j * 64 + lane) * WM + wm] = (uint8_t)bytes[j];
    }
    __syncthreads();
    const int npix = pool ? 64 : 64 * TN;
    if (tid < npix) {
      // global pixel index: pooled window index, or column index (NHWC pixel order)
      const int64_t gp = pool ? (int64_t)ni * 64 + tid : (int64_t)n0 + tid;
      const int64_t limit = pool ? (int64_t)(N >> 2) : (int64_t)N;
      if (gp < limit) {
        if constexpr (WM == 8) {
          const uint2 w = *reinterpret_cast<const uint2 *>(&sO[tid * 8]);
          *reinterpret_cast<uint2 *>(outp + gp * cw_out + mi) = w;
        } else {
          // 32 channels: half of word (mi / 2); a last odd half past D is written as zeros
          const uint32_t w = *reinterpret_cast<const uint32_t *>(&sO[tid * 4]);
          uint32_t *o32 = reinterpret_cast<uint32_t *>(outp) + (gp * cw_out) * 2;
          o32[mi] = w;
          if (mi == kp->tilesM - 1 && (kp->tilesM & 1)) o32[mi + 1] = 0u;  // channels past D: pad bits 0
        }
      }
    }
  }
}


// ---- host side ----------------------------------------------------------------------
template <int TN, int WM, int WN, int MINW, int BMODE, int EMODE, int YIELD>
static bnn_status launch_one(GemmParams &p, hipStream_t s, int kid) {
  using Cfg = GemmCfg<TN, WM, WN>;
  // the last resident set: MINW waves per SIMD, 4 SIMDs per compute unit
  const int64_t resident = (int64_t)(MINW * 4 / (Cfg::THREADS / 64)) * p.n_cu;
  const int64_t nb = (int64_t)p.tilesM * p.tilesN;
  p.prio_from = (int)(nb > resident ? nb - resident : 0);
  ProfScope ps(kid, s);
  hipLaunchKernelGGL((xnor_gemm_kernel<TN, WM, WN, MINW, BMODE, EMODE, YIELD>),
                     dim3((unsigned)(p.tilesM * p.tilesN)), dim3(Cfg::THREADS), 0, s, p);
  return launch_status();
}

template <int TN, int WM, int WN, int MINW>
static bnn_status launch_cfg(GemmParams &p, int bmode, int emode, hipStream_t s, int kid) {
  using Cfg = GemmCfg<TN, WM, WN>;
  p.tilesM = (p.M + Cfg::BM - 1) / Cfg::BM;
  p.tilesN = (p.N + Cfg::BN - 1) / Cfg::BN;
  const int64_t blocks = (int64_t)p.tilesM * p.tilesN;
  if (blocks > 0x7fffffffLL) return BNN_ERR_UNSUPPORTED;
  // The one-cycle yields after each xor/popcount pair pay off only when at least two waves
  // share a SIMD (4 per compute unit); with fewer they cost issue slots.
  const int64_t waves = blocks * (Cfg::THREADS / 64);
  const bool yield = waves >= 2 * 4 * (int64_t)p.n_cu;
  // 256-column tiles writing int32 / fp32: four consecutive columns per lane and 16-byte stores where
  // every group of four columns is whole, inside one image and 16-byte aligned
  p.colperm = (emode == 0 && TN == 4 && WN == 1 && (p.N & 3) == 0 && (!p.C || (p.ldc & 3) == 0) &&
               (!p.Y || (p.ldy & 3) == 0) && (p.img_stride == 0 || ((p.OHW & 3u) == 0 && (p.img_stride & 3) == 0)))
                  ? 1
                  : 0;
  if constexpr ((TN == 4 || TN == 2) && (WM == 8 || WM == 4) && WN == 1) {
    if (emode == 1) {
      if (bmode == 0 || (p.g.pool && TN != 4)) return BNN_ERR_UNSUPPORTED;
      if (bmode == 2)
        return yield ? launch_one<TN, WM, WN, MINW, 2, 1, 1>(p, s, kid) : launch_one<TN, WM, WN, MINW, 2, 1, 0>(p, s, kid);
      return yield ? launch_one<TN, WM, WN, MINW, 1, 1, 1>(p, s, kid) : launch_one<TN, WM, WN, MINW, 1, 1, 0>(p, s, kid);
    }
  }
  if (emode != 0) return BNN_ERR_UNSUPPORTED;
  if (bmode == 2)
    return yield ? launch_one<TN, WM, WN, MINW, 2, 0, 1>(p, s, kid) : launch_one<TN, WM, WN, MINW, 2, 0, 0>(p, s, kid);
  if (bmode == 1)
    return yield ? launch_one<TN, WM, WN, MINW, 1, 0, 1>(p, s, kid) : launch_one<TN, WM, WN, MINW, 1, 0, 0>(p, s, kid);
  return yield ? launch_one<TN, WM, WN, MINW, 0, 0, 1>(p, s, kid) : launch_one<TN, WM, WN, MINW, 0, 0, 0>(p, s, kid);
}

int device_cu_count() {
  // one slot per device id; concurrent first calls write the same value
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cached[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cached[dev] = n;
  }
  return cached[dev];
}

// Whether every row of the maps (every plane, for NCHW maps) starts at a multiple of `ints` 4-byte elements.
bool map_rows_start_every(const GemmParams &p, uint32_t ints) {
  const bool planes = p.img_stride != 0;
  auto ok = [&](const void *base, int64_t ld) {
    return !base || (((uintptr_t)base & (4 * ints - 1)) == 0 && (planes ? p.OHW % ints == 0 : ld % ints == 0));
  };
  return ok(p.C, p.ldc) && ok(p.Y, p.ldy);
}

// Stores of the matrix-core tiles' maps, non-temporal or ordinary.  Measured over 900 random GEMMs and convolutions;
// "words" are 64-bit words of the reduction per stored output, rows that a tile computes for nothing included.
//   Rows of whole 128-byte lines: non-temporal (2 to 9 % faster on average), and so up to 32 rows, half a tile (32 x 14 x
//     14 from 576 bits, 400 MB: 111 us, ordinary 146; 32 x 60 x 60 from 320, 60 MB: 17.4 against 19.9).
//   Rows that start inside a 64-byte half line: a piece of a line written past the L2 costs a line in memory, pieces that
//     meet in the L2 do not.  Ordinary up to 36 words (64 x 128 x 58 x 58 maps from 1152 bits 41 -> 26 us; 1000 x 50004 x
//     700 83 -> 39; 256 x 256 x 14 x 14 from 2304 bits 26 -> 24; on average 1.1 to 2.1 times faster by size); with more,
//     the multiplications hide it and the caches are the operands' (up to 25 % the other way beyond 320 MB).  Up to 56
//     rows the operand's bytes come near the map's and need those caches from half of them on (48 x 1000008 x 1100
//     66 us, ordinary 80; 56 rows 70 against 85; 40 x 200004 x 700 13.2 against 14.3), but not below (56 x 1000004 x
//     576 81 against 66); 64 rows go either way (64 x 400004 x 1600 46 against 41, x 1000008 x 1100 82 against 91).
//     Small calls whose rows are whole 32-byte sectors stay non-temporal from 12 words on: ordinary stores are 0 to 7 %
//     faster alone, but push out the fp32 image that the same call encodes (74 x 128 x 20 x 39, stride 2, both maps:
//     18.1 us, ordinary 19.2; 24 x 157 x 52 x 34 to 128 channels 21.0, 23.0).
//     word: conv_word.hip's kernel has at most 36 words and no tiles to hide such stores behind: rows computed for nothing
//     don't count (256 channels, 163 x 19 x 36 to 435 83 -> 56 us, 45 x 58 x 42 to 160 36.9 -> 26.2, 387 x 37 x 20 to 60
//     37.2 -> 27.1), but up to 56 rows as above (48 x 46 x 18 to 48 9.6 against 10.05 ordinary).
//   Rows of whole half lines (28 x 28 maps): the same where the stores decide, below 12 words, and the call's bytes
//     still fit the last-level cache of 256 MB (64 x 28 x 28 from 576 bits, 240 MB: 55.5 -> 43.1 us; 512 x 117200 x 700
//     60.8 -> 42.0); non-temporal elsewhere (512 x 117200 x 2304 80 us, ordinary 95; 64 x 44 x 44 from 512 bits, 300 MB:
//     20 %; small calls 1 to 5 %).
bool nontemporal_maps(const GemmParams &p, int bmode, bool word) {
  if (map_rows_start_every(p, 32) || p.M <= 32) return true;
  const int64_t words_x_m = (int64_t)p.Kw64 * (((int64_t)p.M + 63) / 64 * 64);
  const int64_t out = (int64_t)p.M * p.N * 4 * ((p.C ? 1 : 0) + (p.Y ? 1 : 0));
  const int64_t in = bmode == 0 ? (int64_t)p.N * p.Kw64 * 8 : (int64_t)p.g.Nimg * p.g.H * p.g.W * p.g.Cw * 8;
  const bool small = out + in <= 50000000, long_rows = words_x_m >= 12 * (int64_t)p.M;
  if (!map_rows_start_every(p, 16))
    return (words_x_m > 36 * (int64_t)p.M && !(word && p.M > 56)) || (p.M <= 56 && 2 * in >= out) ||
           (small && long_rows && map_rows_start_every(p, 8));
  return long_rows || small || out + in > 256000000;
}

bool map_columns_by_four(const GemmParams &p) {
  return (p.N & 3) == 0 && (!p.C || (p.ldc & 3) == 0) && (!p.Y || (p.ldy & 3) == 0) &&
         (p.img_stride == 0 || ((p.OHW & 3u) == 0 && (p.img_stride & 3) == 0));
}

bnn_status run_gemm(GemmParams &p, int bmode, int emode, hipStream_t s, const GemmTune &tune) {
  int cfg = tune.cfg;
  p.n_cu = device_cu_count();
  p.nt_store = map_rows_start_every(p, 32) ? 1 : 0;
  if (bmode == 1 && emode == 0 && p.g.pool == 0 && p.g.kH == 1 && p.g.kW == 1 && p.g.sH == 1 && p.g.sW == 1 &&
      p.g.pH == 0 && p.g.pW == 0) {
    // a stride-1 pointwise convolution over a packed image has nothing to gather: its patch
    // matrix is the packed image itself
    bmode = 0;
    p.B = p.g.act;
    p.ldb = p.g.Cw;
    p.b_vec16 = (p.g.Cw & 1) == 0 ? 1 : 0;
  }
  // a forced value this call cannot use selects the heuristic
  const bool valu = emode == 0 ? (cfg >= 1 && cfg <= 6 && cfg != 5)
                               : (cfg == 3 || cfg == 1 || (!p.g.pool && (cfg == 6 || cfg == 4)));
  const bool short_rows = bmode == 0 && emode == 0 && lowk_applicable(p);
  const bool matrix = (((cfg >= 21 && cfg <= 24) || cfg == 29) && fp4_applicable(p)) || (cfg >= 25 && cfg <= 28);
  const bool few_rows = short_rows && fewrows_applicable(p);
  const bool word = conv_word_applicable(p, bmode);
  const bool lowk = short_rows && ((cfg >= 10 && cfg <= 17) || (cfg >= 30 && cfg <= 37));
  if (!valu && !matrix && !lowk && !(few_rows && cfg == 18) && !(word && cfg == 19)) cfg = -1;
  if (few_rows && (cfg < 0 ? fewrows_faster(p) : cfg == 18)) return launch_fewrows(p, s);
  if (lowk) return launch_lowk(p, cfg % 10, s, cfg < 30 ? 1 : 3);
  if (short_rows && cfg < 0 && lowk_faster(p)) return launch_lowk(p, -1, s);
  if (!valu) {
    // The matrix cores; few outputs split the reduction axis, and so do rows too long for exact fp32 sums.
    p.colperm = emode == 0 && map_columns_by_four(p) ? 1 : 0;
    const bool by_word = word && (cfg < 0 ? tune.lean != 0 && conv_word_faster(p, emode) : cfg == 19);
    p.nt_store = emode == 0 && nontemporal_maps(p, bmode, by_word) ? 1 : 0;
    if (by_word) return launch_conv_word(p, emode, s);
    if (cfg >= 25 && cfg <= 28) return launch_gemm_fp4_split(p, bmode, emode, s, cfg - 25);
    if (cfg < 0 && (fp4_split_applicable(p, bmode) || !fp4_applicable(p))) return launch_gemm_fp4_split(p, bmode, emode, s, -1);
    return launch_gemm_fp4(p, bmode, emode, s, cfg >= 29 ? cfg - 25 : cfg >= 21 ? cfg - 21 : -1, tune.lean != 0);
  }
  // Vector-ALU tiles, with a forced configuration only: the method's own instructions (xor, popcount), measured beside
  // the matrix cores.
  if (bmode == 1 && tune.lean) {
    // lean gather: 16-byte pieces never straddle a tap (even Cw), one validity bit per tap in a
    // 32-bit mask, 32-bit byte offsets into the packed image
    const int64_t taps = (int64_t)p.g.kH * p.g.kW;
    const int64_t img_bytes = (int64_t)p.g.Nimg * p.g.H * p.g.W * p.g.Cw * 8;
    if ((p.g.Cw & 1) == 0 && taps <= 32 && img_bytes <= 0xffffffffLL && (p.Kw64 + 3) / 4 <= LEAN_MAX_STAGES) bmode = 2;
  }
  switch (cfg) {
    case 1: return launch_cfg<4, 4, 1, 4>(p, bmode, emode, s, KID_XNOR_GEMM);        // 32 x 256
    case 2: return launch_cfg<1, 4, 1, 4>(p, bmode, emode, s, KID_XNOR_GEMM_SMALL);  // 32 x 64
    case 3: return launch_cfg<4, 8, 1, 6>(p, bmode, emode, s, KID_XNOR_GEMM);        // 64 x 256
    case 4: return launch_cfg<2, 4, 1, 4>(p, bmode, emode, s, KID_XNOR_GEMM);        // 32 x 128
    case 6: return launch_cfg<2, 8, 1, 4>(p, bmode, emode, s, KID_XNOR_GEMM);        // 64 x 128
    default: return BNN_ERR_UNSUPPORTED;
  }
}

static bnn_status gemm_common(const uint64_t *A, int64_t lda, const uint64_t *B, int64_t ldb, int64_t M, int64_t N,
                              int64_t K, int32_t *C, int64_t ldc, float *Y, int64_t ldy, const float *scale,
                              const float *bias, bnn_ch_axis axis, void *stream, const GemmTune &tune = GemmTune()) {
  if (M < 0 || N < 0 || K <= 0) return BNN_ERR_SHAPE;
  const int64_t Kw = bnn_packed_words(K);
  if (lda < Kw || ldb < Kw) return BNN_ERR_STRIDE;
  if (C && ldc < N) return BNN_ERR_STRIDE;
  if (Y && ldy < N) return BNN_ERR_STRIDE;
  if (M == 0 || N == 0) return BNN_OK;
  if (!A || !B || (!C && !Y)) return BNN_ERR_NULL;
  if (Y && (!scale || !bias)) return BNN_ERR_NULL;
  if (Y && axis != BNN_CH_ROW && axis != BNN_CH_COL) return BNN_ERR_SHAPE;
  if (!aligned16(A) || !aligned16(B) || (C && !aligned16(C)) || (Y && !aligned16(Y))) return BNN_ERR_ALIGN;
  // column indices are ints computed on N rounded up to the tile width (at most 256)
  if (M > 0x7fffffffLL || N > 0x7fffffffLL - 256 || K > 0x7fffffffLL) return BNN_ERR_UNSUPPORTED;
  if (M * 8 * lda > 0xffffffffLL) return BNN_ERR_UNSUPPORTED;  // 32-bit byte offsets into A
  GemmParams p = {};
  p.A = reinterpret_cast<const uint32_t *>(A);
  p.B = B;
  p.lda32 = 2 * lda;
  p.ldb = ldb;
  p.M = (int)M;
  p.N = (int)N;
  p.Kbits = (int)K;
  p.Kformula = (int)K;
  p.Kd = (int)((K + 31) / 32);
  p.Kw64 = (int)Kw;
  p.b_vec16 = (ldb % 2 == 0) ? 1 : 0;
  p.C = C;
  p.Y = Y;
  p.ldc = ldc;
  p.ldy = ldy;
  p.scale = scale;
  p.bias = bias;
  p.axis = (int)axis;
  p.OHW = 0x7fffffffu;
  p.divOHW = FastDiv(0x7fffffffu);
  p.img_stride = 0;
  return run_gemm(p, 0, 0, (hipStream_t)stream, tune);
}

}  // namespace bnn

using namespace bnn;

extern "C" bnn_status bnn_xnor_gemm(const uint64_t *A, int64_t lda, const uint64_t *B, int64_t ldb, int32_t *C,
                                    int64_t ldc, int64_t M, int64_t N, int64_t K, void *stream) {
  if (M > 0 && N > 0 && K > 0 && !C) return BNN_ERR_NULL;
  return gemm_common(A, lda, B, ldb, M, N, K, C, ldc, nullptr, 0, nullptr, nullptr, BNN_CH_NONE, stream);
}

extern "C" bnn_status bnn_xnor_gemm_epilogue(const uint64_t *A, int64_t lda, const uint64_t *B, int64_t ldb, int64_t M,
                                             int64_t N, int64_t K, int32_t *C, int64_t ldc, float *Y, int64_t ldy,
                                             const float *scale, const float *bias, bnn_ch_axis axis, void *stream) {
  return gemm_common(A, lda, B, ldb, M, N, K, C, ldc, Y, ldy, scale, bias, axis, stream);
}

// Declared in bnn_testing.h: the same call with the tile configuration chosen by the caller.
extern "C" bnn_status bnn_testing_xnor_gemm_epilogue(const uint64_t *A, int64_t lda, const uint64_t *B, int64_t ldb,
                                                     int64_t M, int64_t N, int64_t K, int32_t *C, int64_t ldc,
                                                     float *Y, int64_t ldy, const float *scale, const float *bias,
                                                     bnn_ch_axis axis, int cfg, void *stream) {
  GemmTune tune;
  tune.cfg = cfg;
  return gemm_common(A, lda, B, ldb, M, N, K, C, ldc, Y, ldy, scale, bias, axis, stream, tune);
}

// Declared in bnn_testing.h.
extern "C" int bnn_testing_nontemporal_maps(int M, int N, int K, int64_t ldc, int64_t base_bytes) {
  if (M <= 0 || N <= 0 || K <= 0 || ldc < N) return -1;
  GemmParams p = {};
  p.M = M;
  p.N = N;
  p.Kw64 = (int)bnn_packed_words(K);
  p.C = reinterpret_cast<int32_t *>((uintptr_t)4096 + (uintptr_t)base_bytes);
  p.ldc = ldc;
  return nontemporal_maps(p, 0) ? 1 : 0;
}
