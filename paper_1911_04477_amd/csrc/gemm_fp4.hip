// Xnor-Bitcount GEMM (section 3.2) and implicit-GEMM convolution on the matrix cores, operands kept
// at 1 bit per value in memory and in LDS.
//
// sum_k a_k * b_k over +-1 values IS K - 2 * popcount(a XOR b), and V_MFMA_F32_32X32X64_F8F6F4 with both
// operands in E2M1 adds 64 such products per output and instruction, exactly in its fp32 accumulator while
// the sum stays below 2^24.  What decides the speed is turning bits into E2M1 codes: a code is 4 bits,
// sign first, so with x a dword of 32 bits,  (x << s) & 0x88888888 | 0x22222222  (s = 0..3) are four dwords
// of eight codes +1.0 (0x2, bit 0) or -1.0 (0xA, bit 1): 3 shifts + 4 bit-field inserts per 32 values.
// (The signs of both operands are flipped against section 3.1's convention; the products are not.)  The
// order of the values within a dword changes, alike for both operands, which a sum does not see.
//
// Bound: the matrix instructions, with the expansion beside them.  A wave multiplies 32*WTM x 32*WTN
// outputs; per 64 values it needs WTM + WTN expanded fragments (7 vector instructions each) for
// WTM * WTN matrix instructions, so tall wave tiles matter: from registers, with the expansion, 2 x 4
// blocks sustain 8.0 PFLOP/s, 2 x 2 7.5, 1 x 4 6.6, and 9.6 without any expansion.  Expanding in the wave
// that uses a fragment, not when staging it, keeps LDS and its traffic at 1 bit per value, and the
// operand traffic from the L2s, which bounds a GEMM on operands stored at 4 bits, falls by 4.
//
// Values past the end of a row are staged as 0 bits in both operands: each adds (+1)(+1), so the
// accumulators start at -(padded length - K) and end at the result.
//
// Long explicit rows run into the chip's power limit instead: the clock falls as the multipliers' inputs toggle.  Bits
// as the codes 0 and 1 (BitCodes) let half of the products be zero and hold a higher clock; they sum to S = popcount(a AND b),
// and the result is K - 2 popcount(a) - 2 popcount(b) + 4 S (section 3.2's sum, since a XOR b counts a + b - 2 (a AND b)).
// The counts of set bits are taken from the pieces as they are staged.
//
// Lanes of a 32 x 32 block: operand fragments hold row (or column) l % 32 of the block, 64-bit word l / 32
// of the 128-bit piece, one dword of it per instruction; the accumulator's register r holds row
// 8*(r/4) + 4*(l/32) + r%4 of column l % 32.  Column block j, lane l of a wave is tile column WTN*(l%32)+j:
// a lane's WTN columns are consecutive and leave as one 16- or 8-byte store per row, and with columns
// ordered window-major (column = 4 * window + member) a lane of a 4-block wave holds whole pooling windows.
// (Columns that leave one by one, and signs from an LDS region: tile column 32*j + l%32.)
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "fp4_tile.h"

namespace bnn {

typedef const uint32_t __attribute__((address_space(4))) *cu32_args;

// Where operand B comes from.
//   GM_EXPL16 / GM_EXPL8  explicit rows, read with 16-byte / 8-byte loads
//   GM_HALO   packed NHWC image; the input pixels that the tile's output pixels see (halo and padding
//             included) are copied to LDS once and every tap reads them there at a uniform distance
//   GM_ANY    packed NHWC image, every word of every patch gathered from memory (regions that do not fit LDS)
// GM_HALO against gathering per tap through staged tiles: the gather decodes a tap, tests a mask and pads
// every 16 bytes kH*kW times over, about 200 vector instructions per 512 bits of K beside the 336 of the
// expansion.
enum : int { GM_EXPL16 = 0, GM_EXPL8 = 1, GM_HALO = 2, GM_ANY = 3 };
// What leaves: int32 / fp32 maps in one of the three store forms (a kernel each: a choice inside one costs partial row
// tiles 10 %); packed signs; packed signs of the 2x2 maximum.
enum : int { EM_MAPS_NT = MS_NT, EM_MAPS_VEC = MS_VEC, EM_MAPS_ONE = MS_ONE, EM_SIGN = 3, EM_POOL = 4 };

template <int WTM_, int WTN_, int WGM_, int WGN_, int GM_, bool BITS_ = false>
struct Fp4Cfg {
  static constexpr int WTM = WTM_, WTN = WTN_, WGM = WGM_, WGN = WGN_, S = 4;  // S pieces (512 bits of K) per stage
  static constexpr int T = 64 * WGM * WGN;
  static constexpr int BM = 32 * WTM * WGM, BN = 32 * WTN * WGN;
  static constexpr bool STAGEB = GM_ != GM_HALO;
  static constexpr int REGS = BM / 32 + (STAGEB ? BN / 32 : 0);  // 32-row regions of 16-byte pieces
  static constexpr int R16 = 33;                                 // region stride in 16-byte units (one of padding)
  // plane (one piece of every row) stride = 2 mod 8 units: the four pieces of consecutive rows that a
  // staging wave writes then fall on distinct banks
  static constexpr int P16 = REGS * R16 + ((2 - REGS * R16) % 8 + 8) % 8;
  static constexpr int PA = BM * S / T, PB = STAGEB ? BN * S / T : 0;  // pieces per thread and stage
  static constexpr int STAGE_BYTES = 3 * S * P16 * 16;
  // scale and bias of every row; GM_HALO: region offset of every column; bits: corrections of rows and columns
  static constexpr int FIXED_BYTES = STAGE_BYTES + 2 * BM * 4 + (GM_ == GM_HALO ? BN * 4 : 0) + (BITS_ ? (BM + BN) * 4 : 0);
  static_assert(BM * S % T == 0 && BN * S % T == 0 && T % S == 0, "staging must divide evenly");
};

// Copies the input rows 0 .. rows - 1 of a tile's region to LDS planes [word][pixel]; taps outside the image are
// +1 in every real channel.  EVEN: words per pixel in pairs, 16-byte loads.  A lane keeps one word pair of one
// region column, the workgroup's waves walk the rows, and up to BATCH loads are in flight per lane; what depends
// on the row is decoded once, lane i for the wave's i-th row, and read back as scalars.  between() runs after the
// first batch of loads has been issued: work that the loads' latency hides.
template <int T, bool EVEN, class Between>
__device__ __forceinline__ void load_region(const ConvGeom &g, const HaloGeom &hg, char *sReg, int i0, int ih_first, int rows0,
                                            int rows, uint64_t part, int wave, int lane, const Between &between) {
  constexpr int NW = T / 64, BATCH = 8;
  const int rowitems = hg.Wp * hg.ppp;
  const uint32_t rowbytes = (uint32_t)g.W * (uint32_t)g.Cw * 8u;  // host: below 2^32
  bool pending = true;
#pragma unroll 1
  for (int rr = wave; rr < rows; rr += BATCH * NW) {
    // lane i: the wave's i-th row of this batch
    uint32_t alo, ahi, aok;
    {
      const int r = min(rr + lane * NW, rows - 1);
      const int t = max(r - rows0, 0);  // rows past the first image's: `full` rows of each image that follows
      const uint32_t h = __umulhi((uint32_t)t, hg.divFull.mul);
      const int k = (int)((h + (((uint32_t)t - h) >> 1)) >> hg.divFull.shift);  // host: full >= 2
      const bool first = r < rows0;
      const int ih = first ? ih_first + r : t - k * hg.full - g.pH;
      const uint32_t img = (uint32_t)(first ? i0 : i0 + 1 + k);
      const bool ok = ih >= 0 && ih < g.H;
      // host: image rows number fewer than 2^31
      const uint64_t a = reinterpret_cast<uint64_t>(g.act) + (uint64_t)(img * (uint32_t)g.H + (uint32_t)(ok ? ih : 0)) * rowbytes;
      alo = (uint32_t)a;
      ahi = (uint32_t)(a >> 32);
      aok = (uint32_t)(__ballot(ok) & ((1u << BATCH) - 1u));
    }
#pragma unroll 1
    for (int ch = 0; ch < hg.nch; ++ch) {
      const int idx = ch * 64 + lane;
      const uint32_t px = fdiv_sel((uint32_t)idx, hg.divPpp), cw = 2u * ((uint32_t)idx - px * (uint32_t)hg.ppp);
      const int iw = (int)px - g.pW;
      const bool cok = iw >= 0 && iw < g.W;
      const bool two = EVEN || cw + 1u < (uint32_t)g.Cw;
      const uint32_t off = ((cok ? (uint32_t)iw : 0u) * (uint32_t)g.Cw + cw) * 8u;
      u32x4 v[BATCH];
#pragma unroll
      for (int b = 0; b < BATCH; ++b) {
        if (b > 0 && rr + b * NW >= rows) break;  // uniform
        const char *src = reinterpret_cast<const char *>(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)ahi, b) << 32) |
                                                         (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)alo, b));
        if constexpr (EVEN) {
          v[b] = *reinterpret_cast<const u32x4 *>(src + off);
        } else {
          v[b].lo = *reinterpret_cast<const u32x2 *>(src + off);
          v[b].hi = *reinterpret_cast<const u32x2 *>(src + off + (two ? 8u : 0u));
        }
      }
      if (pending) {
        pending = false;
        between();
      }
      const uint64_t p0 = cw + 1u == (uint32_t)g.Cw ? part : ~0ull, p1 = cw + 2u == (uint32_t)g.Cw ? part : ~0ull;
      char *const dst = sReg + cw * hg.plane + px * 8u + (uint32_t)rr * (uint32_t)hg.Wp * 8u;
#pragma unroll
      for (int b = 0; b < BATCH; ++b) {
        if (b > 0 && rr + b * NW >= rows) break;  // uniform
        const bool ok = cok && ((aok >> b) & 1u);
        u32x4 x = v[b];
        x.x = ok ? x.x : (uint32_t)p0;
        x.y = ok ? x.y : (uint32_t)(p0 >> 32);
        x.z = ok ? x.z : (uint32_t)p1;
        x.w = ok ? x.w : (uint32_t)(p1 >> 32);
        char *const d = dst + (uint32_t)(b * NW) * (uint32_t)hg.Wp * 8u;
        if (idx < rowitems) {
          *reinterpret_cast<u32x2 *>(d) = x.lo;
          if (two) *reinterpret_cast<u32x2 *>(d + hg.plane) = x.hi;
        }
      }
    }
  }
  if (pending) between();  // a wave without rows
}

template <int WTM, int WTN, int WGM, int WGN, int GM, int EMODE, int MINW, bool BITS>
__global__ __launch_bounds__(64 * WGM * WGN, MINW) void xnor_gemm_fp4_kernel(GemmParams p) {
  using Cfg = Fp4Cfg<WTM, WTN, WGM, WGN, GM, BITS>;
  // BITS: 0 / 1 codes (see launch_gemm_fp4); the set bits of rows and columns are counted as they are staged
  using Codes = typename std::conditional<BITS, BitCodes, SignCodes>::type;
  constexpr int T = Cfg::T, BM = Cfg::BM, BN = Cfg::BN, PA = Cfg::PA, PB = Cfg::PB, S = Cfg::S;
  constexpr bool POOL = EMODE == EM_POOL;
  // columns of a wave dealt to (block j, lane l): WTN * l + j, so that a lane's columns are consecutive; signs
  // from an LDS region take 32 * j + l (lanes on consecutive pixels: no bank conflicts), and so do 4-byte stores
  constexpr bool DEALT = EMODE != EM_MAPS_ONE && !(GM == GM_HALO && EMODE == EM_SIGN);
  // One dword of every 64-byte line of the arguments, requested at once: they arrive in one memory round trip
  // instead of one per group of arguments that the code below happens to need next (each about 500 cycles).
  {
    const cu32_args ka = (cu32_args)__builtin_amdgcn_kernarg_segment_ptr();
    constexpr int LINES = (int)((sizeof(GemmParams) + 63) / 64);
    static_assert(LINES == 6, "list every line below");
    asm volatile("" ::"s"(ka[0]), "s"(ka[16]), "s"(ka[32]), "s"(ka[48]), "s"(ka[64]), "s"(ka[80]));
  }
  extern __shared__ __attribute__((aligned(16))) char smem[];
  float *const sSc = reinterpret_cast<float *>(smem + Cfg::STAGE_BYTES);
  float *const sBi = sSc + BM;
  uint32_t *const sCol = reinterpret_cast<uint32_t *>(sBi + BM);      // GM_HALO: region offset of every column
  float *const sRow = sBi + BM;                                         // BITS: parts of rows, then of columns
  static_assert(!BITS || (GM == GM_EXPL16 && EMODE < EM_SIGN), "sRow lies where sCol does; only maps know the corrections");
  char *const sReg = smem + Cfg::FIXED_BYTES;                           // GM_HALO: [word][pixel] 8-byte words
  uint32_t *const sOff = reinterpret_cast<uint32_t *>(sReg + p.halo.bytes);  // GM_HALO: distance of every word of a row
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;

  // ---- tile: row tiles of one column tile are neighbours, and each XCD gets a contiguous run ----------
  const uint32_t nwg = gridDim.x;
  uint32_t bid = blockIdx.x;
  {
    const uint32_t q = nwg >> 3, r = nwg & 7u, xcd = bid & 7u, i = bid >> 3;
    bid = xcd * q + min(xcd, r) + i;
  }
  const int ni = (int)fdiv_sel(bid, p.divTilesM), mi = (int)(bid - (uint32_t)ni * (uint32_t)p.tilesM);
  const int m0 = mi * BM, n0 = ni * BN;
  const ConvGeom &g = p.g;
  const HaloGeom &hg = p.halo;

  // ---- staging: thread t moves piece t % S of rows t / S, + T / S, ... --------------------------------
  const int pc = tid % S;           // this thread's piece of every stage
  const int row0 = tid / S;
  const int npieces = (p.Kw64 + 1) >> 1;
  const int nst = (npieces + S - 1) / S;
  uint32_t aoff[PA];                // byte offset of the row (host: operand A is at most 4 GiB)
#pragma unroll
  for (int i = 0; i < PA; ++i) aoff[i] = (uint32_t)min(m0 + row0 + i * (T / S), p.M - 1) * ((uint32_t)p.lda32 * 4u);
  u32x4 ra[PA];
  const bool a16 = GM == GM_EXPL16 || (GM >= GM_HALO && p.b_vec16);  // uniform: whole 16-byte pieces of A
  auto load_a = [&](int st) {
    const int e = st * S + pc;  // piece of the row: words 2e, 2e + 1
    const char *ab = reinterpret_cast<const char *>(p.A);
    if (a16) {
      const uint32_t eo = (uint32_t)min(e, (p.Kw64 >> 1) - 1) * 16u;
#pragma unroll
      for (int i = 0; i < PA; ++i) ra[i] = *reinterpret_cast<const u32x4 *>(ab + (aoff[i] + eo));
    } else {
      const uint32_t wo = (uint32_t)max(min(2 * e, p.Kw64 - 2), 0) * 8u;
      load_pieces_any<PA>(ra, p.Kw64 > 1, [&](int i) { return ab + (size_t)aoff[i] + wo; });
    }
  };
  load_a(0);

  // staged B (explicit rows, or patches gathered word by word)
  constexpr int NB = PB > 0 ? PB : 1;
  const char *brow[NB];   // explicit row, or the pixel's image
  int bih[NB], biw[NB];   // GM_ANY: pixel under tap (0, 0)
  u32x4 rb[NB];
#pragma unroll
  for (int i = 0; i < PB; ++i) {
    const int n = min(n0 + row0 + i * (T / S), p.N - 1);  // columns past N recompute column N - 1
    if constexpr (GM == GM_ANY) {
      uint32_t img, oh, ow;
      column_pixel(g, (uint32_t)n, POOL, img, oh, ow);
      brow[i] = reinterpret_cast<const char *>(g.act + (size_t)img * (size_t)g.H * (size_t)g.W * (size_t)g.Cw);
      bih[i] = (int)oh * g.sH - g.pH;
      biw[i] = (int)ow * g.sW - g.pW;
    } else {
      brow[i] = reinterpret_cast<const char *>(p.B) + (size_t)n * (size_t)p.ldb * 8u;
    }
  }
  const uint64_t part = (g.C & 63) ? (1ull << (g.C & 63)) - 1ull : ~0ull;  // real channels of a tap's last word
  auto load_b = [&](int st) {
    const int e = st * S + pc;
    if constexpr (GM == GM_EXPL16) {
      const uint32_t eo = (uint32_t)min(e, (p.Kw64 >> 1) - 1) * 16u;
#pragma unroll
      for (int i = 0; i < PB; ++i) rb[i] = *reinterpret_cast<const u32x4 *>(brow[i] + eo);
    } else if constexpr (GM == GM_EXPL8) {
      const uint32_t wo = (uint32_t)max(min(2 * e, p.Kw64 - 2), 0) * 8u;
      load_pieces_any<PB>(rb, p.Kw64 > 1, [&](int i) { return brow[i] + wo; });
    } else if constexpr (GM == GM_ANY) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t w = (uint32_t)min(2 * e + h, p.Kw64 - 1);
        const uint32_t tap = fdiv(w, g.divCw), cw = w - tap * (uint32_t)g.Cw;
        const uint32_t kh = fdiv(tap, g.divKW), kw = tap - kh * (uint32_t)g.kW;
        const uint64_t pad = cw + 1u == (uint32_t)g.Cw ? part : ~0ull;  // taps outside the image: +1 in every channel
#pragma unroll
        for (int i = 0; i < PB; ++i) {
          const int ih = bih[i] + (int)kh, iw = biw[i] + (int)kw;
          u32x2 v = {(uint32_t)pad, (uint32_t)(pad >> 32)};
          if (ih >= 0 && ih < g.H && iw >= 0 && iw < g.W)
            v = *reinterpret_cast<const u32x2 *>(brow[i] + (((size_t)ih * (size_t)g.W + (size_t)iw) * (size_t)g.Cw + cw) * 8u);
          if (h == 0) rb[i].lo = v;
          else rb[i].hi = v;
        }
      }
    }
  };
  load_b(0);
  // bits past the end of the row become 0 in both operands (last stage only)
  auto mask_stage = [&](int st) {
    const int e = st * S + pc;
    u32x4 m;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const int left = p.Kbits - (4 * e + d) * 32;  // bits of this dword that exist (host: Kbits < 2^24)
      m[d] = left >= 32 ? 0xffffffffu : (left <= 0 ? 0u : (1u << left) - 1u);
    }
    const bool shifted = 2 * e == p.Kw64 - 1 && e > 0;  // a row's odd last word, read as the second of its piece
    if (!a16 && shifted) {
#pragma unroll
      for (int i = 0; i < PA; ++i) ra[i].lo = ra[i].hi;
    }
    if (GM == GM_EXPL8 && shifted) {
#pragma unroll
      for (int i = 0; i < PB; ++i) rb[i].lo = rb[i].hi;
    }
#pragma unroll
    for (int i = 0; i < PA; ++i) ra[i] &= m;
#pragma unroll
    for (int i = 0; i < PB; ++i) rb[i] &= m;
  };
  // registers -> LDS buffer; T / S rows apart is a constant distance in LDS
  constexpr int RPT = T / S;  // rows between a thread's pieces
  static_assert(RPT % 32 == 0 && (PB == 0 || (32 * WTN) % RPT == 0 || RPT % (32 * WTN) == 0), "constant LDS distances");
  char *const wrA = smem + (pc * Cfg::P16 + (row0 >> 5) * Cfg::R16 + (row0 & 31)) * 16;
  const int col0 = row0 % (32 * WTN);
  const int unitB = DEALT ? (BM / 32 + (row0 / (32 * WTN)) * WTN + col0 % WTN) * Cfg::R16 + col0 / WTN
                          : (BM / 32 + (row0 >> 5)) * Cfg::R16 + (row0 & 31);
  char *const wrB = smem + (pc * Cfg::P16 + unitB) * 16;
  // set bits of this thread's pieces, counted on the way; what lies past the row's end is 0
  uint32_t cntA[PA], cntB[NB];
#pragma unroll
  for (int i = 0; i < PA; ++i) cntA[i] = 0u;
#pragma unroll
  for (int i = 0; i < NB; ++i) cntB[i] = 0u;
  auto count = [](const u32x4 &v, uint32_t n) {
    n += __popc(v.x);
    n += __popc(v.y);
    n += __popc(v.z);
    return n + __popc(v.w);
  };
  auto store_piece = [&](int i, uint32_t buf) {  // i < PA: A, else B
    if (i < PA) {
      if constexpr (BITS) cntA[i] = count(ra[i], cntA[i]);
      *reinterpret_cast<u32x4 *>(wrA + buf + i * (RPT / 32) * Cfg::R16 * 16) = ra[i];
    } else if (i < PA + PB) {
      if constexpr (BITS) cntB[i - PA] = count(rb[i - PA], cntB[i - PA]);
      const int c = (i - PA) * RPT;  // columns from the first one
      const int u = DEALT ? (c / (32 * WTN)) * WTN * Cfg::R16 + (c % (32 * WTN)) / WTN : (c / 32) * Cfg::R16;
      *reinterpret_cast<u32x4 *>(wrB + buf + u * 16) = rb[i - PA];
    }
  };
  // the tile's per-row scale / bias, requested now and written to LDS below; rows past M get the constants whose
  // sign bit is 0, and in maps, where they are row M - 1 once more, that row's
  static_assert(BM <= T, "one row per thread");
  constexpr bool MAPS = EMODE < EM_SIGN;
  const bool affine = !MAPS || (p.Y && p.axis == BNN_CH_ROW);  // uniform
  float fsc = 0.0f, fbi = -1.0f;
  if (affine && tid < BM && (MAPS || m0 + tid < p.M)) {
    fsc = p.scale[min(m0 + tid, p.M - 1)];
    fbi = p.bias[min(m0 + tid, p.M - 1)];
  }

  // ---- GM_HALO: the tile's input region -> LDS -----------------------------------------------------------
  // A unit is an output row (pooled: a pair of them).  An image's units of this tile need consecutive input
  // rows; images follow each other in LDS.  Region row 0 is input row ih_first of image i0.
  if constexpr (GM == GM_HALO) {
    // lane 0 decodes the tile's first column, the others its last one
    const int nlast = min(n0 + BN, p.N) - 1;
    uint32_t cimg, coh, cow;
    column_pixel(g, (uint32_t)(lane == 0 ? n0 : nlast), POOL, cimg, coh, cow);
    const int i0 = __builtin_amdgcn_readlane((int)cimg, 0), i1 = __builtin_amdgcn_readlane((int)cimg, 1);
    const int u0 = __builtin_amdgcn_readlane((int)coh, 0) >> (POOL ? 1 : 0), u1 = __builtin_amdgcn_readlane((int)coh, 1) >> (POOL ? 1 : 0);
    const int ulast0 = i0 == i1 ? u1 : hg.units - 1;           // last unit of the first image
    const int rows0 = (ulast0 - u0) * hg.ustep + hg.uspan;      // its input rows
    const int rows = i0 == i1 ? rows0 : rows0 + (i1 - i0 - 1) * hg.full + u1 * hg.ustep + hg.uspan;
    const int ih_first = u0 * hg.ustep - g.pH;
    auto tables = [&]() {
      // distance of every word of a patch row from the same lane's pixel under tap (0, 0)
      for (int w = tid; w < 2 * npieces; w += T) {
        const uint32_t tap = fdiv_sel((uint32_t)w, g.divCw), cw = (uint32_t)w - tap * (uint32_t)g.Cw;
        const uint32_t kh = fdiv_sel(tap, g.divKW), kw = tap - kh * (uint32_t)g.kW;
        sOff[w] = w < p.Kw64 ? cw * hg.plane + (kh * (uint32_t)hg.Wp + kw) * 8u : (uint32_t)g.Cw * hg.plane;
      }
      // rows of an odd number of words end in the middle of a piece: the missing word is read from a plane of zeros
      if (p.Kw64 & 1)
        for (uint32_t i = (uint32_t)tid * 8u; i < hg.plane; i += T * 8u)
          *reinterpret_cast<u32x2 *>(sReg + (uint32_t)g.Cw * hg.plane + i) = u32x2{0u, 0u};
      // region offset of every column's pixel under tap (0, 0)
      for (int c = tid; c < BN; c += T) {
        uint32_t img, oh, ow;
        column_pixel(g, (uint32_t)min(n0 + c, p.N - 1), POOL, img, oh, ow);
        // row of the pixel's tap (0, 0) inside its image's part of the region
        const int r = (int)img == i0 ? (int)oh * g.sH - u0 * hg.ustep
                                     : rows0 + ((int)img - i0 - 1) * hg.full + (int)oh * g.sH;
        sCol[c] = (uint32_t)(r * hg.Wp + (int)ow * g.sW) * 8u;
      }
    };
    if ((g.Cw & 1) == 0) load_region<T, true>(g, hg, sReg, i0, ih_first, rows0, rows, part, wave, lane, tables);
    else load_region<T, false>(g, hg, sReg, i0, ih_first, rows0, rows, part, wave, lane, tables);
  }
  if (affine && tid < BM) {
    sSc[tid] = fsc;
    sBi[tid] = fbi;
  }

  // SignCodes: the result, less the padding.  BitCodes count S, C = K - 2 * (set bits of the row) - 2 * (set bits of the
  // column) + 4 S: the column's part is added at the end, the row's in the epilogue.
  Fp4Acc<WTM, WTN> acc;
  acc.init(BITS ? 0.0f : -(float)(npieces * 128 - p.Kformula));

  // Stage st sits in LDS buffer st % 3.  It is written during piece 0 of the stage before it, a barrier stands
  // between pieces 1 and 2, and piece 3 already reads ahead into the next stage; the buffer that a stage is
  // written to was last read two stages ago, before the previous barrier.
  constexpr uint32_t BUF = S * Cfg::P16 * 16;  // bytes of a buffer
  const uint32_t fbase = (uint32_t)(lane & 31) * 16u + (uint32_t)(lane >> 5) * 8u;
  const char *const fragA = smem + fbase + (uint32_t)(wm * WTM * Cfg::R16) * 16u;
  const char *const fragB = smem + fbase + (uint32_t)((BM / 32 + wn * WTN) * Cfg::R16) * 16u;
  if (nst == 1) mask_stage(0);
#pragma unroll
  for (int i = 0; i < PA + PB; ++i) store_piece(i, 0u);
  load_a(1);  // past the last stage: its last piece again, not used
  load_b(1);
  __syncthreads();
  const char *regB[WTN];
  const uint32_t *const offp = sOff + (lane >> 5);
  uint32_t woff = 0u;  // of a region: distance of this lane's word of the piece that is read next
  if constexpr (GM == GM_HALO) {
#pragma unroll
    for (int j = 0; j < WTN; ++j)
      regB[j] = sReg + sCol[wn * WTN * 32 + (DEALT ? WTN * (lane & 31) + j : 32 * j + (lane & 31))];
  }
  // fragment f of a piece: bits of the wave's row blocks, then of its column blocks
  auto read_frag = [&](int f, uint32_t plane, u32x2(&a)[WTM], u32x2(&b)[WTN]) {
    if (f < WTM) a[f] = *reinterpret_cast<const u32x2 *>(fragA + plane + f * Cfg::R16 * 16);
    else if (GM == GM_HALO) b[f - WTM] = *reinterpret_cast<const u32x2 *>(regB[f - WTM] + woff);
    else b[f - WTM] = *reinterpret_cast<const u32x2 *>(fragB + plane + (f - WTM) * Cfg::R16 * 16);
  };
  v8i ea[WTM], eb[WTN];         // expanded operands of the next 64 values
  uint32_t ya[WTM], yb[WTN];    // bits of the 64 values after them
  {
    if constexpr (GM == GM_HALO) woff = offp[0];
    u32x2 a[WTM], b[WTN];
#pragma unroll
    for (int f = 0; f < WTM + WTN; ++f) read_frag(f, 0u, a, b);
    if constexpr (GM == GM_HALO) {
      woff = offp[npieces > 1 ? 2 : 0];
    }
#pragma unroll
    for (int i = 0; i < WTM; ++i) {
      ea[i] = Codes::template a<true>(a[i].x);
      ya[i] = a[i].y;
    }
#pragma unroll
    for (int j = 0; j < WTN; ++j) {
      eb[j] = Codes::template b<true>(b[j].x);
      yb[j] = b[j].y;
    }
  }
  uint32_t rbuf = 0u;  // byte offset of the stage's buffer
#pragma unroll 1
  for (int st = 0; st < nst; ++st) {
    const uint32_t wbuf = rbuf == 2 * BUF ? 0u : rbuf + BUF;  // the next stage's
    if (st + 2 == nst || (BITS && st + 1 == nst)) mask_stage(st + 1);  // past the last stage: all 0, nothing more is counted
#pragma unroll
    for (int k = 0; k < S; ++k) {
      const int q = st * S + k;
      if (k > 0 && q >= npieces) break;  // uniform; the first piece of a stage always exists
      if (k == S / 2) __syncthreads();
      constexpr int MM = WTM * WTN, FR = WTM + WTN;
      u32x2 na[WTM], nb[WTN];  // the next piece (past the last one: whatever is there, not used)
      const uint32_t next = k + 1 < S ? rbuf + (k + 1) * Cfg::P16 * 16 : wbuf;
      v8i fa[WTM], fb[WTN];
      multiply_and_expand<Codes, WTM, WTN>(acc, ea, eb, ya, yb, fa, fb, [&](int m) {
#pragma unroll
        for (int f = m * FR / MM; f < (m + 1) * FR / MM; ++f) read_frag(f, next, na, nb);
      });
      uint32_t xa[WTM], xb[WTN];
#pragma unroll
      for (int i = 0; i < WTM; ++i) {
        xa[i] = na[i].x;
        ya[i] = na[i].y;
      }
#pragma unroll
      for (int j = 0; j < WTN; ++j) {
        xb[j] = nb[j].x;
        yb[j] = nb[j].y;
      }
      multiply_and_expand<Codes, WTM, WTN>(acc, fa, fb, xa, xb, ea, eb, [&](int m) {
        if (k == 0) {  // the next stage's pieces, from registers
#pragma unroll
          for (int i = m * (PA + PB) / MM; i < (m + 1) * (PA + PB) / MM; ++i) store_piece(i, wbuf);
        }
        if (k == 1 && m == 0) {
          load_a(st + 2);
          load_b(st + 2);
        }
        if (GM == GM_HALO && m == MM / 2) woff = offp[2 * min(q + 2, npieces - 1)];
      });
    }
    rbuf = wbuf;
  }

  if constexpr (BITS) {
    // the four threads that staged a row add up its bits
    auto sum4 = [](uint32_t n) {
      n += (uint32_t)__builtin_amdgcn_mov_dpp((int)n, 0xB1, 0xF, 0xF, true);
      return n + (uint32_t)__builtin_amdgcn_mov_dpp((int)n, 0x4E, 0xF, 0xF, true);
    };
    static_assert(S == 4, "four threads to a row");
#pragma unroll
    for (int i = 0; i < PA; ++i) {
      const uint32_t n = sum4(cntA[i]);
      if (pc == 0) sRow[row0 + i * RPT] = -2.0f * (float)n;
    }
#pragma unroll
    for (int i = 0; i < PB; ++i) {
      const uint32_t n = sum4(cntB[i]);
      if (pc == 0) sRow[BM + row0 + i * RPT] = 0.25f * (float)p.Kformula - 0.5f * (float)n;
    }
    __syncthreads();
  }
  settle(acc);
  if constexpr (BITS) {  // the columns' part
#pragma unroll
    for (int j = 0; j < WTN; ++j) {
      const float c = sRow[BM + wn * WTN * 32 + (DEALT ? WTN * (lane & 31) + j : 32 * j + (lane & 31))];
#pragma unroll
      for (int i = 0; i < WTM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc.v[i][j][r] += c;
    }
  }
  const int mw = m0 + 32 * WTM * wm, nw = n0 + 32 * WTN * wn;
  const float *sc = sSc + 32 * WTM * wm, *bi = sBi + 32 * WTM * wm;
  if constexpr (MAPS) store_maps<WTM, WTN, EMODE, BITS>(p, acc, mw, nw, lane, sc, bi, sRow + 32 * WTM * wm);
  else if constexpr (EMODE == EM_SIGN) store_signs<WTM, WTN, DEALT>(p, acc, mw, nw, lane, sc, bi);
  else store_signs_pooled<WTM, WTN>(p, acc, mw, nw, lane, sc, bi);
}

// ---- host side -----------------------------------------------------------------------------------------
template <int WTM, int WTN, int WGM, int WGN, int GM, int EMODE, int MINW, bool BITS = false>
static bnn_status launch_fp4(GemmParams &p, hipStream_t s) {
  using Cfg = Fp4Cfg<WTM, WTN, WGM, WGN, GM, BITS>;
  p.tilesM = (p.M + Cfg::BM - 1) / Cfg::BM;
  const int64_t tn = ((int64_t)p.N + Cfg::BN - 1) / Cfg::BN;
  const int64_t blocks = p.tilesM * tn;
  if (blocks > 0x7fffffffLL) return BNN_ERR_UNSUPPORTED;
  p.tilesN = (int)tn;
  p.divTilesM = FastDiv((uint32_t)p.tilesM);
  const size_t lds = Cfg::FIXED_BYTES + (GM == GM_HALO ? (size_t)p.halo.bytes + (size_t)(p.Kw64 + 1) / 2 * 8 : 0);
  ProfScope ps(KID_XNOR_GEMM_FP4, s);
  hipLaunchKernelGGL((xnor_gemm_fp4_kernel<WTM, WTN, WGM, WGN, GM, EMODE, MINW, BITS>), dim3((unsigned)blocks),
                     dim3(Cfg::T), lds, s, p);
  return launch_status();
}

template <int WTM, int WTN, int WGM, int WGN, int GM, int MINW, bool BITS = false>
static bnn_status launch_fp4_maps(GemmParams &p, hipStream_t s) {
  if (!p.colperm) return launch_fp4<WTM, WTN, WGM, WGN, GM, EM_MAPS_ONE, MINW, BITS>(p, s);
  return p.nt_store ? launch_fp4<WTM, WTN, WGM, WGN, GM, EM_MAPS_NT, MINW, BITS>(p, s)
                    : launch_fp4<WTM, WTN, WGM, WGN, GM, EM_MAPS_VEC, MINW, BITS>(p, s);
}

// Upper bound of the number of aligned-grid cells of length `cell` that a run of `len` columns starting at a
// multiple of `len` touches.
static int64_t cells_touched(int64_t len, int64_t cell) {
  if (len % cell == 0) return len / cell;
  if (cell % len == 0) return 1;
  return (len - 2) / cell + 2;
}

// Fills p.halo for column tiles of bn; whether the region (and the table of word distances) is of a size to keep in LDS
// and the image's rows are of a length that the copy into it can step over.  rows: upper bound of a tile's input rows.
bool halo_region(GemmParams &p, int bn, bool pool, int64_t &rows) {
  const ConvGeom &g = p.g;
  HaloGeom &h = p.halo;
  const int us = pool ? 2 : 1;
  const int64_t Wp = (int64_t)(g.OW - 1) * g.sW + g.kW, units = g.OH / us, ustep = (int64_t)us * g.sH,
                uspan = (int64_t)(us - 1) * g.sH + g.kH;
  const int64_t full = (units - 1) * ustep + uspan;
  const int64_t ucols = (int64_t)us * us * (g.OW / us);
  const int64_t nu = cells_touched(bn, ucols);
  const int64_t ni = std::min(nu, cells_touched(bn, ucols * units));
  // the rows of nu units cut into 1 .. ni images: linear in the number of images, so largest at an end
  rows = std::max((nu - 1) * ustep + uspan, (nu - ni) * ustep + ni * uspan);
  const int64_t ppp = (g.Cw + 1) / 2;
  if (p.Kw64 > 4096 || rows > 4096 || Wp > 4096 || ppp > 64 || full < 2 || full > (1 << 24)) return false;
  // load_region's row pitch is a 32-bit number of bytes.  Wp does not bound it: with one output column the image may be
  // any number of columns wider than what its taps read.
  if ((int64_t)g.W * g.Cw * 8 > 0xffffffffLL) return false;
  // plane stride in 8-byte words: the word pairs of one pixel that neighbouring lanes write fall on distinct banks
  const int64_t plane8 = (rows * Wp + 31) / 32 * 32 + std::max<int64_t>(1, 16 / ppp);
  const int64_t bytes = (plane8 * 8 * (g.Cw + (p.Kw64 & 1)) + 15) / 16 * 16;
  if (bytes > 100 * 1024) return false;
  h.Wp = (int)Wp; h.units = (int)units; h.ustep = (int)ustep; h.uspan = (int)uspan; h.full = (int)full;
  h.ppp = (int)ppp;
  h.nch = (int)((Wp * ppp + 63) / 64);
  h.plane = (uint32_t)(plane8 * 8);
  h.bytes = (uint32_t)bytes;
  h.divPpp = FastDiv((uint32_t)h.ppp);
  h.divFull = FastDiv((uint32_t)h.full);
  return true;
}

// Signs leave from any shape; maps, and everything on explicit rows, from the two shapes of 64 x 64 outputs per wave
// on four waves that win there (see below).
template <int WTM, int WTN, int WGM, int WGN, int MINW, bool MAPS>
static bnn_status launch_fp4_shape(GemmParams &p, int bmode, int emode, hipStream_t s, bool region) {
  using H = Fp4Cfg<WTM, WTN, WGM, WGN, GM_HALO>;
  if constexpr (MAPS) {
    if (bmode == 0) {
      const bool v16 = p.Kw64 % 2 == 0 && p.lda32 % 4 == 0 && p.ldb % 2 == 0;
      return v16 ? launch_fp4_maps<WTM, WTN, WGM, WGN, GM_EXPL16, MINW>(p, s)
                 : launch_fp4_maps<WTM, WTN, WGM, WGN, GM_EXPL8, MINW>(p, s);
    }
  }
  p.b_vec16 = p.Kw64 % 2 == 0 && p.lda32 % 4 == 0;
  int64_t rows;
  const bool halo = region && halo_region(p, H::BN, p.g.pool != 0, rows);
  if constexpr (MAPS) {
    if (emode == 0)
      return halo ? launch_fp4_maps<WTM, WTN, WGM, WGN, GM_HALO, MINW>(p, s)
                  : launch_fp4_maps<WTM, WTN, WGM, WGN, GM_ANY, MINW>(p, s);
  }
  if (p.g.pool)
    return halo ? launch_fp4<WTM, WTN, WGM, WGN, GM_HALO, EM_POOL, MINW>(p, s)
                : launch_fp4<WTM, WTN, WGM, WGN, GM_ANY, EM_POOL, MINW>(p, s);
  return halo ? launch_fp4<WTM, WTN, WGM, WGN, GM_HALO, EM_SIGN, MINW>(p, s)
              : launch_fp4<WTM, WTN, WGM, WGN, GM_ANY, EM_SIGN, MINW>(p, s);
}

bool fp4_applicable(const GemmParams &p) {
  // exact fp32 counts: every partial sum is below 2^24 in magnitude
  return p.Kw64 < (1 << 18) - 2;
}

// The 128 x 128 tile of bits (BitCodes): rows of whole 16-byte pieces, partial sums that are multiples of 1/4 exact below 2^22.
static bool bits_applicable(const GemmParams &p, int bmode) {
  return bmode == 0 && p.Kw64 % 2 == 0 && p.lda32 % 4 == 0 && p.ldb % 2 == 0 && p.Kw64 < (1 << 16) - 2;
}

// Workgroups that a compute unit holds with their input regions in LDS, at most three; 0: the region is not for LDS.
// rows: upper bound of a tile's input rows.
template <int WTM, int WTN, int WGM, int WGN>
static int held_with_regions(GemmParams &p, int64_t &rows) {
  using H = Fp4Cfg<WTM, WTN, WGM, WGN, GM_HALO>;
  if (!halo_region(p, H::BN, p.g.pool != 0, rows)) return 0;
  return std::min(3, 160 * 1024 / (H::FIXED_BYTES + (int)p.halo.bytes + (p.Kw64 + 1) / 2 * 8));
}

// Tile of a convolution, and whether its input region is kept in LDS (`region`: allowed to).
static int conv_shape(GemmParams &p, int emode, bool &region) {
  const ConvGeom &g = p.g;
  auto count = [&](int bm, int bn) { return (((int64_t)p.M + bm - 1) / bm) * (((int64_t)p.N + bn - 1) / bn); };
  auto per_unit = [&](int bm, int bn) { return (count(bm, bn) + p.n_cu - 1) / p.n_cu; };
  const int64_t n = per_unit(128, 128), taps = (int64_t)g.kH * g.kW, steps = (int64_t)g.sH * g.sW;
  // No pixel under two taps: a region's pixels are then copied to be read once, and the ones that the stride skips are copied
  // for nothing (1 x 1 by stride 2, 128 x 128 tiles gathering against holding regions: 512 x 4096 x 704 20.9 us against 26.2,
  // 128 x 86016 x 192 packed 10.1 against 12.0).  Where it skips none the copy pays when its lanes, a region row's word
  // pairs at a time, are busy (2 x 2 by stride 2, 256 channels of 32 x 32: 23.6 against 20.9; 192 channels of 8 x 8 16.4
  // against 19.8).  Without a stride it is the copy's latency that counts, while there are few tiles (1 x 1 of 128
  // channels, 1.8 tiles a unit: 5.4 against 6.2; 512 channels, 5.6 tiles: 16.1 against 14.4).
  const bool once = taps < steps || (taps == steps && (steps > 1 ? halo_lanes_idle(g) : emode != 0 && n <= 2));
  // Regions that leave a unit one workgroup where it has several tiles to do cost more than gathering, which a stride of 2
  // makes cheap (3 x 3 by stride 2, 704 channels, three 128 x 128 tiles: 40.4 against 53.7; 512 channels, two of 128 x 256:
  // 34.5 against 37.3); with more taps a pixel it takes the third tile (3 x 3, 1024 channels of 56 x 56: 89.9 against
  // 102.8 with five, but 65.6 against 62.2 on two of 128 x 256).
  auto gather = [&](int held, int64_t tiles, bool third) {
    return held == 0 || once || (held == 1 && tiles >= 2 && (taps < 4 * steps || (third && tiles >= 3)));
  };
  auto held_if = [&](int held) { return region ? held : 0; };
  int64_t rows = 0;
  if (p.M <= 64) {
    // one row of tiles to fill (64 channels, 100352 pixels, K = 576: 7.0 us against 9.0 to 10.9)
    const int held = held_if(held_with_regions<2, 2, 1, 4>(p, rows));
    const int64_t tiles = per_unit(64, 256);
    region = once ? held >= std::min<int64_t>(tiles, 3) : !gather(held, tiles, false);
    return 3;
  }
  const int held128 = held_if(held_with_regions<2, 2, 2, 2>(p, rows));
  if (emode == 0) {
    // Stores of maps want many workgroups in different phases: 64 x 256 tiles while every unit gets two of them and their
    // larger regions do not keep workgroups out (256 x 200704 x 2304 fp32 maps 64.2 us against 68.1 on 128 x 128 and 67.9 on
    // 128 x 256 by four waves; 128 x 131072 x 1152: 16.6, 17.3, 17.7; but 3 x 3 by stride 2 from 512 channels of 8 x 8, one
    // against two held: 119 against 74), else 128 x 128 (512 x 4096 x 2304: 9.9 against 10.3).
    if (!once && count(64, 256) >= 2 * (int64_t)p.n_cu) {
      const int held = held_if(held_with_regions<2, 2, 1, 4>(p, rows));
      if (held > 0 && held >= held128) {
        region = !gather(held, per_unit(64, 256), false);
        return 3;
      }
    }
    region = !gather(held128, n, true);
    return 2;
  }
  // Signs leave little to store, so what counts is expansions per matrix instruction and full rounds of tiles.  128 x 256
  // tiles of 64 x 128 per wave need the fewest expansions, two of them to a compute unit; 128 x 128 tiles fit three times and
  // fill odd counts up to five.  3 x 3 layers, 128 x 128 tiles against 128 x 256, by the number of 128 x 128 tiles per unit:
  // 0.5 9.9 us against 12.9; 1.6 12.3 against 11.6; 2.0 17.5 against 16.0 (pooled 19.5 against 18.4); 2.4 15.9 against 18.5 and
  // 25.3 against 30.1; 3.6 24.0 against 21.8; 4.4 21.2 against 23.3 and 23.7 against 24.8; 5.2 28.0 against 25.0; from there
  // the larger one (7.8 35.6 against 30.2), but for a few per cent either way where the last round is short.
  if (n <= 5 && n % 2 == 1) {
    region = !gather(held128, n, true);
    return 2;
  }
  const int64_t tiles = per_unit(128, 256);
  region = !gather(held_if(held_with_regions<2, 4, 2, 2>(p, rows)), tiles, false);
  // One 128 x 256 tile to a unit: eight waves gather faster than four (3 x 3 by stride 2, 1024 channels: 38.1 against 40.6).
  // Regions they copy faster, four multiply faster, so it is the rows copied (many where the maps are small) against the
  // words of the reduction.  By 197 layers with one tile to a unit and 59 with two, eight waves against four: 3 x 3 by stride 2 of
  // 100 channels of 2 x 2, 320 rows 14.8 against 18.1; of 192 channels of 17 x 16, 40 rows 11.6 against 12.6; pooled of 256
  // channels of 8 x 8, 38 rows 12.5 against 12.7, of 20 x 20 (stride 1), 18 rows 11.5 against 10.8; of 512 channels of 8 x 8 (stride 1),
  // pooled, 40 rows 18.4 against 17.4; two tiles: 128 channels of 2 x 3, 174 rows 16.7 against 18.2, of 6 x 6 pooled, 50 rows
  // 13.2 against 12.6.  At most 4 % (5 % with two) from the better one.
  if (n == 2) return !region || 2 * rows >= 16 + p.Kw64 + (g.pool ? 16 : 0) ? 1 : 0;
  return n == 4 && region && 4 * rows >= 96 + 7 * (int64_t)p.Kw64 ? 1 : 0;
}

bnn_status launch_gemm_fp4(GemmParams &p, int bmode, int emode, hipStream_t s, int shape, bool region) {
  if (shape >= 4 && !bits_applicable(p, bmode)) shape = -1;
  if (bmode == 0) {
    if (shape < 2) {
      // Explicit rows stage B too, which the squarer tile halves (4096^3: 35.1 against 36.6 and 39.3).
      shape = p.M <= 64 ? 3 : 2;
      // Long ones on a full chip, where the sign codes hold the clock down (8192^3 232 -> 211 us, 4096 x 60000 x 2048
      // 273 -> 253, 1000 x 9000 x 4096 26.1 -> 23.8, 512 x 20000 x 2304 18.0 -> 16.3, 4096^3 33.9 -> 32.1).  Counting and the
      // corrections cost a tile about 1000 clocks: shorter rows gain nothing (4096 x 8192 x 1536 38.5 against 38.8, 2048 x
      // 4096 x 1280 10.7 against 11.4), nor do tiles that leave units idle (512 x 4096 x 2304 8.6 against 8.9).
      if (shape == 2 && bits_applicable(p, bmode) && p.Kw64 >= 32 &&
          5 * (((int64_t)p.M + 127) / 128) * (((int64_t)p.N + 127) / 128) >= 6 * (int64_t)p.n_cu)
        shape = 4;
    }
  } else if (shape < 0 || (emode == 0 && shape < 2)) {
    shape = conv_shape(p, emode, region);
  }
  switch (shape) {
    case 0: return launch_fp4_shape<2, 4, 2, 2, 2, false>(p, bmode, emode, s, region);  // 128 x 256, 4 waves of 64 x 128
    case 1: return launch_fp4_shape<2, 2, 2, 4, 2, false>(p, bmode, emode, s, region);  // 128 x 256, 8 waves of 64 x 64
    case 2: return launch_fp4_shape<2, 2, 2, 2, 3, true>(p, bmode, emode, s, region);   // 128 x 128, 4 waves of 64 x 64
    case 4: return launch_fp4_maps<2, 2, 2, 2, GM_EXPL16, 3, true>(p, s);                // 128 x 128, bits
    default: return launch_fp4_shape<2, 2, 1, 4, 2, true>(p, bmode, emode, s, region);  // 64 x 256, 4 waves of 64 x 64
  }
}

}  // namespace bnn
