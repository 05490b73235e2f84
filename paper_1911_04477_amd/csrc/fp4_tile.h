// A wave's tile of the binarized GEMM on the fp4 matrix instruction: bit expansion, accumulators and the
// two epilogues (int32 / fp32 maps; max-pool + affine map + sign packed NHWC).
#pragma once
#include "common.h"

namespace bnn {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// fdiv without the branch on a divisor of 1 (uniform divisors: one select).
__device__ __forceinline__ uint32_t fdiv_sel(uint32_t n, const FastDiv &f) {
  const uint32_t t = __umulhi(n, f.mul);
  const uint32_t q = (t + ((n - t) >> 1)) >> f.shift;
  return f.d == 1 ? n : q;
}

// Output pixel of GEMM column n: image, row and column of the map.
__device__ __forceinline__ void column_pixel(const ConvGeom &g, uint32_t n, bool pool, uint32_t &img, uint32_t &oh,
                                             uint32_t &ow) {
  // window-major when pooling: column = 4 * window + member
  const uint32_t j = pool ? n & 3u : 0u, w = pool ? n >> 2 : n;
  const uint32_t PW = pool ? (uint32_t)g.OW >> 1 : (uint32_t)g.OW, PH = pool ? (uint32_t)g.OH >> 1 : (uint32_t)g.OH;
  const uint32_t t = fdiv_sel(w, g.divOW);
  ow = w - t * PW;
  img = fdiv_sel(t, g.divOH);
  oh = t - img * PH;
  if (pool) {
    ow = 2u * ow + (j & 1u);
    oh = 2u * oh + (j >> 1);
  }
}

// Pieces of rows that are not whole 16-byte pieces (an odd number of words, or rows that start on 8-byte
// boundaries): still one 16-byte load each, global loads need 4-byte alignment only.  A row's odd last word is read
// together with the one before it (the caller moves it), so no load goes past the row's end.  wide: the row has two
// words.  1000 x 3001 x 2321: 14.2 -> 11.6 us against two 8-byte loads per piece.
template <int P, class At>
__device__ __forceinline__ void load_pieces_any(u32x4 *r, bool wide, At at) {
  typedef u32x4 u32x4_any __attribute__((aligned(4)));
  if (wide) {
#pragma unroll
    for (int i = 0; i < P; ++i) r[i] = *reinterpret_cast<const u32x4_any *>(at(i));
  } else {
#pragma unroll
    for (int i = 0; i < P; ++i) {
      r[i].lo = *reinterpret_cast<const u32x2 *>(at(i));
      r[i].hi = u32x2{0u, 0u};
    }
  }
}

// 32 bits -> 32 E2M1 codes (bit 0: +1.0 = 0x2, bit 1: -1.0 = 0xA), value 4j + 3 - s in nibble j of dword s.
// The bit-field insert is written out: the optimizer splits it into an and and an or with literals.
// A matrix instruction may read a register only two wait states after a vector instruction has written it, and the
// compiler does not see that the written-out insert is one.  NOW: the codes may go into a matrix instruction at once,
// the last insert (the others stand before it) is followed by the wait.  Otherwise the caller has at least two
// instructions in between.
template <bool NOW>
__device__ __forceinline__ v8i expand_e2m1(uint32_t x) {
  const uint32_t sign = 0x88888888u, one = 0x22222222u;
  v8i r = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    uint32_t d;
    if (NOW && s == 3) asm volatile("v_bfi_b32 %0, %1, %2, %3\n\ts_nop 1" : "=v"(d) : "s"(sign), "v"(x << s), "v"(one));
    else asm volatile("v_bfi_b32 %0, %1, %2, %3" : "=v"(d) : "s"(sign), "v"(x << s), "v"(one));
    r[s] = (int)d;
  }
  return r;
}

// 32 bits -> 32 codes that are 0 where the bit is 0: the matrix instruction then counts the positions where both bits
// are 1 (S), and the sum of the +-1 products is K - 2 pa - 2 pb + 4 S with the set bits pa, pb of the two rows.  Half of
// the products are 0 and none is negative, so the adders toggle less and the chip holds a higher clock under the same
// loop (with the counting of set bits: 8192^3 232 -> 211 us, 4096^3 33.9 -> 32.1).  Long explicit rows and the chain of
// convolutions use these codes; the tiles of single convolutions do not (2 to 3 % at most, the counting takes it back).  The
// expansion is ands: bit 0, 1, 2 of a nibble alone are the codes 0.5, 1, 2.  A keeps the bits in place (the fourth moves to the
// second's), B swaps the first and the third, so that every product of two set bits is 1.  11 vector instructions per
// pair of dwords against 14.  NOW as above.
template <bool NOW>
__device__ __forceinline__ v8i expand_bits(uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3, uint32_t m0, uint32_t m2) {
  v8i r = {0, 0, 0, 0, 0, 0, 0, 0};
  uint32_t d;
  asm volatile("v_and_b32 %0, %1, %2" : "=v"(d) : "s"(m0), "v"(x0));
  r[0] = (int)d;
  asm volatile("v_and_b32 %0, %1, %2" : "=v"(d) : "s"(0x22222222u), "v"(x1));
  r[1] = (int)d;
  asm volatile("v_and_b32 %0, %1, %2" : "=v"(d) : "s"(m2), "v"(x2));
  r[2] = (int)d;
  if (NOW) asm volatile("v_and_b32 %0, %1, %2\n\ts_nop 1" : "=v"(d) : "s"(0x22222222u), "v"(x3));
  else asm volatile("v_and_b32 %0, %1, %2" : "=v"(d) : "s"(0x22222222u), "v"(x3));
  r[3] = (int)d;
  return r;
}

// What a bit becomes: its sign (above), or itself.
struct SignCodes {
  template <bool NOW>
  static __device__ __forceinline__ v8i a(uint32_t x) { return expand_e2m1<NOW>(x); }
  template <bool NOW>
  static __device__ __forceinline__ v8i b(uint32_t x) { return expand_e2m1<NOW>(x); }
};
struct BitCodes {
  template <bool NOW>
  static __device__ __forceinline__ v8i a(uint32_t x) {  // the fewer fragments: 2 shifts
    return expand_bits<NOW>(x << 2, x, x >> 2, x >> 2, 0x44444444u, 0x11111111u);
  }
  template <bool NOW>
  static __device__ __forceinline__ v8i b(uint32_t x) {
    return expand_bits<NOW>(x, x, x, x >> 2, 0x11111111u, 0x44444444u);
  }
};

// One step of 64 values for a 32 x 32 block: both operands E2M1 (format 4), no block scales.
__device__ __forceinline__ v16f mfma_e2m1(const v8i &a, const v8i &b, const v16f &c) {
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 4, 4, 0, 0, 0, 0);
}

template <int WTM, int WTN>
struct Fp4Acc {
  v16f v[WTM][WTN];
  __device__ __forceinline__ void init(float x) {
#pragma unroll
    for (int i = 0; i < WTM; ++i)
#pragma unroll
      for (int j = 0; j < WTN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) v[i][j][r] = x;
  }
};

// One step of 64 values with the expanded operands (a, b), and beside it the expansion of the next step's
// bits (xa, xb) into (na, nb) and whatever side(k) issues (staging, reading ahead), k = 0 .. WTM * WTN - 1.
// Vector instructions issue in the shadow of a matrix instruction (32 clocks), not beside a run of them, so the
// order is pinned: after each matrix instruction its share of everything else.  (Left to the compiler, the
// expansions of a step form one block and the matrix instructions another, which do not overlap.)  The order also
// keeps the operands' wait states: with several column blocks the first matrix instruction of the next step does not
// read the fragment that was expanded last.
template <class Codes, int WTM, int WTN, class Side>
__device__ __forceinline__ void multiply_and_expand(Fp4Acc<WTM, WTN> &acc, const v8i (&a)[WTM], const v8i (&b)[WTN],
                                                    const uint32_t (&xa)[WTM], const uint32_t (&xb)[WTN], v8i (&na)[WTM],
                                                    v8i (&nb)[WTN], const Side &side) {
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int k = 0; k < WTM * WTN; ++k) {
    const int i = k / WTN, j = k % WTN;
    acc.v[i][j] = mfma_e2m1(a[i], b[j], acc.v[i][j]);
    asm volatile("" : "+v"(acc.v[i][j]));  // emits nothing; keeps the instruction here among the volatile statements
    side(k);
    // fragments k * F / n .. (k + 1) * F / n - 1 of the F = WTM + WTN
#pragma unroll
    for (int f = k * (WTM + WTN) / (WTM * WTN); f < (k + 1) * (WTM + WTN) / (WTM * WTN); ++f) {
      if (f < WTM) na[f] = Codes::template a<false>(xa[f]);
      else nb[f - WTM] = Codes::template b<WTN == 1>(xb[f - WTM]);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// The matrix instructions' results may be read by a written-out instruction only some wait states later (the
// compiler pads only its own).  Two long no-ops, and every accumulator passes through them.
__device__ __forceinline__ void settle(Fp4Acc<2, 4> &a) {
  asm volatile("s_nop 15\n\ts_nop 15"
               : "+v"(a.v[0][0]), "+v"(a.v[0][1]), "+v"(a.v[0][2]), "+v"(a.v[0][3]), "+v"(a.v[1][0]), "+v"(a.v[1][1]),
                 "+v"(a.v[1][2]), "+v"(a.v[1][3]));
}
__device__ __forceinline__ void settle(Fp4Acc<2, 2> &a) {
  asm volatile("s_nop 15\n\ts_nop 15" : "+v"(a.v[0][0]), "+v"(a.v[0][1]), "+v"(a.v[1][0]), "+v"(a.v[1][1]));
}

// How a lane's WTN columns of a map leave: MS_NT / MS_VEC one non-temporal / ordinary store of consecutive columns
// per row; MS_ONE one 4-byte store per column and row, neighbouring lanes on neighbouring columns (columns that are not
// a multiple of 4; against a lane's two columns side by side: 1000 x 3001 x 2321 11.3 -> 10.2 us, 256 x 200001 x 200
// 41.8 -> 34.4, 128 x 31 x 33 maps from 1152 bits 21.7 -> 17.7).
enum : int { MS_NT = 0, MS_VEC = 1, MS_ONE = 2 };

// The result that an accumulator holds; BITS: all but the row's part, over 4 (see BitCodes).
template <bool BITS>
__device__ __forceinline__ float4 row_parts(const float *sRa) {
  return BITS ? *reinterpret_cast<const float4 *>(sRa) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
}
template <bool BITS>
__device__ __forceinline__ float result(float acc, float row) {
  return BITS ? fmaf(4.0f, acc, row) : acc;
}

// One map (int32, or fp32 through the affine map) of a wave's tile.  AFF: 0 int32, 1 fp32 with per-row
// constants, 2 fp32 with per-column constants.  FULL: no row of the tile is past M.
// Rows past M and columns past N hold the values of row M - 1 and column N - 1 once more (the staging clamps them), and
// go to that place: nothing is predicated but whole groups of 8 rows.  (A branch per row and column instead, in code
// that few waves run: 701 x 2113 x 1220 9.7 us, this way 6.4; 701 x 2112 x 1220 7.2, 6.1.)
template <int WTM, int WTN, int AFF, int MS, bool BITS, bool FULL, class P>
__device__ __forceinline__ void store_map(const P &p, const Fp4Acc<WTM, WTN> &acc, int m0, int n, int half,
                                          const float *sSc, const float *sBi, const float *sRa,
                                          const int64_t (&off)[WTN]) {
  typedef int vi __attribute__((ext_vector_type(WTN)));
  constexpr int STEP = MS == MS_ONE ? 32 : 1;  // columns between a lane's
  int32_t *base = AFF == 0 ? p.C : reinterpret_cast<int32_t *>(p.Y);
  const int64_t ld = AFF == 0 ? p.ldc : p.ldy;
  float csc[WTN], cbi[WTN];
  if constexpr (AFF == 2) {
#pragma unroll
    for (int j = 0; j < WTN; ++j) {
      csc[j] = p.scale[min(n + STEP * j, p.N - 1)];
      cbi[j] = p.bias[min(n + STEP * j, p.N - 1)];
    }
  }
  int32_t *ptr[WTN];
#pragma unroll
  for (int j = 0; j < (MS == MS_ONE ? WTN : 1); ++j) ptr[j] = base + off[j] + (int64_t)(FULL ? m0 + 4 * half : m0) * ld;
#pragma unroll
  for (int i = 0; i < WTM; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (!FULL && m0 + 32 * i + 8 * q >= p.M) return;  // uniform
      float4 sc, bi;
      const float4 ra = row_parts<BITS>(sRa + 32 * i + 8 * q + 4 * half);
      if constexpr (AFF == 1) {
        sc = *reinterpret_cast<const float4 *>(sSc + 32 * i + 8 * q + 4 * half);
        bi = *reinterpret_cast<const float4 *>(sBi + 32 * i + 8 * q + 4 * half);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        vi o;
#pragma unroll
        for (int j = 0; j < WTN; ++j) {
          const float v = result<BITS>(acc.v[i][j][4 * q + e], (&ra.x)[e]);
          if constexpr (AFF == 0) o[j] = (int)v;
          else if constexpr (AFF == 1) o[j] = __float_as_int(fmaf((&sc.x)[e], v, (&bi.x)[e]));
          else o[j] = __float_as_int(fmaf(csc[j], v, cbi[j]));
        }
        const int64_t row = FULL ? (int64_t)(32 * i + 8 * q + e) * ld  // uniform
                                 : (int64_t)min(32 * i + 8 * q + 4 * half + e, p.M - 1 - m0) * ld;
        if constexpr (MS == MS_NT) {
          __builtin_nontemporal_store(o, reinterpret_cast<vi *>(ptr[0] + row));
        } else if constexpr (MS == MS_VEC) {
          *reinterpret_cast<vi *>(ptr[0] + row) = o;
        } else {
#pragma unroll
          for (int j = 0; j < WTN; ++j) ptr[j][row] = o[j];
        }
      }
    }
}

template <int WTM, int WTN, int AFF, int MS, bool BITS, class P>
__device__ __forceinline__ void store_map_by(const P &p, const Fp4Acc<WTM, WTN> &acc, int m0, int n, int half,
                                             const float *sSc, const float *sBi, const float *sRa,
                                          const int64_t (&off)[WTN]) {
  if (m0 + 32 * WTM <= p.M) store_map<WTM, WTN, AFF, MS, BITS, true>(p, acc, m0, n, half, sSc, sBi, sRa, off);
  else store_map<WTM, WTN, AFF, MS, BITS, false>(p, acc, m0, n, half, sSc, sBi, sRa, off);
}

// int32 and / or fp32 output of a wave's tile: rows m0.., columns n0.. (row-major, or NCHW planes).  P: the kernel's
// arguments, of which these are read: C, Y, ldc, ldy, M, N, scale, bias, axis, img_stride, OHW, divOHW.
template <int WTM, int WTN, int MS, bool BITS = false, class P>
__device__ __forceinline__ void store_maps(const P &p, const Fp4Acc<WTM, WTN> &acc, int m0, int n0, int lane,
                                           const float *sSc, const float *sBi, const float *sRa = nullptr) {
  constexpr int STEP = MS == MS_ONE ? 32 : 1;
  const int half = lane >> 5;
  const int n = n0 + (MS == MS_ONE ? 1 : WTN) * (lane & 31);
  if (m0 >= p.M || (MS == MS_ONE ? n0 : n) >= p.N) return;
  int64_t off[WTN];
#pragma unroll
  for (int j = 0; j < WTN; ++j) {
    const int nc = min(n + STEP * j, p.N - 1);
    off[j] = nc;
    if (p.img_stride != 0) {  // NCHW planes
      const uint32_t img = fdiv((uint32_t)nc, p.divOHW);
      off[j] = (int64_t)img * p.img_stride + ((uint32_t)nc - img * p.OHW);
    }
  }
  if (p.C) store_map_by<WTM, WTN, 0, MS, BITS>(p, acc, m0, n, half, sSc, sBi, sRa, off);
  if (p.Y && p.axis == BNN_CH_ROW) store_map_by<WTM, WTN, 1, MS, BITS>(p, acc, m0, n, half, sSc, sBi, sRa, off);
  else if (p.Y) store_map_by<WTM, WTN, 2, MS, BITS>(p, acc, m0, n, half, sSc, sBi, sRa, off);
}

// nibble q of a 16-bit mask -> bits 8q .. 8q + 3
__device__ __forceinline__ uint32_t spread_nibbles(uint32_t m) {
  return (m & 0xFu) | ((m & 0xF0u) << 4) | ((m & 0xF00u) << 8) | ((m & 0xF000u) << 12);
}

// 64 channel bits of one column from the two row halves' bits (bit 16 i + 4 q + e of half h = row
// 32 i + 8 q + 4 h + e).
__device__ __forceinline__ uint64_t sign_word(uint32_t h0, uint32_t h1) {
  const uint32_t lo = spread_nibbles(h0 & 0xFFFFu) | (spread_nibbles(h1 & 0xFFFFu) << 4);
  const uint32_t hi = spread_nibbles(h0 >> 16) | (spread_nibbles(h1 >> 16) << 4);
  return ((uint64_t)hi << 32) | lo;
}

// Binarizing epilogue: affine map, sign; packed NHWC words.  Tile rows are output channels, 64 of them
// (WTM = 2): one word per output pixel.
template <int WTM, int WTN, bool DEALT>
__device__ __forceinline__ void store_signs(const GemmParams &p, const Fp4Acc<WTM, WTN> &acc, int m0, int n0, int lane,
                                            const float *sSc, const float *sBi) {
  static_assert(WTM == 2 && (WTN == 2 || WTN == 4), "one 64-channel word per wave");
  const int half = lane >> 5, l32 = lane & 31;
  const int word = m0 >> 6;
  if (word >= p.cw_out) return;  // wave-uniform
  uint32_t bits[WTN];  // rows are taken in descending order
#pragma unroll
  for (int j = 0; j < WTN; ++j) bits[j] = 0u;
#pragma unroll
  for (int i = 1; i >= 0; --i)
#pragma unroll
    for (int q = 3; q >= 0; --q) {
      const float4 sc = *reinterpret_cast<const float4 *>(sSc + 32 * i + 8 * q + 4 * half);
      const float4 bi = *reinterpret_cast<const float4 *>(sBi + 32 * i + 8 * q + 4 * half);
      constexpr int ROWS = 4 / WTN;  // four signs at a time
#pragma unroll
      for (int e = 3; e >= 0; e -= ROWS) {
        float y[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int r = e - k / WTN;
          y[k] = fmaf((&sc.x)[r], acc.v[i][k % WTN][4 * q + r], (&bi.x)[r]);
        }
        shift_in_signs<WTN>(bits, y);
      }
    }
  settle_signs(bits);
  // lanes l and l + 32 hold the two row halves of the same columns: the lower lanes assemble the first half of
  // the columns, the upper lanes the second
#pragma unroll
  for (int j = 0; j < WTN / 2; ++j) {
    const auto x = __builtin_amdgcn_permlane32_swap(bits[j], bits[j + WTN / 2], false, false);
    const int jj = half ? j + WTN / 2 : j;
    const int n = n0 + (DEALT ? WTN * l32 + jj : 32 * jj + l32);
    if (n < p.N) p.outp[(int64_t)n * p.cw_out + word] = sign_word(x[0], x[1]);
  }
}

// The same on the 2x2 maximum.  Columns are window-major: a lane of a 4-block wave holds whole windows, a
// lane of a 2-block wave one row of a window, its neighbour the other.
template <int WTM, int WTN>
__device__ __forceinline__ void store_signs_pooled(const GemmParams &p, const Fp4Acc<WTM, WTN> &acc, int m0, int n0,
                                                   int lane, const float *sSc, const float *sBi) {
  static_assert(WTM == 2 && (WTN == 2 || WTN == 4), "one 64-channel word per wave");
  const int half = lane >> 5, l32 = lane & 31;
  const int word = m0 >> 6;
  if (word >= p.cw_out) return;  // wave-uniform
  // rows are taken in descending order
  uint32_t bits[1] = {0u};
#pragma unroll
  for (int i = 1; i >= 0; --i)
#pragma unroll
    for (int q = 3; q >= 0; --q) {
      const float4 sc = *reinterpret_cast<const float4 *>(sSc + 32 * i + 8 * q + 4 * half);
      const float4 bi = *reinterpret_cast<const float4 *>(sBi + 32 * i + 8 * q + 4 * half);
      float y[4];
#pragma unroll
      for (int e = 3; e >= 0; --e) {
        const int r = 4 * q + e;
        float m;
        // the counts are finite: no need for the canonicalization that fmaxf brings
        asm("v_max_f32 %0, %1, %2" : "=v"(m) : "v"(acc.v[i][0][r]), "v"(acc.v[i][1][r]));
        if constexpr (WTN == 4) {
          asm("v_max3_f32 %0, %0, %1, %2" : "+v"(m) : "v"(acc.v[i][2][r]), "v"(acc.v[i][3][r]));
        } else {
          const float o = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(m), 0xB1, 0xF, 0xF, true));
          asm("v_max_f32 %0, %0, %1" : "+v"(m) : "v"(o));
        }
        y[3 - e] = fmaf((&sc.x)[e], m, (&bi.x)[e]);
      }
      shift_in_signs<1>(bits, y);
    }
  settle_signs(bits);
  const auto x = __builtin_amdgcn_permlane32_swap(bits[0], bits[0], false, false);
  const int w = WTN == 4 ? (n0 >> 2) + l32 : (n0 >> 2) + (l32 >> 1);  // pooled pixel
  if (half == 0 && (WTN == 4 || (l32 & 1) == 0) && w < (p.N >> 2))
    p.outp[(int64_t)w * p.cw_out + word] = sign_word(x[0], x[1]);
}

}  // namespace bnn
