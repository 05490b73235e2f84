// Internal helpers shared by the translation units of libbnn (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bnn.h"

namespace bnn {

// Kernel ids reported by the timing hook.
enum KernelId : int {
  KID_ENCODE_ROWS = 0,
  KID_PACK_CONV_WEIGHT = 1,
  KID_ENCODE_NCHW = 2,
  KID_IM2COL_GATHER = 3,
  KID_XNOR_GEMM = 4,
  KID_MAXPOOL = 5,
  KID_CONV_F32 = 6,
  KID_FC_F32 = 7,
  KID_VALU_PROBE = 8,
  KID_COPY_PROBE = 9,
  KID_XNOR_GEMM_SMALL = 10,
  KID_CONV_F32_SIGN = 11,
  KID_XNOR_GEMM_MFMA = 12,
  KID_CONTROL_CONV_F32 = 13,
  KID_XNOR_GEMM_MFMA_FP4 = 14,
  KID_XNOR_GEMM_LOWK = 15,
  KID_EXPAND_FP4 = 17,
  KID_XNOR_GEMM_MFMA_FP4X = 18,
  KID_XNOR_GEMM_FP4 = 19,
  KID_XNOR_GEMM_FP4_SPLIT = 20,
  KID_IM2COL_BAND = 21,
  KID_CONV_CHAIN = 22,
  KID_CONV_POINTWISE = 23,
  KID_XNOR_GEMM_FEWROWS = 24,
  KID_COUNT = 25
};

// Timing hook: records an event pair around a launch when profiling is on.
void prof_begin(int kernel_id, hipStream_t s);
void prof_end(hipStream_t s);

struct ProfScope {
  hipStream_t s;
  ProfScope(int kid, hipStream_t st) : s(st) { prof_begin(kid, st); }
  ~ProfScope() { prof_end(s); }
};

inline bnn_status launch_status() {
  return hipGetLastError() == hipSuccess ? BNN_OK : BNN_ERR_HIP;
}

inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Division of a 32-bit unsigned value by a runtime constant with one mulhi and one
// shift (round-up method; exact for every n < 2^31 and 1 <= d < 2^31).
struct FastDiv {
  uint32_t d, mul, shift;
  __host__ __device__ FastDiv() : d(1), mul(0), shift(0) {}
  __host__ __device__ explicit FastDiv(uint32_t div) : d(div) {
    if (div == 1) {
      mul = 0;
      shift = 0;
      return;
    }
    uint32_t l = 0;
    while ((1ull << l) < div) ++l;  // l = ceil(log2 d)
    shift = l - 1;
    // m = floor(2^32 * (2^l - d) / d) + 1, used as q = (mulhi(n, m) + n) >> l, rewritten
    // below so that no 33-bit intermediate is needed for n < 2^31.
    mul = (uint32_t)(((1ull << 32) * ((1ull << l) - div)) / div + 1);
  }
};

__device__ __forceinline__ uint32_t fdiv(uint32_t n, const FastDiv &f) {
  if (f.d == 1) return n;
  uint32_t t = __umulhi(n, f.mul);
  return (t + ((n - t) >> 1)) >> f.shift;
}

// ---- cross-file internals ---------------------------------------------------------------
// Geometry of an implicit-GEMM B operand: column n of the GEMM is output pixel n of a
// convolution over a packed NHWC image (ceil(C/64) words per pixel), and word w of its
// row is word (w mod Cw) of tap (w div Cw), taps ordered (kh, kw).
struct ConvGeom {
  const uint64_t *act;  // [Nimg, H, W, Cw]
  int Nimg, C, H, W, Cw, OH, OW, kH, kW, sH, sW, pH, pW;
  int pool;             // 0, or 2: columns are ordered window-major (see decode_col in gemm.hip)
  FastDiv divCw, divKW;
  FastDiv divOW, divOH; // output dims, or pooled output dims when pool == 2
};

// Matrix-core convolution: the input region of a tile of output pixels, kept in LDS as [word][pixel].
struct HaloGeom {
  int Wp;              // region pixels per row: every column a tap of any output column of a row reads
  int units;           // units per image: output rows, or pairs of them when pooling
  int ustep, uspan;    // input rows between units, input rows of one unit
  int full;            // input rows of a whole image's units
  int ppp;             // word pairs per pixel
  int nch;             // runs of 64 word pairs per region row
  uint32_t plane;      // bytes between the planes of two words
  uint32_t bytes;      // of the region
  FastDiv divPpp, divFull;
};

struct GemmParams {
  const uint32_t *A;   // [M, lda32] dwords
  const uint64_t *B;   // [N, ldb] words (explicit B only)
  int64_t lda32, ldb;
  int M, N;
  int Kd;              // dwords per row that hold bits of the reduction (ceil(Kbits/32))
  int Kbits;           // bits per row taking part in the exclusive-or
  int Kformula;        // K of the formula (true reduction length)
  int Kw64;            // words per row that may be read (ceil(Kbits/64))
  int b_vec16;         // B rows may be read with 16-byte loads
  int32_t *C;
  float *Y;
  int64_t ldc, ldy;    // row (m) strides of C and Y
  const float *scale, *bias;
  int axis;
  uint32_t OHW;        // columns per image; n -> (img, pix) = (n / OHW, n % OHW)
  FastDiv divOHW;
  int64_t img_stride;  // elements between images in C / Y
  int tilesM, tilesN;
  FastDiv divTilesM;   // matrix-core GEMM only
  int prio_from;       // workgroups with id >= prio_from lower their wave priority as they advance through K
  int n_cu;            // compute units of the device (host only: launch heuristics)
  int nt_store;        // int32 / fp32 tile stores are non-temporal
  int colperm;         // int32 / fp32 output whose columns and strides are multiples of 4: a lane's columns are
                       // consecutive and go out as one store per row (vector ALU: in 256-column tiles, LDS row
                       // 64 * j + l holds tile column 4 * l + j)
  int pairs;           // split-K kernel: two consecutive columns of a row are 8 aligned bytes of a map
  ConvGeom g;          // implicit B only
  HaloGeom halo;       // matrix-core convolution only
  uint64_t *outp;      // packed-sign output [pixels, cw_out] (packed epilogue only)
  int cw_out;
};

// Per-call choice of the GEMM variant.  The entry points of bnn.h always pass the defaults (size
// heuristic, table-driven gather where the geometry allows it); only the entry points of
// bnn_testing.h pass anything else.  Every variant computes the same values.
struct GemmTune {
  int cfg = -1;   // tile configuration (numbering in bnn_testing.h); -1 = heuristic
  int lean = 1;   // 0 = always the general implicit-GEMM gather
};

// Compute units of the current device (queried once per device, then cached).
int device_cu_count();

// Launch the exclusive-or / popcount GEMM described by p (tilesM / tilesN are filled in).
// bmode 0: B is an explicit [N, ldb] matrix; 1: B is gathered from p.g (implicit GEMM; the
// launcher switches to the lean gather, kernel mode 2, when the geometry allows it).
// emode 0: int32 / fp32 store; 1: packed sign(fma(scale, acc, bias)) store, optional 2x2 pool.
bnn_status run_gemm(GemmParams &p, int bmode, int emode, hipStream_t s, const GemmTune &tune = GemmTune());

// Convolution of an image of one to four words per pixel (conv_word.hip), taps straight from memory.
bool conv_word_applicable(const GemmParams &p, int bmode);
bool conv_word_faster(const GemmParams &p, int emode);  // its rule against the other matrix-core kernels
bnn_status launch_conv_word(GemmParams &p, int emode, hipStream_t s);

// Short-row GEMM (gemm_lowk.hip): rows of at most four words, explicit B, maps; form: see there, -1: its rule's.
bool lowk_applicable(const GemmParams &p);
bool lowk_faster(const GemmParams &p);  // its rule against the other matrix-core kernels
bnn_status launch_lowk(GemmParams &p, int form, hipStream_t s, int rounds = 1);

// Short rows, few of them, by very many columns (gemm_fewrows.hip).
bool fewrows_applicable(const GemmParams &p);
bool fewrows_faster(const GemmParams &p);  // its rule, for applicable problems
bnn_status launch_fewrows(GemmParams &p, hipStream_t s);

// Matrix-core GEMM on packed operands (gemm_fp4.hip): bmode / emode as for run_gemm; shape: tile number or -1;
// region: convolutions may keep a tile's input region in LDS (false: always the general gather).
bool fp4_applicable(const GemmParams &p);
// Whether the copy of a region row, its word pairs at a time, leaves more than half of the lanes idle.
inline bool halo_lanes_idle(const ConvGeom &g) {
  const int64_t pairs = ((int64_t)(g.OW - 1) * g.sW + g.kW) * ((g.Cw + 1) / 2);
  return 2 * pairs < (pairs + 63) / 64 * 64;
}
bool halo_region(GemmParams &p, int bn, bool pool, int64_t &rows);  // host only: p.halo from p.g and p.Kw64
bnn_status launch_gemm_fp4(GemmParams &p, int bmode, int emode, hipStream_t s, int shape, bool region);
// The same with the reduction axis split over the waves of a workgroup, for few outputs (gemm_fp4_split.hip).
bool fp4_split_applicable(const GemmParams &p, int bmode);  // whether its rule on sizes takes the problem
bnn_status launch_gemm_fp4_split(GemmParams &p, int bmode, int emode, hipStream_t s, int shape);

// Convolution from the fp32 image in one launch, by the split kernel (gemm_fp4_split.hip): K split 4 or 8 ways (0, 1;
// asked for, or -1: by its rule), -1 where it does not apply.
int conv_image_shape(const GemmParams &p, int shape);
void conv_image_rows(const GemmParams &p, int pixel, int64_t *rows);  // as bnn_testing_conv_image has it
bnn_status launch_conv_image(const GemmParams &p, const float *x, uint64_t *img, int shape, hipStream_t s);

// How the matrix-core kernels store int32 / fp32 maps (gemm.hip): past the caches; whether columns and strides are
// multiples of 4, so that a lane's columns can leave together.
bool nontemporal_maps(const GemmParams &p, int bmode, bool word = false);  // word: conv_word.hip's kernel
bool map_columns_by_four(const GemmParams &p);
bool map_rows_start_every(const GemmParams &p, uint32_t ints);  // multiples of `ints` 4-byte elements

// Pointwise convolution from the fp32 image in one launch (conv_pointwise.hip).
bool pointwise_applicable(const GemmParams &p);
bnn_status launch_conv_pointwise(GemmParams &p, const float *x, uint64_t *img, hipStream_t s);

// The binarization predicate: +0.0 and -0.0 -> 1, negative and NaN -> 0.
__device__ __forceinline__ bool sign_bit(float v) { return v >= 0.0f; }

// Four signs, y[0] first, shifted into R registers in turn: bits[k % R] = 2 * bits[k % R] + (y[k] >= 0), a compare and an
// add-with-carry each.  A vector instruction may read a carry only two wait states after the vector instruction that
// wrote it, and inside one asm statement nothing but its own instructions stands between them: the four compares come
// first, into a carry register each, so that every one has three instructions to its reader.  (256 x 128 x 16 x 16 to 256
// channels: 12.4 us; compare, s_nop 1, add-with-carry sign by sign: 12.8.)
template <int R>
__device__ __forceinline__ void shift_in_signs(uint32_t (&bits)[R], const float (&y)[4]) {
  static_assert(R == 1 || R == 2 || R == 4, "four signs");
  uint64_t c0, c1, c2;
#define BNN_COMPARE4(C0, C1, C2, Y0, Y1, Y2, Y3)                                                              \
  "v_cmp_le_f32 " C0 ", 0, " Y0 "\n\tv_cmp_le_f32 " C1 ", 0, " Y1 "\n\tv_cmp_le_f32 " C2 ", 0, " Y2           \
  "\n\tv_cmp_le_f32 vcc, 0, " Y3 "\n\t"
#define BNN_ADDC(B, C) "v_addc_co_u32 " B ", " C ", " B ", " B ", " C "\n\t"
  if constexpr (R == 4) {
    asm(BNN_COMPARE4("%4", "%5", "%6", "%7", "%8", "%9", "%10") BNN_ADDC("%0", "%4") BNN_ADDC("%1", "%5")
            BNN_ADDC("%2", "%6") BNN_ADDC("%3", "vcc")
        : "+v"(bits[0]), "+v"(bits[1]), "+v"(bits[2]), "+v"(bits[3]), "=&s"(c0), "=&s"(c1), "=&s"(c2)
        : "v"(y[0]), "v"(y[1]), "v"(y[2]), "v"(y[3])
        : "vcc");
  } else if constexpr (R == 2) {
    asm(BNN_COMPARE4("%2", "%3", "%4", "%5", "%6", "%7", "%8") BNN_ADDC("%0", "%2") BNN_ADDC("%1", "%3")
            BNN_ADDC("%0", "%4") BNN_ADDC("%1", "vcc")
        : "+v"(bits[0]), "+v"(bits[1]), "=&s"(c0), "=&s"(c1), "=&s"(c2)
        : "v"(y[0]), "v"(y[1]), "v"(y[2]), "v"(y[3])
        : "vcc");
  } else {
    asm(BNN_COMPARE4("%1", "%2", "%3", "%4", "%5", "%6", "%7") BNN_ADDC("%0", "%1") BNN_ADDC("%0", "%2")
            BNN_ADDC("%0", "%3") BNN_ADDC("%0", "vcc")
        : "+v"(bits[0]), "=&s"(c0), "=&s"(c1), "=&s"(c2)
        : "v"(y[0]), "v"(y[1]), "v"(y[2]), "v"(y[3])
        : "vcc");
  }
#undef BNN_COMPARE4
#undef BNN_ADDC
}

// Lane exchanges read a register two wait states after it was written at the earliest; the compiler does not see the
// writes above.
template <int R>
__device__ __forceinline__ void settle_signs(uint32_t (&bits)[R]) {
#pragma unroll
  for (int j = 0; j < R; ++j) asm("s_nop 1" : "+v"(bits[j]));
}

// Conv helpers (im2col.hip).  check_conv_geometry validates shapes and 32-bit limits;
// run_im2col launches encode (+ gather), or both in one kernel, with already validated arguments.
bnn_status check_conv_geometry(int N, int C, int H, int W, int kH, int kW, int sH, int sW, int pH, int pW);
bnn_status run_im2col(const float *x, int N, int C, int H, int W, int kH, int kW, int sH, int sW, int pH, int pW,
                      uint64_t *cols, void *workspace, hipStream_t s);

// 3x3 convolution of a 3-channel image with fp32 NCHW output (conv.hip); validated arguments.
bnn_status launch_conv2d_f32_k27(const float *x, const float *w, int N, int H, int W, int D, int sH, int sW, int pH,
                                 int pW, const float *scale, const float *bias, float *out, hipStream_t s);

// Signs of the 3x3x3 layer for more than a few pixels (conv_first_sign.hip), by workgroups of 4, 8 or 16 waves (0, 1, 2; -1: not).
int first_sign_f16(int N, int H, int W, int D, int sH, int sW, int pH, int pW, int units);
bnn_status launch_first_sign_f16(const float *x, const float *w, int N, int H, int W, int D, int sH, int sW, int pH, int pW,
                                 const float *scale, const float *bias, uint64_t *out, int shape, hipStream_t s);

}  // namespace bnn
