/*
 * bnn_testing.h -- entry points for tests and measurements; NOT part of the library's ABI and
 * not meant for applications.  The *_testing_* calls are the calls of bnn.h with the kernel
 * variant chosen by the caller instead of by the size heuristic; every variant computes the
 * values bnn.h specifies, and nothing set here outlives the call.  Only the kernel-timing hook
 * (bnn_prof_*) keeps state between calls: a list of HIP events, which never changes what a
 * call computes or launches.
 */
#ifndef BNN_TESTING_H_
#define BNN_TESTING_H_

#include "bnn.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * Tile configurations of the Xnor-Bitcount GEMM (section 3.2), argument `cfg` below:
 *   -1  the size heuristic (what bnn.h's entry points use)
 *   vector-ALU tiles (xor + popcount), which the size heuristic does not use:
 *    1  32 x 256 tile      2  32 x 64       3  64 x 256      4  32 x 128      6  64 x 128
 *   21 .. 24  the matrix-core GEMM (packed operands, expanded to 4-bit floating point in the wave that
 *       multiplies them): 128 x 256 tiles on four waves, 128 x 256 on eight (both only with the packed epilogue),
 *       128 x 128, 64 x 256
 *   25 .. 28  the same for few outputs, the reduction axis split over the waves of a workgroup:
 *       32 x 32 tiles split 4 / 8 ways, 64 x 64 tiles split 4 / 8 ways
 *   29  23 with the operands' bits expanded to 0 and 1 instead of +1 and -1 and the sums corrected by the counts of set
 *       bits (explicit rows in 16-byte pieces, int32 / fp32 output, K below 2^22)
 *   10 .. 17  the short-row kernel on the matrix cores (rows of at most four words): blocks of 32 x 32 outputs per
 *       wave, +1 of 64 x 64, +2 a workgroup's waves side by side, +4 contiguous runs of workgroups per XCD;
 *       30 .. 37  the same with three blocks of rows per wave
 *   18  the kernel for at most 16 such rows by very many columns (two or four words, columns and strides multiples of 4)
 *   19  convolutions of at most 256 channels, 1 x 1 or 3 x 3, whose taps go straight from memory to the matrix cores
 *   40, 41  bnn_conv2d in one launch, the tile encoding the input rows that it reads, the reduction split 4 / 8 ways
 * A value that a call cannot use (the packed epilogue needs a 32- or 64-row tile with two or
 * four column groups, or one of 21 to 28; 10 to 18 and 30 to 37 exist for an explicit B with int32 / fp32 output only;
 * 21 to 24 need K below 2^24, 29 what it says)
 * selects the heuristic for that call, and so does any other value.
 * `lean`: 1 = convolutions whose geometry allows it keep a tile's input region in LDS (matrix cores; with cfg = -1 where
 * it also pays, what bnn.h's entry points do) or gather their patches with the table-driven loader (vector ALU);
 * 0 = always the general gather.
 */

/* bnn_xnor_gemm_epilogue (and, with Y == NULL, bnn_xnor_gemm) on tile configuration cfg. */
BNN_API bnn_status bnn_testing_xnor_gemm_epilogue(const uint64_t *A, int64_t lda, const uint64_t *B, int64_t ldb,
                                                  int64_t M, int64_t N, int64_t K, int32_t *C, int64_t ldc, float *Y,
                                                  int64_t ldy, const float *scale, const float *bias,
                                                  bnn_ch_axis axis, int cfg, void *stream);

/* bnn_conv2d on tile configuration cfg and gather `lean`. */
BNN_API bnn_status bnn_testing_conv2d(const float *x, const uint64_t *w_packed, int N, int C, int H, int W, int D,
                                      int kH, int kW, int sH, int sW, int pH, int pW, int32_t *out_i32,
                                      float *out_f32, const float *scale, const float *bias, void *workspace,
                                      size_t workspace_bytes, int cfg, int lean, void *stream);

/* bnn_conv2d_packed on tile configuration cfg and gather `lean`. */
BNN_API bnn_status bnn_testing_conv2d_packed(const uint64_t *x_packed, const uint64_t *w_packed, int N, int C, int H,
                                             int W, int D, int kH, int kW, int sH, int sW, int pH, int pW, int pool,
                                             int32_t *out_i32, float *out_f32, uint64_t *out_packed,
                                             const float *scale, const float *bias, int cfg, int lean,
                                             void *stream);

/*
 * bnn_testing_conv_region -- host only, launches nothing: the input region that the matrix-core convolution
 * keeps in LDS for tiles of `columns` output pixels (128 or 256).  Returns 1 and fills region[] with
 *   0 the bound on a tile's input rows   1 pixels per region row   2 bytes between the planes of two words
 *   3 bytes of the region,
 * 0 where such a convolution gathers from memory instead, -1 for arguments bnn_conv2d_packed refuses.
 */
#define BNN_TESTING_REGION_VALUES 4
BNN_API int bnn_testing_conv_region(int N, int C, int H, int W, int kH, int kW, int sH, int sW, int pH, int pW,
                                    int pool, int columns, int64_t *region);

/*
 * bnn_testing_conv_word -- host only, launches nothing: whether a convolution of a packed image (packed 1: packed output, 0: an
 * int32 map, 2: an int32 and an fp32 map) goes to the kernel of configuration 19 on a device of `units` compute units: 2 it does, 1 it could, 0 it cannot,
 * -1 for arguments bnn_conv2d_packed refuses.  (A pointwise map without stride or padding is an explicit GEMM before that.)
 */
BNN_API int bnn_testing_conv_word(int N, int C, int H, int W, int D, int kH, int kW, int sH, int sW, int pH, int pW, int pool,
                                  int packed, int units);

/*
 * bnn_testing_conv_word_nontemporal -- host only, launches nothing: whether that kernel stores an int32 map of whole 16-byte
 * pieces with non-temporal (1) or ordinary (0) stores; -1 where it cannot take the call.
 */
BNN_API int bnn_testing_conv_word_nontemporal(int N, int C, int H, int W, int D, int kH, int kW, int sH, int sW, int pH, int pW);

/*
 * bnn_testing_nontemporal_maps -- host only, launches nothing: whether the matrix-core GEMM stores an int32 map
 * [M, N] of row stride ldc, starting base_bytes past a multiple of 128 bytes, with non-temporal (1) or ordinary
 * (0) stores; -1 for sizes below 1 or ldc < N.
 */
BNN_API int bnn_testing_nontemporal_maps(int M, int N, int K, int64_t ldc, int64_t base_bytes);

/*
 * bnn_xnor_gemm_mfma_fp4_expanded on a chosen workgroup tile (rows x columns of C):
 *   -1 the choice of bnn.h's entry point;  0 128 x 128;  1 256 x 128;  2 128 x 256.
 * Other values: BNN_ERR_SHAPE.
 */
BNN_API bnn_status bnn_testing_xnor_gemm_mfma_fp4_expanded(const uint8_t *A4, int64_t lda_bytes, const uint8_t *B4,
                                                           int64_t ldb_bytes, int32_t *C, int64_t ldc, int64_t M,
                                                           int64_t N, int64_t K, int tile, void *stream);

/* ---- measurement helpers ------------------------------------------------------------ */

/*
 * Kernel timing.  While enabled, every kernel the library launches is bracketed by a
 * pair of HIP events recorded on the caller's stream (host objects, created on first
 * use and kept until bnn_prof_enable(0)).  At most BNN_PROF_MAX_RECORDS launches are
 * recorded between two resets; later ones run untimed.  Not thread-safe.
 */
#define BNN_PROF_MAX_RECORDS 4096
BNN_API bnn_status bnn_prof_enable(int enable);
BNN_API bnn_status bnn_prof_reset(void);
BNN_API int64_t bnn_prof_count(void);
/* Synchronises on record i's end event, then returns its kernel id and duration. */
BNN_API bnn_status bnn_prof_get(int64_t i, int *kernel_id, float *milliseconds);
BNN_API const char *bnn_kernel_name(int kernel_id);

/*
 * bnn_valu_peak_probe -- a microbenchmark, not part of the method: every lane issues
 * 2 * 64 * iters vector lane-operations (xor + popcount-accumulate pairs) from registers,
 * no loads; the grid is `blocks` workgroups of 256 threads.  sink [blocks*256] int32
 * receives a value that depends on all of them.
 *   kind 0  independent pairs, both operands in vector registers, scheduled by the compiler
 *   kind 2 / 4  the GEMM's own row statements for 2 / 4 column groups per lane (xor operand
 *           in a scalar register, each xor directly followed by its popcount, one-cycle
 *           yield after each pair); iters should be a multiple of kind
 * Other kinds: BNN_ERR_SHAPE.
 */
BNN_API bnn_status bnn_valu_peak_probe(int32_t *sink, int blocks, int iters, int kind, void *stream);

/*
 * bnn_copy_probe -- plain device copy of n_bytes (multiple of 16) used as the yardstick
 * for achievable HBM bandwidth and for scaling hardware byte counters.
 */
BNN_API bnn_status bnn_copy_probe(const void *src, void *dst, size_t n_bytes, void *stream);

/* Convolutions from the fp32 image in one launch, K split 4 or 8 ways (shapes 0, 1): the one that bnn_conv2d takes on a device
 * of `units` compute units, or for shape >= 0 that one where it can be taken; -1 where it is not, or for invalid arguments.
 * rows receives the first and the last input row, counted over all images, of the tile that begins at output pixel `pixel`, and
 * the most rows that the launch has room for. */
BNN_API int bnn_testing_conv_image(int N, int C, int H, int W, int D, int kH, int kW, int sH, int sW, int pH, int pW,
                                   int units, int shape, int pixel, int64_t *rows);

/* The form in which bnn_conv2d_f32_sign takes a 3 x 3 layer of three channels on a device of `units` compute units: 0 fused
 * multiply-add chains for every output, one group of 32 channels a workgroup, 1 four groups; 2, 3, 4 half-precision products by workgroups of 4, 8, 16
 * waves; -1 for invalid arguments.  Host only, launches nothing. */
BNN_API int bnn_testing_first_sign(int N, int H, int W, int D, int sH, int sW, int pH, int pW, int units);

#ifdef __cplusplus
}
#endif
#endif /* BNN_TESTING_H_ */
