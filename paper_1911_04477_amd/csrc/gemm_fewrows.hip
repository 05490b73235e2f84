// Xnor-Bitcount GEMM (section 3.2) of at most 16 rows of two or four words by very many columns, explicit B, int32 / fp32
// output, on the vector ALU.
//
// Bound by memory: the columns' bits in, 4 bytes per row and column out, and nothing is used twice.  The matrix-core kernel
// of such rows (gemm_lowk.hip) multiplies blocks of 32 or 64 rows whatever M is, which takes it longer than the memory from
// some 30,000 to 600,000 columns on.  Here a lane owns four consecutive columns: their rows are requested up front, the rows of A are
// the same for all lanes and come by scalar loads, and every row leaves as one 16-byte store per lane.  2 x 4194304 x 128: 43 ->
// 17 us (6.0 TB/s), 8 x 1048576 x 256 14.4 -> 10.8.
#include "common.h"

namespace bnn {

typedef uint32_t few_u32x4 __attribute__((ext_vector_type(4)));
typedef int32_t few_i32x4 __attribute__((ext_vector_type(4)));

template <int GROUPS, int KD>  // groups of 8 rows; dwords per row: 4 or 8
__global__ __launch_bounds__(256) void xnor_gemm_few_kernel(GemmParams p) {
  typedef const uint32_t __attribute__((address_space(4))) *cu32_ptr;
  typedef const float __attribute__((address_space(4))) *cf32_ptr;
  const uint32_t n = (blockIdx.x * 256u + threadIdx.x) * 4u;  // first of this lane's four columns; N is a multiple of 4
  const bool col_ok = n < (uint32_t)p.N;
  const uint32_t nc = col_ok ? n : 0u;

  // bits past K are 0 in both operands
  const int tail_bits = p.Kbits & 63;
  const uint64_t tail_mask = tail_bits ? (1ull << tail_bits) - 1ull : ~0ull;
  const uint32_t tm_lo = (uint32_t)tail_mask, tm_hi = (uint32_t)(tail_mask >> 32);
  uint32_t b[4][KD];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint64_t *const src = p.B + (size_t)(nc + (uint32_t)j) * (size_t)p.ldb;
    if (p.b_vec16) {  // uniform
#pragma unroll
      for (int q = 0; q < KD / 4; ++q) {
        const few_u32x4 v = *reinterpret_cast<const few_u32x4 *>(src + 2 * q);
#pragma unroll
        for (int d = 0; d < 4; ++d) b[j][4 * q + d] = v[d];
      }
    } else {
#pragma unroll
      for (int w = 0; w < KD / 2; ++w) {
        const uint2 v = *reinterpret_cast<const uint2 *>(src + w);
        b[j][2 * w] = v.x;
        b[j][2 * w + 1] = v.y;
      }
    }
  }
  uint32_t img = 0u, pix = nc;  // NCHW planes: four columns are of one image
  if (p.img_stride != 0) {
    img = fdiv(nc, p.divOHW);
    pix = nc - img * p.OHW;
  }
  const int64_t off = (int64_t)img * p.img_stride + pix;
  float csc[4], cbi[4];
  const bool col_affine = p.Y && p.axis == BNN_CH_COL;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    csc[j] = col_affine ? p.scale[nc + (uint32_t)j] : 0.0f;
    cbi[j] = col_affine ? p.bias[nc + (uint32_t)j] : 0.0f;
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    b[j][KD - 2] &= tm_lo;
    b[j][KD - 1] &= tm_hi;
  }

  const cu32_ptr A = (cu32_ptr)(uintptr_t)p.A;
  const cf32_ptr scale = (cf32_ptr)(uintptr_t)p.scale, bias = (cf32_ptr)(uintptr_t)p.bias;
#pragma unroll
  for (int g = 0; g < GROUPS; ++g) {
    if (8 * g >= p.M) break;  // uniform
    uint32_t a[8][KD];        // rows past M are row M - 1 once more
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int d = 0; d < KD; ++d) a[i][d] = A[(size_t)min(8 * g + i, p.M - 1) * (size_t)p.lda32 + (size_t)d];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int m = 8 * g + i;
      if (m >= p.M) break;  // uniform
      a[i][KD - 2] &= tm_lo;
      a[i][KD - 1] &= tm_hi;
      few_i32x4 v;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        int acc = 0;
#pragma unroll
        for (int d = 0; d < KD; ++d) acc += __popc(a[i][d] ^ b[j][d]);
        v[j] = p.Kformula - 2 * acc;
      }
      if (!col_ok) continue;
      if (p.C) __builtin_nontemporal_store(v, reinterpret_cast<few_i32x4 *>(p.C + off + (int64_t)m * p.ldc));
      if (p.Y) {
        const float s = col_affine ? 0.0f : scale[m], t = col_affine ? 0.0f : bias[m];
        few_i32x4 y;
#pragma unroll
        for (int j = 0; j < 4; ++j)
          y[j] = __float_as_int(col_affine ? fmaf(csc[j], (float)v[j], cbi[j]) : fmaf(s, (float)v[j], t));
        __builtin_nontemporal_store(y, reinterpret_cast<few_i32x4 *>(p.Y + off + (int64_t)m * p.ldy));
      }
    }
  }
}

// Whether the kernel can run the problem described by p (explicit B).
bool fewrows_applicable(const GemmParams &p) {
  return p.M <= 16 && (p.Kw64 == 2 || p.Kw64 == 4) && map_columns_by_four(p);
}

// The vector instructions grow with the rows and their words, the matrix-core kernel's blocks do not.  us, here against there:
// 1 x 32768 x 128 2.8, 3.3; 2 x 65536 x 256 3.5, 3.5; 4 x 65536 x 128 3.2, 3.5; 8 x 131072 x 128 4.2, 4.3; 9 x 131072 x 256 5.4, 4.6;
// 8 x 200000 x 256 5.2, 5.5; 16 x 262144 x 128 6.2, 6.4; 12 x 400004 x 256 8.4, 8.2; 12 x 1048576 x 256 13.5, 16.6.  From 13 rows
// on the other way again where the result no longer fits the caches (16 x 4194304 x 128 65, 54; 16 x 1048576 x 128 14.1, 16.0).
bool fewrows_faster(const GemmParams &p) {
  return p.N >= 32768 && p.N >= (int64_t)9216 * p.M * p.Kw64 && (p.M <= 12 || p.N <= 1 << 21);
}

bnn_status launch_fewrows(GemmParams &p, hipStream_t s) {
  p.b_vec16 = p.ldb % 2 == 0;
  const dim3 grid((unsigned)(((int64_t)p.N + 1023) / 1024)), block(256);
  ProfScope ps(KID_XNOR_GEMM_FEWROWS, s);
  if (p.M <= 8) {
    if (p.Kw64 == 2) hipLaunchKernelGGL((xnor_gemm_few_kernel<1, 4>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((xnor_gemm_few_kernel<1, 8>), grid, block, 0, s, p);
  } else {
    if (p.Kw64 == 2) hipLaunchKernelGGL((xnor_gemm_few_kernel<2, 4>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((xnor_gemm_few_kernel<2, 8>), grid, block, 0, s, p);
  }
  return launch_status();
}

}  // namespace bnn
