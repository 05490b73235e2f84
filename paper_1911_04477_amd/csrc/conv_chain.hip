// Consecutive binarized 3x3 convolutions (stride 1, padding 1; packed NHWC in and out, optional 2x2 max-pool, affine map
// and sign after each) in one launch: a workgroup takes an image through all of them.
//
// A packed map is small (32 x 32 x 128 channels: 16 KB), so an image's activations never leave the compute unit: two LDS
// buffers of padded planes [word][row][column] take turns, the border holds the +1 of the padding, and every tap of
// every column is an LDS read at a constant distance.  Layer by layer in separate launches, a 128 x 256 tile spends a
// third of its time on what is not multiplication (arguments, region loads, tables, a cold instruction cache, the tail
// of the launch); here that is paid once, a layer costs two barriers, and the eight waves run free in between.
// 256 images through the five layers of the stack: 84 us one by one -> 57 (4.9 PBOPS, half the fp4 peak; of 128,000 clocks
// per unit 74,000 are matrix instructions, 10,000 the start, 8,000 a layer's barriers, tables, first and last steps).
//
// A wave owns tiles of 64 channels x 128 or 64 pixels.  Filters come straight from memory in the order in which the
// waves multiply them (bnn_pack_conv_chain_weight: 1 KB per 64 rows and 128 bits, one coalesced load three steps ahead,
// running on into the wave's next tile or layer), so nothing of them is staged and the loop has no barrier.
//
// Bits are multiplied as 0 / 1 codes (BitCodes): the accumulators start at (K - 2 * set bits of the patch) / 4, the set
// bits of the filter row are known from packing, and both meet in the sign: bit = (scale * C + bias >= 0) is a
// threshold on the integer C, found once per channel with the map's own fma, so the epilogue is one fma and one shift
// per output instead of fma, compare and add-with-carry.
#include <algorithm>

#include "common.h"
#include "fp4_tile.h"

namespace bnn {

typedef const uint32_t __attribute__((address_space(4))) *cu32_args;

constexpr int CHAIN_T = 512, CHAIN_WAVES = CHAIN_T / 64, CHAIN_MAX_LAYERS = 8, CHAIN_MAX_CHANNELS = CHAIN_T;
constexpr int CHAIN_AHEAD = 3;  // pieces of a filter row in flight: a row of taps

struct ChainLayer {
  const u32x4 *w;        // filter fragments [D / 64][Cw / 2][tap][lane] of 16 bytes
  const int32_t *ones;   // set bits of every filter row
  const float *scale, *bias;
  int W, Cw, D, pool;
  int P;                 // output columns of the multiplication: pixels of the map
  int pitch, pixels;     // padded columns; padded pixels of the input map
  uint32_t plane;        // bytes of a plane: one dword of every pixel, as codes
  int opitch, opixels;   // of the output map
  uint32_t oplane;
  int wide;              // tiles of 128 columns, else 64
  int rows64, tiles;
  FastDiv divW, divRows64, divPitchIn, divOpitch;  // divW: of a pixel's index, pooled: of a window's
};

struct ChainParams {
  const uint64_t *x;
  uint64_t *out;
  int layers, opix, cw_out;            // pixels and words per pixel of the last output
  int H, W;
  uint32_t buf1, pop, col, thr;        // LDS offsets: second map, set bits per pixel (two), column tables, thresholds
  uint32_t pop_bytes, col_bytes;
  FastDiv divW, divPairs;
  ChainLayer l[CHAIN_MAX_LAYERS];
};

// The codes (BitCodes::b) of a dword of an activation, four bits each: expanded once where a map is written, not under
// every tap of every tile.
__device__ __forceinline__ u32x4 chain_codes(uint32_t x) {
  return u32x4{x & 0x11111111u, x & 0x22222222u, x & 0x44444444u, (x >> 2) & 0x22222222u};
}

// Smallest integer d in [-K, K + 1] (K + 1: none) from which fma(|scale|, d, bias) >= 0 holds; the predicate does not fall
// with d (NaN: never true).  An estimate first, bisection over what it leaves.
__device__ __forceinline__ int sign_threshold(float scale, float bias, int K) {
  const float s = fabsf(scale);
  auto holds = [&](int d) { return fmaf(s, (float)d, bias) >= 0.0f; };
  const float top = (float)(K + 1);
  const int c = (int)fminf(fmaxf(-bias * __builtin_amdgcn_rcpf(s), -top), top);  // NaN: -top
  int lo = max(c - 2, -K - 1), hi = min(c + 2, K + 1);
  if (lo > -K - 1 && holds(lo)) lo = -K - 1;
  if (hi < K + 1 && !holds(hi)) hi = K + 1;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (holds(mid)) hi = mid;
    else lo = mid;
  }
  return hi;
}

// acc += the 9 * nc2 pieces of a tile.  ring holds the first CHAIN_AHEAD pieces on entry, those of `next` on return.
// col: LDS offset of every column block's codes under tap (0, 0): the word of this lane's half of the piece, its first
// dword; the second is a plane further.  A row of three taps (one turn of the ring, six steps of 64 values) per round of
// the loop: all nine taps in line are 13 KB of code that a tile of 18 words passes once.
template <int WTN>
__device__ __forceinline__ void chain_multiply(Fp4Acc<2, WTN> &acc, u32x4 (&ring)[CHAIN_AHEAD], const char *smem,
                                               const u32x4 *a, const u32x4 *next, const uint32_t (&col)[WTN],
                                               uint32_t pitch16, uint32_t plane, int nc2, int lane) {
  constexpr int MM = 2 * WTN;
  constexpr int NB = WTN == 4 ? 2 : 3;  // codes of a step are requested NB - 1 steps ahead: 256 clocks of multiplication
  u32x4 b[NB][WTN];
  v8i ea[2];
  uint32_t ya[2];
#pragma unroll
  for (int h = 0; h < NB - 1; ++h)
#pragma unroll
    for (int j = 0; j < WTN; ++j) b[h][j] = *reinterpret_cast<const u32x4 *>(smem + (col[j] + (uint32_t)h * plane));
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    ea[i] = BitCodes::a<true>(ring[0][2 * i]);
    ya[i] = ring[0][2 * i + 1];
  }
  uint32_t off = 0u;  // of the row of taps, from col
  int kh = 0, left = 3 * nc2;
#pragma unroll 1
  do {
    const bool last = --left == 0;
    const u32x4 *const an = last ? next : a + 3 * 64;
    uint32_t noff = off + pitch16;
    if (++kh == 3) {
      kh = 0;
      noff = off + 4u * plane - 2u * pitch16;
    }
    if (last) noff = off;  // past the last piece: taps once more, not used
#pragma unroll
    for (int h = 0; h < 6; ++h) {  // tap h / 2, dword h % 2
      constexpr int AHEAD = NB - 1;
      const int hl = h + AHEAD;  // the step whose codes are requested
      const uint32_t o = (hl < 6 ? off + 16u * (uint32_t)(hl / 2) : noff + 16u * (uint32_t)((hl - 6) / 2)) + (hl % 2 ? plane : 0u);
      const u32x4 &rn = ring[((h + 1) / 2) % 3];  // bits of the next step
      v8i na[2];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 0; k < MM; ++k) {
        const int i = k / WTN, j = k % WTN;
        const u32x4 &c = b[h % NB][j];
        acc.v[i][j] = mfma_e2m1(ea[i], v8i{(int)c.x, (int)c.y, (int)c.z, (int)c.w, 0, 0, 0, 0}, acc.v[i][j]);
        asm volatile("" : "+v"(acc.v[i][j]));  // emits nothing; keeps the order, as in multiply_and_expand
        if (k < WTN) b[hl % NB][k] = *reinterpret_cast<const u32x4 *>(smem + (col[k] + o));
        if (k % WTN == WTN - 1) na[i] = BitCodes::a<false>(h % 2 ? rn[2 * i] : ya[i]);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (h % 2) {
#pragma unroll
        for (int i = 0; i < 2; ++i) ya[i] = rn[2 * i + 1];
        ring[h / 2] = an[(h / 2) * 64 + lane];  // this tap's place is free
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) ea[i] = na[i];
    }
    a = an;
    off = noff;
  } while (left != 0);
  settle(acc);
}

// Signs of a tile's 64 channels -> one word per column (pool: per window) for the lanes that store it; bits are
// collected as sign bits of threshold differences, last channel first.
template <int WTN, bool POOL>
__device__ __forceinline__ void chain_signs(const Fp4Acc<2, WTN> &acc, const float *sg, const float *th,
                                            uint32_t (&bits)[POOL ? 1 : WTN]) {
#pragma unroll
  for (int j = 0; j < (POOL ? 1 : WTN); ++j) bits[j] = 0u;
#pragma unroll
  for (int i = 1; i >= 0; --i)
#pragma unroll
    for (int q = 3; q >= 0; --q) {
      const float4 s = *reinterpret_cast<const float4 *>(sg + 32 * i + 8 * q);
      const float4 t = *reinterpret_cast<const float4 *>(th + 32 * i + 8 * q);
#pragma unroll
      for (int e = 3; e >= 0; --e) {
        const int r = 4 * q + e;
        if constexpr (POOL) {
          float m;
          asm("v_max_f32 %0, %1, %2" : "=v"(m) : "v"(acc.v[i][0][r]), "v"(acc.v[i][1][r]));
          if constexpr (WTN == 4) {
            asm("v_max3_f32 %0, %0, %1, %2" : "+v"(m) : "v"(acc.v[i][2][r]), "v"(acc.v[i][3][r]));
          } else {
            const float o = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(m), 0xB1, 0xF, 0xF, true));
            asm("v_max_f32 %0, %0, %1" : "+v"(m) : "v"(o));
          }
          const float y = fmaf((&s.x)[e], m, (&t.x)[e]);
          bits[0] = __builtin_amdgcn_alignbit(bits[0], (uint32_t)__float_as_int(y), 31);
        } else {
#pragma unroll
          for (int j = 0; j < WTN; ++j) {
            const float y = fmaf((&s.x)[e], acc.v[i][j][r], (&t.x)[e]);
            bits[j] = __builtin_amdgcn_alignbit(bits[j], (uint32_t)__float_as_int(y), 31);
          }
        }
      }
    }
}

// One wave's tile t of layer L: multiplication and sign epilogue.  store(index of the output pixel, word, bits).
template <int WTN, class Store>
__device__ __forceinline__ void chain_tile(const ChainLayer &L, int t, u32x4 (&ring)[CHAIN_AHEAD], const u32x4 *a,
                                           const u32x4 *next, const char *smem, uint32_t in, const float *sCol,
                                           const uint32_t *sPix, const float *sThr, int lane, const Store &store) {
  asm("" : "+v"(lane));  // what depends on the lane is computed here, not kept across tiles in spilled registers
  const int half = lane >> 5, l32 = lane & 31;
  const int nb = (int)fdiv_sel((uint32_t)t, L.divRows64), mt = t - nb * L.rows64;
  const int n0 = nb * 32 * WTN;
  const bool pool = L.pool != 0;
  Fp4Acc<2, WTN> acc;
  uint32_t col[WTN];
#pragma unroll
  for (int j = 0; j < WTN; ++j) {
    const int c = min(n0 + (pool ? WTN * l32 + j : 32 * j + l32), L.P - 1);  // columns past the map repeat its last one
    col[j] = in + (uint32_t)half * 2u * L.plane + sPix[c];
    const float v = sCol[c];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc.v[i][j][r] = v;
  }
  chain_multiply<WTN>(acc, ring, smem, a, next, col, (uint32_t)L.pitch * 16u, L.plane, L.Cw >> 1, lane);
  const float *sg = sThr + 64 * mt + 4 * half, *th = sg + L.D;
  if (pool) {
    uint32_t bits[1];
    chain_signs<WTN, true>(acc, sg, th, bits);
    const auto x = __builtin_amdgcn_permlane32_swap(bits[0], bits[0], false, false);
    const int w = (n0 >> 2) + (WTN == 4 ? l32 : l32 >> 1);
    if (half == 0 && (WTN == 4 || (l32 & 1) == 0) && w < (L.P >> 2)) store(w, mt, ~sign_word(x[0], x[1]));
  } else {
    uint32_t bits[WTN];
    chain_signs<WTN, false>(acc, sg, th, bits);
    // lanes l and l + 32 hold the two row halves of the same columns: the lower lanes assemble the first half of the
    // columns, the upper lanes the second
#pragma unroll
    for (int j = 0; j < WTN / 2; ++j) {
      const auto x = __builtin_amdgcn_permlane32_swap(bits[j], bits[j + WTN / 2], false, false);
      const int n = n0 + 32 * (half ? j + WTN / 2 : j) + l32;
      if (n < L.P) store(n, mt, ~sign_word(x[0], x[1]));
    }
  }
}

__global__ __launch_bounds__(CHAIN_T, 2) void conv_chain_kernel(ChainParams p) {
  // Every 64-byte line of the arguments is requested at once (see xnor_gemm_fp4_kernel): layer by layer they are a
  // memory round trip each.
  {
    const cu32_args ka = (cu32_args)__builtin_amdgcn_kernarg_segment_ptr();
    constexpr int LINES = (int)((sizeof(ChainParams) + 63) / 64);
    static_assert(LINES > 16 && LINES <= 24, "every line below");
    constexpr int E = LINES - 1;
    asm volatile("" ::"s"(ka[0]), "s"(ka[16]), "s"(ka[32]), "s"(ka[48]), "s"(ka[64]), "s"(ka[80]), "s"(ka[96]),
                 "s"(ka[112]), "s"(ka[128]), "s"(ka[144]), "s"(ka[160]), "s"(ka[176]));
    asm volatile("" ::"s"(ka[192]), "s"(ka[208]), "s"(ka[224]), "s"(ka[240]), "s"(ka[256]), "s"(ka[16 * (E < 17 ? E : 17)]),
                 "s"(ka[16 * (E < 18 ? E : 18)]), "s"(ka[16 * (E < 19 ? E : 19)]), "s"(ka[16 * (E < 20 ? E : 20)]),
                 "s"(ka[16 * (E < 21 ? E : 21)]), "s"(ka[16 * (E < 22 ? E : 22)]), "s"(ka[16 * E]));
  }
  extern __shared__ __attribute__((aligned(16))) char smem[];
  int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint32_t *const sPix = reinterpret_cast<uint32_t *>(smem + p.col);
  uint32_t *const sOut = reinterpret_cast<uint32_t *>(smem + p.col + p.col_bytes);
  float *const sCol = reinterpret_cast<float *>(smem + p.col + 2 * p.col_bytes);
  float *const sThr = reinterpret_cast<float *>(smem + p.thr);
  auto fragments = [&](const ChainLayer &L, int t) {  // of tile t
    const int nb = (int)fdiv_sel((uint32_t)t, L.divRows64);
    return L.w + (size_t)(t - nb * L.rows64) * (size_t)(9 * (L.Cw >> 1) * 64);
  };
  // the codes of a word (64 channels of a pixel) -> the map's planes [word][dword][pixel]
  auto put_word = [&](uint32_t buf, uint32_t plane, int word, int at, uint32_t lo, uint32_t hi) {
    char *const d = smem + buf + 2u * (uint32_t)word * plane + (uint32_t)at * 16u;
    *reinterpret_cast<u32x4 *>(d) = chain_codes(lo);
    *reinterpret_cast<u32x4 *>(d + plane) = chain_codes(hi);
  };
  // a map's border is the +1 of the padding; its pixels' set bits are counted from 0
  auto clear_map = [&](uint32_t buf, uint32_t pop, int pitch, int pixels, uint32_t plane, int words, const FastDiv &divPitch) {
    uint32_t *const sPop = reinterpret_cast<uint32_t *>(smem + pop);
    for (int i = CHAIN_T - 1 - tid; i < pixels; i += CHAIN_T) {  // the first waves have the column tables to fill
      const int y = (int)fdiv_sel((uint32_t)i, divPitch), x = i - y * pitch;
      const bool border = x == 0 || x == pitch - 1 || i < pitch || i >= pixels - pitch;
      sPop[i] = border ? 64u * (uint32_t)words : 0u;
      if (border)
        for (int w = 0; w < words; ++w)
          put_word(buf, plane, w, i, ~0u, ~0u);
    }
  };

  // scale, bias, set bits -> direction, threshold
  auto thresholds = [&](float *d, const ChainLayer &L, int threads) {
    if (tid >= threads) return;
    for (int c = tid; c < L.D; c += threads) {
      const float scale = d[c];
      const int t = sign_threshold(scale, d[L.D + c], 576 * L.Cw), ones2 = 2 * __float_as_int(d[2 * L.D + c]);
      d[c] = scale < 0.0f ? -1.0f : 1.0f;
      // From an integer: never -0.  The epilogue keeps the sign bit of direction * acc + this, and -1 * 0 + -0 has it set.
      d[L.D + c] = 0.25f * (float)(scale < 0.0f ? ones2 - t : -ones2 - t);
    }
  };

  // ---- the image, the first filters and every layer's affine map are requested together -----------------
  const ChainLayer &F = p.l[0];
  const int pairs = F.Cw >> 1;
  const uint64_t *const xi = p.x + (size_t)blockIdx.x * (size_t)(p.H * p.W) * (size_t)F.Cw;
  u32x4 ring[CHAIN_AHEAD];
  {
    int nl = 0;
    while (nl + 1 < p.layers && wave >= p.l[nl].tiles) ++nl;
    const u32x4 *const a = fragments(p.l[nl], min(wave, p.l[nl].tiles - 1));
#pragma unroll
    for (int i = 0; i < CHAIN_AHEAD; ++i) ring[i] = a[i * 64 + lane];
  }
  float sc[CHAIN_MAX_LAYERS], bi[CHAIN_MAX_LAYERS];
  int ones[CHAIN_MAX_LAYERS];
#pragma unroll
  for (int l = 0; l < CHAIN_MAX_LAYERS; ++l)
    if (l < p.layers) {  // uniform
      const int c = min(tid, p.l[l].D - 1);
      sc[l] = p.l[l].scale[c];
      bi[l] = p.l[l].bias[c];
      ones[l] = p.l[l].ones[c];
    }
  constexpr int IN = 4;  // pieces of the image per thread and round
  const int npieces = p.H * p.W * pairs;
  u32x4 v[IN];
  auto load_image = [&](int i0) {
#pragma unroll
    for (int b = 0; b < IN; ++b)
      if (i0 + b * CHAIN_T < npieces)  // uniform
        v[b] = reinterpret_cast<const u32x4 *>(xi)[min(i0 + b * CHAIN_T + tid, npieces - 1)];
  };
  load_image(0);
  uint32_t warm = 0u;
  {
    // Every workgroup of a chiplet (consecutive ones go to different chiplets) asks for its share of the filters, one
    // dword of every 128-byte line, so that they are in the chiplet's L2 when their turn comes: from the waves' own
    // loads each line would be a miss for all of them at once, and three pieces ahead do not cover that.
    const int share = (int)blockIdx.x >> 3, shares = ((int)gridDim.x + 7) >> 3;
    int line = share * CHAIN_T + tid;
    const int step = shares * CHAIN_T;
    for (int l = 0; l < p.layers; ++l) {
      const int lines = (9 * p.l[l].Cw * p.l[l].D + 15) >> 4;
      for (; line < lines; line += step) warm ^= reinterpret_cast<const uint32_t *>(p.l[l].w)[min(line * 32, 18 * p.l[l].Cw * p.l[l].D - 1)];
      line -= lines;
    }
  }
  clear_map(0u, p.pop, F.pitch, F.pixels, F.plane, F.Cw, F.divPitchIn);
  __syncthreads();
  {
    uint32_t *const sPop = reinterpret_cast<uint32_t *>(smem + p.pop);
#pragma unroll 1
    for (int i0 = 0; i0 < npieces; i0 += IN * CHAIN_T) {
      if (i0 > 0) load_image(i0);
#pragma unroll
      for (int b = 0; b < IN; ++b) {
        const int i = i0 + b * CHAIN_T + tid;
        if (i >= npieces) break;
        const int px = (int)fdiv_sel((uint32_t)i, p.divPairs), c2 = i - px * pairs;
        const int y = (int)fdiv_sel((uint32_t)px, p.divW), x = px - y * p.W;
        const int at = (y + 1) * F.pitch + x + 1;
        put_word(0u, F.plane, 2 * c2, at, v[b].x, v[b].y);
        put_word(0u, F.plane, 2 * c2 + 1, at, v[b].z, v[b].w);
        atomicAdd(&sPop[at], (uint32_t)(__popc(v[b].x) + __popc(v[b].y) + __popc(v[b].z) + __popc(v[b].w)));
      }
    }
  }
  asm volatile("" ::"v"(warm));
  {
    float *d = sThr;
#pragma unroll
    for (int l = 0; l < CHAIN_MAX_LAYERS; ++l)
      if (l < p.layers) {
        const int D = p.l[l].D;
        if (tid < D) {
          d[tid] = sc[l];
          d[D + tid] = bi[l];
          d[2 * D + tid] = __int_as_float(ones[l]);
        }
        d += 3 * D;
      }
  }
  thresholds(sThr, F, CHAIN_T);  // a thread's own values

  uint32_t in = 0u, out = p.buf1;
  float *thr = sThr;  // per layer: scale, then direction; bias, then threshold; set bits of the rows
#pragma unroll 1
  for (int l = 0; l < p.layers; ++l) {
    const ChainLayer &L = p.l[l];
    const bool final = l + 1 == p.layers;
    const uint32_t pop = p.pop + (l & 1 ? p.pop_bytes : 0u), opop = p.pop + (l & 1 ? 0u : p.pop_bytes);
    asm("" : "+v"(tid));  // as in chain_tile
    __syncthreads();  // this layer's input is complete, the buffers of its output are free
    if (!final) clear_map(out, opop, L.opitch, L.opixels, L.oplane, L.D >> 6, L.divOpitch);
    {
      const uint32_t *const sPop = reinterpret_cast<const uint32_t *>(smem + pop);
      const int PW = L.pool ? L.W >> 1 : L.W;
      for (int c = tid; c < L.P; c += CHAIN_T) {
        const int w = L.pool ? c >> 2 : c;  // pooled: columns are window-major
        const int wy = (int)fdiv_sel((uint32_t)w, L.divW), wx = w - wy * PW;
        const int y = L.pool ? 2 * wy + ((c >> 1) & 1) : wy, x = L.pool ? 2 * wx + (c & 1) : wx;
        const uint32_t *const q = sPop + y * L.pitch + x;
        uint32_t n = 0u;
#pragma unroll
        for (int k = 0; k < 9; ++k) n += q[(k / 3) * L.pitch + k % 3];
        sPix[c] = (uint32_t)(y * L.pitch + x) * 16u;
        sCol[c] = 0.25f * (float)(576 * L.Cw) - 0.5f * (float)n;
        if (!L.pool || (c & 3) == 0) sOut[w] = (uint32_t)((wy + 1) * L.opitch + wx + 1);
      }
    }
    __syncthreads();
    uint32_t *const sPopOut = reinterpret_cast<uint32_t *>(smem + opop);
    auto store = [&](int n, int word, uint64_t v) {
      if (final) {
        p.out[((size_t)blockIdx.x * (size_t)p.opix + (size_t)n) * (size_t)p.cw_out + (size_t)word] = v;
      } else {
        const uint32_t at = sOut[n];
        put_word(out, L.oplane, word, (int)at, (uint32_t)v, (uint32_t)(v >> 32));
        atomicAdd(&sPopOut[at], (uint32_t)__popcll(v));
      }
    };
#pragma unroll 1
    for (int t = wave; t < L.tiles; t += CHAIN_WAVES) {
      const u32x4 *const a = fragments(L, t);
      const u32x4 *next = a;  // no further tile: loaded again, not used
      if (t + CHAIN_WAVES < L.tiles) {
        next = fragments(L, t + CHAIN_WAVES);
      } else {
        int nl = l + 1;
        while (nl < p.layers && wave >= p.l[nl].tiles) ++nl;
        if (nl < p.layers) next = fragments(p.l[nl], wave);
      }
      if (L.wide) chain_tile<4>(L, t, ring, a, next, smem, in, sCol, sPix, thr, lane, store);
      else chain_tile<2>(L, t, ring, a, next, smem, in, sCol, sPix, thr, lane, store);
    }
    const uint32_t s = in;
    in = out;
    out = s;
    thr += 3 * L.D;
    // by the first wave of every SIMD, which the arbiter prefers: the second ones still multiply
    if (!final) thresholds(thr, p.l[l + 1], CHAIN_T / 2);
  }
}

// Filter rows [D, 9 * Cw] in tap order -> fragments in the order of multiplication (see the kernel), 8 bytes a thread.
__global__ __launch_bounds__(256) void pack_chain_weight_kernel(const uint64_t *__restrict__ w, int Cw, uint32_t total,
                                                                FastDiv divPieces, uint64_t *__restrict__ frag) {
  const uint32_t o = blockIdx.x * 256u + threadIdx.x;
  if (o >= total) return;
  const int i = (int)(o & 1u), lane = (int)(o >> 1) & 63;
  const uint32_t piece = o >> 7, rb = fdiv_sel(piece, divPieces), q = piece - rb * divPieces.d;
  const int c2 = (int)(q / 9u), tap = (int)(q - 9u * (uint32_t)c2);
  const size_t row = (size_t)rb * 64u + 32u * (size_t)i + (size_t)(lane & 31);
  frag[o] = w[row * (size_t)(9 * Cw) + (size_t)(tap * Cw + 2 * c2 + (lane >> 5))];
}

__global__ __launch_bounds__(64) void count_row_bits_kernel(const uint64_t *__restrict__ w, int words, int32_t *__restrict__ ones) {
  int n = 0;
  for (int i = threadIdx.x; i < words; i += 64) n += __popcll(w[(size_t)blockIdx.x * (size_t)words + (size_t)i]);
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) n += __shfl_xor(n, d);
  if (threadIdx.x == 0) ones[blockIdx.x] = n;
}

}  // namespace bnn

using namespace bnn;

static size_t chain_fragment_bytes(int C, int D) { return (size_t)D * 9 * (size_t)(C / 64) * 8; }

static bool chain_channels_ok(int C, int D) {
  return C > 0 && D > 0 && C % 128 == 0 && D % 64 == 0 && C <= CHAIN_MAX_CHANNELS && D <= CHAIN_MAX_CHANNELS;
}

extern "C" size_t bnn_conv_chain_weight_bytes(int C, int D) {
  return chain_channels_ok(C, D) ? chain_fragment_bytes(C, D) + (size_t)D * 4 : 0;
}

extern "C" bnn_status bnn_pack_conv_chain_weight(const uint64_t *w_packed, int D, int C, void *w_chain, void *stream) {
  if (D < 0 || C <= 0) return BNN_ERR_SHAPE;
  if (D == 0) return BNN_OK;
  if (!chain_channels_ok(C, D)) return BNN_ERR_UNSUPPORTED;
  if (!w_packed || !w_chain) return BNN_ERR_NULL;
  if (!aligned16(w_packed) || !aligned16(w_chain)) return BNN_ERR_ALIGN;
  hipStream_t s = (hipStream_t)stream;
  const int Cw = C / 64;
  const uint32_t total = (uint32_t)D * 9u * (uint32_t)Cw;
  ProfScope ps(KID_PACK_CONV_WEIGHT, s);
  hipLaunchKernelGGL(pack_chain_weight_kernel, dim3((total + 255) / 256), dim3(256), 0, s, w_packed, Cw, total,
                     FastDiv((uint32_t)(9 * (Cw / 2))), reinterpret_cast<uint64_t *>(w_chain));
  hipLaunchKernelGGL(count_row_bits_kernel, dim3((unsigned)D), dim3(64), 0, s, w_packed, 9 * Cw,
                     reinterpret_cast<int32_t *>(reinterpret_cast<char *>(w_chain) + chain_fragment_bytes(C, D)));
  return launch_status();
}

// Fills p but for the pointers; LDS bytes, or 0 where the chain does not fit the kernel.  checked: the arguments' status.
static size_t chain_plan(ChainParams &p, int N, int C, int H, int W, int n_layers, const bnn_chain_layer *layers,
                         bnn_status &checked) {
  checked = BNN_ERR_SHAPE;
  if (N < 0 || C <= 0 || H <= 0 || W <= 0 || n_layers <= 0) return 0;
  checked = BNN_ERR_NULL;
  if (!layers) return 0;
  checked = BNN_ERR_UNSUPPORTED;
  if (n_layers > CHAIN_MAX_LAYERS) return 0;
  const int C0 = C, H0 = H, W0 = W;
  p.layers = n_layers;
  p.H = H;
  p.W = W;
  p.divW = FastDiv((uint32_t)W);
  p.divPairs = FastDiv((uint32_t)std::max(C / 128, 1));
  size_t buf[2] = {0, 0}, pop = 0, col = 0, thr = 0;
  auto pixels = [](int h, int w) { return (h + 2) * (w + 2); };
  auto plane = [&](int h, int w) { return (uint32_t)pixels(h, w) * 16u; };
  for (int i = 0; i < n_layers; ++i) {
    const int D = layers[i].D, pool = layers[i].pool;
    if (D <= 0 || (pool != 0 && pool != 2) || (pool && ((H | W) & 1))) {
      checked = BNN_ERR_SHAPE;
      return 0;
    }
    if (!chain_channels_ok(C, D) || H > 256 || W > 256) return 0;
    ChainLayer &L = p.l[i];
    const int OH = pool ? H / 2 : H, OW = pool ? W / 2 : W;
    L.W = W;
    L.Cw = C / 64;
    L.D = D;
    L.pool = pool;
    L.P = H * W;
    L.pitch = W + 2;
    L.pixels = pixels(H, W);
    L.plane = plane(H, W);
    L.opitch = OW + 2;
    L.opixels = pixels(OH, OW);
    L.oplane = plane(OH, OW);
    L.rows64 = D / 64;
    // wide tiles expand fewer fragments per matrix instruction; narrow ones where a wide one would be half empty
    const int wide = L.rows64 * ((L.P + 127) / 128), narrow = L.rows64 * ((L.P + 63) / 64);
    L.wide = 20 * ((wide + CHAIN_WAVES - 1) / CHAIN_WAVES) <= 11 * ((narrow + CHAIN_WAVES - 1) / CHAIN_WAVES) ? 1 : 0;
    L.tiles = L.wide ? wide : narrow;
    L.divW = FastDiv((uint32_t)OW);
    L.divRows64 = FastDiv((uint32_t)L.rows64);
    L.divPitchIn = FastDiv((uint32_t)L.pitch);
    L.divOpitch = FastDiv((uint32_t)L.opitch);
    buf[i & 1] = std::max(buf[i & 1], 2 * (size_t)L.plane * (size_t)L.Cw);
    pop = std::max(pop, (size_t)L.pixels * 4);
    col = std::max(col, (size_t)L.P * 4);
    thr += (size_t)D * 12;
    C = D;
    H = OH;
    W = OW;
  }
  p.opix = H * W;
  p.cw_out = C / 64;
  auto up16 = [](size_t b) { return (b + 15) & ~(size_t)15; };
  size_t at = up16(buf[0]);
  p.buf1 = (uint32_t)at;
  at += up16(buf[1]);
  p.pop = (uint32_t)at;
  p.pop_bytes = (uint32_t)up16(pop);
  at += 2 * up16(pop);
  p.col = (uint32_t)at;
  p.col_bytes = (uint32_t)up16(col);
  at += 3 * up16(col);
  p.thr = (uint32_t)at;
  at += thr;
  if (at > 160 * 1024) return 0;
  if ((int64_t)N * H0 * W0 * (C0 / 64) > 0x7fffffffLL) return 0;  // H0 and W0 are at most 256 here
  checked = BNN_OK;
  return at;
}

extern "C" int bnn_conv_chain_pays(int N, int C, int H, int W, int n_layers, const bnn_chain_layer *layers) {
  ChainParams p = {};
  bnn_status st;
  if (N <= 0 || !chain_plan(p, N, C, H, W, n_layers, layers, st)) return 0;
  // Both sides from their measured parts, in ns, of one chain: 32 x 32 maps, 128-128-256-256-512-512 channels, N images on
  // 256 units.  For smaller maps the fixed parts are too large.  120 random chains of 2 to 6 layers, 4 x 4 to 32 x 32: the 33 that
  // are taken run 1.18 times as fast as their layers (0.95 to 1.46; two are more than 3 % slower), 12 of 87 that are refused
  // would gain (130 images of 16 x 16, 256 channels, three layers: 24.6 us against 31.9; 223 of 8 x 8 18.6, 24.9).
  // The chain: 8 us of launch, image and first filters, per layer 3.3 us of barriers, tables and epilogue, and the two
  // waves of a SIMD share its matrix unit (64 clocks of 2.4 GHz per matrix instruction of both); as often as images need
  // the units.  Measured 57 us for up to 256 images, whatever their number.
  int64_t chain = 8000, layered = 0;
  const int64_t cu = device_cu_count(), rounds = (N + cu - 1) / cu;
  for (int i = 0; i < n_layers; ++i) {
    const ChainLayer &L = p.l[i];
    const int64_t turns = (L.tiles + CHAIN_WAVES - 1) / CHAIN_WAVES, pieces = 9 * (L.Cw / 2);
    chain += 3300 + turns * pieces * (L.wide ? 16 : 8) * 64 * 10 / 24;
    // Layer by layer: 4 us for a launch and a tile's ends, and 0.41 us per 10^9 multiply-adds of the tiles of 128 x 128
    // that a unit gets at most (256 images: 20.1, 12.1, 17.6, 12.5, 19.5 us).  The pass of the whole stack, layers against
    // chain: 128 images, the last that fill the units evenly, 83.8 us against 83.9; 130 105.5, 87.8; 200 114, 93; 257, a
    // second round of images, 147, 151; 320 153, 155; 384 164, 157; 512 191, 166.
    const int64_t bm = L.D <= 64 ? 64 : 128;
    const int64_t t = ((L.D + bm - 1) / bm) * (((int64_t)N * L.P + 127) / 128), each = (t + cu - 1) / cu;
    layered += 4000 + each * cu * bm * 128 / 1000 * (576 * L.Cw) / 1000 * 41 / 100;
  }
  return rounds * chain < layered ? 1 : 0;
}

extern "C" bnn_status bnn_conv_chain(const uint64_t *x_packed, int N, int C, int H, int W, int n_layers,
                                     const bnn_chain_layer *layers, uint64_t *out_packed, void *stream) {
  ChainParams p = {};
  bnn_status st;
  const size_t lds = chain_plan(p, N, C, H, W, n_layers, layers, st);
  if (st != BNN_OK) return st;
  if (N == 0) return BNN_OK;
  if (!x_packed || !out_packed) return BNN_ERR_NULL;
  if (!aligned16(x_packed) || !aligned16(out_packed)) return BNN_ERR_ALIGN;
  for (int i = 0; i < n_layers; ++i) {
    const bnn_chain_layer &L = layers[i];
    if (!L.w_chain || !L.scale || !L.bias) return BNN_ERR_NULL;
    if (!aligned16(L.w_chain)) return BNN_ERR_ALIGN;
    p.l[i].w = reinterpret_cast<const u32x4 *>(L.w_chain);
    p.l[i].ones = reinterpret_cast<const int32_t *>(reinterpret_cast<const char *>(L.w_chain) +
                                                    chain_fragment_bytes(64 * p.l[i].Cw, L.D));
    p.l[i].scale = L.scale;
    p.l[i].bias = L.bias;
  }
  p.x = x_packed;
  p.out = out_packed;
  hipStream_t s = (hipStream_t)stream;
  ProfScope ps(KID_CONV_CHAIN, s);
  hipLaunchKernelGGL(conv_chain_kernel, dim3((unsigned)N), dim3(CHAIN_T), lds, s, p);
  return launch_status();
}
