// The three batched complex slice products of one iteration (per stored frequency b):
//   Z~_b = X~_b Y~_b                       (step 3)                   k_zgemm
//   A_b  = W~_b Y~_b^*  and the X-update, or its right-hand side       k_agemm
//          R_b = eta A_b G_Y^+ + H_rho1 X~_b (I - eta P_Y)   (step 1, eq. (updataXYW1))
//   X~_b^* W~_b (step 2), and in extra blocks of the same launch
//   G_X = X~_b^* X~_b + rho1 (H X~_b)^*(H X~_b), G_X^+ and I - eta P_X   k_bgemm
// The complex products run on the matrix cores as real FP32 products (16 x 16 x 4 tiles):
// a complex m x k by k x n product is an m x 2k by 2k x n' real one whose operands are the
// interleaved (re, im) storage itself, with the signs of the complex product placed in the
// operand that is built on the fly.  X~^* W~ and the X-update's r x r products run on the FP64
// matrix cores; r x r Grams are FP64.  Mixed mode reads W~ from its
// BF16 storage (stochastically rounded by the slice kernel) and converts to FP32 before
// the product.
#include <type_traits>
#include "kernels.h"
#include "pinv.h"

namespace tctf {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef double v4d __attribute__((ext_vector_type(4)));

// D += A B on one 16 x 16 x 4 FP32 tile: lane l supplies A[l % 16][l / 16] and
// B[l / 16][l % 16], and holds D[4 (l / 16) + t][l % 16] in element t.
__device__ __forceinline__ v4f mfma4(float a, float b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
// The FP64 16 x 16 x 4 tile: operands as above; lane l holds D[l / 16 + 4 t][l % 16].
__device__ __forceinline__ v4d mfma4d(double a, double b, v4d c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// ---------------------------------------------------------------- Z~ = X~ Y~
// Real form: Z'[i][2j + c] = sum_kk X'[i][kk] Y'[kk][2j + c] with kk = 2s + d,
// X'[i][2s + d] = (re, im)_d X~(i, s) and Y' carrying the signs of the complex product:
// Y'[2s][2j] = Yr, Y'[2s+1][2j] = -Yi, Y'[2s][2j+1] = Yi, Y'[2s+1][2j+1] = Yr.
// Block: 64 rows x 32 columns of one frequency, 4 wavefronts of 16 rows; Y~ staged in LDS, each
// wavefront forms four 16-column tiles, and output tiles go straight to the interleaved Z~ rows.
// The product writes Z~ and reads little, so it is bound by the stores once enough blocks are
// there; a block is short enough that its loads, LDS stage and stores are one latency each.  us
// with 128 / 64 / 32 columns per block: 144 x 288 x 28, r 8 6.7 / 4.8 / 4.0 (12.3 with the 288
// columns of a row tile in one block); 300 x 120 x 24, r 24 16.7 / 10.3 / 7.0; 529 x 96 x 112, r 16
// 12.0 / 11.4 / 11.6; 36 x 48 x 7, r 3 4.2 / 4.1 / 3.1.
// PINV: the first npinv blocks instead form G_Y^+ and I - eta P_Y of frequency blockIdx.x for
// the next X-step (pinvy_block): independent work that runs beside the product (an instance of
// its own, since the inverse takes more registers than a product of r <= 16).
#define ZG_ROWS 64
#define ZG_COLS 32
template <int RM, bool PINV>   // r <= RM: every loop below has a compile-time trip count
__global__ void __launch_bounds__(256) k_zgemm(const float2* __restrict__ xt, const float2* __restrict__ yt,
                                               float2* __restrict__ zt, int n1, int n2, int r, int nb,
                                               int npinv, PinvyArgs pa) {
  extern __shared__ __align__(16) unsigned char zsm[];
  if constexpr (PINV) {
    if ((int)blockIdx.x < npinv) {
      pinvy_block(blockIdx.x, pa, zsm);
      return;
    }
  }
  float2* ysh = (float2*)zsm;   // [s][j] of the column chunk
  const int bid = blockIdx.x - npinv, ntile = (n1 + ZG_ROWS - 1) / ZG_ROWS, tb = bid / ntile;
  const int i0 = (bid % ntile) * ZG_ROWS, b = tb % nb, j0 = tb / nb * ZG_COLS, nc = min(ZG_COLS, n2 - j0), tid = threadIdx.x;
  const int lane = tid & 63, w = tid >> 6, m = lane & 15, q = lane >> 4;
  constexpr int KS = RM / 2;   // K steps of 4 over 2r <= 2 RM
  constexpr int YPER = RM * ZG_COLS / 256;
  float2 yv[YPER];   // this thread's share of the block's Y~ columns, loaded ahead of its LDS store
#pragma unroll
  for (int u = 0; u < YPER; ++u) {
    const int e = tid + 256 * u, s = e / ZG_COLS, jj = e % ZG_COLS;
    yv[u] = ld_or(yt, ((size_t)b * r + s) * n2 + j0 + jj, s < r && jj < nc, make_float2(0.f, 0.f));
  }
  // A operands for every K step: X'[row][4 ks + q] (0 past the ends; loads clamped in range)
  const int row = i0 + 16 * w + m;
  float a[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const int kk = 4 * ks + q, s = kk >> 1;
    const float2 x = xt[((size_t)b * r + min(s, r - 1)) * n1 + min(row, n1 - 1)];
    a[ks] = (s < r && row < n1) ? ((kk & 1) ? x.y : x.x) : 0.f;
  }
  // Tile u of a group of four covers the group's 64 output floats 4 m + u (lane m's B
  // column), so a lane ends with four consecutive floats of a row: one 16-byte store.  The
  // operand pick of Y' is fixed by (kk & 1, column & 1) = (q & 1, u & 1).
  const int d = q & 1;
  float* zf = (float*)zt;
  const bool vec4 = (n2 & 1) == 0;   // rows start 16-byte aligned
#pragma unroll
  for (int u = 0; u < YPER; ++u) ysh[tid + 256 * u] = yv[u];
  __syncthreads();
  v4f acc[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) acc[u] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const int s = min((4 * ks + q) >> 1, r - 1);   // rows past 2r meet a zero A operand
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int cpar = u & 1;
      const int jj = 2 * m + (u >> 1);
      const float2 y = ysh[s * ZG_COLS + jj];
      const float bv = (d == 1 && cpar == 0) ? -y.y : (d != cpar ? y.y : y.x);
      acc[u] = mfma4(a[ks], bv, acc[u]);
    }
  }
  const int col = 4 * m;   // first of this lane's four floats of the block's 2 nc
  if (col < 2 * nc) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int i = i0 + 16 * w + 4 * q + t;
      if (i < n1) {
        float* dst = zf + (((size_t)i * nb + b) * n2 + j0) * 2 + col;
        if (col + 4 <= 2 * nc) {
          if (vec4) {
            *(float4*)dst = make_float4(acc[0][t], acc[1][t], acc[2][t], acc[3][t]);
          } else {
            ((float2*)dst)[0] = make_float2(acc[0][t], acc[1][t]);
            ((float2*)dst)[1] = make_float2(acc[2][t], acc[3][t]);
          }
        } else {   // 2 nc is even: the last two floats of the row
          *(float2*)dst = make_float2(acc[0][t], acc[1][t]);
        }
      }
    }
  }
}

// Mixed precision: the same product on the BF16 matrix cores (16 x 16 x 16 tiles, FP32
// accumulation).  Each FP32 factor value v is split into v_hi = bf16(v) and v_lo =
// bf16(v - v_hi) (round to nearest), and Z' = X'_hi Y'_hi + X'_hi Y'_lo + X'_lo Y'_hi: three
// BF16 products that keep about 16 bits of each operand, so Z~ carries errors near 2^-17
// relative instead of BF16's 2^-9.  Z~ feeds the W-step directly: BF16-sized noise there,
// new every iteration, made the iterate wander along the weakly determined directions of
// the completion (the RSE drifting by a few percent over thousands of iterations), while the
// split products leave it where the FP32 iteration goes.
// Lane (m, q) supplies A[m][4 q + e] and B[4 q + e][m], e = 0..3, of each 16-deep K chunk:
// in chunk c, K index 16 c + 4 q + e is (s, d) = (8 c + 2 q + e / 2, e % 2), so the lane's A
// values are (re, im) of X~(row, s0) and X~(row, s0 + 1), s0 = 8 c + 2 q, and its B values
// the signed parts of Y~(s0, j) and Y~(s0 + 1, j) (see Y' above).  Output tiles as k_zgemm's.
typedef short v4s __attribute__((ext_vector_type(4)));
__device__ __forceinline__ v4f mfma16bf(v4s a, v4s b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}
// (hi, lo) BF16 parts of x, as the low and high halves of one word
__device__ __forceinline__ uint32_t bf16_split(float x) {
  const uint16_t h = f32_to_bf16(x);
  return (uint32_t)h | ((uint32_t)f32_to_bf16(x - bf16_to_f32(h)) << 16);
}
template <int RM, bool PINV>
__global__ void __launch_bounds__(256) k_zgemm_bf(const float2* __restrict__ xt, const float2* __restrict__ yt,
                                                  float2* __restrict__ zt, int n1, int n2, int r, int nb,
                                                  int npinv, PinvyArgs pa) {
  extern __shared__ __align__(16) unsigned char zsm[];
  if constexpr (PINV) {
    if ((int)blockIdx.x < npinv) {
      pinvy_block(blockIdx.x, pa, zsm);
      return;
    }
  }
  uint2* ysh = (uint2*)zsm;   // [s][j] of the column chunk: (re, im) split words
  const int bid = blockIdx.x - npinv, ntile = (n1 + ZG_ROWS - 1) / ZG_ROWS, tb = bid / ntile;
  const int i0 = (bid % ntile) * ZG_ROWS, b = tb % nb, j0 = tb / nb * ZG_COLS, nc = min(ZG_COLS, n2 - j0), tid = threadIdx.x;
  const int lane = tid & 63, w = tid >> 6, m = lane & 15, q = lane >> 4;
  constexpr int KC = RM / 8;   // 16-deep K chunks over 2 RM
  constexpr int YPER = RM * ZG_COLS / 256;
  float2 yv[YPER];
#pragma unroll
  for (int u = 0; u < YPER; ++u) {
    const int e = tid + 256 * u, s = e / ZG_COLS, jj = e % ZG_COLS;
    yv[u] = ld_or(yt, ((size_t)b * r + s) * n2 + j0 + jj, s < r && jj < nc, make_float2(0.f, 0.f));
  }
  // A operands: X~(row, s0), X~(row, s0 + 1) of each chunk, split
  const int row = i0 + 16 * w + m;
  v4s ahi[KC], alo[KC];
#pragma unroll
  for (int c = 0; c < KC; ++c) {
    uint32_t h[4];
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      const int s = 8 * c + 2 * q + d;
      const float2 xv = xt[((size_t)b * r + min(s, r - 1)) * n1 + min(row, n1 - 1)];   // clamped, unconditional
      const float2 x = (s < r && row < n1) ? xv : make_float2(0.f, 0.f);
      h[2 * d] = bf16_split(x.x);
      h[2 * d + 1] = bf16_split(x.y);
    }
    ahi[c] = v4s{(short)(h[0] & 0xffffu), (short)(h[1] & 0xffffu), (short)(h[2] & 0xffffu), (short)(h[3] & 0xffffu)};
    alo[c] = v4s{(short)(h[0] >> 16), (short)(h[1] >> 16), (short)(h[2] >> 16), (short)(h[3] >> 16)};
  }
  float* zf = (float*)zt;
  const bool vec4 = (n2 & 1) == 0;   // rows start 16-byte aligned
#pragma unroll
  for (int u = 0; u < YPER; ++u) ysh[tid + 256 * u] = make_uint2(bf16_split(yv[u].x), bf16_split(yv[u].y));
  __syncthreads();
  v4f acc[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) acc[u] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < KC; ++c) {
    const int s0 = 8 * c + 2 * q;   // rows past r are zero in the chunk
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int jj = 2 * m + (u >> 1);
      const uint2 y0 = ysh[s0 * ZG_COLS + jj], y1 = ysh[(s0 + 1) * ZG_COLS + jj];   // (re, im) split words
      v4s bh, bl;
      if (u & 1) {   // column 2 j + 1: (Yi, Yr, Yi', Yr')
        bh = v4s{(short)(y0.y & 0xffffu), (short)(y0.x & 0xffffu), (short)(y1.y & 0xffffu), (short)(y1.x & 0xffffu)};
        bl = v4s{(short)(y0.y >> 16), (short)(y0.x >> 16), (short)(y1.y >> 16), (short)(y1.x >> 16)};
      } else {       // column 2 j: (Yr, -Yi, Yr', -Yi')
        bh = v4s{(short)(y0.x & 0xffffu), (short)((y0.y & 0xffffu) ^ 0x8000u), (short)(y1.x & 0xffffu),
                 (short)((y1.y & 0xffffu) ^ 0x8000u)};
        bl = v4s{(short)(y0.x >> 16), (short)((y0.y >> 16) ^ 0x8000u), (short)(y1.x >> 16),
                 (short)((y1.y >> 16) ^ 0x8000u)};
      }
      acc[u] = mfma16bf(alo[c], bh, acc[u]);
      acc[u] = mfma16bf(ahi[c], bl, acc[u]);
      acc[u] = mfma16bf(ahi[c], bh, acc[u]);
    }
  }
  const int col = 4 * m;   // first of this lane's four floats of the block's 2 nc
  if (col < 2 * nc) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int i = i0 + 16 * w + 4 * q + t;
      if (i < n1) {
        float* dst = zf + (((size_t)i * nb + b) * n2 + j0) * 2 + col;
        if (col + 4 <= 2 * nc) {
          if (vec4) {
            *(float4*)dst = make_float4(acc[0][t], acc[1][t], acc[2][t], acc[3][t]);
          } else {
            ((float2*)dst)[0] = make_float2(acc[0][t], acc[1][t]);
            ((float2*)dst)[1] = make_float2(acc[2][t], acc[3][t]);
          }
        } else {
          *(float2*)dst = make_float2(acc[0][t], acc[1][t]);
        }
      }
    }
  }
}

void zgemm_set_attr(int r) {
  if (pinv_lds_bytes(r) > 65536) {
    (void)hipFuncSetAttribute((const void*)k_zgemm<32, true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)pinv_lds_bytes(r));
    (void)hipFuncSetAttribute((const void*)k_zgemm_bf<32, true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)pinv_lds_bytes(r));
  }
}

template <int RM>
static void zgemm(const Plan& p, int npinv) {
  const int grid = npinv + (p.n1 + ZG_ROWS - 1) / ZG_ROWS * p.nb * ((p.n2 + ZG_COLS - 1) / ZG_COLS);
  size_t lds = (size_t)RM * ZG_COLS * sizeof(float2);
  if (npinv && pinv_lds_bytes(p.r) > lds) lds = pinv_lds_bytes(p.r);
  const auto k = p.mixed ? (npinv ? k_zgemm_bf<RM, true> : k_zgemm_bf<RM, false>)
                         : (npinv ? k_zgemm<RM, true> : k_zgemm<RM, false>);
  k<<<grid, 256, lds, p.stream>>>(p.xt, p.yt, p.zt, p.n1, p.n2, p.r, p.nb, npinv, pinvy_args(p));
}

// with_pinv: G_Y^+ too, in blocks ahead of the product's.  One iteration in us, in this launch / in one
// before it: 288 x 28 x 144 66.1 / 69.9, 12 x 12 x 2016 63.0 / 66.1, 40 x 40 x 1100, r = 30 340 / 353,
// 12 x 12 x 8064 134.6 / 135.7.
void launch_zgemm(const Plan& p, int with_pinv) {
  const int npinv = with_pinv ? p.nb : 0;
  if (p.r <= 8) zgemm<8>(p, npinv);
  else if (p.r <= 16) zgemm<16>(p, npinv);
  else zgemm<32>(p, npinv);
}

// ---------------------------------------------------------------- A = W~ Y~^* and the X-update
// Real form: A'[i][2s + e] = sum_kk W'[i][kk] Y'[kk][2s + e], kk = 2j + c, W' the
// interleaved W~ row and Y'[2j][2s] = Yr, Y'[2j+1][2s] = Yi, Y'[2j][2s+1] = -Yi,
// Y'[2j+1][2s+1] = Yr (Y = Y~(s, j)).  Within a group of 16 K values the K order is
// permuted so that lane (m, q) feeds the four products of the group from the four
// consecutive floats W'[m][16 g + 4 q ..] (two complex entries of W~), and the matching
// Y' values are the same two complex entries of Y~ row s (with the sign pattern).
// Block: 16 RT rows x one frequency, RT x WC wavefronts; wavefront (rt, c) takes 16 rows and
// every WC-th run of up to AG_GROUPS groups of 8 columns, all its W~ loads of a pass issued
// before the products.  FP32 sums run over one pass (at most 48 columns) and are added in
// FP64 across passes and wavefronts: FP32 sums over all 288 columns of 144 x 288 x 28 were the
// largest error of the iteration (W after six iterations 5e-7 from the FP64 result, 1.8e-7 so).
// Epilogue on the FP64 matrix cores, with U = X~ (I - eta P_Y) (absent when I - eta P_Y is
// exactly 0):
// * hk >= 0: the whole X-update.  Since X~_new = H_rho1^{-1} (eta A G_Y^+ + H_rho1 U) =
//   U + eta H_rho1^{-1} V with V = A G_Y^+, and H_rho1^{-1} is the stencil of hinv_stencil,
//   the block forms V on its rows (zero outside the matrix), multiplies it by the banded
//   matrix of the stencil's taps and writes X~_new on the 16 RT - 2 hk rows whose stencil lies
//   inside the block; consecutive blocks overlap by 2 hk rows.  U needs X~ on the output rows
//   only, which no other block writes, so X~ is updated in place.  Real bins (b = 0, n3 / 2)
//   keep a zero imaginary part.
// * hk = -1: the right-hand side R = eta A G_Y^+ + H_rho1 U for k_hsolve.
// What bounds it: at 529 x 96 x 112, r = 16 no single unit (21.2 us; 19 without any product, 10
// without loads and stores of the epilogue either): the chain of loads, products and two LDS
// hand-overs of blocks that all start together.  Before (one wavefront column, the epilogue on
// the VALU) 20.5 us with FP32 sums over all columns; 144 x 288 x 28, r = 8 16.2 before, 10.1 now;
// 300 x 120 x 24, r = 24 16.2 before, 13.3 now.
#define AG_GROUPS 6   // groups of 8 columns per wavefront and pass
struct HStencil {
  int k;                            // half-width, -1: right-hand side only
  double tap[2 * HINV_KMAX + 2];    // c lambda^d
};
// LDS of a block: the Y~ chunk as the products' B operands (a column pair of row s with the
// signs of e = 0 and of e = 1, 16 bytes each; mixed: hi and lo BF16 parts), then in its place
// the FP64 partial A' of each wavefront column (the sums in the first, V in the second); rows of
// both padded against bank conflicts.
__host__ __device__ constexpr int ag_ystride(int wc) { return wc * AG_GROUPS * 4 + 1; }   // column pairs
__host__ __device__ constexpr int ag_astride(int rm) { return 2 * rm + 1; }
static size_t agemm_lds_bytes(int rm, int rt, int wc) {
  const size_t y = (size_t)2 * rm * ag_ystride(wc) * sizeof(float4);
  const size_t a = (size_t)(wc > 2 ? wc : 2) * 16 * rt * ag_astride(rm) * sizeof(double);
  return y > a ? y : a;
}
template <int RM, bool MIXED, int RT>   // r <= RM; MIXED: W~ stored as packed bf16 pairs
__global__ void __launch_bounds__(RM == 32 ? 512 : 1024) k_agemm(const void* wt, const float2* __restrict__ yt,
                                                const float2* xt, const cd* __restrict__ gyp,   // xt may be xout
                                                const cd* __restrict__ qy, const int* __restrict__ qy_zero,
                                                float2* __restrict__ rhs, int n1, int n2, int r, int nb,
                                                double eta, double rho1, int raw_a, uint32_t* ctr,
                                                float2* xout, int n3, HStencil hs) {
  constexpr int ROWS = 16 * RT, NNT = RM / 8, CT = RM / 8, LDA = ag_astride(RM), KV = RM / 2;
  constexpr int YPER = (RM * AG_GROUPS * 4 + 64 * RT - 1) / (64 * RT);
  extern __shared__ __align__(16) unsigned char asm_[];
  __shared__ double tsh[2 * HINV_KMAX + 2];   // the stencil's taps
  float4* ysh = (float4*)asm_;                // [2 s + e][column pair]
  double* ash = (double*)asm_;                // [c][row][2s + e]
  const int tid = threadIdx.x, nt = blockDim.x, wc = nt / (64 * RT);
  const int lane = tid & 63, w = tid >> 6, m = lane & 15, q = lane >> 4, rt = w % RT, cg = w / RT;
  const int ystride = ag_ystride(wc);
  const int hk = raw_a ? -1 : hs.k;
#pragma unroll
  for (int d = 0; d < 2 * HINV_KMAX + 2; ++d)   // constant indices: the taps stay in the argument segment
    if (tid == d && d <= 2 * hk + 1) tsh[d] = hs.tap[d];   // read after the first barrier
  // with the stencil, block x covers rows x (ROWS - 2 hk) - hk .. (some outside the matrix)
  const int i0 = hk >= 0 ? (int)blockIdx.x * (ROWS - 2 * hk) - hk : (int)blockIdx.x * ROWS;
  const int b = blockIdx.y;
  const int row = i0 + 16 * rt + m;
  const bool row_in = row >= 0 && row < n1;
  // one thread of the launch advances the counter of the rounding bits that this
  // iteration's slice kernel (a later launch) uses for the BF16 W~
  if (ctr && blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) ctr[0] += 1u;
  // G_Y^+ as the B operand of V = A G_Y^+ for this wavefront's column tile, in real form
  // G'[2s][2t] = Gr, G'[2s+1][2t] = -Gi, G'[2s][2t+1] = Gi, G'[2s+1][2t+1] = Gr; likewise Q
  auto load_g = [&](const cd* mat, int ct, double (&bg)[KV]) {
    const double* base = (const double*)(mat + (size_t)b * r * r);
    const int sc = (16 * ct + m) >> 1, dd = q & 1, ee = m & 1;
#pragma unroll
    for (int ks = 0; ks < KV; ++ks) {
      const int sr = (4 * ks + q) >> 1;
      const bool ok = sr < r && sc < r;
      const double v = base[ok ? (uint32_t)(2 * (sr * r + sc) + (dd != ee)) : 0u];
      bg[ks] = ok ? (dd > ee ? -v : v) : 0.0;
    }
  };
  v4f acc[NNT];
  v4d accd[NNT];
#pragma unroll
  for (int u = 0; u < NNT; ++u) accd[u] = v4d{0.0, 0.0, 0.0, 0.0};
  const int pcols = wc * AG_GROUPS * 8;   // columns per pass
  for (int j0 = 0; j0 < n2; j0 += pcols) {
    using raw_t = typename std::conditional<MIXED, uint32_t, float2>::type;
    const int nc = min(pcols, n2 - j0);
    // The Y~ chunk is loaded first (its LDS stage must not wait for the W~ loads, the memory
    // counter being in order): the threads of a wavefront column load its own columns.
    float2 y0[YPER], y1[YPER];
    const int jw = cg * AG_GROUPS * 8, tl = tid - cg * 64 * RT;
#pragma unroll
    for (int u = 0; u < YPER; ++u) {
      const int e = tl + 64 * RT * u, sx = e / (AG_GROUPS * 4), jj = jw + 2 * (e % (AG_GROUPS * 4));
      const float2* src = yt + ((size_t)b * r + min(sx, r - 1)) * n2 + j0;
      y0[u] = src[min(jj, nc - 1)];
      y1[u] = src[min(jj + 1, nc - 1)];
    }
    // Every W~ load of the pass: unconditional from one base (row clamped into range; the buffer
    // has slack past its end), kept raw so that the products of group g wait for its own loads.
    // Group g of this wavefront covers columns jw + 8 g .. + 7; this lane takes 2
    const int ng = min(AG_GROUPS, (nc - jw + 7) / 8);   // <= 0: no columns left
    raw_t lo[AG_GROUPS], hi[AG_GROUPS];
    const raw_t* wrow = (const raw_t*)wt + ((size_t)min(max(row, 0), n1 - 1) * nb + b) * n2 + j0 + (ng > 0 ? jw : 0) + 2 * q;
#pragma unroll
    for (int g = 0; g < AG_GROUPS; ++g) {
      const int gc = max(0, min(g, ng - 1));
      lo[g] = wrow[8 * gc];
      hi[g] = wrow[8 * gc + 1];
    }
    if (j0 > 0) __syncthreads();   // every wavefront is done with the previous chunk
#pragma unroll
    for (int u = 0; u < YPER; ++u) {
      const int e = tl + 64 * RT * u, sx = e / (AG_GROUPS * 4), pr = cg * AG_GROUPS * 4 + e % (AG_GROUPS * 4), jj = 2 * pr;
      const float2 z = make_float2(0.f, 0.f), a = sx < r && jj < nc ? y0[u] : z, c = sx < r && jj + 1 < nc ? y1[u] : z;
      if (sx < RM) {
        // e = 0: (Yr, Yi, Yr', Yi');  e = 1: (-Yi, Yr, -Yi', Yr')
        float4 o0, o1;
        if constexpr (MIXED) {   // four hi parts, then four lo parts
          const uint32_t ar = bf16_split(a.x), ai = bf16_split(a.y), cr = bf16_split(c.x), ci = bf16_split(c.y), sg = 0x80008000u;
          const uint32_t an = ai ^ sg, cn = ci ^ sg;
          auto his = [](uint32_t x, uint32_t y) { return __uint_as_float((x & 0xffffu) | (y << 16)); };
          auto los = [](uint32_t x, uint32_t y) { return __uint_as_float((x >> 16) | (y & 0xffff0000u)); };
          o0 = make_float4(his(ar, ai), his(cr, ci), los(ar, ai), los(cr, ci));
          o1 = make_float4(his(an, ar), his(cn, cr), los(an, ar), los(cn, cr));
        } else {
          o0 = make_float4(a.x, a.y, c.x, c.y);
          o1 = make_float4(-a.y, a.x, -c.y, c.x);
        }
        ysh[(2 * sx) * ystride + pr] = o0;
        ysh[(2 * sx + 1) * ystride + pr] = o1;
      }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NNT; ++u) acc[u] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int g = 0; g < AG_GROUPS; ++g) {
      if (g < ng) {
        // columns past the end hold other data: dropped in the last group only (rows outside
        // the matrix hold a clamped row's product, dropped when A' is stored)
        if (jw + 8 * g + 8 > nc) {
          const int valid = nc - jw - (8 * g + 2 * q);
          const raw_t z = raw_t();
          lo[g] = valid > 0 ? lo[g] : z;
          hi[g] = valid > 1 ? hi[g] : z;
        }
        const float4* yg = ysh + m * ystride + (jw >> 1) + 4 * g + q;
        if constexpr (MIXED) {
          // BF16 matrix cores: this lane's four K values are the two packed W~ words as they
          // are (exact), Y~ enters split into its hi and lo BF16 parts (two products)
          const v4s av = __builtin_bit_cast(v4s, make_uint2(lo[g], hi[g]));
#pragma unroll
          for (int u = 0; u < NNT; ++u) {
            const float4 y2 = yg[16 * u * ystride];
            acc[u] = mfma16bf(av, __builtin_bit_cast(v4s, make_float2(y2.z, y2.w)), acc[u]);
            acc[u] = mfma16bf(av, __builtin_bit_cast(v4s, make_float2(y2.x, y2.y)), acc[u]);
          }
        } else {
          const float2 a0 = lo[g], a1 = hi[g];
#pragma unroll
          for (int u = 0; u < NNT; ++u) {
            const float4 y2 = yg[16 * u * ystride];
            acc[u] = mfma4(a0.x, y2.x, acc[u]);
            acc[u] = mfma4(a0.y, y2.y, acc[u]);
            acc[u] = mfma4(a1.x, y2.z, acc[u]);
            acc[u] = mfma4(a1.y, y2.w, acc[u]);
          }
        }
      }
    }
#pragma unroll
    for (int u = 0; u < NNT; ++u)
#pragma unroll
      for (int t = 0; t < 4; ++t) accd[u][t] += (double)acc[u][t];
  }
  double bg[KV];
  if (!raw_a) load_g(gyp, cg % CT, bg);
  const int noqy = raw_a || qy_zero[b];
  __syncthreads();   // every wavefront is done with the Y~ chunk
  // partial A' of this wavefront: element t of tile u is A'[16 rt + 4 q + t][16 u + m]
#pragma unroll
  for (int u = 0; u < NNT; ++u)
#pragma unroll
    for (int t = 0; t < 4; ++t)
      {
        const int ro = 16 * rt + 4 * q + t;
        ash[(cg * ROWS + ro) * LDA + 16 * u + m] = 16 * u + m < 2 * r && i0 + ro >= 0 && i0 + ro < n1 ? accd[u][t] : 0.0;
      }
  __syncthreads();
  if (wc > 1) {
    for (int e = tid; e < ROWS * 2 * RM; e += nt) {   // the sum over the wavefront columns, in order
      const int at = e / (2 * RM) * LDA + e % (2 * RM);
      double v = ash[at];
      for (int c = 1; c < wc; ++c) v += ash[c * ROWS * LDA + at];
      ash[at] = v;
    }
    __syncthreads();
  }
  if (raw_a) {
    for (int e = tid; e < ROWS * r; e += nt) {
      const int s = e / ROWS, rr = e % ROWS;
      if (i0 + rr < n1)
        rhs[((size_t)b * r + s) * n1 + i0 + rr] = make_float2((float)ash[rr * LDA + 2 * s], (float)ash[rr * LDA + 2 * s + 1]);
    }
    return;
  }
  // V' = A' G' tile by tile: lane (m, q) holds rows q + 4 t, column m of its tile
  double* vsh = ash + ROWS * LDA;
  v4d res[CT];
#pragma unroll
  for (int k = 0; k < CT; ++k) {
    const int ct = cg + k * wc;
    if (ct >= CT) break;   // the same in the whole wavefront
    if (k > 0) load_g(gyp, ct, bg);
    v4d v = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int ks = 0; ks < KV; ++ks) v = mfma4d(ash[(16 * rt + m) * LDA + 4 * ks + q], bg[ks], v);
    res[k] = v;
    if (hk >= 0) {
#pragma unroll
      for (int t = 0; t < 4; ++t) vsh[(16 * rt + q + 4 * t) * LDA + 16 * ct + m] = v[t];
    }
  }
  __syncthreads();   // V of every row of the block is in LDS
  if (hk >= 0) {
    // (H_rho1^{-1} V)(i, s): direct tap c lambda^|i - j| plus the reflections in the two
    // ends, c lambda^(i + j + 1) and c lambda^(2 n1 - 1 - i - j), where within the table
#pragma unroll
    for (int k = 0; k < CT; ++k) res[k] = v4d{0.0, 0.0, 0.0, 0.0};
    const int k0 = max(0, 16 * rt - hk) >> 2, k1 = (min(ROWS, 16 * rt + 16 + hk) + 3) >> 2, tmax = 2 * hk + 1;
    const bool ends = i0 <= hk || i0 + ROWS >= n1 - hk - 1;   // the same in the whole block
    for (int kk = k0; kk < k1; ++kk) {
      const int j = i0 + 4 * kk + q, dist = abs(row - j);
      double wgt = tsh[min(dist, tmax)];
      if (ends) {
        const int e1 = row + j + 1, e2 = 2 * n1 - 1 - row - j;
        wgt += (e1 >= 0 && e1 <= tmax ? tsh[min(max(e1, 0), tmax)] : 0.0) +
               (e2 >= 0 && e2 <= tmax ? tsh[min(max(e2, 0), tmax)] : 0.0);
        if (j < 0 || j >= n1) wgt = 0.0;
      }
      wgt = dist <= hk ? wgt : 0.0;
#pragma unroll
      for (int k = 0; k < CT; ++k) {
        const int ct = cg + k * wc;
        if (ct >= CT) break;
        res[k] = mfma4d(wgt, vsh[(4 * kk + q) * LDA + 16 * ct + m], res[k]);
      }
    }
  }
#pragma unroll
  for (int k = 0; k < CT; ++k) {
    const int ct = cg + k * wc;
    if (ct >= CT) break;
#pragma unroll
    for (int t = 0; t < 4; ++t) res[k][t] *= eta;
    if (!noqy) {   // + U, or + H_rho1 U = (H_rho1 X~) (I - eta P_Y)
      load_g(qy, ct, bg);
      const double deg = (n1 == 1) ? 0.0 : ((row == 0 || row == n1 - 1) ? 1.0 : 2.0);
#pragma unroll
      for (int ks = 0; ks < KV; ++ks) {
        const int kk = 4 * ks + q, s = min(kk >> 1, r - 1), ic = min(max(row, 0), n1 - 1);
        const float2* xc = xt + ((size_t)b * r + s) * n1;
        const float2 x0 = xc[ic];
        double xv = (kk & 1) ? x0.y : x0.x;
        if (hk < 0) {
          const float2 xm = xc[max(ic - 1, 0)], xp = xc[min(ic + 1, n1 - 1)];
          xv = (1.0 + rho1 * deg) * xv - rho1 * ((ic > 0 ? (double)((kk & 1) ? xm.y : xm.x) : 0.0) +
                                                (ic + 1 < n1 ? (double)((kk & 1) ? xp.y : xp.x) : 0.0));
        }
        res[k] = mfma4d(kk < 2 * r && row_in ? xv : 0.0, bg[ks], res[k]);
      }
    }
  }
  __syncthreads();   // every X~ read of the block is done before X~ is overwritten
  const bool real_bin = hk >= 0 && bin_is_real(b, n3);
  float* out = (float*)(hk >= 0 ? xout : rhs);
#pragma unroll
  for (int k = 0; k < CT; ++k) {
    const int ct = cg + k * wc, col = 16 * ct + m;
    if (ct >= CT || col >= 2 * r) break;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int ro = 16 * rt + q + 4 * t, io = i0 + ro;
      const bool in = io >= 0 && io < n1 && (hk < 0 || (ro >= hk && ro < ROWS - hk));
      if (in) out[(((size_t)b * r + (col >> 1)) * n1 + io) * 2 + (col & 1)] = (real_bin && (col & 1)) ? 0.0f : (float)res[k][t];
    }
  }
}

// H_rho1 = I + rho1 D^T D (D: first differences along mode 1) is tridiagonal with
// diagonal 1 + 2 rho1 (1 + rho1 in the end rows) and off-diagonal -rho1.  Away from the
// ends its inverse is c lambda^|i - j|, lambda the root in (0, 1) of
// rho1 lambda^2 - (1 + 2 rho1) lambda + rho1 = 0 and c = lambda / (rho1 (1 - lambda^2));
// an end row is a mirror (the row equation holds with a ghost entry equal to the end
// entry), which adds the image terms c lambda^(i + j + 1) and c lambda^(2 n1 - 1 - i - j).
// The images of images are below lambda^(2 n1), and dropping every tap with |i - j| > k
// changes a result by at most c lambda^(k + 1) / (1 - lambda) times the largest |V| there:
// k is the least with lambda^(k + 1) <= 2^-40: below FP32's rounding unit even where
// neighbouring rows differ in scale by 10^4 (k = 5 at rho1 = 0.01, 11 at rho1 = 0.1).
int hinv_stencil(double rho1, int n1, int r, double* tap) {
  if (r > 16 || !(rho1 >= 0.0)) return -1;
  double lam = 0.0, c = 1.0;
  if (rho1 > 0.0) {
    const double a = 1.0 + 2.0 * rho1;
    lam = 2.0 * rho1 / (a + sqrt(a * a - 4.0 * rho1 * rho1));   // the small root, without cancellation
    c = lam / (rho1 * (1.0 - lam * lam));
  }
  int k = 0;
  double p = lam;   // lambda^(k + 1)
  while (p > 0x1p-40 && k <= HINV_KMAX) {
    p *= lam;
    ++k;
  }
  if (k > HINV_KMAX || n1 < 2 * k + 2) return -1;
  double v = c;
  for (int d = 0; d <= 2 * k + 1; ++d) {
    tap[d] = v;
    v *= lam;
  }
  return k;
}

// Row tiles and wavefront columns of an X-update block.  64 rows while that gives the device
// two rounds of blocks, else 32 (the stencil's halo permitting: 1.5 times the rows read, but
// twice the blocks; 144 x 288 x 28 10.1 us against 13.0), and 32 where they hold the matrix
// (12 x 12 x 8064 18.2 us against 28.6).  The columns of W~ are split over wavefronts, 48 each,
// while the grid has fewer than 2048 of them (144 x 288 x 28 12.9 us with one column, 10.1 with
// three or more; 529 x 96 x 112, whose grid fills the device, 21.2 with one, 26.6 with two).
// The epilogue has rm / 8 column tiles, which 2 or 4 wavefront columns share even where the columns
// of W~ need fewer, within the same bound (the X-update alone in us with 1 / 2 / 4: 40 x 33 x 7, r =
// 32 17.9 / 14.2 / 12.6; 678 x 32 x 25, r = 30 19.8 / 17.0 / 26.0; 20 x 17 x 9, r = 16 10.1 / 9.0 / -).
static void agemm_shape(const Plan& p, int hk, int rm, int* rt, int* wc) {
  const int halo = hk >= 0 ? 2 * hk : 0;
  const long blocks4 = (long)((p.n1 + 63 - halo) / (64 - halo)) * p.nb;
  *rt = rm == 32 || (halo <= 16 && (blocks4 < 512 || p.n1 <= 32 - halo)) ? 2 : 4;
  const long waves = (long)((p.n1 + 16 * *rt - halo - 1) / (16 * *rt - halo)) * p.nb * *rt;
  const int most = (rm == 32 ? 8 : 16) / *rt, want = (p.n2 + 8 * AG_GROUPS - 1) / (8 * AG_GROUPS);
  int tiles = rm / 8;
  while (tiles > 1 && waves * tiles > 2048) tiles >>= 1;
  *wc = (int)(2048 / waves);
  if (*wc < 1) *wc = 1;
  if (*wc > want) *wc = want > tiles ? want : tiles;
  if (*wc > most) *wc = most;
}

typedef void (*AgemmKernel)(const void*, const float2*, const float2*, const cd*, const cd*, const int*, float2*, int, int,
                            int, int, double, double, int, uint32_t*, float2*, int, HStencil);
template <int RM>
static AgemmKernel agemm_kernel(int mixed, int rt) {
  if constexpr (RM == 32) return mixed ? k_agemm<32, true, 2> : k_agemm<32, false, 2>;
  else if (rt == 4) return mixed ? k_agemm<RM, true, 4> : k_agemm<RM, false, 4>;
  else return mixed ? k_agemm<RM, true, 2> : k_agemm<RM, false, 2>;
}

void launch_agemm(const Plan& p, int raw_a, int advance, int scratch_out) {
  HStencil hs;
  hs.k = raw_a ? -1 : p.hk;
  for (int d = 0; d < 2 * HINV_KMAX + 2; ++d) hs.tap[d] = d <= 2 * hs.k + 1 ? p.htap[d] : 0.0;
  const int rm = p.r <= 8 ? 8 : (p.r <= 16 ? 16 : 32);
  int rt, wc;
  agemm_shape(p, hs.k, rm, &rt, &wc);
  const int rows = hs.k >= 0 ? 16 * rt - 2 * hs.k : 16 * rt;
  float2* xout = scratch_out ? p.rhs : p.xt;
  const dim3 grid((p.n1 + rows - 1) / rows, p.nb);
  const AgemmKernel kernel = rm == 8 ? agemm_kernel<8>(p.mixed, rt) : (rm == 16 ? agemm_kernel<16>(p.mixed, rt) : agemm_kernel<32>(p.mixed, rt));
  const size_t lds = agemm_lds_bytes(rm, rt, wc);
  if (lds > 65536) (void)hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  kernel<<<grid, 64 * rt * wc, lds, p.stream>>>(p.wt, p.yt, p.xt, p.gyp, p.qy, p.qy_zero, p.rhs, p.n1, p.n2, p.r, p.nb,
                                                p.eta, p.rho1, raw_a, advance ? p.ctr : nullptr, xout, p.n3, hs);
}

// ---------------------------------------------------------------- X~^* W~ and G_X in one launch
// Outputs of the G_X blocks, per frequency b ([nb][r][r] FP64 complex unless noted).
struct GramOut {
  cd* gxm;       // G_X
  cd* dmat;      // (H X~)^*(H X~)
  cd* gxp;       // G_X^+
  cd* qx;        // I - eta G_X^+ G_X (not written when it is exactly 0)
  int* qx_zero;  // [nb] 1 when I - eta P_X = 0
  double rho1, eta;
  int force_eigen;
  double2* part; // S and D of npart row groups [nb][npart][2][r][r], upper tiles, or npart = 0
  int npart;
};

// (re, im) tiles of a complex product conj(x) w summed over rows: lane (m, q) supplies
// x = X(row q of the K step, column m) and w = W(row q, column m).
struct BgTile {
  v4d re, im;
};
__device__ __forceinline__ void bg_fma(BgTile& t, double xr, double xi, double wr, double wi) {
  t.re = mfma4d(xr, wr, t.re);
  t.im = mfma4d(xr, wi, t.im);
  t.re = mfma4d(xi, wi, t.re);
  t.im = mfma4d(-xi, wr, t.im);
}
// Adds the tiles of the W wavefronts into wavefront 0's, in a fixed tree order through LDS
// (buf: W / 2 x NT x 4 x 64 double2): the result does not depend on timing.
template <int W, int NT>
__device__ __forceinline__ void bg_reduce(BgTile (&t)[NT], double2* buf, int w, int lane) {
#pragma unroll
  for (int h = W / 2; h >= 1; h >>= 1) {
    if (w >= h && w < 2 * h) {
#pragma unroll
      for (int k = 0; k < NT; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e) buf[(((w - h) * NT + k) * 4 + e) * 64 + lane] = make_double2(t[k].re[e], t[k].im[e]);
    }
    __syncthreads();
    if (w < h) {
#pragma unroll
      for (int k = 0; k < NT; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const double2 o = buf[((w * NT + k) * 4 + e) * 64 + lane];
          t[k].re[e] += o.x;
          t[k].im[e] += o.y;
        }
    }
    __syncthreads();
  }
}

// X~^* W~.  Block: one frequency b and CW = 16 WL complex columns, reduced over every row i in
// the block: its W wavefronts take contiguous ranges of 4-row K steps, with two groups of
// loads in flight; each lane loads X~(i, s) and W~(i, j) once per K step and feeds both parts
// to the FP64 matrix cores.  X~ and W~ are FP32 or BF16 values, exact in FP64, so the sums
// carry FP64 rounding only (the Y-step's G_X^+ amplifies any rounding of X~^* W~).
template <int XL, int WL>
struct BgShape {
  static constexpr int KG = 16 / (XL + WL);   // K steps per load group (two groups in flight)
};
template <int XL, int WL, bool MX>
__device__ __forceinline__ void bg_load(const void* __restrict__ wt, const float2* __restrict__ xt, int ks, int ks1,
                                        int q, int m, int b, int r, int n1, int n2, int nb, int j0,
                                        float2 (&xv)[BgShape<XL, WL>::KG][XL], float2 (&wv)[BgShape<XL, WL>::KG][WL]) {
  constexpr int KG = BgShape<XL, WL>::KG;
#pragma unroll
  for (int k = 0; k < KG; ++k) {
    const int i = 4 * (ks + k) + q;
    const bool rowok = ks + k < ks1 && i < n1;
#pragma unroll
    for (int a = 0; a < XL; ++a) {
      const int s = 16 * a + m;
      xv[k][a] = ld_or(xt, ((size_t)b * r + s) * n1 + i, rowok && s < r, make_float2(0.f, 0.f));
    }
#pragma unroll
    for (int u = 0; u < WL; ++u) {
      const int j = j0 + 16 * u + m;
      const size_t idx = ((size_t)i * nb + b) * n2 + j;
      if constexpr (MX) wv[k][u] = unpack_bf16x2(ld_or((const uint32_t*)wt, idx, rowok && j < n2, 0u));
      else wv[k][u] = ld_or((const float2*)wt, idx, rowok && j < n2, make_float2(0.f, 0.f));
    }
  }
}
template <int XL, int WL>
__device__ __forceinline__ void bg_mfma(const float2 (&xv)[BgShape<XL, WL>::KG][XL],
                                        const float2 (&wv)[BgShape<XL, WL>::KG][WL], int cnt, BgTile (&acc)[XL * WL]) {
  constexpr int KG = BgShape<XL, WL>::KG;
#pragma unroll
  for (int k = 0; k < KG; ++k) {
    if (k < cnt) {   // the same in the whole wavefront
#pragma unroll
      for (int a = 0; a < XL; ++a)
#pragma unroll
        for (int u = 0; u < WL; ++u) bg_fma(acc[a * WL + u], xv[k][a].x, xv[k][a].y, wv[k][u].x, wv[k][u].y);
    }
  }
}

// G_X of frequency b: S = X~^* X~ and D = (H X~)^*(H X~) over every row (H X~: differences of
// neighbouring rows, exact in FP64; none past the last row), in 16 x 16 tiles (a, c), c >= a,
// of the real part re_a re_c + im_a im_c and of M = re_a im_c (on the diagonal, where the
// imaginary part is M - M^T) or M - im_a re_c (beside it); then G_X = S + rho1 D (= X~^* H_rho1
// X~), its pseudo-inverse (Lemma SVPMPI, pinv_herm) and I - eta P_X, all by one block.  Lane
// (m, q) holds the rows i, i + 1 and i + 2 (i = 2 q of a run of eight), which serve two K steps
// and their differences.  What bounds it is a chain: at 529 rows and r = 16 about 5 us of FP64
// matrix-core work on one compute unit, then 8 pivot steps; the product blocks of the same
// launch take as long.  Launch at 529 x 96 x 112, r = 16: 19.6 us, product blocks alone 17.6;
// before, the Gram in two launches on a graph branch beside the product: 7.3 + 11.5 us beside
// 16.6, and 14 us for the branch's fork and join.  144 x 288 x 28, r = 8: 10.4 us (5.1 + 7.6
// beside 6.6, and the fork and join, before).
//
// gramx_rows: the tiles of S and D over the runs of eight rows k0 .. k1 - 1, by the W wavefronts.
template <int XL, int W>
__device__ __forceinline__ void gramx_rows(const float2* __restrict__ xt, int b, int n1, int r, int k0, int k1,
                                           BgTile (&gs)[XL * (XL + 1) / 2], BgTile (&gd)[XL * (XL + 1) / 2]) {
  constexpr int KG = XL == 1 ? 4 : 2;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, m = lane & 15, q = lane >> 4;
  const int per = (k1 - k0 + W - 1) / W, ks0 = min(k1, k0 + w * per), ks1 = min(k1, ks0 + per);
  const float2* xb = xt + (size_t)b * r * n1;
  float2 xa[KG][XL][3], xn[KG][XL][3];
  auto load = [&](int ks, float2 (&x)[KG][XL][3]) {
#pragma unroll
    for (int k = 0; k < KG; ++k) {
      const int i = 8 * min(ks + k, max(ks1 - 1, 0)) + 2 * q;
#pragma unroll
      for (int a = 0; a < XL; ++a)
#pragma unroll
        for (int h = 0; h < 3; ++h) x[k][a][h] = xb[(uint32_t)(min(16 * a + m, r - 1) * n1 + min(i + h, n1 - 1))];
    }
  };
  auto prod = [&](int ks, const float2 (&x)[KG][XL][3]) {
#pragma unroll
    for (int k = 0; k < KG; ++k) {
      if (ks + k < ks1) {   // the same in the whole wavefront
        const int i = 8 * (ks + k) + 2 * q;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          double xr[XL], xi[XL], dr[XL], di[XL];
#pragma unroll
          for (int a = 0; a < XL; ++a) {
            const bool ok = i + h < n1 && 16 * a + m < r;   // past the last row its copies meet: no difference
            xr[a] = ok ? x[k][a][h].x : 0.0f;
            xi[a] = ok ? x[k][a][h].y : 0.0f;
            dr[a] = ok ? (double)x[k][a][h + 1].x - (double)x[k][a][h].x : 0.0;
            di[a] = ok ? (double)x[k][a][h + 1].y - (double)x[k][a][h].y : 0.0;
          }
          int t = 0;
#pragma unroll
          for (int a = 0; a < XL; ++a)
#pragma unroll
            for (int c = a; c < XL; ++c, ++t) {
              gs[t].re = mfma4d(xr[a], xr[c], gs[t].re);
              gd[t].re = mfma4d(dr[a], dr[c], gd[t].re);
              gs[t].im = mfma4d(xr[a], xi[c], gs[t].im);
              gd[t].im = mfma4d(dr[a], di[c], gd[t].im);
              gs[t].re = mfma4d(xi[a], xi[c], gs[t].re);
              gd[t].re = mfma4d(di[a], di[c], gd[t].re);
              if (c > a) {
                gs[t].im = mfma4d(-xi[a], xr[c], gs[t].im);
                gd[t].im = mfma4d(-di[a], dr[c], gd[t].im);
              }
            }
        }
      }
    }
  };
  load(ks0, xa);
  for (int ks = ks0; ks < ks1; ks += 2 * KG) {
    load(ks + KG, xn);   // clamped: past the wavefront's rows nothing new is read
    prod(ks, xa);
    if (ks + KG >= ks1) break;
    load(ks + 2 * KG, xa);
    prod(ks + KG, xn);
  }
}

template <int XL, int W>
__device__ __forceinline__ void gramx_block(const float2* __restrict__ xt, int b, int n1, int r, const GramOut& go,
                                            unsigned char* sm) {
  constexpr int NT = XL * (XL + 1) / 2;
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, w = tid >> 6, m = lane & 15, q = lane >> 4, rr = r * r;
  BgTile gs[NT], gd[NT];
#pragma unroll
  for (int k = 0; k < NT; ++k) gs[k].re = gs[k].im = gd[k].re = gd[k].im = v4d{0.0, 0.0, 0.0, 0.0};
  if (go.npart == 0) {
    gramx_rows<XL, W>(xt, b, n1, r, 0, (n1 + 7) >> 3, gs, gd);
  } else {
    const double2* part = go.part + (size_t)b * go.npart * 2 * rr;
    for (int g = w; g < go.npart; g += W) {
      int t = 0;
#pragma unroll
      for (int a = 0; a < XL; ++a)
#pragma unroll
        for (int c = a; c < XL; ++c, ++t) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int s = 16 * a + q + 4 * e, u = 16 * c + m;
            const bool in = s < r && u < r;
            const double2 vs = ld_or(part, (size_t)2 * g * rr + s * r + u, in, make_double2(0.0, 0.0));
            const double2 vd = ld_or(part, (size_t)(2 * g + 1) * rr + s * r + u, in, make_double2(0.0, 0.0));
            gs[t].re[e] += vs.x;
            gs[t].im[e] += vs.y;
            gd[t].re[e] += vd.x;
            gd[t].im[e] += vd.y;
          }
        }
    }
  }
  bg_reduce<W>(gs, (double2*)sm, w, lane);
  bg_reduce<W>(gd, (double2*)sm, w, lane);
  // (the reductions end with a barrier: their LDS is free again)
  cd* gx = (cd*)sm;
  cd* gp = gx + rr;
  PinvScratch ps;
  ps.work = gp + rr;
  ps.vec = ps.work + rr;
  ps.rot = (double*)(ps.vec + rr);
  ps.red = ps.rot + 96;
  cd* dx = gp;   // D and G_X by way of LDS: the diagonal tiles' imaginary parts need M^T
  if (w == 0) {
    int t = 0;
#pragma unroll
    for (int a = 0; a < XL; ++a)
#pragma unroll
      for (int c = a; c < XL; ++c, ++t) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          // element e of lane (q, m): row q + 4 e, column m of the tile
          const int s = 16 * a + q + 4 * e, u = 16 * c + m;
          if (s < r && u < r) {
            const cd d = cd_make(gd[t].re[e], gd[t].im[e]);
            const cd v = cd_add(cd_make(gs[t].re[e], gs[t].im[e]), cd_scale(d, go.rho1));
            ps.work[s * r + u] = v;
            dx[s * r + u] = d;
            if (c > a) {
              ps.work[u * r + s] = cd_conj(v);
              dx[u * r + s] = cd_conj(d);
            }
          }
        }
      }
  }
  __syncthreads();
  for (int e = tid; e < rr; e += nt) {
    const int s = e / r, u = e - s * r;
    cd v = ps.work[e], d = dx[e];
    if (XL == 1 || (s >> 4) == (u >> 4)) {
      v.im -= ps.work[u * r + s].im;
      d.im -= dx[u * r + s].im;
    }
    gx[e] = v;
    go.gxm[(size_t)b * rr + e] = v;
    go.dmat[(size_t)b * rr + e] = d;
  }
  __syncthreads();
  const int fullr = pinv_herm(gx, gp, r, go.force_eigen, ps);
  const bool qzero = fullr && go.eta == 1.0;
  for (int e = tid; e < rr; e += nt) {
    go.gxp[(size_t)b * rr + e] = gp[e];
    if (!qzero) {   // q = I - eta G_X^+ G_X
      const int s = e / r, t = e % r;
      cd acc = cd_make(0.0, 0.0);
      for (int u = 0; u < r; ++u) cd_fma(acc, gp[s * r + u], gx[u * r + t]);
      go.qx[(size_t)b * rr + e] = cd_make((s == t ? 1.0 : 0.0) - go.eta * acc.re, -go.eta * acc.im);
    }
  }
  if (tid == 0) go.qx_zero[b] = qzero ? 1 : 0;
}

// S and D of row group blockIdx.x of frequency blockIdx.y, runs of eight rows g per .. (g + 1) per,
// for the G_X blocks of the next launch to add up.
template <int XL>
__global__ void __launch_bounds__(512) k_gramx_part(const float2* __restrict__ xt, int n1, int r, int per, double2* __restrict__ part) {
  constexpr int NT = XL * (XL + 1) / 2;
  extern __shared__ __align__(16) unsigned char psm[];
  const int g = blockIdx.x, b = blockIdx.y, lane = threadIdx.x & 63, w = threadIdx.x >> 6, m = lane & 15, q = lane >> 4, rr = r * r;
  BgTile gs[NT], gd[NT];
#pragma unroll
  for (int k = 0; k < NT; ++k) gs[k].re = gs[k].im = gd[k].re = gd[k].im = v4d{0.0, 0.0, 0.0, 0.0};
  const int nks = (n1 + 7) >> 3, k0 = min(nks, g * per);
  gramx_rows<XL, 8>(xt, b, n1, r, k0, min(nks, k0 + per), gs, gd);
  bg_reduce<8>(gs, (double2*)psm, w, lane);
  bg_reduce<8>(gd, (double2*)psm, w, lane);
  if (w != 0) return;
  double2* out = part + ((size_t)b * gridDim.x + g) * 2 * rr;
  int t = 0;
#pragma unroll
  for (int a = 0; a < XL; ++a)
#pragma unroll
    for (int c = a; c < XL; ++c, ++t) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int s = 16 * a + q + 4 * e, u = 16 * c + m;
        if (s < r && u < r) {
          out[s * r + u] = make_double2(gs[t].re[e], gs[t].im[e]);
          out[rr + s * r + u] = make_double2(gd[t].re[e], gd[t].im[e]);
        }
      }
    }
}

// Blocks 0 .. nb - 1: G_X of frequency blockIdx.x (the longest chain, so they start first);
// the others: the product.  Block order of the product: the column groups of one frequency run
// on one XCD (blocks are dealt to the eight XCDs in turn), so each XCD's L2 holds the X~ rows of
// its own frequencies only.
// The bound of 2 keeps the two-wavefront instances from the accumulator registers, whose moves cost
// more than they save (12 x 12 x 8064: 37 us with them, 26 without).
template <int XL, int WL, bool MX, int W>   // r <= 16 XL, 16 WL complex columns and W wavefronts per block, MX: W~ in BF16
__global__ void __launch_bounds__(64 * W, 2) k_bgemm(const void* __restrict__ wt, const float2* __restrict__ xt,
                                                      double2* __restrict__ bout, int n1, int n2, int r, int nb,
                                                      int ncg, GramOut go) {
  constexpr int KG = BgShape<XL, WL>::KG;
  extern __shared__ __align__(16) unsigned char bsm[];
  if ((int)blockIdx.x < nb) {
    gramx_block<XL, W>(xt, (int)blockIdx.x, n1, r, go, bsm);
    return;
  }
  // XCD-aware order: block id -> (frequency, column group)
  const int nblk = (int)gridDim.x - nb, id = (int)blockIdx.x - nb, x = id & 7, qd = nblk >> 3, rem = nblk & 7;
  const int lid = x * qd + min(x, rem) + (id >> 3);
  const int b = lid / ncg, cg = lid % ncg, j0 = 16 * WL * cg;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, m = lane & 15, q = lane >> 4;
  const int nks = (n1 + 3) >> 2, per = (nks + W - 1) / W;
  const int ks0 = min(nks, w * per), ks1 = min(nks, ks0 + per);
  BgTile acc[XL * WL];
#pragma unroll
  for (int k = 0; k < XL * WL; ++k) acc[k].re = acc[k].im = v4d{0.0, 0.0, 0.0, 0.0};
  float2 xa[KG][XL], wa[KG][WL], xb[KG][XL], wb[KG][WL];
  bg_load<XL, WL, MX>(wt, xt, ks0, ks1, q, m, b, r, n1, n2, nb, j0, xa, wa);
  for (int ks = ks0; ks < ks1; ks += 2 * KG) {
    if (ks + KG < ks1) bg_load<XL, WL, MX>(wt, xt, ks + KG, ks1, q, m, b, r, n1, n2, nb, j0, xb, wb);
    bg_mfma<XL, WL>(xa, wa, ks1 - ks, acc);
    if (ks + KG >= ks1) break;
    if (ks + 2 * KG < ks1) bg_load<XL, WL, MX>(wt, xt, ks + 2 * KG, ks1, q, m, b, r, n1, n2, nb, j0, xa, wa);
    bg_mfma<XL, WL>(xb, wb, ks1 - ks - KG, acc);
  }
  bg_reduce<W>(acc, (double2*)bsm, w, lane);
  if (w != 0) return;
#pragma unroll
  for (int a = 0; a < XL; ++a)
#pragma unroll
    for (int u = 0; u < WL; ++u)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int s = 16 * a + q + 4 * t, j = j0 + 16 * u + m;
        if (s < r && j < n2) bout[((size_t)b * r + s) * n2 + j] = make_double2(acc[a * WL + u].re[t], acc[a * WL + u].im[t]);
      }
}

// Wavefronts per block: 8, or 2 where there are many frequencies of few rows (12 x 12 x 8064:
// 139 us with 8, 26 with 2).
static int bgemm_waves(const Plan& p) { return p.n1 <= 64 && p.nb >= 256 ? 2 : 8; }

static size_t bgemm_lds_bytes(int r, int bcg, int waves) {
  const int xl = r <= 16 ? 1 : 2, tiles = xl * (bcg / 16), gtiles = xl * (xl + 1) / 2;
  const size_t red = (size_t)(waves / 2) * (tiles > gtiles ? tiles : gtiles) * 4 * 64 * sizeof(double2);
  return red > pinv_lds_bytes(r) ? red : pinv_lds_bytes(r);
}
// More than half a compute unit's LDS: blocks of a launch with no more of them than units, in which
// the matrix cores bound each, do not meet on one (three of 3600 x 2 x 26, r = 2, together 184 us per
// iteration with the LDS that they use, 180 so).
#define BG_LDS_ALONE (84 * 1024)

bool bgemm_cols_valid(int r, int bcg) { return (bcg == 16 || bcg == 32) && r <= 32; }

typedef void (*BgemmKernel)(const void*, const float2*, double2*, int, int, int, int, int, GramOut);
template <int XL, int W>
static BgemmKernel bgemm_kernel(int bcg, int mixed) {
  if (bcg == 32) return mixed ? k_bgemm<XL, 2, true, W> : k_bgemm<XL, 2, false, W>;
  return mixed ? k_bgemm<XL, 1, true, W> : k_bgemm<XL, 1, false, W>;
}
template <int XL>
static BgemmKernel bgemm_kernel_of(int bcg, int mixed, int waves) {
  return waves == 2 ? bgemm_kernel<XL, 2>(bcg, mixed) : bgemm_kernel<XL, 8>(bcg, mixed);
}

// Row groups of G_X in a launch of their own, 0: all rows in the block that inverts it.  Up to r = 16
// that block's sums are no longer than the product's beside it, but at r > 16, or for thousands of
// rows with few frequencies or an inverse by the eigen route after them, they are the launch's chain
// (and members of a batch whose chains meet on a compute unit share its matrix cores): groups of at
// least 96 rows, four or more, and no more blocks than compute units.  One iteration in us, one
// block / groups: 8192 x 32 x 3, r = 32 533 / 388; 1500 x 24 x 112, r = 17 206 / 190; 384 x 24 x 5, r =
// 24 83.4 / 78.7; 600 x 24 x 200, r = 24 (two groups) 198 / 207; 8192 x 16 x 7, r = 16 170 / 165; 2000 x
// 12 x 28, r = 12 76.3 / 76.2; 4000 x 24 x 112, r = 16 199 / 220, by the eigen route 507 / 467; 1000 x 16
// x 12, r = 16, eigen 402 / 401; three of 6591 x 7 x 2, r = 4, together 250 / 190.
static int gramx_groups(const Plan& p) {
  if (p.r <= 16 && !(p.n1 >= 2000 && (p.force_eigen || p.nb <= 16))) return 0;
  int g = p.n1 / 96;
  if (g > 256 / p.nb) g = 256 / p.nb;
  // the partials lie in Z~'s buffer: 32 r^2 bytes each in 8 n1 n2 per frequency
  const long room = (long)p.n1 * p.n2 / (4 * p.r * p.r);
  if (g > room) g = (int)room;
  return g >= 4 ? g : 0;
}

// X~^* W~ -> bpart [nb][r][n2]; G_X, (H X~)^*(H X~), G_X^+ and I - eta P_X.
void launch_bgemm(const Plan& p) {
  GramOut go;
  go.gxm = p.gxm;
  go.dmat = p.dmat;
  go.gxp = p.gxp;
  go.qx = p.qx;
  go.qx_zero = p.qx_zero;
  go.rho1 = p.rho1;
  go.eta = p.eta;
  go.force_eigen = p.force_eigen;
  go.part = (double2*)p.zt;   // Z~ is formed anew after this launch
  go.npart = gramx_groups(p);
  if (go.npart > 0) {
    const int per = ((p.n1 + 7) / 8 + go.npart - 1) / go.npart;
    const dim3 grid(go.npart, p.nb);
    const size_t lds = bgemm_lds_bytes(p.r, 16, 8);
    if (p.r <= 16) k_gramx_part<1><<<grid, 512, lds, p.stream>>>(p.xt, p.n1, p.r, per, go.part);
    else k_gramx_part<2><<<grid, 512, lds, p.stream>>>(p.xt, p.n1, p.r, per, go.part);
  }
  const int ncg = (p.n2 + p.bcg - 1) / p.bcg, waves = bgemm_waves(p);
  size_t lds = bgemm_lds_bytes(p.r, p.bcg, waves);
  if ((1 + ncg) * p.nb <= 256 && lds < BG_LDS_ALONE) lds = BG_LDS_ALONE;
  const BgemmKernel kernel = p.r <= 16 ? bgemm_kernel_of<1>(p.bcg, p.mixed, waves) : bgemm_kernel_of<2>(p.bcg, p.mixed, waves);
  if (lds > 65536) (void)hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  kernel<<<p.nb + ncg * p.nb, 64 * waves, lds, p.stream>>>(p.wt, p.xt, p.bpart, p.n1, p.n2, p.r, p.nb, ncg, go);
}

}  // namespace tctf
