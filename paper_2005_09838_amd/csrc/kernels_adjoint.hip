// Reverse-mode derivatives of one TCTF2R iteration, in FP64 throughout.
//
// The forward iteration (section 4.1, algorithm box steps 1-4 and 7) with full-rank Grams
// and the common step eta maps (X~, Y~, W) to
//   X~+ = (1 - eta) X~ + eta H_rho1^{-1} W~ Y~^* G_Y^{-1},        G_Y = Y~ Y~^*,
//   Y~+ = (1 - eta) Y~ + eta G_X^{-1} X~+^* W~,                   G_X = X~+^* H_rho1 X~+,
//   Z   = Re idft(X~+ Y~+)                                         (eq. (barAAk)),
//   W+  = the W-step of eq. (subquKKT) at Z,  W~ = dft(W)          (eq. (bar BA-k)),
// (the pseudo-inverse updates of eq. (updataXYW1) reduce to these when the Grams have full
// rank, since grad_X = H_rho1 X~ G_Y - W~ Y~^* and grad_Y = G_X Y~ - X~^* W~).
// The kernels below run the reverse pass of that map.  Adjoint convention for a real loss
// L: the adjoint of a complex entry z is dL/dRe z + i dL/dIm z; a stored frequency b
// carries the adjoint it has in the sum over all n3 frequencies.  Per frequency the rules
// are those of products (C = A B: A_bar += C_bar B^*, B_bar += A^* C_bar), inverses
// (C = G^{-1}: G_bar = -C^* C_bar C^*) and Grams (G = Y Y^*: Y_bar += (G_bar + G_bar^*) Y);
// across frequencies only the tube transforms and the weight adjoints couple them, through
// the bin weights c_b.  The W-step's adjoint solves the same tridiagonal system restricted
// to the unobserved entries of each row (i, :, k) (K_{mu rho2} is symmetric).
//
// The parts: a batched complex GEMM on the FP64 matrix cores over strided views (FP32 forward
// values or FP64 adjoints), tridiagonal H_rho1 applications and solves along n1, the FP64
// tube transforms, FP64 Gram inverses by the library's Hermitian pseudo-inverse, and
// fixed-order reductions for the weights' adjoints.
#include "kernels.h"
#include "pinv.h"

namespace tctf {

// ---------------------------------------------------------------- batched complex GEMM
template <bool F32>
__device__ __forceinline__ cd ld_view(const CView& v, long e) {
  if constexpr (F32) {
    const float2 f = ((const float2*)v.p)[e];
    return cd_make(f.x, f.y);
  } else {
    const double2 d = ((const double2*)v.p)[e];
    return cd_make(d.x, d.y);
  }
}

typedef double v4d __attribute__((ext_vector_type(4)));

// C = alpha A B + beta D for every batch b (blockIdx.z); A is M x K, B is K x N, C and D are M x N
// FP64 complex at b cbs + i crs + j ccs (D may be C; beta = 0 does not read it).
//
// A wavefront forms a 16 x 16 tile on the FP64 matrix cores, 16 of K (four steps of four products)
// per turn with the turn's eight loads in flight at once and no LDS: lane (m, q) holds A(m, 4 s + q)
// and B(4 s + q, m).  The products of this file are small (the tiles of M x N are fewer than the
// compute units) and latency bounds them, so where K > 64 the NW = 8 wavefronts of a block share a
// tile's K and their sums are added in LDS in a fixed order; else a block's four wavefronts take
// four tiles along N.  The products of one step at 144 x 288 x 28, r 8: 3.6 to 7.9 us, 6.0 on
// average (10.4 on 16 x 16 LDS tiles with two barriers per 16 of K).
struct Gemm64 {
  int M, N, K;
  cd alpha, beta;
  CView A, B;
  const double2* D;
  double2* C;
  long cbs, crs, ccs;
};
__device__ __forceinline__ void gemm64_out(const Gemm64& g, int b, int i, int j, cd acc) {
  if (i >= g.M || j >= g.N) return;
  const long e = (long)b * g.cbs + (long)i * g.crs + (long)j * g.ccs;
  cd v = cd_mul(g.alpha, acc);
  if (g.beta.re != 0.0 || g.beta.im != 0.0) v = cd_add(v, cd_mul(g.beta, cd_make(g.D[e].x, g.D[e].y)));
  g.C[e] = make_double2(v.re, v.im);
}

template <bool AF, bool BF, bool SPLIT>
__global__ void __launch_bounds__(SPLIT ? 512 : 256) k_zgemm64(Gemm64 g) {
  constexpr int NW = SPLIT ? 8 : 1;   // wavefronts on one tile's K
  __shared__ double sums[SPLIT ? 8 * 256 * 2 : 1];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, m = lane & 15, q = lane >> 4, b = blockIdx.z;
  const int i0 = blockIdx.y * 16, j0 = (SPLIT ? blockIdx.x : blockIdx.x * 4 + wid) * 16;
  const long ra = b * g.A.bs + min(i0 + m, g.M - 1) * g.A.rs, rb = b * g.B.bs + min(j0 + m, g.N - 1) * g.B.cs;
  const double ca = g.A.conj ? -1.0 : 1.0, cb = g.B.conj ? -1.0 : 1.0;
  v4d re = {0.0, 0.0, 0.0, 0.0}, im = re;
  for (int k0 = 16 * (SPLIT ? wid : 0); k0 < g.K; k0 += 16 * NW) {
    cd x[4], y[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int k = min(k0 + 4 * s + q, g.K - 1);
      x[s] = ld_view<AF>(g.A, ra + k * g.A.cs);
      y[s] = ld_view<BF>(g.B, rb + k * g.B.rs);
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      if (k0 + 4 * s < g.K) {
        const bool in = k0 + 4 * s + q < g.K;
        const double xr = in ? x[s].re : 0.0, xi = in ? ca * x[s].im : 0.0;
        const double yr = in ? y[s].re : 0.0, yi = in ? cb * y[s].im : 0.0;
        re = __builtin_amdgcn_mfma_f64_16x16x4f64(xr, yr, re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(xr, yi, im, 0, 0, 0);
        re = __builtin_amdgcn_mfma_f64_16x16x4f64(-xi, yi, re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(xi, yr, im, 0, 0, 0);
      }
    }
  }
  if constexpr (SPLIT) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {   // row q + 4 t, column m
      const int e = (q + 4 * t) * 16 + m;
      sums[2 * (wid * 256 + e)] = re[t];
      sums[2 * (wid * 256 + e) + 1] = im[t];
    }
    __syncthreads();
    if (threadIdx.x < 256) {
      const int f = threadIdx.x, i = g.crs == 1 ? f & 15 : f >> 4, j = g.crs == 1 ? f >> 4 : f & 15;
      cd acc = cd_make(0.0, 0.0);
#pragma unroll
      for (int w = 0; w < 8; ++w) {
        const int e = 2 * (w * 256 + i * 16 + j);
        acc = cd_add(acc, cd_make(sums[e], sums[e + 1]));
      }
      gemm64_out(g, b, i0 + i, j0 + j, acc);
    }
  } else {
#pragma unroll
    for (int t = 0; t < 4; ++t) gemm64_out(g, b, i0 + q + 4 * t, j0 + m, cd_make(re[t], im[t]));
  }
}

template <bool AF, bool BF>
static void gemm64(const Plan& p, const Gemm64& g) {
  const unsigned tm = (g.M + 15) / 16, tn = (g.N + 15) / 16;
  if (g.K > 64) k_zgemm64<AF, BF, true><<<dim3(tn, tm, p.nb), 512, 0, p.stream>>>(g);
  else k_zgemm64<AF, BF, false><<<dim3((tn + 3) / 4, tm, p.nb), 256, 0, p.stream>>>(g);
}
static void gemm_add(const Plan& p, int M, int N, int K, cd alpha, CView A, CView B, cd beta, const double2* D, double2* C,
                     long cbs, long crs, long ccs) {
  Gemm64 g;
  g.M = M;
  g.N = N;
  g.K = K;
  g.alpha = alpha;
  g.beta = beta;
  g.A = A;
  g.B = B;
  g.D = D;
  g.C = C;
  g.cbs = cbs;
  g.crs = crs;
  g.ccs = ccs;
  if (A.f32 && B.f32) gemm64<true, true>(p, g);
  else if (A.f32) gemm64<true, false>(p, g);
  else if (B.f32) gemm64<false, true>(p, g);
  else gemm64<false, false>(p, g);
}
static void gemm(const Plan& p, int M, int N, int K, cd alpha, CView A, CView B, cd beta, double2* C, long cbs, long crs,
                 long ccs) {
  gemm_add(p, M, N, K, alpha, A, B, beta, C, C, cbs, crs, ccs);
}

static CView view(const void* ptr, long bs, long rs, long cs, int f32) {
  CView v;
  v.p = ptr;
  v.bs = bs;
  v.rs = rs;
  v.cs = cs;
  v.f32 = f32;
  v.conj = 0;
  return v;
}
static CView ctr(CView v) {   // conjugate transpose of a view
  const long t = v.rs;
  v.rs = v.cs;
  v.cs = t;
  v.conj ^= 1;
  return v;
}

// ---------------------------------------------------------------- elementwise helpers
// The step length's share of an adjoint: u <- (1 - eta) a, v <- eta a for a: [nb][per] complex, after
// the imaginary parts of the real frequencies (b = 0 and the Nyquist bin) are set to 0 (the forward
// update does this to its results, and the map is its own adjoint).
__global__ void k_adj_split(const double2* __restrict__ a, long per, int nb, int n3, double eta, double2* __restrict__ u,
                            double2* __restrict__ v) {
  const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= per * nb) return;
  double2 x = a[e];
  if (bin_is_real((int)(e / per), n3)) x.y = 0.0;
  u[e] = make_double2((1.0 - eta) * x.x, (1.0 - eta) * x.y);
  v[e] = make_double2(eta * x.x, eta * x.y);
}
static void split(const Plan& p, const double2* a, long per, double2* u, double2* v) {
  k_adj_split<<<(unsigned)((per * p.nb + 255) / 256), 256, 0, p.stream>>>(a, per, p.nb, p.n3, p.eta, u, v);
}

// The inverse's rule on the r x r adjoints, one block per frequency: G_bar = -C^* C_bar C^* and
// S = G_bar + G_bar^*, C = G^{-1}.
__global__ void __launch_bounds__(256) k_adj_gram(const double2* __restrict__ gi, const double2* __restrict__ gib,
                                                  double2* __restrict__ gb, double2* __restrict__ s, int r) {
  extern __shared__ __align__(16) unsigned char sm[];
  const int rr = r * r;
  cd* c = (cd*)sm;
  cd* x = c + rr;
  cd* y = x + rr;
  const long o = (long)blockIdx.x * rr;
  for (int e = threadIdx.x; e < rr; e += blockDim.x) {
    c[e] = cd_make(gi[o + e].x, gi[o + e].y);
    x[e] = cd_make(gib[o + e].x, gib[o + e].y);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < rr; e += blockDim.x) {   // C^* C_bar
    const int i = e / r, j = e % r;
    cd acc = cd_make(0.0, 0.0);
    for (int k = 0; k < r; ++k) cd_fma(acc, cd_make(c[k * r + i].re, -c[k * r + i].im), x[k * r + j]);
    y[e] = acc;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < rr; e += blockDim.x) {   // times -C^*
    const int i = e / r, j = e % r;
    cd acc = cd_make(0.0, 0.0);
    for (int k = 0; k < r; ++k) cd_fma(acc, y[i * r + k], cd_make(-c[j * r + k].re, c[j * r + k].im));
    x[e] = acc;
    gb[o + e] = make_double2(acc.re, acc.im);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < rr; e += blockDim.x) {
    const cd u = x[e], v = x[(e % r) * r + e / r];
    s[o + e] = make_double2(u.re + v.re, u.im - v.im);
  }
}
static void gram_adjoint(const Plan& p, const double2* gi, const double2* gib, double2* gb, double2* s) {
  k_adj_gram<<<p.nb, 256, 3 * (size_t)p.r * p.r * sizeof(cd), p.stream>>>(gi, gib, gb, s, p.r);
}

// out(b, s, i) = (a + c deg_i) x_i - c (x_{i-1} + x_{i+1}) along n1 for X-shaped arrays
// [nb][r][n1] (deg_i = number of neighbours of row i): H_rho1 with (1, rho1), D^T D with (0, 1).
template <typename T>
__global__ void k_adj_happly(const T* __restrict__ x, double2* __restrict__ out, int n1, long total, double a,
                             double c) {
  const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= total) return;
  const int i = (int)(e % n1);
  const double deg = (n1 == 1) ? 0.0 : ((i == 0 || i == n1 - 1) ? 1.0 : 2.0);
  auto get = [&](long k) { return cd_make((double)x[k].x, (double)x[k].y); };
  cd v = cd_scale(get(e), a + c * deg);
  if (i > 0) v = cd_sub(v, cd_scale(get(e - 1), c));
  if (i + 1 < n1) v = cd_sub(v, cd_scale(get(e + 1), c));
  out[e] = make_double2(v.re, v.im);
}

// y = H_rho1^{-1} x for every column (b, s) of two X-shaped arrays (blockIdx.y), one wavefront per
// column: d_i = (x_i + rho1 d_{i-1}) / alpha_i down the column, then y_i = d_i + (rho1 / alpha_i)
// y_{i+1} up, as scans of affine maps over 64 entries at a time.  120 columns of 144 entries, both
// arrays: 5.7 us (131 with a thread per column).
__device__ __forceinline__ void hscan(double& a, double& br, double& bi, int dir) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int from = lane - dir * off;
    const double ao = __shfl(a, from & 63), ro = __shfl(br, from & 63), io = __shfl(bi, from & 63);
    if (from >= 0 && from < 64) {
      br = fma(a, ro, br);
      bi = fma(a, io, bi);
      a *= ao;
    }
  }
}
__global__ void __launch_bounds__(256) k_adj_hsolve(const double2* __restrict__ x0, double2* __restrict__ y0,
                                                    const double2* __restrict__ x1, double2* __restrict__ y1, int n1,
                                                    long ncol, const double* __restrict__ htab) {
  const long col = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (col >= ncol) return;
  const int lane = threadIdx.x & 63, nch = (n1 + 63) / 64;
  const double2* xc = (blockIdx.y ? x1 : x0) + col * n1;
  double2* yc = (blockIdx.y ? y1 : y0) + col * n1;
  double cr = 0.0, ci = 0.0;
  for (int ch = 0; ch < nch; ++ch) {
    const int i = 64 * ch + lane, at = min(i, n1 - 1);
    const double2 v = xc[at];
    const double inv = htab[n1 + at];
    double a = at > 0 ? htab[2 * n1 + at] : 0.0, br = v.x * inv, bi = v.y * inv;
    hscan(a, br, bi, 1);
    br = fma(a, cr, br);
    bi = fma(a, ci, bi);
    if (i < n1) yc[i] = make_double2(br, bi);
    cr = __shfl(br, 63);
    ci = __shfl(bi, 63);
  }
  cr = ci = 0.0;
  for (int ch = nch - 1; ch >= 0; --ch) {
    const int i = 64 * ch + lane;
    double a = 0.0, br = 0.0, bi = 0.0;   // past the end: 0
    if (i < n1) {
      const double2 d = yc[i];
      a = i + 1 < n1 ? htab[2 * n1 + i] : 0.0;
      br = d.x;
      bi = d.y;
    }
    hscan(a, br, bi, -1);
    br = fma(a, cr, br);
    bi = fma(a, ci, bi);
    if (i < n1) yc[i] = make_double2(br, bi);
    cr = __shfl(br, 0);
    ci = __shfl(bi, 0);
  }
}

// G^{-1} of every frequency's r x r Gram (FP64 pseudo-inverse of Lemma SVPMPI, which is
// the inverse at full rank); flag[0] = 1 if some Gram is rank deficient.
__global__ void __launch_bounds__(256) k_adj_inv(const double2* __restrict__ g, double2* __restrict__ gi, int r,
                                                 int* flag) {
  extern __shared__ __align__(16) unsigned char sm[];
  const int b = blockIdx.x, rr = r * r;
  cd* a = (cd*)sm;
  cd* p = a + rr;
  PinvScratch ps;
  ps.work = p + rr;
  ps.vec = ps.work + rr;
  ps.rot = (double*)(ps.vec + rr);
  ps.red = ps.rot + 96;
  for (int e = threadIdx.x; e < rr; e += blockDim.x) a[e] = cd_make(g[(long)b * rr + e].x, g[(long)b * rr + e].y);
  __syncthreads();
  const int full = pinv_herm(a, p, r, 0, ps);
  for (int e = threadIdx.x; e < rr; e += blockDim.x) gi[(long)b * rr + e] = make_double2(p[e].re, p[e].im);
  if (threadIdx.x == 0 && !full) flag[0] = 1;
}

// ---------------------------------------------------------------- W-step adjoint
// For every row (i, :, k): lambda solves K_uu lambda_u = w_bar_u with lambda_o = 0
// (K_{mu rho2} = (1 + mu) I + rho2 K^T K restricted to the unobserved entries), z_bar = lambda;
// partial sums of -<lambda, w> (mu) and -<lambda, K^T K w> = -sum of products of differences
// (rho2) per block.
//
// Block (x, i): S = 2^ls segments of at most L columns of the rows (i, :, k), k = x KB .. + KB,
// KB = 256 / S, a thread per (segment, row).  With the tabulated pivots elimination and back
// substitution are affine maps of the value that enters a segment, so each thread forms its
// segment's map, takes the incoming value through the maps before it from LDS, and repeats its
// columns.  What bounds it: the latency of the loads (all in flight at once) and of the chains of
// L + S steps.  144 x 288 x 28: 18.4 us (516 with a thread per row and a division per entry).
template <int L>
__global__ void __launch_bounds__(256) k_adj_wstep(const double* __restrict__ wbar, const double* __restrict__ w,
                                                   const float* __restrict__ gp, double* __restrict__ zbar,
                                                   const double* __restrict__ wtab, int n2, int n3, double rho2,
                                                   int gseg, int ls, double* __restrict__ part) {
  __shared__ double red[48];
  __shared__ double ma[256], mb[256], na[256], nb[256];
  const int S = 1 << ls, KB = 256 >> ls, tid = threadIdx.x, s = tid >> (8 - ls), kk = tid & (KB - 1);
  const int k = blockIdx.x * KB + kk, kc = min(k, n3 - 1), len = (n2 + S - 1) >> ls;
  const int j0 = s * len, cnt = k < n3 ? min(len, n2 - j0) : 0;   // may be negative: no columns
  const long i = blockIdx.y, base = i * n2 * n3 + kc;
  double x[L], wj[L], inv[L];
  float g[L];
#pragma unroll
  for (int u = 0; u < L; ++u) {
    const int j = min(j0 + u, n2 - 1);
    x[u] = wbar[base + (long)j * n3];
    wj[u] = w[base + (long)j * n3];
    g[u] = gp[packed_g_at(i, j, kc, n2, n3, gseg)];
  }
  const double wr = w[base + (long)min(j0 + max(cnt, 0), n2 - 1) * n3];   // right of the segment
#pragma unroll
  for (int u = 0; u < L; ++u) {
    const bool un = u < cnt && is_unobserved(g[u]);
    const double t = wtab[un ? unobs_index(g[u]) : 0];
    inv[u] = un ? t : 0.0;   // 0: lambda = 0, and nothing passes
    if (!un) x[u] = 0.0;
  }
  double a = 1.0, b = 0.0;
#pragma unroll
  for (int u = 0; u < L; ++u) {
    if (u < cnt) {
      b = inv[u] * fma(rho2, b, x[u]);
      a *= rho2 * inv[u];
    }
  }
  ma[tid] = a;
  mb[tid] = b;
  __syncthreads();
  double d = 0.0;
  for (int t = kk; t < s * KB; t += KB) d = fma(ma[t], d, mb[t]);
#pragma unroll
  for (int u = 0; u < L; ++u) {
    if (u < cnt) d = inv[u] * fma(rho2, d, x[u]);
    x[u] = d;
  }
  a = cnt > 0 ? 1.0 : 0.0;
  b = 0.0;
#pragma unroll
  for (int u = L - 1; u >= 0; --u) {
    if (u < cnt) {
      const double c = rho2 * inv[u];
      b = fma(c, b, x[u]);
      a *= c;
    }
  }
  na[tid] = a;
  nb[tid] = b;
  __syncthreads();
  double lam = 0.0, smu = 0.0, srho = 0.0;
  for (int t = 256 - KB + kk; t > tid; t -= KB) lam = fma(na[t], lam, nb[t]);
#pragma unroll
  for (int u = L - 1; u >= 0; --u) {
    if (u < cnt) {
      const double right = lam, wn = u + 1 < cnt ? wj[u + 1 < L ? u + 1 : u] : wr;
      lam = fma(rho2 * inv[u], lam, x[u]);
      zbar[base + (long)(j0 + u) * n3] = lam;
      smu -= lam * wj[u];
      if (j0 + u + 1 < n2) srho -= (right - lam) * (wn - wj[u]);
    }
  }
  double zero = 0.0;
  block_sum3_d(smu, srho, zero, red);
  if (tid == 0) {
    const long blk = i * gridDim.x + blockIdx.x;
    part[2 * blk] = smu;
    part[2 * blk + 1] = srho;
  }
}

// Segments of at most 16 columns; no more of them than that needs, so that as many lanes as
// possible read consecutive words.  Returns the number of partials.
static int wstep_adjoint(const Plan& p, const AdjWork& w, const double* w_bar) {
  int ls = 0;
  while (((p.n2 + (1 << ls) - 1) >> ls) > 16) ++ls;   // n2 <= 1024: ls <= 6
  const int len = (p.n2 + (1 << ls) - 1) >> ls, KB = 256 >> ls;
  const dim3 grid((p.n3 + KB - 1) / KB, p.n1);
  const auto kernel = len <= 9 ? k_adj_wstep<9> : (len <= 12 ? k_adj_wstep<12> : k_adj_wstep<16>);
  kernel<<<grid, 256, 0, p.stream>>>(w_bar, w.w1s, p.gp, w.zbar, w.wtab, p.n2, p.n3, p.rho2, p.gseg, ls, w.wpart);
  return (int)(grid.x * grid.y);
}

// theta[k0] += sum of part[2 b], theta[k1] += sum of part[2 b + 1] (fixed order)
__global__ void k_adj_reduce2(const double* __restrict__ part, int nblk, double* theta, int k0, int k1) {
  __shared__ double red[16];
  double a = 0.0, c = 0.0;
  for (int b = threadIdx.x; b < nblk; b += blockDim.x) {
    a += part[2 * b];
    c += part[2 * b + 1];
  }
  a = block_sum_d(a, red);
  c = block_sum_d(c, red);
  if (threadIdx.x == 0) {
    theta[k0] += a;
    theta[k1] += c;
  }
}

// theta[k] += coef sum_b c_b Re sum_e conj(A(b, e)) B(b, e); A, B: [nb][per] complex.
// Partials per block in part[], then one block adds them in a fixed order.
__global__ void __launch_bounds__(256) k_adj_wdot(const double2* __restrict__ A, const double2* __restrict__ B,
                                                  long per, int nb, int n3, double* __restrict__ part) {
  __shared__ double red[16];
  double s = 0.0;
  const long n = per * nb;
  for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (long)gridDim.x * blockDim.x) {
    const double2 a = A[e], b = B[e];
    s += bin_weight((int)(e / per), n3) * (a.x * b.x + a.y * b.y);
  }
  s = block_sum_d(s, red);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}
__global__ void k_adj_reduce1(const double* __restrict__ part, int nblk, double coef, double* theta, int k) {
  __shared__ double red[16];
  double a = 0.0;
  for (int b = threadIdx.x; b < nblk; b += blockDim.x) a += part[b];
  a = block_sum_d(a, red);
  if (threadIdx.x == 0) theta[k] += coef * a;
}

__global__ void k_adj_flag_zero(int* flag) {
  if (threadIdx.x == 0 && blockIdx.x == 0) flag[0] = 0;
}

// ---------------------------------------------------------------- host side
#define ADJ_DOT_BLOCKS 256

size_t adjoint_work_bytes(const Plan& p) {
  const size_t N = (size_t)p.n1 * p.n2 * p.n3, nh = (size_t)p.nb * p.n1 * p.n2;
  const size_t fx = (size_t)p.nb * p.r * p.n1, fy = (size_t)p.nb * p.r * p.n2, g = (size_t)p.nb * p.r * p.r;
  auto al = [](size_t b) { return (b + 255) & ~(size_t)255; };
  return 2 * al(N * 8) + 2 * al(nh * 16) + 9 * al(fx * 16) + 4 * al(fy * 16) + 10 * al(g * 16) +
         al(3 * (size_t)p.n1 * 8) + al(4 * (size_t)p.n2 * 8) + al(ADJ_DOT_BLOCKS * 8) + al(64);
}

void adjoint_carve(const Plan& p, void* ws, AdjWork* w) {
  const size_t N = (size_t)p.n1 * p.n2 * p.n3, nh = (size_t)p.nb * p.n1 * p.n2;
  const size_t fx = (size_t)p.nb * p.r * p.n1, fy = (size_t)p.nb * p.r * p.n2, g = (size_t)p.nb * p.r * p.r;
  unsigned char* o = (unsigned char*)ws;
  auto take = [&](size_t bytes) { unsigned char* at = o; o += (bytes + 255) & ~(size_t)255; return (void*)at; };
  w->w1s = (double*)take(N * 8);
  w->zbar = (double*)take(N * 8);
  w->ztb = (double2*)take(nh * 16);
  w->wtb = (double2*)take(nh * 16);
  double2** xs[9] = {&w->x1b, &w->hx1, &w->a, &w->pp, &w->q, &w->pb, &w->qb, &w->ab, &w->dt};
  for (auto q : xs) *q = (double2*)take(fx * 16);
  double2** ys[4] = {&w->y1b, &w->bm, &w->bb, &w->rb};
  for (auto q : ys) *q = (double2*)take(fy * 16);
  double2** gs[10] = {&w->gy, &w->gyi, &w->gx, &w->gxi, &w->gyib, &w->gxib, &w->gyb, &w->gxb, &w->S, &w->T};
  for (auto q : gs) *q = (double2*)take(g * 16);
  w->htab = (double*)take(3 * (size_t)p.n1 * 8);
  w->wtab = (double*)take(4 * (size_t)p.n2 * 8);
  w->part = (double*)take(ADJ_DOT_BLOCKS * 8);
  w->wpart = (double*)w->ztb;   // the W-step's partials, read before ztb is written
  w->flag = (int*)take(64);
}

void adjoint_set_attr(int r) {
  if (pinv_lds_bytes(r) > 65536)
    (void)hipFuncSetAttribute((const void*)k_adj_inv, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)pinv_lds_bytes(r));
}

static void inv(const Plan& p, const AdjWork& w, const double2* g, double2* gi) {
  k_adj_inv<<<p.nb, 256, pinv_lds_bytes(p.r), p.stream>>>(g, gi, p.r, w.flag);
}

static void wdot_add(const Plan& p, const AdjWork& w, const double2* A, const double2* B, long per, double coef,
                     double* theta, int k) {
  k_adj_wdot<<<ADJ_DOT_BLOCKS, 256, 0, p.stream>>>(A, B, per, p.nb, p.n3, w.part);
  k_adj_reduce1<<<1, 256, 0, p.stream>>>(w.part, ADJ_DOT_BLOCKS, coef, theta, k);
}

template <typename T>
static void happly(const Plan& p, const T* x, double2* out, double a, double c) {
  const long total = (long)p.nb * p.r * p.n1;
  k_adj_happly<T><<<(unsigned)((total + 255) / 256), 256, 0, p.stream>>>(x, out, p.n1, total, a, c);
}

static void hsolve2(const Plan& p, const AdjWork& w, const double2* x0, double2* y0, const double2* x1, double2* y1) {
  const long ncol = (long)p.nb * p.r;
  k_adj_hsolve<<<dim3((unsigned)((ncol + 3) / 4), 2), 256, 0, p.stream>>>(x0, y0, x1, y1, p.n1, ncol, w.htab);
}

void launch_adjoint_step(const Plan& p, const AdjWork& w, const AdjState& in, const AdjState& out, double2* xt_bar,
                         double2* yt_bar, double* w_bar, double* theta) {
  const int n1 = p.n1, n2 = p.n2, n3 = p.n3, r = p.r, nb = p.nb;
  const cd one = cd_make(1.0, 0.0), zero = cd_make(0.0, 0.0);
  // matrix views of the forward values (FP32): X [nb][r][n1] as n1 x r, Y [nb][r][n2] as
  // r x n2, W~ [n1][nb][n2] as n1 x n2
  const CView X = view(in.xt, (long)r * n1, 1, n1, 1), Y = view(in.yt, (long)r * n2, n2, 1, 1);
  const CView Wt = view(in.wt, n2, (long)nb * n2, 1, 1);
  const CView X1 = view(out.xt, (long)r * n1, 1, n1, 1), Y1 = view(out.yt, (long)r * n2, n2, 1, 1);
  (void)X;
  auto xv = [&](const double2* a) { return view(a, (long)r * n1, 1, n1, 0); };      // n1 x r, [nb][r][n1]
  auto yv = [&](const double2* a) { return view(a, (long)r * n2, n2, 1, 0); };      // r x n2
  auto gv = [&](const double2* a) { return view(a, (long)r * r, r, 1, 0); };        // r x r
  auto hv = [&](const double2* a) { return view(a, (long)n1 * n2, n2, 1, 0); };     // n1 x n2, [nb][n1][n2]

  k_adj_flag_zero<<<1, 64, 0, p.stream>>>(w.flag);
  launch_tables64(p, w.wtab, w.htab);
  // W+ in the spatial domain, from its stored spectrum
  launch_tube_inv64(p, SPEC_F32, out.wt, n2, (long)nb * n2, 1, w.w1s, (long)n2 * n3, n3, n1, n2, 1.0 / n3);
  // step 4: W-step adjoint -> z_bar, and the mu, rho2 adjoints
  const int wblk = wstep_adjoint(p, w, w_bar);
  k_adj_reduce2<<<1, 256, 0, p.stream>>>(w.wpart, wblk, theta, 0, 2);
  // step 3: Z~_bar = ifft(Z_bar) on the stored frequencies; X~+_bar += Z~_bar Y~+^*,
  // Y~+_bar += X~+^* Z~_bar
  launch_tube_fwd64(p, w.zbar, w.ztb, (long)n1 * n2, n2, 1, (long)n2 * n3, n3, n1, n2, 1.0 / n3);
  gemm_add(p, n1, r, n2, one, hv(w.ztb), ctr(Y1), one, xt_bar, w.x1b, (long)r * n1, 1, n1);
  gemm_add(p, r, n2, n1, one, ctr(X1), hv(w.ztb), one, yt_bar, w.y1b, (long)r * n2, n2, 1);
  // step 2: Y~+ = (1 - eta) Y~ + eta G_X^{-1} B,  B = X~+^* W~,  G_X = X~+^* H_rho1 X~+
  split(p, w.y1b, (long)r * n2, yt_bar, w.rb);
  happly<float2>(p, (const float2*)out.xt, w.hx1, 1.0, p.rho1);
  gemm(p, r, r, n1, one, ctr(X1), xv(w.hx1), zero, w.gx, (long)r * r, r, 1);
  inv(p, w, w.gx, w.gxi);
  gemm(p, r, n2, n1, one, ctr(X1), Wt, zero, w.bm, (long)r * n2, n2, 1);
  gemm(p, r, r, n2, one, yv(w.rb), ctr(yv(w.bm)), zero, w.gxib, (long)r * r, r, 1);
  gemm(p, r, n2, r, one, ctr(gv(w.gxi)), yv(w.rb), zero, w.bb, (long)r * n2, n2, 1);
  gram_adjoint(p, w.gxi, w.gxib, w.gxb, w.S);
  gemm(p, n1, r, n2, one, Wt, ctr(yv(w.bb)), one, w.x1b, (long)r * n1, 1, n1);
  gemm(p, n1, n2, r, one, X1, yv(w.bb), zero, w.wtb, (long)n1 * n2, n2, 1);
  gemm(p, n1, r, r, one, xv(w.hx1), gv(w.S), one, w.x1b, (long)r * n1, 1, n1);
  happly<float2>(p, (const float2*)out.xt, w.dt, 0.0, 1.0);
  gemm(p, r, r, n1, one, ctr(X1), xv(w.dt), zero, w.T, (long)r * r, r, 1);
  wdot_add(p, w, w.gxb, w.T, (long)r * r, 1.0, theta, 1);
  // step 1: X~+ = (1 - eta) X~ + eta Q,  Q = H_rho1^{-1} P,  P = A G_Y^{-1},  A = W~ Y~^*
  split(p, w.x1b, (long)r * n1, xt_bar, w.qb);
  gemm(p, r, r, n2, one, Y, ctr(Y), zero, w.gy, (long)r * r, r, 1);
  inv(p, w, w.gy, w.gyi);
  gemm(p, n1, r, n2, one, Wt, ctr(Y), zero, w.a, (long)r * n1, 1, n1);
  gemm(p, n1, r, r, one, xv(w.a), gv(w.gyi), zero, w.pp, (long)r * n1, 1, n1);
  hsolve2(p, w, w.pp, w.q, w.qb, w.pb);
  happly<double2>(p, w.q, w.dt, 0.0, 1.0);
  wdot_add(p, w, w.pb, w.dt, (long)r * n1, -1.0, theta, 1);
  gemm(p, n1, r, r, one, xv(w.pb), ctr(gv(w.gyi)), zero, w.ab, (long)r * n1, 1, n1);
  gemm(p, r, r, n1, one, ctr(xv(w.a)), xv(w.pb), zero, w.gyib, (long)r * r, r, 1);
  gram_adjoint(p, w.gyi, w.gyib, w.gyb, w.S);
  gemm(p, n1, n2, r, one, xv(w.ab), Y, one, w.wtb, (long)n1 * n2, n2, 1);
  gemm(p, r, n2, n1, one, ctr(xv(w.ab)), Wt, one, yt_bar, (long)r * n2, n2, 1);
  gemm(p, r, n2, r, one, gv(w.S), Y, one, yt_bar, (long)r * n2, n2, 1);
  // step 7 of the previous iteration: W~ = dft(W), so W_bar = sum_b c_b Re(omega^{-b l} W~_bar_b)
  launch_tube_inv64(p, SPEC_F64, w.wtb, (long)n1 * n2, n2, 1, w_bar, (long)n2 * n3, n3, n1, n2, 1.0);
}

void launch_adjoint_initial(const Plan& p, const double2* xt_bar, const double2* yt_bar, double* x0_bar,
                            double* y0_bar) {
  const int n1 = p.n1, n2 = p.n2, n3 = p.n3, r = p.r;
  // X~ [nb][r][n1] -> X0 [n1][r][n3];  Y~ [nb][r][n2] -> Y0 [r][n2][n3]
  if (x0_bar) launch_tube_inv64(p, SPEC_F64, xt_bar, (long)r * n1, n1, 1, x0_bar, n3, (long)r * n3, r, n1, 1.0);
  if (y0_bar) launch_tube_inv64(p, SPEC_F64, yt_bar, (long)r * n2, n2, 1, y0_bar, (long)n2 * n3, n3, r, n2, 1.0);
}

void launch_objective_gradient(const Plan& p, const AdjWork& w, double* x_grad, double* y_grad) {
  const int n1 = p.n1, n2 = p.n2, n3 = p.n3, r = p.r, nb = p.nb;
  const cd one = cd_make(1.0, 0.0), zero = cd_make(0.0, 0.0), mone = cd_make(-1.0, 0.0);
  const CView X = view(p.xt, (long)r * n1, 1, n1, 1), Y = view(p.yt, (long)r * n2, n2, 1, 1);
  const CView Wt = view(p.wt, n2, (long)nb * n2, 1, 1);
  auto xv = [&](const double2* a) { return view(a, (long)r * n1, 1, n1, 0); };
  auto gv = [&](const double2* a) { return view(a, (long)r * r, r, 1, 0); };
  // grad_X = H_rho1 X~ G_Y - W~ Y~^*,  grad_Y = G_X Y~ - X~^* W~  (eq. (hkXYDer))
  happly<float2>(p, p.xt, w.hx1, 1.0, p.rho1);
  gemm(p, r, r, n2, one, Y, ctr(Y), zero, w.gy, (long)r * r, r, 1);
  gemm(p, n1, r, n2, mone, Wt, ctr(Y), zero, w.a, (long)r * n1, 1, n1);
  gemm(p, n1, r, r, one, xv(w.hx1), gv(w.gy), one, w.a, (long)r * n1, 1, n1);
  gemm(p, r, r, n1, one, ctr(X), xv(w.hx1), zero, w.gx, (long)r * r, r, 1);
  gemm(p, r, n2, n1, mone, ctr(X), Wt, zero, w.bm, (long)r * n2, n2, 1);
  gemm(p, r, n2, r, one, gv(w.gx), Y, one, w.bm, (long)r * n2, n2, 1);
  // d f0 / d X = Re idft(grad_X): the inverse transform with the 1 / n3 of eq. (barAAk)
  launch_tube_inv64(p, SPEC_F64, w.a, (long)r * n1, n1, 1, x_grad, n3, (long)r * n3, r, n1, 1.0 / n3);
  launch_tube_inv64(p, SPEC_F64, w.bm, (long)r * n2, n2, 1, y_grad, (long)n2 * n3, n3, r, n2, 1.0 / n3);
}

}  // namespace tctf
