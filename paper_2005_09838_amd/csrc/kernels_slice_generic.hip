// The slice work (steps 3, 4 and 7 of the algorithm box) for any tube length n3 and any
// slice size: used where the fused LDS slice kernel does not apply (n3 outside the generated
// transform lengths, or an n2 x n3 slice larger than its LDS).  Three launches through the
// spatial buffers Z and W ([n1][n2][n3] FP32 in the workspace): the FP64 inverse tube transform
// (eq. (barAAk)), the W-step of eq. (subquKKT) along every row (i, :, k) with the objective's
// per-row partial sums (fit, ridge, K term) or, for the stationarity check, the KKT residual
// maxima, and the FP64 forward transform (eq. (bar BA-k)).
#include "kernels.h"

namespace tctf {

struct GenWArgs {
  const float* z;
  const float* gp;       // packed G in G's own order
  const float* wtab;     // pivots, at the index an unobserved entry of gp carries
  float* w;
  float* w_out;
  double* part;          // [n1][gridDim.x][3] sums (SLICE_KKT: maxima)
  int n2, n3;
  double mu, rho2;
  int mode, w_from_g;
  int ls, lk;            // 2^ls segments of a row, 2^lk rows of a block
};

// Block (x, i): S = 2^ls segments of at most L columns of the rows (i, :, k), k = x KB .. + KB, KB =
// 2^lk, a thread per (segment, row); a wavefront's loads are runs of KB words.  Observed entries are
// identity equations (w = g), unobserved ones (1 + mu + rho2 deg_j) w_j - rho2 (w_{j-1} + w_{j+1}) =
// z_j; with the tabulated reciprocal pivots elimination and back substitution are affine maps of
// the value that enters a segment, chained through LDS.  What bounds it: the loads' latency (all of
// a segment in flight at once) and the chains of L + S steps.  w_from_g: W is P_Omega(G).
// 288 x 28 x 144: 9.4 us (10.2 with a thread per row); the whole slice stage at 144 x 288 x 25 55.0
// (102.9), at 100 x 200 x 50 32.8 (70.4).
template <int L>
__global__ void __launch_bounds__(256) k_gen_wstep(GenWArgs a) {
  __shared__ double red[48];
  __shared__ float ma[256], mb[256], na[256], nb[256];
  const int S = 1 << a.ls, KB = 1 << a.lk, n2 = a.n2, n3 = a.n3, tid = threadIdx.x, s = tid >> a.lk, kk = tid & (KB - 1);
  const int k = blockIdx.x * KB + kk, len = (n2 + S - 1) >> a.ls;
  const int j0 = s * len, cnt = k < n3 ? min(len, n2 - j0) : 0;   // may be negative: no columns
  const long i = blockIdx.y, base = i * n2 * n3 + min(k, n3 - 1);  // entry (i, j, k) at base + j n3
  const float r2 = (float)a.rho2;
  const bool solve = a.mode != SLICE_INIT && !a.w_from_g;
  float z[L], g[L], c[L], y[L];
#pragma unroll
  for (int u = 0; u < L; ++u) {
    const long e = base + (long)min(j0 + u, n2 - 1) * n3;
    z[u] = a.z[e];
    g[u] = a.gp[e];
  }
#pragma unroll
  for (int u = 0; u < L; ++u) {
    const bool un = is_unobserved(g[u]);
    const float inv = a.wtab[un ? unobs_index(g[u]) : 0];
    c[u] = un && solve ? r2 * inv : 0.0f;
    y[u] = un ? (solve ? z[u] * inv : 0.0f) : g[u];
  }
  float p = 1.0f, q = 0.0f;
#pragma unroll
  for (int u = 0; u < L; ++u) {
    if (u < cnt) {
      q = fmaf(c[u], q, y[u]);
      p *= c[u];
    }
  }
  ma[tid] = p;
  mb[tid] = q;
  __syncthreads();
  float in = 0.0f;
  for (int t = kk; t < s * KB; t += KB) in = fmaf(ma[t], in, mb[t]);
#pragma unroll
  for (int u = 0; u < L; ++u) {
    if (u < cnt) in = fmaf(c[u], in, y[u]);
    y[u] = in;
  }
  p = cnt > 0 ? 1.0f : 0.0f;
  q = 0.0f;
#pragma unroll
  for (int u = L - 1; u >= 0; --u) {
    if (u < cnt) {
      q = fmaf(c[u], q, y[u]);
      p *= c[u];
    }
  }
  na[tid] = p;
  nb[tid] = q;
  __syncthreads();
  float w = 0.0f;
  for (int t = (S - 1) * KB + kk; t > tid; t -= KB) w = fmaf(na[t], w, nb[t]);
  double fit = 0.0, ridge = 0.0, sm = 0.0;
#pragma unroll
  for (int u = L - 1; u >= 0; --u) {
    if (u < cnt) {
      const float right = w;
      w = fmaf(c[u], w, y[u]);
      const long e = base + (long)(j0 + u) * n3;
      a.w[e] = w;
      if (a.w_out) a.w_out[e] = w;
      const double d = (double)z[u] - (double)w;
      fit += d * d;
      ridge += (double)w * w;
      if (j0 + u + 1 < n2) sm += ((double)right - (double)w) * ((double)right - (double)w);
    }
  }
  if (a.mode == SLICE_RESULT) return;
  if (a.mode == SLICE_KKT) {   // residual maxima instead, from the stored row
    __syncthreads();
    fit = ridge = sm = 0.0;
    for (int u = 0; u < cnt; ++u) {
      const int j = j0 + u;
      const long e = base + (long)j * n3;
      const double wj = a.w[e], zj = a.z[e], l = j > 0 ? (double)a.w[e - n3] : 0.0, r = j + 1 < n2 ? (double)a.w[e + n3] : 0.0;
      const double deg = (j > 0 ? 1.0 : 0.0) + (j + 1 < n2 ? 1.0 : 0.0);
      const float gj = a.gp[e];
      if (!is_unobserved(gj)) ridge = fmax(ridge, fabs(wj - (double)gj));
      else if (solve) fit = fmax(fit, fabs((1.0 + a.mu + a.rho2 * deg) * wj - a.rho2 * (l + r) - zj));
      sm = fmax(sm, fabs(zj));
    }
    fit = block_max_d(fit, red);
    ridge = block_max_d(ridge, red);
    sm = block_max_d(sm, red);
  } else {
    block_sum3_d(fit, ridge, sm, red);
  }
  if (tid == 0) {
    double* out = a.part + 3 * (i * gridDim.x + blockIdx.x);
    out[0] = fit;
    out[1] = ridge;
    out[2] = sm;
  }
}

// The partials of each OD row in a fixed order: sums, or maxima.
__global__ void k_gen_rows(const double* __restrict__ part, int n1, int nchunk, int maxima, double* __restrict__ out) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= 3 * n1) return;
  const int i = e / 3, c = e % 3;
  double v = 0.0;
  for (int x = 0; x < nchunk; ++x) {
    const double p = part[3 * ((long)i * nchunk + x) + c];
    v = maxima ? fmax(v, p) : v + p;
  }
  out[e] = v;
}

// Blocks of k_gen_wstep: segments of at most 16 columns and no more of them than that needs, so that
// the runs of rows are long; no more rows per block than there are, in whole wavefronts.
struct WstepShape {
  int ls, lk, nchunk;
};
static WstepShape wstep_shape(int n2, int n3) {
  WstepShape w = {0, 8, 0};
  while (((n2 + (1 << w.ls) - 1) >> w.ls) > 16) ++w.ls;   // n2 <= 1024: ls <= 6
  w.lk -= w.ls;
  while (w.lk > 0 && w.ls + w.lk > 6 && (1 << (w.lk - 1)) >= n3) --w.lk;
  w.nchunk = (n3 + (1 << w.lk) - 1) >> w.lk;
  return w;
}
size_t slice_generic_part_doubles(int n1, int n2, int n3) {
  const size_t nchunk = wstep_shape(n2, n3).nchunk;
  return nchunk > 1 ? 3 * nchunk * n1 : 0;
}

void launch_slice_generic(const Plan& p, int mode, float* w_out, float* z_out, int w_from_g) {
  const long n = (long)p.n1 * p.n2 * p.n3, slice = (long)p.n2 * p.n3;
  const bool need_z = !(mode == SLICE_RESULT && w_from_g && z_out == nullptr);
  if (need_z)
    launch_tube_inv(p, SPEC_F32, p.zt, p.n2, (long)p.nb * p.n2, 1, p.zsp, z_out, slice, p.n3, p.n1, p.n2, 1.0 / p.n3);
  else
    launch_zero(p, p.zsp, (size_t)n * 4);
  const WstepShape ws = wstep_shape(p.n2, p.n3);
  const int ls = ws.ls, lk = ws.lk, nchunk = ws.nchunk, threads = 1 << (ls + lk), len = (p.n2 + (1 << ls) - 1) >> ls;
  double* rows = mode == SLICE_KKT ? p.kkt : p.slice_obj;
  GenWArgs a;
  a.z = p.zsp;
  a.gp = p.gp;
  a.wtab = p.wtab;
  a.w = p.wsp;
  a.w_out = w_out;
  a.part = nchunk > 1 ? p.rowpart : rows;
  a.n2 = p.n2;
  a.n3 = p.n3;
  a.mu = p.mu;
  a.rho2 = p.rho2;
  a.mode = mode;
  a.w_from_g = w_from_g;
  a.ls = ls;
  a.lk = lk;
  const auto wstep = len <= 9 ? k_gen_wstep<9> : (len <= 12 ? k_gen_wstep<12> : k_gen_wstep<16>);
  wstep<<<dim3(nchunk, p.n1), threads, 0, p.stream>>>(a);
  bool sums = nchunk > 1 && mode != SLICE_RESULT;   // still to be formed
  if (mode == SLICE_INIT || mode == SLICE_ITER) {
    RowSums r = {sums ? a.part : nullptr, rows, nchunk};
    if (launch_tube_fwd(p, p.mixed ? SPEC_BF16 : SPEC_F32, p.wsp, p.wt, p.n2, (long)p.nb * p.n2, 1, slice, p.n3, p.n1, p.n2, 1.0, r))
      sums = false;
  }
  if (sums) k_gen_rows<<<(3 * p.n1 + 255) / 256, 256, 0, p.stream>>>(a.part, p.n1, nchunk, mode == SLICE_KKT, rows);
}

}  // namespace tctf
