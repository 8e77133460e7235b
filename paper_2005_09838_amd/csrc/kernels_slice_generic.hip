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
};

// Block (x, i): rows (i, :, k), k = 256 x + thread; a wavefront's loads are consecutive words.
// Thomas elimination over the row with the tabulated reciprocal pivots: observed entries are
// identity equations (w = g), unobserved ones (1 + mu + rho2 deg_j) w_j - rho2 (w_{j-1} +
// w_{j+1}) = z_j.  NC > 0 (n2 <= NC): the row in registers, every load in flight at once; else
// chunks of 16 columns, the forward results through w.  w_from_g: W is P_Omega(G).
// 288 x 28 x 144: 10.0 us (38.5 with one block per OD row, a division per entry and c' through
// memory); 12 x 12 x 8064: 7.2 us and 5.2 for k_gen_rows (463).
template <int NC>
__global__ void __launch_bounds__(256) k_gen_wstep(GenWArgs a) {
  __shared__ double red[48];
  extern __shared__ float tab[];   // [4][n2]
  const int n2 = a.n2, n3 = a.n3, k = blockIdx.x * 256 + threadIdx.x;
  const long i = blockIdx.y;
  for (int e = threadIdx.x; e < 4 * n2; e += blockDim.x) tab[e] = a.wtab[e];
  __syncthreads();
  const float r2 = (float)a.rho2;
  const bool solve = a.mode != SLICE_INIT && !a.w_from_g;
  double fit = 0.0, ridge = 0.0, sm = 0.0;
  if (k < n3) {
    const long base = i * n2 * n3 + k;   // entry (i, j, k) at base + j n3
    auto terms = [&](float z, float w, float wr, bool has_r) {   // an entry and its right neighbour
      const double d = (double)z - (double)w;
      fit += d * d;
      ridge += (double)w * w;
      if (has_r) sm += ((double)wr - (double)w) * ((double)wr - (double)w);
    };
    // (pivot factor, constant) of the forward recurrence y = c y' + d
    auto coef = [&](float g, float z, float& c, float& d) {
      const bool un = is_unobserved(g);
      const float inv = tab[un ? unobs_index(g) : 0];
      c = un && solve ? r2 * inv : 0.0f;
      d = un ? (solve ? z * inv : 0.0f) : g;
    };
    if constexpr (NC > 0) {
      float z[NC], g[NC], c[NC], y[NC];
#pragma unroll
      for (int j = 0; j < NC; ++j) {
        const long e = base + (long)min(j, n2 - 1) * n3;
        z[j] = a.z[e];
        g[j] = a.gp[e];
      }
      float yp = 0.0f;
#pragma unroll
      for (int j = 0; j < NC; ++j) {
        if (j < n2) {
          coef(g[j], z[j], c[j], y[j]);
          y[j] = fmaf(c[j], yp, y[j]);
          yp = y[j];
        }
      }
      float wn = 0.0f;
#pragma unroll
      for (int j = NC - 1; j >= 0; --j) {
        if (j < n2) {
          const bool has_r = j + 1 < n2;
          const float w = has_r ? fmaf(c[j], wn, y[j]) : y[j];
          y[j] = w;
          a.w[base + (long)j * n3] = w;
          if (a.w_out) a.w_out[base + (long)j * n3] = w;
          terms(z[j], w, wn, has_r);
          wn = w;
        }
      }
    } else {
      constexpr int C = 16;
      float yp = 0.0f;
      for (int j0 = 0; j0 < n2; j0 += C) {
        float z[C], g[C];
#pragma unroll
        for (int u = 0; u < C; ++u) {
          const long e = base + (long)min(j0 + u, n2 - 1) * n3;
          z[u] = a.z[e];
          g[u] = a.gp[e];
        }
#pragma unroll
        for (int u = 0; u < C; ++u) {
          if (j0 + u < n2) {
            float c, d;
            coef(g[u], z[u], c, d);
            yp = fmaf(c, yp, d);
            a.w[base + (long)(j0 + u) * n3] = yp;
          }
        }
      }
      float wn = 0.0f;
      for (int j0 = (n2 - 1) / C * C; j0 >= 0; j0 -= C) {
        float z[C], g[C], y[C];
#pragma unroll
        for (int u = 0; u < C; ++u) {
          const long e = base + (long)min(j0 + u, n2 - 1) * n3;
          z[u] = a.z[e];
          g[u] = a.gp[e];
          y[u] = a.w[e];
        }
#pragma unroll
        for (int u = C - 1; u >= 0; --u) {
          if (j0 + u < n2) {
            const bool has_r = j0 + u + 1 < n2;
            float c, d;
            coef(g[u], z[u], c, d);
            const float w = has_r ? fmaf(c, wn, y[u]) : y[u];
            a.w[base + (long)(j0 + u) * n3] = w;
            if (a.w_out) a.w_out[base + (long)(j0 + u) * n3] = w;
            terms(z[u], w, wn, has_r);
            wn = w;
          }
        }
      }
    }
    if (a.mode == SLICE_KKT) {   // residual maxima instead, from the stored row
      fit = ridge = sm = 0.0;
      for (int j = 0; j < n2; ++j) {
        const long e = base + (long)j * n3;
        const double w = a.w[e], z = a.z[e], l = j > 0 ? (double)a.w[e - n3] : 0.0,
                     r = j + 1 < n2 ? (double)a.w[e + n3] : 0.0;
        const double deg = (j > 0 ? 1.0 : 0.0) + (j + 1 < n2 ? 1.0 : 0.0);
        const float g = a.gp[e];
        if (!is_unobserved(g)) ridge = fmax(ridge, fabs(w - (double)g));
        else if (solve) fit = fmax(fit, fabs((1.0 + a.mu + a.rho2 * deg) * w - a.rho2 * (l + r) - z));
        sm = fmax(sm, fabs(z));
      }
    }
  }
  if (a.mode == SLICE_RESULT) return;
  if (a.mode == SLICE_KKT) {
    fit = block_max_d(fit, red);
    ridge = block_max_d(ridge, red);
    sm = block_max_d(sm, red);
  } else {
    block_sum3_d(fit, ridge, sm, red);
  }
  if (threadIdx.x == 0) {
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

void launch_slice_generic(const Plan& p, int mode, float* w_out, float* z_out, int w_from_g) {
  const long n = (long)p.n1 * p.n2 * p.n3, slice = (long)p.n2 * p.n3;
  const bool need_z = !(mode == SLICE_RESULT && w_from_g && z_out == nullptr);
  if (need_z)
    launch_tube_inv(p, SPEC_F32, p.zt, p.n2, (long)p.nb * p.n2, 1, p.zsp, z_out, slice, p.n3, p.n1, p.n2, 1.0 / p.n3);
  else
    launch_zero(p, p.zsp, (size_t)n * 4);
  const int nchunk = (p.n3 + 255) / 256, threads = p.n3 >= 256 ? 256 : (p.n3 + 63) / 64 * 64;
  double* rows = mode == SLICE_KKT ? p.kkt : p.slice_obj;
  GenWArgs a;
  a.z = p.zsp;
  a.gp = p.gp;
  a.wtab = p.wtab;
  a.w = p.wsp;
  a.w_out = w_out;
  a.part = nchunk > 1 ? (double*)p.csp : rows;   // csp holds 24 n1 ceil(n3 / 256) bytes wherever n3 > 256
  a.n2 = p.n2;
  a.n3 = p.n3;
  a.mu = p.mu;
  a.rho2 = p.rho2;
  a.mode = mode;
  a.w_from_g = w_from_g;
  const dim3 grid(nchunk, p.n1);
  const size_t lds = 4 * (size_t)p.n2 * sizeof(float);
  if (p.n2 <= 16) k_gen_wstep<16><<<grid, threads, lds, p.stream>>>(a);
  else if (p.n2 <= 32) k_gen_wstep<32><<<grid, threads, lds, p.stream>>>(a);
  else k_gen_wstep<0><<<grid, threads, lds, p.stream>>>(a);
  if (nchunk > 1 && mode != SLICE_RESULT)
    k_gen_rows<<<(3 * p.n1 + 255) / 256, 256, 0, p.stream>>>((const double*)p.csp, p.n1, nchunk, mode == SLICE_KKT, rows);
  if (mode == SLICE_INIT || mode == SLICE_ITER)
    launch_tube_fwd(p, p.mixed ? SPEC_BF16 : SPEC_F32, p.wsp, p.wt, p.n2, (long)p.nb * p.n2, 1, slice, p.n3, p.n1, p.n2, 1.0);
}

}  // namespace tctf
