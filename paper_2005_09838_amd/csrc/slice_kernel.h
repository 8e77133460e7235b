#pragma once
// The slice kernel: for one OD row i (a horizontal slice, n2 x n3) it
//   1. brings Z~(i,:,b) back to the tube domain (eq. (barAAk), step 3 of the algorithm box),
//   2. solves the W-step of every row (i, k) along mode 2 (eq. (subquKKT) / eq. (Wkiom), step 4),
//   3. transforms W(i,:,:) along the tube (eq. (bar BA-k), step 7) and stores W~(i,:,b),
// and emits the FP64 partial sums of the objective terms it can see (fit, ridge, K term).
//
// W-step of a row: observed entries are fixed (w_j = g_j); the unobserved ones solve
//   (1 + mu + rho2 deg_j) w_j - rho2 (w_{j-1} + w_{j+1}) = z_j,
// a tridiagonal system with the observed neighbours on the right-hand side.  Thomas
// elimination needs no pivoting (strict diagonal dominance); its reciprocal pivots depend
// only on the position in the run of unobserved entries, on whether the run starts at the
// first slot and on whether the entry is the last slot, so they come from the precomputed
// table wtab, at the index that the packed G carries in each unobserved entry:
//   forward  y_j = (z_j + rho2 y_{j-1}) / alpha_j      (y = g on observed entries)
//   backward w_j = y_j + rho2 / alpha_j * w_{j+1}       (w = g on observed entries)
#include "kernels.h"
#include "pinv.h"
#define TUBE_TWIDDLES
#include "tube_dft_gen.h"
#include "tube_lds.h"

namespace tctf {

struct SliceArgs {
  const float2* zt;
  const float* gp;
  const float* wtab;
  void* wt;
  double* slice_obj;
  double* kkt;
  float* w_out;
  float* z_out;
  int n1, n2, nb;
  float rho2;
  double mu, rho2d;
  int mode, mixed, w_from_g;
  int nseg;      // segments per row of the W-step (and of the packed G's row order)
  int npinv;     // SLICE_ITER: blocks 0 .. npinv - 1 form G_Y^+ of frequency blockIdx.x
  const uint32_t* ctr;   // counter of the BF16 rounding bits (mixed precision)
  PinvyArgs pa;
};

// Value of the lane d below (up) or above (down) within a 16-lane DPP row: a row shift of the
// VALU (lanes whose source falls outside the row read 0; callers only use lanes whose source
// is in their group).
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}

// Inclusive scan of the affine maps x -> A x + B over the S lanes of a row (S a power of two
// that divides 64, lane s of the row): UP composes lane s's map after those of lanes < s, else
// after those of lanes > s.  Within 16 lanes by DPP row shifts; rows of 32 or 64 lanes add the
// totals of the other 16-lane groups by cross-lane reads.
template <bool UP, int D>
__device__ __forceinline__ void scan_step(float& A, float& B, int s16, int w16) {
  const float a2 = dpp_mov<(UP ? 0x110 : 0x100) + D>(A), b2 = dpp_mov<(UP ? 0x110 : 0x100) + D>(B);
  if (UP ? s16 >= D : s16 + D < w16) {
    B = fmaf(A, b2, B);
    A *= a2;
  }
}
template <bool UP>
__device__ __forceinline__ void affine_scan(float& A, float& B, int s, int S) {
  const int s16 = s & 15, w16 = S < 16 ? S : 16;
  if (S > 1) scan_step<UP, 1>(A, B, s16, w16);
  if (S > 2) scan_step<UP, 2>(A, B, s16, w16);
  if (S > 4) scan_step<UP, 4>(A, B, s16, w16);
  if (S > 8) scan_step<UP, 8>(A, B, s16, w16);
  for (int h = 16; h < S; h <<= 1) {   // join neighbouring groups of h lanes
    const int lane = threadIdx.x & 63, base = lane & ~(2 * h - 1);
    const float a2 = __shfl(A, base + (UP ? h - 1 : h)), b2 = __shfl(B, base + (UP ? h - 1 : h));
    if (((lane & h) != 0) == UP) {
      B = fmaf(A, b2, B);
      A *= a2;
    }
  }
}
// value of the next lane of the row below / above, 0 at the row's end
template <bool UP>
__device__ __forceinline__ float lane_shift(float v, int s, int S) {
  float x;
  if (S <= 16) x = dpp_mov<(UP ? 0x111 : 0x101)>(v);
  else x = UP ? __shfl_up(v, 1) : __shfl_down(v, 1);
  return s == (UP ? 0 : S - 1) ? 0.0f : x;
}

// W-step of every row (i, :, k) with S lanes per row: lane (k, s) takes the columns
// [j0, j0 + len) of segment s (the first n2 % S segments hold one column more).  Both Thomas
// passes are first-order affine recurrences,
//   forward  y_j = a_j y_{j-1} + b_j  (a = rho2 / alpha_j, b = z_j / alpha_j; a = 0, b = g_j observed)
//   backward w_j = c_j w_{j+1} + y_j  (c = a_j; c = 0 at the last column),
// so each lane composes its segment's map, the maps of a row are combined by a scan across
// its lanes, and each lane then runs its segment once more from the right boundary value.
// The packed G of the next item is loaded while the current one is solved; its order
// (packed_g_at) makes each load a run of consecutive words.
// The terms of f0 come from the values still in registers (the neighbours across segment ends
// from the adjacent lanes): ridge sum w_j^2, K term sum (w_{j+1} - w_j)^2 and the fit residual
// z_j - w_j, which on unobserved entries the row's equation gives as
// (mu + rho2 deg_j) w_j - rho2 (w_{j-1} + w_{j+1}).  SLICE_KKT: ff and fr take the maxima of
// the residuals of eq. (subquKKT) (unobserved (W K_{mu rho2} - Z)_ij, observed W - G) and fs
// that of |Z| instead.  solve = false: W = P_Omega(G).
// FULL: every segment holds exactly L columns; else at most L, and the entries past a segment
// are the identity map, which leaves every scan and pass unchanged.
template <int L, bool ITER, bool FULL>
__device__ __forceinline__ void wstep_rows(float* zs, int LD, const float* tab, const float* __restrict__ grow, int n2,
                                           int N, int S, const SliceArgs& a, bool solve, double& fr, double& fs,
                                           double& ff) {
  const int tid = threadIdx.x, nt = blockDim.x, items = N * S, sh = __ffs(S) - 1;
  const int Lf = FULL ? L : n2 >> sh, rem = FULL ? 0 : n2 & (S - 1);
  const float rho2 = a.rho2, cin = fmaf(2.0f, rho2, (float)a.mu);
  float g[L];
  // Every load is unconditional (past the segment: word 0, dropped): a load under a branch
  // would be waited for at the branch's end.
  auto load_g = [&](int it) {
    const int k = it >> sh, s = it & (S - 1);
    const int part = s < rem ? Lf * items + k * rem + s : 0;
#pragma unroll
    for (int u = 0; u < L; ++u) g[u] = FULL || u < Lf ? (grow + u * items)[(uint32_t)it] : grow[(uint32_t)(u == Lf ? part : 0)];
  };
  if (tid < items) load_g(tid);
  for (int it = tid; it < items; it += nt) {
    const int k = it >> sh, s = it & (S - 1);
    const int j0 = s * Lf + min(s, rem), len = Lf + (s < rem ? 1 : 0);
    float* col = zs + j0 * LD + k;
    float z[L], av[L], bv[L];
    bool un[L];
#pragma unroll
    for (int u = 0; u < L; ++u) z[u] = col[FULL || u < Lf ? u * LD : (u < len ? u * LD : 0)];
#pragma unroll
    for (int u = 0; u < L; ++u) {
      un[u] = g[u] != g[u];   // unobserved entries are NaNs
      av[u] = tab[un[u] ? unobs_index(g[u]) : 0];
    }
    float A = 1.0f, B = 0.0f, pf = 0.0f;
#pragma unroll
    for (int u = 0; u < L; ++u) {
      const bool in = FULL || u < len;
      bv[u] = un[u] ? (ITER || solve ? z[u] * av[u] : 0.0f) : g[u];
      av[u] = un[u] ? rho2 * av[u] : 0.0f;
      const float d = un[u] && (ITER || solve) ? 0.0f : z[u] - (un[u] ? 0.0f : g[u]);
      pf = in ? fmaf(d, d, pf) : pf;
      if (!FULL) {
        av[u] = in ? av[u] : 1.0f;
        bv[u] = in ? bv[u] : 0.0f;
      }
      B = fmaf(av[u], B, bv[u]);
      A *= av[u];
    }
    if (it + nt < items && (ITER || a.mode != SLICE_KKT)) load_g(it + nt);   // these loads fly during the solve
    if (ITER || solve) {
      // c_j = a_j except at the last column
      float C = s == S - 1 ? 0.0f : A;
      affine_scan<true>(A, B, s, S);
      float y = lane_shift<true>(B, s, S), D = 0.0f;
#pragma unroll
      for (int u = 0; u < L; ++u) {
        y = fmaf(av[u], y, bv[u]);
        bv[u] = FULL || u < len ? y : 0.0f;   // y_j
        if (FULL ? u == L - 1 : true) av[u] = s == S - 1 && (FULL || u == len - 1) ? 0.0f : av[u];
      }
#pragma unroll
      for (int u = L - 1; u >= 0; --u) D = fmaf(av[u], D, bv[u]);
      affine_scan<false>(C, D, s, S);
      float w = lane_shift<false>(D, s, S);
#pragma unroll
      for (int u = L - 1; u >= 0; --u) {
        w = fmaf(av[u], w, bv[u]);
        bv[u] = w;   // w_j (past the segment: the right neighbour's first value)
      }
    }
#pragma unroll
    for (int u = 0; u < L; ++u)
      if (FULL || u < len) col[u * LD] = bv[u];
    if (ITER || a.mode != SLICE_RESULT) {
      float last = bv[FULL ? L - 1 : 0];
      if (!FULL) {
#pragma unroll
        for (int u = 1; u < L; ++u) last = u < len ? bv[u] : last;
      }
      float wl = lane_shift<true>(last, s, S);
      const float right = lane_shift<false>(bv[0], s, S);
      if (ITER || a.mode != SLICE_KKT) {
        float pr = 0.0f, ps = 0.0f;
#pragma unroll
        for (int u = 0; u < L; ++u) {
          const bool in = FULL || u < len, end = FULL ? u + 1 == L : u + 1 >= len;   // end of the segment
          const float wq = in ? bv[u] : 0.0f, wr = end ? right : bv[u + 1 < L ? u + 1 : u];
          const bool has_r = !(end && s == S - 1);
          const float cj = cin - (u == 0 && s == 0 ? rho2 : 0.0f) - (has_r ? 0.0f : rho2);
          if (ITER || solve) {
            const float d = un[u] && in ? fmaf(cj, wq, -rho2 * (wl + wr)) : 0.0f;
            pf = fmaf(d, d, pf);
          }
          const float dr = in && has_r ? wr - wq : 0.0f;
          pr = fmaf(wq, wq, pr);
          ps = fmaf(dr, dr, ps);
          wl = wq;
        }
        fr += (double)pr;
        fs += (double)ps;
        ff += (double)pf;
      } else {
#pragma unroll
        for (int u = 0; u < L; ++u) {
          if (u < len) {
            const int j = j0 + u;
            const float wq = bv[u], wr = (u + 1 < len) ? bv[u + 1 < L ? u + 1 : u] : right;
            const bool has_l = j > 0, has_r = j + 1 < n2;
            const double cj = a.mu + a.rho2d * ((has_l ? 1.0 : 0.0) + (has_r ? 1.0 : 0.0));
            const double nbr = (has_l ? (double)wl : 0.0) + (has_r ? (double)wr : 0.0);
            if (!un[u]) fr = fmax(fr, fabs((double)wq - (double)g[u]));
            else if (solve) ff = fmax(ff, fabs((1.0 + cj) * wq - a.rho2d * nbr - (double)z[u]));
            fs = fmax(fs, fabs((double)z[u]));
            wl = wq;
          }
        }
        if (it + nt < items) load_g(it + nt);
      }
    }
  }
}

// Threads per tube: short tubes are transformed by one thread in registers; longer ones by
// four or eight neighbouring lanes of one wavefront through the tube's LDS row (at most two
// groups of each four-step stage per lane), so that no stage needs a block barrier.  Outside the
// iteration (ITER false) short even tubes take the four-step form as well: the rounding of the
// first W~ to BF16 turns a last FP32 bit of the transform into 2^-8 of an entry, and with this
// form the first W~ of a mixed-precision run, and a checkpoint of it, keep the bits that they
// had before the iteration's transforms moved to registers.
template <int N, bool ITER>
__host__ __device__ constexpr int slice_tube_threads() {
  constexpr int m1 = TubePlan<N>::M1, m2 = TubePlan<N>::M2;
  return m1 == 0 || (ITER && N <= 32) ? 1 : (m1 > 5 && m2 > 5 ? 8 : 4);
}

// LDS row stride of one tube: odd where one thread owns a tube, so that a run of tubes does not
// meet in one bank; where lanes share a tube, rows of (re, im) pairs whose stride spreads the
// tubes of 16 lanes over the 32 banks (short tubes: the least, within the LDS of the rule on
// slice sizes).
template <int N, bool ITER>
__host__ __device__ constexpr int slice_ld() {
  constexpr int T = slice_tube_threads<N, ITER>();
  int ld = (N % 2 == 0) ? N + 3 : N + 2;
  if (T > 1) {
    ld = N + 2;
    while (N > 32 && (T == 8 ? (ld % 32 < 14 || ld % 32 > 22) : ((ld + 2) % 16 < 8))) ld += 2;
  }
  return ld;
}

// Orders this wavefront's LDS accesses: what its lanes wrote before is read after.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

template <int N>
__device__ __forceinline__ void load_inverse_tube(const float2* __restrict__ src, int n2, int j, float (&z)[N]) {
  constexpr int NB = N / 2 + 1;
  float re[NB], im[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const float2 v = src[b * n2 + j];
    re[b] = v.x;
    im[b] = v.y;
  }
  tube_inv<N>(re, im, z);
}

// One block per OD row, the slice in LDS: Z~ in and W~ out once, two block barriers.  What
// bounds it: the VALU (about 13 thousand wave instructions per 96 x 112 slice, two thirds of
// them the transforms) and, at 529 rows on 256 compute units, the units that hold three rows;
// three blocks fit a unit's LDS, so a register cap that let more wavefronts in only spilled
// (42 us at six wavefronts per SIMD, 29 at four).  In an iteration the first nb blocks form
// G_Y^+ and I - eta P_Y for the next X-step (pinvy_block).
// 529 x 96 x 112: 42.0 us before (flags, W-step and transforms of a tube over four wavefronts,
// seven block barriers), 28.7 now; 144 x 288 x 28: 86.7 before (one lane per row of the
// W-step), 9.5 now; 36 x 48 x 7: 19.2 before, 5.7 now.
template <int N, int L, bool ITER>
__global__ void __launch_bounds__(640) k_slice(SliceArgs a) {
  constexpr int T = slice_tube_threads<N, ITER>(), LD = slice_ld<N, ITER>(), NB = N / 2 + 1, M = N / 2, PN = (M / 2 + T) / T;
  extern __shared__ __align__(16) float smem[];
  if constexpr (ITER) {
    if ((int)blockIdx.x < a.npinv) {
      pinvy_block((int)blockIdx.x, a.pa, (unsigned char*)smem);
      return;
    }
  }
  const int n2 = a.n2, tid = threadIdx.x, nt = blockDim.x;
  float* zs = smem;                           // [n2][LD]
  float* tab = zs + (size_t)n2 * LD;          // [4][n2]
  size_t off = (size_t)n2 * (LD + 4);
  off += off & 1;
  float2* twm = (float2*)(smem + off);        // [M], twn [M + 1]: the LDS transforms only
  float2* twn = twm + (T > 1 ? M : 0);
  double* red = (double*)(twn + (T > 1 ? M + 1 : 0));
  const size_t i = ITER ? blockIdx.x - a.npinv : blockIdx.x;
  const float* grow = a.gp + i * n2 * N;
  const bool solve = ITER || (a.mode != SLICE_INIT && !a.w_from_g);

  // ---- 1. inverse transform of Z~(i, j, :) (times M for the LDS transforms)
  const bool need_z = ITER || !(a.mode == SLICE_RESULT && a.w_from_g && a.z_out == nullptr);
  const int t = tid & (T - 1);
  if constexpr (T > 1) {
    using FC = FftStepC<TubePlan<N>::M1, TubePlan<N>::M2, T>;
    // the first tubes' loads fly while the tables are copied
    const float2* zrow = a.zt + i * a.nb * n2;
    float2 xb[PN], xm[PN];
    const int jw0 = (tid >> 6) * (64 / T), jl = (tid & 63) / T;
    if (need_z && jw0 < n2) tube_inv_load<N, T>(zrow, n2, min(jw0 + jl, n2 - 1), t, xb, xm);
    for (int e = tid; e < 4 * n2; e += nt) tab[e] = a.wtab[e];
    for (int e = tid; e <= N; e += nt) twm[e] = TubeTwiddles<N>::w[e];   // M of one, then M + 1 of the other
    __syncthreads();
    if (need_z) {
      for (int jw = jw0; jw < n2; jw += nt / T) {   // the wavefront's tubes
        const int j = jw + jl;
        const bool act = j < n2;
        float* row = zs + j * LD;
        if (act) tube_inv_pre<N, T>((float2*)row, twn, t, xb, xm);
        wave_sync();
        if (jw + nt / T < n2) tube_inv_load<N, T>(zrow, n2, min(j + nt / T, n2 - 1), t, xb, xm);
        if (act) fft4_step_a<TubePlan<N>::M1, TubePlan<N>::M2, -1, T>((float2*)row, twm, t);
        wave_sync();
        FC sc;
        if (act) sc.read((float2*)row, t);
        wave_sync();
        if (act) sc.template write<-1>((float2*)row, t);
      }
    }
  } else {
    for (int e = tid; e < 4 * n2; e += nt) tab[e] = a.wtab[e];
    if (need_z) {
      for (int j = tid; j < n2; j += nt) {
        float* row = zs + j * LD;
        float z[N];
        load_inverse_tube<N>(a.zt + i * a.nb * n2, n2, j, z);
#pragma unroll
        for (int q = 0; q < N; ++q) row[q] = z[q];
      }
    }
  }
  __syncthreads();
  if constexpr (!ITER) {
    if (a.z_out) {
      float* dst = a.z_out + i * n2 * N;
      for (int e = tid; e < n2 * N; e += nt) dst[e] = zs[(e / N) * LD + e % N];
      __syncthreads();
    }
  }

  // ---- 2. W-step along mode 2 for the rows (i, :, k), with the objective terms
  double fit = 0.0, ridge = 0.0, sm = 0.0;
  if (n2 == L * a.nseg) wstep_rows<L, ITER, true>(zs, LD, tab, grow, n2, N, a.nseg, a, solve, ridge, sm, fit);
  else wstep_rows<L, ITER, false>(zs, LD, tab, grow, n2, N, a.nseg, a, solve, ridge, sm, fit);
  __syncthreads();

  // ---- 3. forward transform of W(i, j, :)
  if (ITER || a.mode == SLICE_INIT) {
    uint32_t key = 0;
    if (a.mixed) key = fmix32(a.ctr[0] * 0x9e3779b9u + 0x7f4a7c15u);
    const size_t base = i * a.nb * n2;
    uint32_t* wrow16 = (uint32_t*)a.wt + base;
    float2* wrow32 = (float2*)a.wt + base;
    auto store = [&](int j, int b, float re, float im) {
      const int at = b * n2 + j;
      if (a.mixed) wrow16[at] = pack_bf16x2_sr(re, im, fmix32((uint32_t)(base + at) ^ key));
      else wrow32[at] = make_float2(re, im);
    };
    if constexpr (T > 1) {
      using FC = FftStepC<TubePlan<N>::M1, TubePlan<N>::M2, T>;
      for (int jw = (tid >> 6) * (64 / T); jw < n2; jw += nt / T) {
        const int j = jw + ((tid & 63) / T);
        const bool act = j < n2;
        float* row = zs + j * LD;
        if (act) fft4_step_a<TubePlan<N>::M1, TubePlan<N>::M2, +1, T>((float2*)row, twm, t);
        wave_sync();
        FC sc;
        if (act) sc.read((float2*)row, t);
        wave_sync();
        if (act) sc.template write<+1>((float2*)row, t);
        wave_sync();
        if (act) {
          tube_fwd_post<N, T>((const float2*)row, twn, t, [&](int b, float re, float im) { store(j, b, re, im); });
        }
      }
    } else {
      for (int j = tid; j < n2; j += nt) {
        const float* row = zs + j * LD;
        float w[N], re[NB], im[NB];
#pragma unroll
        for (int q = 0; q < N; ++q) w[q] = row[q];
        tube_fwd<N>(w, re, im);
#pragma unroll
        for (int b = 0; b < NB; ++b) store(j, b, re[b], im[b]);
      }
    }
  }
  if constexpr (!ITER) {
    if (a.mode == SLICE_RESULT) {
      if (a.w_out) {
        float* dst = a.w_out + i * n2 * N;
        for (int e = tid; e < n2 * N; e += nt) dst[e] = zs[(e / N) * LD + e % N];
      }
      return;
    }
    if (a.mode == SLICE_KKT) {
      fit = block_max_d(fit, red);
      ridge = block_max_d(ridge, red);
      sm = block_max_d(sm, red);
      if (tid == 0) {
        a.kkt[3 * i + 0] = fit;
        a.kkt[3 * i + 1] = ridge;
        a.kkt[3 * i + 2] = sm;
      }
      return;
    }
  }
  block_sum3_d(fit, ridge, sm, red);
  if (tid == 0) {
    a.slice_obj[3 * i + 0] = fit;
    a.slice_obj[3 * i + 1] = ridge;
    a.slice_obj[3 * i + 2] = sm;
  }
}

}  // namespace tctf
