// Moore-Penrose inverse of a small Hermitian positive-semidefinite Gram matrix in FP64,
// computed cooperatively by one thread block (Lemma SVPMPI: A^+ = V diag(1/lambda) V^*
// over the kept eigenvalues).
//
// Rule: eigenvalues lambda_i <= tau = r * eps64 * lambda_max are dropped (a zero matrix
// gives 0).  Fast path: Gauss-Jordan elimination (the sweep operator, no pivoting, valid
// for positive-definite input) in LDS, pinv_sweep.  Its result is accepted only if it proves that every eigenvalue exceeds 8 tau:
// lambda_min >= 1/||A^-1||_F > 8 r eps ||A||_F >= 8 tau.  Then the rule keeps every
// eigenvalue and A^+ = A^-1.  Otherwise (or when forced) a cyclic Jacobi
// eigen-decomposition with parallel (round-robin) pair ordering is used by the whole block
// and the rule is applied to its eigenvalues.
//
// The routines are forced inline: called out of line they take their LDS through generic
// addresses and give every kernel that hosts them 152 registers (r = 30 by the eigen route: 761 us
// beside the Z~ product and 824 in the X~^* W~ launch, 535 and 491 inline).
#pragma once
#include "common.h"
#include "kernels.h"

#define TCTF_EPS64 2.220446049250313e-16

struct PinvScratch {
  cd* work;    // r*r
  cd* vec;     // r*r
  double* rot; // 6 * 16 doubles (rotation parameters of one round)
  double* red; // >= 48 doubles
};

// Fast path: the sweep operator on the 2 x 2 pivot blocks K = {k, k + 1} (a last 1 x 1 block at
// odd r), every thread of the block on its own entries:
//   A_KK -> -E, A_Kj -> E A_Kj, A_iK -> A_iK E, A_ij -> A_ij - A_iK E A_Kj,  E = A_KK^-1;
// sweeping every index gives -A^-1.  Each step reads one LDS copy and writes another, so it
// costs one barrier, and every thread forms E for itself: about 0.6 us a step at r <= 16 (r = 16
// with its Gram read and results written 8.5 us; one wavefront with the matrix in registers,
// passing pivots by cross-lane moves, 10.1; r = 24 19.4 us, 33 with two barriers and 1 x 1
// pivots).  Returns 1 when every pivot was positive; then *out holds -A^-1 (one of w0, w1).
template <int PER>   // entries of a thread in flight
__device__ __forceinline__ int pinv_sweep(const cd* A, cd* w0, cd* w1, int r, const cd** out) {
  const int tid = threadIdx.x, nt = blockDim.x, rr = r * r;
  const int p0 = tid / r, q0 = tid - p0 * r, dp = nt / r, dq = nt - dp * r;
  const cd* src = A;
  cd* dst = w0;
  int ok = 1;
  for (int k = 0; k < r; k += 2) {
    const bool two = k + 1 < r;
    const int k1 = two ? k + 1 : k;
    const cd pa = src[k * r + k], pb = src[k * r + k1], pd = src[k1 * r + k1];
    int p = p0, q = q0;
    for (int e0 = tid; e0 < rr; e0 += PER * nt) {
      // every LDS read of the batch is issued before any use
      cd c0[PER], c1[PER], u0[PER], u1[PER], v[PER];
      int ph[PER], qh[PER];
#pragma unroll
      for (int h = 0; h < PER; ++h) {
        const bool in = e0 + h * nt < rr;
        ph[h] = in ? p : 0;
        qh[h] = in ? q : 0;
        p += dp;
        q += dq;
        if (q >= r) {
          q -= r;
          ++p;
        }
        c0[h] = src[ph[h] * r + k];
        c1[h] = src[ph[h] * r + k1];
        u0[h] = src[k * r + qh[h]];
        u1[h] = src[k1 * r + qh[h]];
        v[h] = src[ph[h] * r + qh[h]];
      }
      const double det = two ? pa.re * pd.re - (pb.re * pb.re + pb.im * pb.im) : pa.re;
      const double idet = 1.0 / det, e00 = two ? pd.re * idet : idet, e11 = two ? pa.re * idet : 0.0;
      const cd e01 = cd_make(two ? -pb.re * idet : 0.0, two ? -pb.im * idet : 0.0), e10 = cd_conj(e01);
#pragma unroll
      for (int h = 0; h < PER; ++h) {
        const bool row0 = ph[h] == k, row1 = ph[h] == k1, col0 = qh[h] == k, col1 = qh[h] == k1;
        // (R0, R1): A_pK E, or in a pivot row minus that row of E
        cd r0 = cd_add(cd_scale(c0[h], e00), cd_mul(c1[h], e10)), r1 = cd_add(cd_mul(c0[h], e01), cd_scale(c1[h], e11));
        r0.re = row0 ? -e00 : (row1 ? -e10.re : r0.re);
        r0.im = row0 ? 0.0 : (row1 ? -e10.im : r0.im);
        r1.re = row0 ? -e01.re : (row1 ? -e11 : r1.re);
        r1.im = row0 ? -e01.im : (row1 ? 0.0 : r1.im);
        cd o = row0 || row1 ? cd_make(0.0, 0.0) : v[h];
        o = cd_sub(cd_sub(o, cd_mul(r0, u0[h])), cd_mul(r1, u1[h]));
        o.re = col0 ? r0.re : (col1 ? r1.re : o.re);
        o.im = col0 ? r0.im : (col1 ? r1.im : o.im);
        if (e0 + h * nt < rr) dst[e0 + h * nt] = o;
      }
    }
    // the same in every thread
    ok &= pa.re > 0.0 && (two ? pa.re * pd.re - (pb.re * pb.re + pb.im * pb.im) : pa.re) > 0.0;
    __syncthreads();
    src = dst;
    dst = dst == w0 ? w1 : w0;
  }
  *out = src;
  return ok;
}

// Cyclic Jacobi eigen-decomposition of a Hermitian r x r matrix A by the whole block, with
// parallel (round-robin) pair ordering: on return s.work holds the rotated matrix (the
// eigenvalues on its diagonal, unsorted) and s.vec the eigenvectors as columns.  fro is
// ||A||_F (the sweeps stop when the off-diagonal part falls below 1e-14 fro).
__device__ __forceinline__ void jacobi_herm(const cd* A, int r, double fro, PinvScratch s) {
  const int tid = threadIdx.x, nt = blockDim.x, rr = r * r;
  for (int e = tid; e < rr; e += nt) {
    s.work[e] = A[e];
    s.vec[e] = cd_make((e / r == e % r) ? 1.0 : 0.0, 0.0);
  }
  __syncthreads();
  const int rp = r + (r & 1), npair = rp / 2;
  for (int sweep = 0; sweep < 30; ++sweep) {
    double off = 0.0;
    for (int e = tid; e < rr; e += nt)
      if (e / r != e % r) off += s.work[e].re * s.work[e].re + s.work[e].im * s.work[e].im;
    off = block_sum_d(off, s.red);
    if (sqrt(off) <= 1e-14 * fro) break;
    for (int m = 0; m < rp - 1; ++m) {
      // rotation parameters of every disjoint pair of this round
      for (int i = tid; i < npair; i += nt) {
        int p, q;
        if (i == 0) { p = rp - 1; q = m; }
        else { p = (m + i) % (rp - 1); q = (m - i + rp - 1) % (rp - 1); }
        if (p > q) { int t = p; p = q; q = t; }
        double* R = s.rot + 6 * i;
        R[0] = -1.0;   // p < 0 marks "no rotation"
        if (q < r) {
          const double a = s.work[p * r + p].re, d = s.work[q * r + q].re;
          const cd b = s.work[p * r + q];
          const double ab = hypot(b.re, b.im);
          if (ab > 1e-300 && ab > TCTF_EPS64 * 1e-3 * sqrt(fabs(a * d))) {
            const double ph_re = b.re / ab, ph_im = b.im / ab;
            const double zeta = (d - a) / (2.0 * ab);
            double t;
            if (fabs(zeta) > 1e150) t = 0.5 / zeta;
            else t = (zeta >= 0.0 ? 1.0 : -1.0) / (fabs(zeta) + sqrt(1.0 + zeta * zeta));
            const double c = 1.0 / sqrt(1.0 + t * t), sn = t * c;
            R[0] = p; R[1] = q; R[2] = c; R[3] = sn; R[4] = ph_re; R[5] = ph_im;
          }
        }
      }
      __syncthreads();
      // columns: A <- A U and V <- V U with U_pp = c, U_pq = s, U_qp = -s conj(phi), U_qq = c conj(phi)
      for (int e = tid; e < npair * r; e += nt) {
        const double* R = s.rot + 6 * (e / r);
        if (R[0] < 0.0) continue;
        const int p = (int)R[0], q = (int)R[1], row = e % r;
        const double c = R[2], sn = R[3];
        const cd phc = cd_make(R[4], -R[5]);
        const cd upq = cd_make(sn, 0.0), uqp = cd_scale(phc, -sn), uqq = cd_scale(phc, c);
        for (int pass = 0; pass < 2; ++pass) {
          cd* M = pass ? s.vec : s.work;
          const cd xp = M[row * r + p], xq = M[row * r + q];
          M[row * r + p] = cd_add(cd_scale(xp, c), cd_mul(xq, uqp));
          M[row * r + q] = cd_add(cd_mul(xp, upq), cd_mul(xq, uqq));
        }
      }
      __syncthreads();
      // rows: A <- U^* A
      for (int e = tid; e < npair * r; e += nt) {
        const double* R = s.rot + 6 * (e / r);
        if (R[0] < 0.0) continue;
        const int p = (int)R[0], q = (int)R[1], col = e % r;
        const double c = R[2], sn = R[3];
        const cd ph = cd_make(R[4], R[5]);
        // conj(U_qp) = -s phi, conj(U_qq) = c phi
        const cd xp = s.work[p * r + col], xq = s.work[q * r + col];
        s.work[p * r + col] = cd_add(cd_scale(xp, c), cd_scale(cd_mul(xq, ph), -sn));
        s.work[q * r + col] = cd_add(cd_scale(xp, sn), cd_scale(cd_mul(xq, ph), c));
      }
      __syncthreads();
    }
  }
}

// Returns 1 (to every thread) if all eigenvalues were kept, 0 otherwise.
__device__ __forceinline__ int pinv_herm(const cd* A, cd* P, int r, int force_eigen, PinvScratch s) {
  const int tid = threadIdx.x, nt = blockDim.x, rr = r * r;
  if (!force_eigen) {
    const cd* swept;
    // a matrix that is not finite, zero or indefinite has no positive pivot somewhere: not ok
    const int ok = rr <= nt ? pinv_sweep<1>(A, s.work, s.vec, r, &swept) : pinv_sweep<2>(A, s.work, s.vec, r, &swept);
    if (ok) {
      // the norms, by every wavefront for itself: no barrier
      double f2 = 0.0, g2 = 0.0;
      for (int e = tid & 63; e < rr; e += 64) {
        const cd a = A[e], v = swept[e];
        f2 += a.re * a.re + a.im * a.im;
        g2 += v.re * v.re + v.im * v.im;
      }
      for (int off = 32; off > 0; off >>= 1) {
        f2 += __shfl_xor(f2, off);
        g2 += __shfl_xor(g2, off);
      }
      if (isfinite(g2) && isfinite(f2) && 8.0 * r * TCTF_EPS64 * sqrt(f2) * sqrt(g2) < 1.0) {
        for (int e = tid; e < rr; e += nt) P[e] = cd_make(-swept[e].re, -swept[e].im);
        __syncthreads();
        return 1;
      }
    }
    __syncthreads();   // the other paths write over the copies
  }
  double f2 = 0.0, dmax = -1.0;
  for (int e = tid; e < rr; e += nt) {
    cd a = A[e];
    f2 += a.re * a.re + a.im * a.im;
    if (e / r == e % r) dmax = fmax(dmax, a.re);
  }
  f2 = block_sum_d(f2, s.red);
  dmax = block_max_d(dmax, s.red);
  if (!isfinite(f2)) {
    for (int e = tid; e < rr; e += nt) P[e] = cd_make(NAN, NAN);
    __syncthreads();
    return 0;
  }
  if (!(dmax > 0.0)) {   // PSD with a non-positive diagonal: the zero matrix
    for (int e = tid; e < rr; e += nt) P[e] = cd_make(0.0, 0.0);
    __syncthreads();
    return 0;
  }
  const double fro = sqrt(f2);

  // Jacobi eigen-decomposition of A into work (eigenvalues on the diagonal) and vec.
  jacobi_herm(A, r, fro, s);
  double lmax = -1e300;
  for (int i = tid; i < r; i += nt) lmax = fmax(lmax, s.work[i * r + i].re);
  lmax = block_max_d(lmax, s.red);
  const double tau = fmax(r * TCTF_EPS64 * lmax, 0.0);
  int kept = 0;
  for (int i = 0; i < r; ++i) kept += (s.work[i * r + i].re > tau) ? 1 : 0;
  for (int e = tid; e < rr; e += nt) {
    const int p = e / r, q = e % r;
    cd acc = cd_make(0.0, 0.0);
    for (int i = 0; i < r; ++i) {
      const double l = s.work[i * r + i].re;
      if (l > tau) acc = cd_add(acc, cd_scale(cd_mulc(s.vec[p * r + i], s.vec[q * r + i]), 1.0 / l));
    }
    P[e] = acc;
  }
  __syncthreads();
  return kept == r ? 1 : 0;
}

// Bytes of LDS of a Gram, its pseudo-inverse and the scratch at rank r.
__host__ __device__ inline size_t pinv_lds_bytes(int r) {
  return (size_t)(4 * r * r) * sizeof(cd) + 144 * sizeof(double);
}

// Inputs and outputs of pinvy_block ([nb][r][r] FP64 complex unless noted).
struct PinvyArgs {
  const cd* gyq;      // [nb][ny][r][r] partial Grams of Y~ over column blocks
  int ny;
  const cd* dmat;     // (H X~)^*(H X~)
  double* bin_obj;    // [nb] c_b tr((H X~)^*(H X~) G_Y): the rho1 term of eq. (fun-XYW)
  int n3;
  cd* gyp;            // G_Y^+
  cd* qy;             // I - eta P_Y
  int* qy_zero;       // [nb] 1 when I - eta P_Y is exactly 0
  int r;
  double eta;
  int force_eigen;
};

static inline PinvyArgs pinvy_args(const tctf::Plan& p) {
  PinvyArgs a;
  a.gyq = p.gym;
  a.ny = p.ny;
  a.dmat = p.dmat;
  a.bin_obj = p.bin_obj;
  a.n3 = p.n3;
  a.gyp = p.gyp;
  a.qy = p.qy;
  a.qy_zero = p.qy_zero;
  a.r = p.r;
  a.eta = p.eta;
  a.force_eigen = p.force_eigen;
  return a;
}

// Per frequency b, by a whole block: G_Y as the sum of the column-block partials (fixed
// order), the objective term c_b tr(D G_Y), G_Y^+ and, unless it is exactly 0,
// q = I - eta G_Y G_Y^+ for the next X-update (first line of eq. (updataXYW1)); qy_zero[b] = 1
// marks q = 0.  sm: pinv_lds_bytes(r) bytes of LDS.
__device__ __forceinline__ void pinvy_block(int b, const PinvyArgs& a, unsigned char* sm) {
  const int tid = threadIdx.x, nt = blockDim.x, r = a.r, rr = r * r;
  cd* gy = (cd*)sm;
  cd* gp = gy + rr;
  PinvScratch ps;
  ps.work = gp + rr;
  ps.vec = ps.work + rr;
  ps.rot = (double*)(ps.vec + rr);
  ps.red = ps.rot + 96;
  for (int e = tid; e < rr; e += nt) {
    const cd* src = a.gyq + (size_t)b * a.ny * rr + e;
    cd g = src[0];
    for (int k0 = 1; k0 < a.ny; k0 += 8) {   // eight partials' loads in flight, added in order
      cd v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = src[(size_t)min(k0 + k, a.ny - 1) * rr];
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (k0 + k < a.ny) g = cd_add(g, v[k]);
    }
    gy[e] = g;
  }
  __syncthreads();
  const int fully = pinv_herm(gy, gp, r, a.force_eigen, ps);
  const bool qyz = fully && a.eta == 1.0;
  for (int e = tid; e < rr; e += nt) {
    cd qv = cd_make(0.0, 0.0);
    if (!qyz) {
      const int s = e / r, t = e % r;
      cd acc = cd_make(0.0, 0.0);
      for (int u = 0; u < r; ++u) cd_fma(acc, gy[s * r + u], gp[u * r + t]);
      qv = cd_make((s == t ? 1.0 : 0.0) - a.eta * acc.re, -a.eta * acc.im);
    }
    a.qy[(size_t)b * rr + e] = qv;
    a.gyp[(size_t)b * rr + e] = gp[e];
  }
  if (tid == 0) a.qy_zero[b] = qyz ? 1 : 0;
  if (tid < 64) {   // tr(D G_Y), by one wavefront
    double tr = 0.0;
    for (int e = tid; e < rr; e += 64) {
      const cd d = a.dmat[(size_t)b * rr + (e % r) * r + e / r], g = gy[e];   // D(t, s) for G_Y(s, t)
      tr += d.re * g.re - d.im * g.im;
    }
    for (int off = 32; off > 0; off >>= 1) tr += __shfl_xor(tr, off);
    if (tid == 0) a.bin_obj[b] = bin_weight(b, a.n3) * tr;
  }
}
