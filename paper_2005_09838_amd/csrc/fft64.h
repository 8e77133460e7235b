// FP64 tube transforms of any length in LDS: P complex sequences of length N at once, N the
// product of the plan's radices, as autosorting (Stockham) passes.  Two real tubes share one
// complex sequence (c = x_0 + i x_1), which serves odd lengths as well as even ones.
#pragma once
#include "common.h"
#include "kernels.h"

namespace tctf {

#define FFT64_PER 8   // complex values per thread: P N <= FFT64_PER blockDim.x

// f / d for 0 <= f < 2^20 with rd = 1.0f / d: the quotient of f + 1/2 is at least 1 / (2 d) away
// from every integer, more than its rounding error
__device__ __forceinline__ int fft64_div(int f, float rd) { return (int)(((float)f + 0.5f) * rd); }

__device__ __forceinline__ cd cmul2(cd a, cd b) { return cd_make(fma(a.re, b.re, -a.im * b.im), fma(a.re, b.im, a.im * b.re)); }
// sigma i a, sigma = +1 or -1
__device__ __forceinline__ cd cmuli(cd a, double sg) { return cd_make(-sg * a.im, sg * a.re); }

// In-place DFT of length R with exponent sign sg.
template <int R>
__device__ __forceinline__ void dft_small(cd (&v)[R], double sg) {
  if constexpr (R == 2) {
    const cd t = v[1];
    v[1] = cd_sub(v[0], t);
    v[0] = cd_add(v[0], t);
  } else if constexpr (R == 4) {
    const cd a = cd_add(v[0], v[2]), b = cd_sub(v[0], v[2]), c = cd_add(v[1], v[3]), d = cmuli(cd_sub(v[1], v[3]), sg);
    v[0] = cd_add(a, c);
    v[1] = cd_add(b, d);
    v[2] = cd_sub(a, c);
    v[3] = cd_sub(b, d);
  } else if constexpr (R == 8) {
    cd e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
    dft_small<4>(e, sg);
    dft_small<4>(o, sg);
    const double h = 0.70710678118654752440;
    o[1] = cmul2(o[1], cd_make(h, sg * h));
    o[2] = cmuli(o[2], sg);
    o[3] = cmul2(o[3], cd_make(-h, sg * h));
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[k] = cd_add(e[k], o[k]);
      v[k + 4] = cd_sub(e[k], o[k]);
    }
  } else if constexpr (R == 9) {   // 3 x 3 with twiddles: n = 3 n1 + n2, k = k1 + 3 k2
    constexpr double C9[5] = {1.0, 0.766044443118978, 0.17364817766693041, 0.0, -0.9396926207859083}, S9[5] = {0.0, 0.6427876096865393, 0.984807753012208, 0.0, 0.3420201433256689};   // exp(2 pi i e / 9), e = n2 k1
    cd t[3][3];
#pragma unroll
    for (int b = 0; b < 3; ++b) {
#pragma unroll
      for (int a = 0; a < 3; ++a) t[b][a] = v[3 * a + b];
      dft_small<3>(t[b], sg);
#pragma unroll
      for (int k = 1; k < 3; ++k)
        if (b > 0) t[b][k] = cmul2(t[b][k], cd_make(C9[b * k], sg * S9[b * k]));
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      cd u[3] = {t[0][k], t[1][k], t[2][k]};
      dft_small<3>(u, sg);
#pragma unroll
      for (int l = 0; l < 3; ++l) v[k + 3 * l] = u[l];
    }
  } else if constexpr (R == 6 || R == 10 || R == 12) {   // coprime factors need no twiddles
    constexpr int A = R == 6 ? 3 : (R == 10 ? 5 : 3), B = R / A;
    constexpr int EA = R == 6 ? 4 : (R == 10 ? 6 : 4), EB = R == 6 ? 3 : (R == 10 ? 5 : 9);   // 1 mod A, 0 mod B and the reverse
    cd t[B][A];
#pragma unroll
    for (int b = 0; b < B; ++b) {
#pragma unroll
      for (int a = 0; a < A; ++a) t[b][a] = v[(B * a + A * b) % R];
      dft_small<A>(t[b], sg);
    }
#pragma unroll
    for (int k = 0; k < A; ++k) {
      cd u[B];
#pragma unroll
      for (int b = 0; b < B; ++b) u[b] = t[b][k];
      dft_small<B>(u, sg);
#pragma unroll
      for (int l = 0; l < B; ++l) v[(EA * k + EB * l) % R] = u[l];
    }
  } else {   // odd R through the sums and differences of the pairs (q, R - q)
    constexpr int H = (R - 1) / 2;
    // cos and sin of 2 pi k / R, k = 1..H
    constexpr double C3[1] = {-0.5}, S3[1] = {0.86602540378443864676};
    constexpr double C5[2] = {0.30901699437494742410, -0.80901699437494742410}, S5[2] = {0.95105651629515357212, 0.58778525229247312917};
    constexpr double C7[3] = {0.62348980185873353053, -0.22252093395631440429, -0.90096886790241912624};
    constexpr double S7[3] = {0.78183148246802980871, 0.97492791218182360702, 0.43388373911755812048};
    cd s[H], d[H], x0 = v[0], sum = v[0];
#pragma unroll
    for (int q = 1; q <= H; ++q) {
      s[q - 1] = cd_add(v[q], v[R - q]);
      d[q - 1] = cd_sub(v[q], v[R - q]);
      sum = cd_add(sum, s[q - 1]);
    }
    v[0] = sum;
#pragma unroll
    for (int k = 1; k <= H; ++k) {
      cd a = x0, b = cd_make(0.0, 0.0);
#pragma unroll
      for (int q = 1; q <= H; ++q) {
        const int t = (k * q) % R, u = t <= H ? t : R - t;
        const double c = R == 3 ? C3[u > 1 ? 0 : u - 1] : (R == 5 ? C5[u > 2 ? 0 : u - 1] : C7[u - 1]);
        const double sn = (R == 3 ? S3[u > 1 ? 0 : u - 1] : (R == 5 ? S5[u > 2 ? 0 : u - 1] : S7[u - 1])) * (t <= H ? 1.0 : -1.0);
        a = cd_make(fma(c, s[q - 1].re, a.re), fma(c, s[q - 1].im, a.im));
        b = cd_make(fma(sn, d[q - 1].re, b.re), fma(sn, d[q - 1].im, b.im));
      }
      const cd ib = cmuli(b, sg);
      v[k] = cd_add(a, ib);
      v[R - k] = cd_sub(a, ib);
    }
  }
}

// One pass of radix R: butterfly j of a sequence reads j + r N / R, twiddles by
// exp(sg 2 pi i r (j mod Ns) / (Ns R)) and writes (j / Ns) Ns R + j mod Ns + r Ns.  Every thread
// reads all of its butterflies before any thread writes.
template <int R>
__device__ __forceinline__ void fft64_pass(cd* x, int N, int P, int Ns, const cd* tw, int ts, double sg) {
  constexpr int B = (FFT64_PER + R - 1) / R;
  const int tid = threadIdx.x, nt = blockDim.x, nr = N / R, tot = P * nr, step = nr / Ns;   // N / (Ns R)
  const float rnr = 1.0f / nr, rns = 1.0f / Ns;
  cd v[B][R];
  int at[B];
#pragma unroll
  for (int h = 0; h < B; ++h) {
    const int f = tid + h * nt;
    at[h] = -1;
    if (f < tot) {
      const int pr = fft64_div(f, rnr), j = f - pr * nr, jd = fft64_div(j, rns), jm = j - jd * Ns;
      const cd* src = x + pr * N + j;
      at[h] = pr * N + jd * Ns * R + jm;
#pragma unroll
      for (int r = 0; r < R; ++r) v[h][r] = src[r * nr];
      if (Ns > 1) {   // powers of the twiddle as an even and an odd chain
        cd w = tw[jm * step * ts];
        w.im *= sg;
        const cd w2 = cmul2(w, w);
        cd po = w, pe = w2;
#pragma unroll
        for (int r = 1; r < R; r += 2) {
          v[h][r] = cmul2(v[h][r], po);
          if (r + 1 < R) v[h][r + 1] = cmul2(v[h][r + 1], pe);
          if (r + 2 < R) po = cmul2(po, w2);
          if (r + 3 < R) pe = cmul2(pe, w2);
        }
      }
      dft_small<R>(v[h], sg);
    }
  }
  __syncthreads();
#pragma unroll
  for (int h = 0; h < B; ++h) {
    if (at[h] >= 0) {
#pragma unroll
      for (int r = 0; r < R; ++r) x[at[h] + r * Ns] = v[h][r];
    }
  }
  __syncthreads();
}

// The same for any radix: output by output, sum_u x_u exp(sg 2 pi i u (jm + t Ns) / (Ns R)).
__device__ __forceinline__ void fft64_pass_any(cd* x, int N, int P, int R, int Ns, const cd* tw, int ts, double sg) {
  const int tid = threadIdx.x, nt = blockDim.x, nr = N / R, tot = P * N, step = nr / Ns;
  const float rn = 1.0f / N, rnsr = 1.0f / (Ns * R), rns = 1.0f / Ns;
  cd v[FFT64_PER];
#pragma unroll
  for (int h = 0; h < FFT64_PER; ++h) {
    const int f = tid + h * nt;
    v[h] = cd_make(0.0, 0.0);
    if (f < tot) {
      const int pr = fft64_div(f, rn), o = f - pr * N, jd = fft64_div(o, rnsr), oo = o - jd * Ns * R;
      const int t = fft64_div(oo, rns), jm = oo - t * Ns, e1 = (jm + t * Ns) * step;
      const cd* src = x + pr * N + jd * Ns + jm;
      int e = 0;   // u e1 mod N
      cd acc = cd_make(0.0, 0.0);
      for (int u = 0; u < R; ++u) {
        cd w = tw[e * ts];
        w.im *= sg;
        cd_fma(acc, src[u * nr], w);
        e += e1;
        if (e >= N) e -= N;
      }
      v[h] = acc;
    }
  }
  __syncthreads();
#pragma unroll
  for (int h = 0; h < FFT64_PER; ++h) {
    const int f = tid + h * nt;
    if (f < tot) x[f] = v[h];
  }
  __syncthreads();
}

// All passes; x holds the sequences in natural order before and after.  tw[ts e] = exp(2 pi i e / N).
// Begins and ends with a block barrier.
__device__ inline void fft64(cd* x, int P, const Fft64Plan& pl, const cd* tw, int ts, double sg) {
  int Ns = 1;
  __syncthreads();
  for (int k = 0; k < pl.passes; ++k) {
    const int R = pl.radix[k], N = pl.n;
    switch (R) {
      case 2: fft64_pass<2>(x, N, P, Ns, tw, ts, sg); break;
      case 3: fft64_pass<3>(x, N, P, Ns, tw, ts, sg); break;
      case 4: fft64_pass<4>(x, N, P, Ns, tw, ts, sg); break;
      case 5: fft64_pass<5>(x, N, P, Ns, tw, ts, sg); break;
      case 6: fft64_pass<6>(x, N, P, Ns, tw, ts, sg); break;
      case 7: fft64_pass<7>(x, N, P, Ns, tw, ts, sg); break;
      case 8: fft64_pass<8>(x, N, P, Ns, tw, ts, sg); break;
      case 9: fft64_pass<9>(x, N, P, Ns, tw, ts, sg); break;
      case 10: fft64_pass<10>(x, N, P, Ns, tw, ts, sg); break;
      case 12: fft64_pass<12>(x, N, P, Ns, tw, ts, sg); break;
      default: fft64_pass_any(x, N, P, R, Ns, tw, ts, sg); break;
    }
    Ns *= R;
  }
}

}  // namespace tctf
