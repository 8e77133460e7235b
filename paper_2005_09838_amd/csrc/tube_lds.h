// Tube transforms that run in the tube's own LDS row (for the longer even tube lengths).
//
// A real tube of even length N = 2M is handled through the complex sequence
// c[m] = x[2m] + i x[2m+1] of length M (the half-length form of eq. (bar BA-k)), and the
// length-M complex transform is a four-step FFT with M = M1 * M2:
//   step A, for each n1 < M1: a length-M2 DFT over x[n1 + M1 n2], times exp(S 2 pi i n1 k2 / M),
//           stored back at complex position n1 + M1 k2;
//   step C, for each k2 < M2: a length-M1 DFT over those M1 values, result C[k2 + M2 k1]
//           stored at complex position k2 + M2 k1 (natural order).
// The small DFTs are generated straight-line code (tube_dft_gen.h).  T lanes of one wavefront
// share a tube: lane t takes the groups t, t + T, ... of each stage, and the caller orders the
// wavefront's LDS accesses between the stages.  row: the tube's M complex positions;
// twm[n1 + M1 k2] = exp(+2 pi i n1 k2 / M); twn[b] = exp(+2 pi i b / N), b <= M.
#pragma once
#include "common.h"
#include "tube_dft_gen.h"

// Step A: groups n1 = t, t + T, ...  A group's values stay at its own positions.
template <int M1, int M2, int S, int T>
__device__ __forceinline__ void fft4_step_a(float2* row, const float2* __restrict__ twm, int t) {
#pragma unroll
  for (int h = 0; h < (M1 + T - 1) / T; ++h) {
    const int n1 = t + h * T;
    if (n1 < M1) {
      float re[M2], im[M2];
#pragma unroll
      for (int n2 = 0; n2 < M2; ++n2) {
        const float2 v = row[n1 + M1 * n2];
        re[n2] = v.x;
        im[n2] = v.y;
      }
      dftc<M2, S>(re, im);
#pragma unroll
      for (int k2 = 0; k2 < M2; ++k2) {
        const float2 w = twm[n1 + M1 * k2];
        const float c = w.x, s = S > 0 ? w.y : -w.y;
        row[n1 + M1 * k2] = make_float2(fmaf(re[k2], c, -im[k2] * s), fmaf(re[k2], s, im[k2] * c));
      }
    }
  }
}

// Step C: groups k2 = t, t + T, ...  Every lane reads all of its groups' inputs before any lane
// writes (the caller orders the two), since C[k2 + M2 k1] goes to complex position k2 + M2 k1.
template <int M1, int M2, int T>
struct FftStepC {
  static constexpr int G = (M2 + T - 1) / T;
  float re[G][M1], im[G][M1];
  __device__ __forceinline__ void read(const float2* row, int t) {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      const int g = t + h * T;
      if (g < M2) {
#pragma unroll
        for (int n1 = 0; n1 < M1; ++n1) {
          const float2 v = row[n1 + M1 * g];
          re[h][n1] = v.x;
          im[h][n1] = v.y;
        }
      }
    }
  }
  template <int S>
  __device__ __forceinline__ void write(float2* row, int t) {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      const int g = t + h * T;
      if (g < M2) {
        dftc<M1, S>(re[h], im[h]);
#pragma unroll
        for (int k1 = 0; k1 < M1; ++k1) row[g + M2 * k1] = make_float2(re[h][k1], im[h][k1]);
      }
    }
  }
};

// Inverse transform (eq. (barAAk)) of the stored frequencies X[b], b = 0..M (imaginary parts of
// X[0] and X[M] taken as 0), of column j of src (frequency b at src[b n2 + j]).
//   E[b] = (X[b] + conj X[M-b]) / 2,  O[b] = (X[b] - conj X[M-b]) exp(-2 pi i b / N) / 2,
//   C[b] = E[b] + i O[b],  C[M-b] = conj E[b] + i conj O[b],  c = inverse DFT_M(C).
// The pairs (b, M - b), b = t, t + T, ... <= M / 2, of lane t: all loads first (clamped and
// unconditional), then C[b] and C[M-b] to the row.  After the four-step transform, x[2m] + i x[2m+1]
// sits at row[m].
template <int N, int T, int P>
__device__ __forceinline__ void tube_inv_load(const float2* __restrict__ src, int n2, int j, int t, float2 (&xb)[P],
                                              float2 (&xm)[P]) {
  constexpr int M = N / 2;
#pragma unroll
  for (int u = 0; u < P; ++u) {
    const int b = min(t + u * T, M / 2);
    xb[u] = src[b * n2 + j];
    xm[u] = src[(M - b) * n2 + j];
  }
}
template <int N, int T, int P>
__device__ __forceinline__ void tube_inv_pre(float2* row, const float2* __restrict__ twn, int t, const float2 (&xb)[P],
                                             const float2 (&xm)[P]) {
  constexpr int M = N / 2;
#pragma unroll
  for (int u = 0; u < P; ++u) {
    const int b = t + u * T;
    if (b <= M / 2) {
      const int mb = M - b;
      const float xbr = xb[u].x, xbi = (b == 0) ? 0.0f : xb[u].y;
      const float xmr = xm[u].x, xmi = (b == 0) ? 0.0f : xm[u].y;
      constexpr float h = 1.0f / N;   // the half of E and O and the 1 / M of the inverse
      const float er = h * (xbr + xmr), ei = h * (xbi - xmi);
      const float dr = h * (xbr - xmr), di = h * (xbi + xmi);
      const float2 w = twn[b];
      const float orr = fmaf(dr, w.x, di * w.y), oi = fmaf(di, w.x, -dr * w.y);
      row[b] = make_float2(er - oi, ei + orr);
      if (b != 0 && mb != b) row[mb] = make_float2(er + oi, orr - ei);
    }
  }
}

// Last stage of the forward transform (eq. (bar BA-k)) of the tube (row[m] = c[m] =
// x[2m] + i x[2m+1] at first) with C = DFT_M(c) in natural order: calls store(b, re, im) for the pairs
// (b, M - b), b = t, t + T, ... <= M / 2, of lane t.
//   E = (C[b] + conj C[M-b]) / 2,  O = (C[b] - conj C[M-b]) / (2i),
//   X[b] = E + exp(2 pi i b / N) O,  X[M-b] = conj(E - exp(2 pi i b / N) O),  X[M] = E[0] - O[0].
template <int N, int T, class Store>
__device__ __forceinline__ void tube_fwd_post(const float2* row, const float2* __restrict__ twn, int t, Store store) {
  constexpr int M = N / 2;
#pragma unroll
  for (int u = 0; u < (M / 2 + T) / T; ++u) {
    const int b = t + u * T;
    if (b > M / 2) break;
    const int mb = (b == 0) ? 0 : M - b;
    const float2 cb = row[b], cm = row[mb];
    const float cbr = cb.x, cbi = cb.y, cmr = cm.x, cmi = cm.y;
    const float er = 0.5f * (cbr + cmr), ei = 0.5f * (cbi - cmi);
    const float dr = 0.5f * (cbr - cmr), di = 0.5f * (cbi + cmi);
    const float orr = di, oi = -dr;   // D / i
    const float2 w = twn[b];
    const float wr = fmaf(w.x, orr, -w.y * oi), wi = fmaf(w.x, oi, w.y * orr);
    if (b == 0) {
      store(0, er + wr, 0.0f);
      store(M, er - wr, 0.0f);
    } else {
      store(b, er + wr, ei + wi);
      if (mb != b) store(mb, er - wr, wi - ei);
    }
  }
}
