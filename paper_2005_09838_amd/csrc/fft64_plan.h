// Host side: the passes of a complex FP64 transform (fft64.h).
#pragma once

namespace tctf {

// Passes of a transform of length n, the product of the radices.
#define FFT64_MAX_PASSES 14   // the search goes down to 2^13; no length up to 8192 needs more than 5
struct Fft64Plan {
  int n, passes;
  int radix[FFT64_MAX_PASSES];
};

// The fewest passes over the radices of dft_small, and of two such plans the one with the smaller
// largest radix (the slice stage in us with the first found / this: 288 x 28 x 288 as 12 12 2 49.2, 8 6
// 6 48.0; 144 x 28 x 36 as 12 3 17.3, 6 6 16.4; 20 x 20 x 2016 as 12 12 7 2 33.8, 8 7 6 6 32.8; 100 x 20 x
// 336 as 12 7 4 23.9, 8 7 6 24.4), prime factors past 7 as passes of their own.  Odd radices first: the
// first pass writes its outputs R apart, which an even R would put into few LDS banks.  The radices
// of cur and best do not increase: the first is the largest.
inline void fft64_factor(int n, int cap, int* cur, int depth, int* best, int* passes) {
  if (n == 1) {
    if (depth == *passes && depth > 0 && cur[0] >= best[0]) return;
    *passes = depth;
    for (int k = 0; k < depth; ++k) best[k] = cur[k];
    return;
  }
  if (depth == *passes) return;
  static const int radices[] = {12, 10, 9, 8, 7, 6, 5, 4, 3, 2};
  for (int r : radices)
    if (r <= cap && n % r == 0) {
      cur[depth] = r;
      fft64_factor(n / r, r, cur, depth + 1, best, passes);
    }
}
inline Fft64Plan fft64_plan(int n) {
  Fft64Plan pl;
  pl.n = n;
  pl.passes = 0;
  for (int r = 11; r <= n; r += 2)
    while (n % r == 0 && r % 3 && r % 5 && r % 7) {   // what is left of r's smaller factors is gone: r is prime
      pl.radix[pl.passes++] = r;
      n /= r;
    }
  int cur[FFT64_MAX_PASSES], best[FFT64_MAX_PASSES] = {13}, passes = FFT64_MAX_PASSES;
  fft64_factor(n, 12, cur, 0, best, &passes);
  for (int odd = 1; odd >= 0; --odd)
    for (int k = 0; k < passes; ++k)
      if ((best[k] & 1) == odd) pl.radix[pl.passes++] = best[k];
  return pl;
}

}  // namespace tctf
