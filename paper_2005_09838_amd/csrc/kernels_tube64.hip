// FP64 tube transforms between spatial tubes and stored frequencies for any tube length and any
// strides: the initial factors and the factor results, the three-launch slice path and the
// adjoint.  Forward (eq. (bar BA-k)): X[b] = s sum_k x[k] exp(+2 pi i b k / n3), b = 0 .. n3 / 2;
// inverse (eq. (barAAk)): x[k] = s sum_b c_b Re(exp(-2 pi i b k / n3) X[b]).
#include "fft64.h"
#include "kernels.h"

namespace tctf {

template <int KIND> struct SpecOf { typedef float2 type; };
template <> struct SpecOf<SPEC_F64> { typedef double2 type; };

template <int KIND>
__device__ __forceinline__ cd spec_load(const void* in, size_t at) {
  const typename SpecOf<KIND>::type v = ((const typename SpecOf<KIND>::type*)in)[at];
  return cd_make(v.x, v.y);
}
// key: of the BF16 rounding bits (SPEC_BF16)
template <int KIND>
__device__ __forceinline__ void spec_store(void* out, size_t at, double re, double im, uint32_t key) {
  if constexpr (KIND == SPEC_F64) ((double2*)out)[at] = make_double2(re, im);
  else if constexpr (KIND == SPEC_F32) ((float2*)out)[at] = make_float2((float)re, (float)im);
  else ((uint32_t*)out)[at] = pack_bf16x2_sr((float)re, (float)im, fmix32((uint32_t)at ^ key));
}

// Block (x, y): up to 2 PP tubes (y, q), q = 2 PP x ..., as PP complex sequences in LDS, then the
// roots of unity unless the caller's table holds them.  A sequence carries two tubes: on the
// inverse C[k] = A[k] + i B[k] over the conjugate-symmetric extension of both spectra, on the
// forward A = (C[k] + conj C[N - k]) / 2, B = (C[k] - conj C[N - k]) / (2 i); either tube carries the
// FP64 rounding of the larger.  What bounds it: LDS traffic and the barriers of the passes (288 x 28
// x 144: 10.9 us with two passes, 16.7 with four and twice the values per block, direct sums 115;
// 72 pairs of 8064, too few for pairs, 25.3 us with four passes, 29.6 with six of radices up to 8).
// NT: at most 256 threads hold a butterfly of 12 in registers, 1024 would not at the others' expense.
struct Tube64 {
  long bs, ps, qs;   // strides of the spectrum
  long sp, sq;       // strides of the spatial tubes
  int Q, PP;
  int lds_tw;          // the roots are in LDS
  double s;
  const double2* tw;   // exp(2 pi i e / n3), or NULL
  RowSums rows;        // of the rows y, summed by the first block of each (k_tube64_fwd)
};
// The roots of unity: in LDS behind the sequences (from the caller's table, or formed), or the table
// itself where a sequence leaves no room.
__device__ __forceinline__ const cd* tube64_roots(const Tube64& t, cd* w, int N) {
  if (!t.lds_tw) return (const cd*)t.tw;
  for (int e = threadIdx.x; e < N; e += blockDim.x) {
    double sn, c;
    if (t.tw) {
      c = t.tw[e].x;
      sn = t.tw[e].y;
    } else {
      sincospi(2.0 * e / N, &sn, &c);
    }
    w[e] = cd_make(c, sn);
  }
  return w;
}

// The partial sums of row blockIdx.y, by the row's first block.
__device__ __forceinline__ void tube64_rows(const Tube64& t) {
  const int tid = threadIdx.x;
  if (t.rows.part && blockIdx.x == 0 && tid < 3) {
    const double* part = t.rows.part + 3 * (size_t)blockIdx.y * t.rows.nchunk + tid;
    double v = 0.0;
    for (int c = 0; c < t.rows.nchunk; ++c) v += part[3 * c];
    t.rows.out[3 * blockIdx.y + tid] = v;
  }
}

template <int KIND, typename T, int NT>
__global__ void __launch_bounds__(NT) k_tube64_inv(const void* __restrict__ in, T* __restrict__ out, T* __restrict__ out2,
                                                     Tube64 t, Fft64Plan pl) {
  extern __shared__ __align__(16) unsigned char sm[];
  cd* x = (cd*)sm;
  const int N = pl.n, nb = N / 2 + 1, q0 = 2 * t.PP * blockIdx.x, tid = threadIdx.x, nt = blockDim.x;
  const int nq = min(2 * t.PP, t.Q - q0), np = (nq + 1) >> 1;
  const float rp = 1.0f / np, rn = 1.0f / N;
  const cd* tw = tube64_roots(t, x + t.PP * N, N);
  for (int e = tid; e < nb * np; e += nt) {
    const int b = fft64_div(e, rp), pp = e - b * np;
    const size_t at = b * t.bs + blockIdx.y * t.ps + (q0 + 2 * pp) * t.qs;
    const bool two = 2 * pp + 1 < nq;
    cd a = spec_load<KIND>(in, at), c = spec_load<KIND>(in, at + (two ? t.qs : 0));
    if (!two) c = cd_make(0.0, 0.0);
    if (b == 0 || 2 * b == N) a.im = c.im = 0.0;
    x[pp * N + b] = cd_make(a.re - c.im, a.im + c.re);
    if (b > 0 && 2 * b != N) x[pp * N + N - b] = cd_make(a.re + c.im, c.re - a.im);
  }
  fft64(x, np, pl, tw, 1, -1.0);
  for (int e = tid; e < nq * N; e += nt) {
    const int q = fft64_div(e, rn), k = e - q * N;
    const cd v = x[(q >> 1) * N + k];
    const T z = (T)(t.s * ((q & 1) ? v.im : v.re));
    const size_t at = blockIdx.y * t.sp + (q0 + q) * t.sq + k;
    out[at] = z;
    if (out2) out2[at] = z;
  }
}

template <int KIND, typename T, int NT>
__global__ void __launch_bounds__(NT) k_tube64_fwd(const T* __restrict__ in, void* __restrict__ out, Tube64 t, Fft64Plan pl,
                                                     const uint32_t* __restrict__ ctr) {
  extern __shared__ __align__(16) unsigned char sm[];
  cd* x = (cd*)sm;
  const int N = pl.n, nb = N / 2 + 1, q0 = 2 * t.PP * blockIdx.x, tid = threadIdx.x, nt = blockDim.x;
  const int nq = min(2 * t.PP, t.Q - q0), np = (nq + 1) >> 1;
  const float rp = 1.0f / np, rn = 1.0f / N;
  tube64_rows(t);
  const cd* tw = tube64_roots(t, x + t.PP * N, N);
  for (int e = tid; e < np * N; e += nt) {
    const int pp = fft64_div(e, rn), k = e - pp * N;
    const size_t at = blockIdx.y * t.sp + (q0 + 2 * pp) * t.sq + k;
    const bool two = 2 * pp + 1 < nq;
    const T a = in[at], c = in[at + (two ? t.sq : 0)];
    x[pp * N + k] = cd_make((double)a, two ? (double)c : 0.0);
  }
  fft64(x, np, pl, tw, 1, +1.0);
  uint32_t key = 0;
  if constexpr (KIND == SPEC_BF16) key = fmix32(ctr[0] * 0x9e3779b9u + 0x7f4a7c15u);
  for (int e = tid; e < nb * np; e += nt) {
    const int b = fft64_div(e, rp), pp = e - b * np;
    const cd c = x[pp * N + b], d = x[pp * N + (b ? N - b : 0)];
    const bool real = b == 0 || 2 * b == N;
    const double h = 0.5 * t.s;
    const size_t at = b * t.bs + blockIdx.y * t.ps + (q0 + 2 * pp) * t.qs;
    spec_store<KIND>(out, at, h * (c.re + d.re), real ? 0.0 : h * (c.im - d.im), key);
    if (2 * pp + 1 < nq) spec_store<KIND>(out, at + t.qs, h * (c.im + d.im), real ? 0.0 : h * (d.re - c.re), key);
  }
}

// ---- one even tube per block through the complex sequence c[m] = x[2 m] + i x[2 m + 1] of half its
// length M: long tubes that are too few to fill the device as pairs.  512 threads of up to eight
// values, which leaves each the registers of its widest butterfly.  12 x 12 x 8064: 19.1 us inverse
// and 23.4 forward for 144 blocks, 25.3 and 24.7 for 72 of pairs.
template <int KIND, typename T>
__global__ void __launch_bounds__(512) k_tube64_half_inv(const void* __restrict__ in, T* __restrict__ out,
                                                          T* __restrict__ out2, Tube64 t, Fft64Plan pl) {
  extern __shared__ __align__(16) unsigned char sm[];
  cd* x = (cd*)sm;
  const int M = pl.n, tid = threadIdx.x, nt = blockDim.x;
  const cd* tw = (const cd*)t.tw;
  const size_t src = blockIdx.y * t.ps + blockIdx.x * t.qs, dst = blockIdx.y * t.sp + blockIdx.x * t.sq;
  for (int b = tid; b < M; b += nt) {
    // C[b] = X[b] + conj X[M - b] + i exp(-2 pi i b / N) (X[b] - conj X[M - b])
    cd p = spec_load<KIND>(in, src + b * t.bs), q = spec_load<KIND>(in, src + (M - b) * t.bs);
    if (b == 0) p.im = q.im = 0.0;
    q.im = -q.im;
    cd w = tw[b];
    w.im = -w.im;
    const cd o = cmul2(cd_sub(p, q), w), e = cd_add(p, q);
    x[b] = cd_make(e.re - o.im, e.im + o.re);
  }
  fft64(x, 1, pl, tw, 2, -1.0);
  for (int k = tid; k < 2 * M; k += nt) {
    const T z = (T)(t.s * ((const double*)x)[k]);
    out[dst + k] = z;
    if (out2) out2[dst + k] = z;
  }
}

template <int KIND, typename T>
__global__ void __launch_bounds__(512) k_tube64_half_fwd(const T* __restrict__ in, void* __restrict__ out, Tube64 t,
                                                          Fft64Plan pl, const uint32_t* __restrict__ ctr) {
  extern __shared__ __align__(16) unsigned char sm[];
  cd* x = (cd*)sm;
  const int M = pl.n, tid = threadIdx.x, nt = blockDim.x;
  const cd* tw = (const cd*)t.tw;
  tube64_rows(t);
  const size_t src = blockIdx.y * t.sp + blockIdx.x * t.sq, dst = blockIdx.y * t.ps + blockIdx.x * t.qs;
  for (int k = tid; k < 2 * M; k += nt) ((double*)x)[k] = (double)in[src + k];
  fft64(x, 1, pl, tw, 2, +1.0);
  uint32_t key = 0;
  if constexpr (KIND == SPEC_BF16) key = fmix32(ctr[0] * 0x9e3779b9u + 0x7f4a7c15u);
  for (int b = tid; b <= M; b += nt) {
    // E = (C[b] + conj C[M - b]) / 2, O = (C[b] - conj C[M - b]) / (2 i), X[b] = E + exp(2 pi i b / N) O
    const cd c = x[b == M ? 0 : b];
    cd d = x[b == 0 || b == M ? 0 : M - b];
    d.im = -d.im;
    const cd e = cd_add(c, d), f = cd_sub(c, d), o = cd_make(f.im, -f.re);
    const cd v = b == M ? cd_sub(e, o) : cd_add(e, cmul2(o, tw[b]));
    const bool real = b == 0 || b == M;
    spec_store<KIND>(out, dst + b * t.bs, 0.5 * t.s * v.re, real ? 0.0 : 0.5 * t.s * v.im, key);
  }
}

// ---- direct sums, one thread per output: lengths with a large prime factor and few tubes.  TAB: the
// roots come from the caller's table (an instance of its own: with the choice inside the loop its
// loads wait for each other; both transforms of 4 tubes of 3347 and the W-step 464 us, 801 so).
template <bool TAB>
__device__ __forceinline__ double2 direct_root(const Tube64& t, int m, int n3) {
  if constexpr (TAB) return t.tw[m];
  double2 w;
  sincospi(2.0 * m / n3, &w.y, &w.x);
  return w;
}
template <int KIND, typename T, bool TAB>
__global__ void __launch_bounds__(256) k_tube_direct_inv(const void* __restrict__ in, T* __restrict__ out, T* __restrict__ out2,
                                                         Tube64 t, int P, int n3) {
  const long g = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= (long)P * t.Q * n3) return;
  const int k = (int)(g % n3), nb = n3 / 2 + 1;
  const long tube = g / n3, p = tube / t.Q, q = tube % t.Q;
  double acc = 0.0;
  int m = 0;   // (b k) mod n3
#pragma unroll 4
  for (int b = 0; b < nb; ++b) {
    const cd v = spec_load<KIND>(in, b * t.bs + p * t.ps + q * t.qs);
    const double2 w = direct_root<TAB>(t, m, n3);
    acc += bin_weight(b, n3) * (v.re * w.x + (bin_is_real(b, n3) ? 0.0 : v.im * w.y));   // Re(e^{-i th} v)
    m += k;
    if (m >= n3) m -= n3;
  }
  const size_t at = p * t.sp + q * t.sq + k;
  out[at] = (T)(t.s * acc);
  if (out2) out2[at] = (T)(t.s * acc);
}
template <int KIND, typename T, bool TAB>
__global__ void __launch_bounds__(256) k_tube_direct_fwd(const T* __restrict__ in, void* __restrict__ out, Tube64 t, int P,
                                                         int n3, const uint32_t* __restrict__ ctr) {
  const long g = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const int nb = n3 / 2 + 1;
  if (g >= (long)P * t.Q * nb) return;
  const int b = (int)(g % nb);
  const long tube = g / nb, p = tube / t.Q, q = tube % t.Q;
  const T* src = in + p * t.sp + q * t.sq;
  double re = 0.0, im = 0.0;
  int m = 0;   // (b k) mod n3
#pragma unroll 4
  for (int k = 0; k < n3; ++k) {
    const double2 w = direct_root<TAB>(t, m, n3);
    const double v = src[k];
    re += w.x * v;
    im += w.y * v;
    m += b;
    if (m >= n3) m -= n3;
  }
  if (bin_is_real(b, n3)) im = 0.0;
  uint32_t key = 0;
  if constexpr (KIND == SPEC_BF16) key = fmix32(ctr[0] * 0x9e3779b9u + 0x7f4a7c15u);
  spec_store<KIND>(out, b * t.bs + p * t.ps + q * t.qs, t.s * re, t.s * im, key);
}

// ---- host side
// Whether tubes go through sequences of half their length, a block each: long even ones (with the
// table of roots) of which a compute unit holds one.  Both transforms and the W-step in us, pairs /
// halves: 12 x 12 x 8064 57.5 / 47.5, 10 x 10 x 4032 34.4 / 29.1, 12 x 12 x 2688 30.4 / 26.6,
// 12 x 12 x 2048 25.9 / 25.0, 16 x 16 x 2048 29.6 / 28.2; 22 x 22 x 2048 (242 pairs) 34.5 / 36.4.
static bool tube64_half(const Plan& p, long pairs) { return p.n3 % 2 == 0 && p.n3 >= 2048 && pairs <= 128; }

// Threads of a block on a sequence of half the length, of M values.
static int tube64_half_threads(int M) { return M >= 2048 ? 512 : (M / 4 + 63) / 64 * 64; }

static Tube64 tube64_args(const Plan& p, long bs, long ps, long qs, long sp, long sq, int Q, double s) {
  Tube64 t;
  t.bs = bs;
  t.ps = ps;
  t.qs = qs;
  t.sp = sp;
  t.sq = sq;
  t.Q = Q;
  t.PP = 1;
  t.s = s;
  t.tw = p.twg;
  t.rows = {nullptr, nullptr, 0};
  return t;
}

// Pairs per block (up to 1024 values, and at least two blocks per compute unit where there are
// enough pairs), threads (four values each) and LDS.  Both transforms and the W-step in us with up
// to 512 / 1024 / 2048 values: 288 x 28 x 144 34.3 / 31.7 / 39.5, 144 x 28 x 288 42.2 / 35.9 / 45.4,
// 144 x 288 x 25 104.0 / 104.9 / 110.8; with 2 / 4 / 8 values per thread, of 1024: 12 x 12 x 2016
// 28.3 / 28.2 / 31.9, 288 x 28 x 144 - / 31.7 / 33.6.
static dim3 tube64_shape(Tube64* t, int n3, int P, int* threads, size_t* lds) {
  const int per_p = (t->Q + 1) / 2;
  const long pairs = (long)per_p * P;
  int pp = n3 >= 1024 ? 1 : 1024 / n3;
  if (pp > (pairs + 511) / 512) pp = (int)((pairs + 511) / 512);
  if (pp > per_p) pp = per_p;
  t->PP = pp;
  int nt = ((pp * n3 + 3) / 4 + 63) / 64 * 64;
  if (nt > 1024) nt = 1024;
  *threads = nt;
  t->lds_tw = n3 <= 1024;
  *lds = ((size_t)pp * n3 + (t->lds_tw ? n3 : 0)) * sizeof(cd);
  return dim3((per_p + pp - 1) / pp, P);
}

// Sum of the radices that are passes of direct sums (fft64_pass_any).
static int sum_radices(int n) {
  int sum = 0;
  for (int f = 2; f * f <= n; ++f)
    while (n % f == 0) {
      if (f > 7) sum += f;
      n /= f;
    }
  return n > 7 ? sum + n : sum;
}

// Whether the passes beat the direct sums.  With radices up to 7 they do from 32 entries on (24 where
// the sums have no table of roots): below, their barriers cost as much as the sums.  Both transforms
// and the W-step in us, direct / passes, for 144 x 28 tubes: of 18 entries 13.6 / 15.8, 25 15.2 /
// 15.8, 30 16.3 / 16.2, 36 19.3 / 18.4, 60 30.7 / 19.4.
// A prime radix past 7 is itself a direct sum of N radix terms by the one block that holds the
// sequence, while the direct sums spread over the device, so few tubes of such lengths are better off
// with them.  The two times in us, fitted to 471 shapes (1 to 8192 tubes; lengths up to 8192 with a prime
// factor past 7), in 11 of which the choice costs a tenth and 10 us more than the better side:
// * a direct sum's thread waits 0.13 us for each term of both transforms, however few tubes there
//   are, once per round of one 256-thread block per compute unit (0.7 of that from the second on;
//   more where the table of roots leaves the caches);
// * a pass costs 0.072 us per radix term and value of a thread (four, or eight past 4096; 0.3 of
//   that more for each further block of a compute unit), or where the blocks fill the device 0.45 ns
//   per term, 0.6 with the roots in memory.
// Direct / passes: 1 x 1021 129 / 425, 128 x 1021 136 / 434, 1024 x 1021 1369 / 539; 4 x 1527 201 /
// 440, 256 x 1527 803 / 449; 64 x 5105 4153 / 3059; 455 x 1481 1340 / 2400; 6 x 7115 1270 / 6110.
static bool tube64_fast(const Plan& p, int P, int Q) {
  const int n3 = p.n3;
  if (n3 > 1024 && !p.twg) return false;   // the roots would not fit beside the sequence
  const int terms = sum_radices(n3);
  if (terms == 0) return n3 >= (p.twg ? 32 : 24);
  const long tubes = (long)P * Q, pairs = (long)((Q + 1) / 2) * P;
  int threads;
  long blocks, values;
  if (tube64_half(p, pairs)) {
    threads = tube64_half_threads(n3 / 2);
    blocks = tubes;
    values = n3 / 2;
  } else {
    Tube64 t;
    t.Q = Q;
    size_t lds;
    const dim3 grid = tube64_shape(&t, n3, P, &threads, &lds);
    blocks = (long)grid.x * grid.y;
    values = (long)t.PP * n3;
  }
  if (terms > 4096) return false;   // one pass over nearly the whole length
  const long rounds = (tubes * n3 + 65535) / 65536;
  double per_round = 2.5e-4 * n3;
  per_round = per_round < 0.7 ? 0.7 : (per_round > 1.35 ? 1.35 : per_round);
  const double direct = 6.0 + 0.13 * n3 * (per_round * rounds > 1.0 ? per_round * rounds : 1.0);
  const double shared = n3 > 1024 ? 1.0 : 1.0 + 0.3 * ((blocks + 255) / 256 - 1);
  const double chain = 0.072 * ((values + threads - 1) / threads) * terms * shared;
  const double full = n3 > 1024 ? 6e-4 * ((blocks + 255) / 256) : 4.5e-4 * (blocks > 512 ? blocks / 512.0 : 1.0);
  const double passes = 14.0 + (chain > full * values * terms ? chain : full * values * terms);
  return passes < direct;
}

template <int KIND, typename T>
static void tube_inv(const Plan& p, const void* in, T* out, T* out2, Tube64 t, int P) {
  const long pairs = (long)((t.Q + 1) / 2) * P;
  if (!tube64_fast(p, P, t.Q)) {
    const long n = (long)P * t.Q * p.n3;
    const auto k = t.tw ? k_tube_direct_inv<KIND, T, true> : k_tube_direct_inv<KIND, T, false>;
    k<<<(unsigned)((n + 255) / 256), 256, 0, p.stream>>>(in, out, out2, t, P, p.n3);
    return;
  }
  if (tube64_half(p, pairs)) {
    const int M = p.n3 / 2, threads = tube64_half_threads(M);
    k_tube64_half_inv<KIND, T><<<dim3(t.Q, P), threads, M * sizeof(cd), p.stream>>>(in, out, out2, t, p.fft_half);
    return;
  }
  int nt;
  size_t lds;
  const dim3 grid = tube64_shape(&t, p.n3, P, &nt, &lds);
  const auto k = nt <= 256 ? k_tube64_inv<KIND, T, 256> : k_tube64_inv<KIND, T, 1024>;
  if (lds > 65536) (void)hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  k<<<grid, nt, lds, p.stream>>>(in, out, out2, t, p.fft);
}
template <int KIND, typename T>
static bool tube_fwd(const Plan& p, const T* in, void* out, Tube64 t, int P) {
  const long pairs = (long)((t.Q + 1) / 2) * P;
  if (!tube64_fast(p, P, t.Q)) {
    const long n = (long)P * t.Q * (p.n3 / 2 + 1);
    const auto k = t.tw ? k_tube_direct_fwd<KIND, T, true> : k_tube_direct_fwd<KIND, T, false>;
    k<<<(unsigned)((n + 255) / 256), 256, 0, p.stream>>>(in, out, t, P, p.n3, p.ctr);
    return false;
  }
  if (tube64_half(p, pairs)) {
    const int M = p.n3 / 2, threads = tube64_half_threads(M);
    k_tube64_half_fwd<KIND, T><<<dim3(t.Q, P), threads, M * sizeof(cd), p.stream>>>(in, out, t, p.fft_half, p.ctr);
    return true;
  }
  int nt;
  size_t lds;
  const dim3 grid = tube64_shape(&t, p.n3, P, &nt, &lds);
  const auto k = nt <= 256 ? k_tube64_fwd<KIND, T, 256> : k_tube64_fwd<KIND, T, 1024>;
  if (lds > 65536) (void)hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  k<<<grid, nt, lds, p.stream>>>(in, out, t, p.fft, p.ctr);
  return true;
}

// grid.y counts P (n1 <= 8192 or r <= 32)
void launch_tube_inv(const Plan& p, int kind, const void* in, long bs, long ps, long qs, float* out, float* out2, long sp,
                     long sq, int P, int Q, double s) {
  const Tube64 t = tube64_args(p, bs, ps, qs, sp, sq, Q, s);
  if (kind == SPEC_F64) tube_inv<SPEC_F64, float>(p, in, out, out2, t, P);
  else tube_inv<SPEC_F32, float>(p, in, out, out2, t, P);
}
void launch_tube_inv64(const Plan& p, int kind, const void* in, long bs, long ps, long qs, double* out, long sp, long sq,
                       int P, int Q, double s) {
  const Tube64 t = tube64_args(p, bs, ps, qs, sp, sq, Q, s);
  if (kind == SPEC_F64) tube_inv<SPEC_F64, double>(p, in, out, (double*)nullptr, t, P);
  else tube_inv<SPEC_F32, double>(p, in, out, (double*)nullptr, t, P);
}
bool launch_tube_fwd(const Plan& p, int kind, const float* in, void* out, long bs, long ps, long qs, long sp, long sq, int P,
                     int Q, double s, RowSums rows) {
  Tube64 t = tube64_args(p, bs, ps, qs, sp, sq, Q, s);
  t.rows = rows;
  return kind == SPEC_BF16 ? tube_fwd<SPEC_BF16, float>(p, in, out, t, P) : tube_fwd<SPEC_F32, float>(p, in, out, t, P);
}
void launch_tube_fwd64(const Plan& p, const double* in, double2* out, long bs, long ps, long qs, long sp, long sq, int P,
                       int Q, double s) {
  tube_fwd<SPEC_F64, double>(p, in, out, tube64_args(p, bs, ps, qs, sp, sq, Q, s), P);
}

// twg[m] = (cos, sin)(2 pi m / n3), m = 0..n3-1
__global__ void k_roots(double2* __restrict__ twg, int n3) {
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= n3) return;
  double s, c;
  sincospi(2.0 * (double)m / n3, &s, &c);
  twg[m] = make_double2(c, s);
}
void launch_roots(const Plan& p) { k_roots<<<(p.n3 + 255) / 256, 256, 0, p.stream>>>(p.twg, p.n3); }

}  // namespace tctf
