// Shared device-side definitions of the TCTF2R gfx950 library.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#define TCTF_RMAX 32          // largest tubal rank r supported by the r x r kernels
#define TCTF_N2MAX 1024       // largest n2 (slice kernel: one thread per tube of a slice)
#define TCTF_N1MAX 8192       // largest n1 (tridiagonal H_rho1 solve held in LDS)
#define TCTF_N3MAX 8192       // largest tube length n3
#define TCTF_SLICE_LDS_MAX (150 * 1024)
#define TCTF_LDS_BYTES (160 * 1024)   // of a compute unit

// Complex numbers: planar pairs in registers, float2 / double2 in memory.
struct cf { float re, im; };
struct cd { double re, im; };

__host__ __device__ __forceinline__ cd cd_make(double r, double i) { cd z; z.re = r; z.im = i; return z; }
__host__ __device__ __forceinline__ cd cd_add(cd a, cd b) { return cd_make(a.re + b.re, a.im + b.im); }
__host__ __device__ __forceinline__ cd cd_sub(cd a, cd b) { return cd_make(a.re - b.re, a.im - b.im); }
__host__ __device__ __forceinline__ cd cd_mul(cd a, cd b) {
  return cd_make(a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re);
}
// a * conj(b)
__host__ __device__ __forceinline__ cd cd_mulc(cd a, cd b) {
  return cd_make(a.re * b.re + a.im * b.im, a.im * b.re - a.re * b.im);
}
// conj(a) * b
__host__ __device__ __forceinline__ cd cd_cmul(cd a, cd b) {
  return cd_make(a.re * b.re + a.im * b.im, a.re * b.im - a.im * b.re);
}
__host__ __device__ __forceinline__ cd cd_conj(cd a) { return cd_make(a.re, -a.im); }
__host__ __device__ __forceinline__ cd cd_scale(cd a, double s) { return cd_make(a.re * s, a.im * s); }
// acc += a * b
__host__ __device__ __forceinline__ void cd_fma(cd& acc, cd a, cd b) {
  acc.re = fma(a.re, b.re, fma(-a.im, b.im, acc.re));
  acc.im = fma(a.re, b.im, fma(a.im, b.re, acc.im));
}

// BF16 with round-to-nearest-even (NaN kept quiet); stored as the upper half of a float.
__host__ __device__ __forceinline__ uint16_t f32_to_bf16(float x) {
  uint32_t u = __float_as_uint(x);
  if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x007fffffu)) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__host__ __device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }
__host__ __device__ __forceinline__ float bf16_round(float x) { return bf16_to_f32(f32_to_bf16(x)); }
__host__ __device__ __forceinline__ uint32_t pack_bf16x2(float re, float im) {
  return (uint32_t)f32_to_bf16(re) | ((uint32_t)f32_to_bf16(im) << 16);
}
// MurmurHash3's 32-bit finaliser (Appleby): a bijective mixer, used as a counter-based
// generator of rounding bits.
__host__ __device__ __forceinline__ uint32_t fmix32(uint32_t h) {
  h ^= h >> 16;
  h *= 0x85ebca6bu;
  h ^= h >> 13;
  h *= 0xc2b2ae35u;
  h ^= h >> 16;
  return h;
}
// BF16 by stochastic rounding: the 16 dropped bits are compared with 16 uniform random bits
// (added, then truncated), so the result rounds up with probability equal to the dropped
// fraction and its expectation is x.  Unlike round-to-nearest, its error is not the same
// every time a slowly changing value is rounded.  NaN/Inf as round-to-nearest.
__host__ __device__ __forceinline__ uint16_t f32_to_bf16_sr(float x, uint32_t rnd16) {
  const uint32_t u = __float_as_uint(x);
  if ((u & 0x7f800000u) == 0x7f800000u) return f32_to_bf16(x);
  return (uint16_t)((u + (rnd16 & 0xffffu)) >> 16);
}
__host__ __device__ __forceinline__ uint32_t pack_bf16x2_sr(float re, float im, uint32_t rnd) {
  return (uint32_t)f32_to_bf16_sr(re, rnd) | ((uint32_t)f32_to_bf16_sr(im, rnd >> 16) << 16);
}
__host__ __device__ __forceinline__ float2 unpack_bf16x2(uint32_t v) {
  return make_float2(bf16_to_f32((uint16_t)(v & 0xffffu)), bf16_to_f32((uint16_t)(v >> 16)));
}

// Unobserved entries of the packed observation tensor are quiet NaNs whose payload is the
// entry's index into the W-step's table of reciprocal pivots (Plan::wtab, below 4 n2): its
// position in its run of consecutive unobserved entries along mode 2, in the table for the
// kind of run (starting at the first slot of the row or after an observed entry) and of entry
// (the last slot or not).
__host__ __device__ __forceinline__ uint32_t pack_unobserved(uint32_t index) {
  return 0x7fc00000u | (index & 0x3fffffu);
}
__device__ __forceinline__ bool is_unobserved(float g) { return (__float_as_uint(g) & 0x7f800000u) == 0x7f800000u; }
__device__ __forceinline__ uint32_t unobs_index(float g) { return __float_as_uint(g) & 0x3fffffu; }

// Offset of entry (i, j, k) in the packed G.  seg = 0: as in G, [n1][n2][n3].  seg = S > 0: each
// OD row in the order in which the fused slice kernel's lanes read it.  S lanes share a row
// (i, :, k); segment s holds n2 / S consecutive columns and the first n2 % S segments one more.
// Column u of every segment comes before column u + 1, at (u n3 + k) S + s; the odd columns
// u = n2 / S of the longer segments are last, at k (n2 % S) + s.
__host__ __device__ __forceinline__ size_t packed_g_at(long i, int j, int k, int n2, int n3, int seg) {
  if (seg == 0) return ((size_t)i * n2 + j) * n3 + k;
  const int lf = n2 / seg, rem = n2 % seg, cut = rem * (lf + 1);
  const int s = j < cut ? j / (lf + 1) : rem + (j - cut) / lf;
  const int u = j < cut ? j % (lf + 1) : (j - cut) % lf;
  return (size_t)i * n2 * n3 + (u < lf ? (size_t)(u * n3 + k) * seg + s : (size_t)lf * n3 * seg + (size_t)k * rem + s);
}

// Weight of stored frequency b in a sum over all n3 frequencies (conjugate pairs).
__host__ __device__ __forceinline__ double bin_weight(int b, int n3) {
  return (b == 0 || (n3 % 2 == 0 && b == n3 / 2)) ? 1.0 : 2.0;
}
__host__ __device__ __forceinline__ bool bin_is_real(int b, int n3) {
  return b == 0 || (n3 % 2 == 0 && b == n3 / 2);
}

// Block-wide FP64 sum of one value per thread (blockDim.x <= 1024); all threads get it.
__device__ __forceinline__ double block_sum_d(double v, double* red) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  __syncthreads();
  if (lane == 0) red[wid] = v;
  __syncthreads();
  double s = 0.0;
  for (int w = 0; w < nw; ++w) s += red[w];   // fixed order
  __syncthreads();
  return s;
}
// Three block-wide FP64 sums at once (blockDim.x <= 1024; red holds >= 48 doubles).
__device__ __forceinline__ void block_sum3_d(double& a, double& b, double& c, double* red) {
  for (int off = 32; off > 0; off >>= 1) {
    a += __shfl_xor(a, off);
    b += __shfl_xor(b, off);
    c += __shfl_xor(c, off);
  }
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  __syncthreads();
  if (lane == 0) {
    red[wid] = a;
    red[16 + wid] = b;
    red[32 + wid] = c;
  }
  __syncthreads();
  double sa = 0.0, sb = 0.0, sc = 0.0;
  for (int w = 0; w < nw; ++w) {   // fixed order
    sa += red[w];
    sb += red[16 + w];
    sc += red[32 + w];
  }
  a = sa;
  b = sb;
  c = sc;
}
__device__ __forceinline__ double block_max_d(double v, double* red) {
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off));
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  __syncthreads();
  if (lane == 0) red[wid] = v;
  __syncthreads();
  double s = red[0];
  for (int w = 1; w < nw; ++w) s = fmax(s, red[w]);
  __syncthreads();
  return s;
}

// p[i] when ok, else z.  The load itself is unconditional (from p[0] when !ok, which must
// be a valid element) and only its value is selected: a load under a branch is waited for
// at the branch's end, so a batch of guarded loads would otherwise cost one memory latency
// per load instead of one for the batch.
template <typename T>
__device__ __forceinline__ T ld_or(const T* __restrict__ p, size_t i, bool ok, T z) {
  const T v = p[ok ? i : 0];
  return ok ? v : z;
}

// Block-cooperative copy of n elements, dst[e] = load(e) for e < n, in batches of PER
// elements per thread whose loads are all issued before any of their stores (a loop of
// load-then-store would wait out one memory latency per element).  Lanes past n load
// element n - 1 and drop it, so no load sits under a branch.
template <int PER, typename T, typename F>
__device__ __forceinline__ void stage_batched(T* dst, int n, F load) {
  const int nt = blockDim.x;
  for (int e0 = 0; e0 < n; e0 += PER * nt) {
    T v[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = e0 + threadIdx.x + u * nt;
      v[u] = load(e < n ? e : n - 1);
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = e0 + threadIdx.x + u * nt;
      if (e < n) dst[e] = v[u];
    }
  }
}

// The same with a store functor: store(e, value) for e < n.
template <int PER, typename T, typename L, typename S>
__device__ __forceinline__ void stage_batched_to(int n, L load, S store) {
  const int nt = blockDim.x;
  for (int e0 = 0; e0 < n; e0 += PER * nt) {
    T v[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = e0 + threadIdx.x + u * nt;
      v[u] = load(e < n ? e : n - 1);
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = e0 + threadIdx.x + u * nt;
      if (e < n) store(e, v[u]);
    }
  }
}
