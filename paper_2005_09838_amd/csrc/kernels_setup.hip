// Setup kernels: packing of the observations, constant tables, initial transforms,
// the objective reduction and the termination / stationarity measures.
#include "kernels.h"

#include <cstring>

namespace tctf {

size_t wt_elem_bytes(const Plan& p) { return p.mixed ? 4 : 8; }

// One thread per row (i, k) along mode 2.  Observed entries keep their value (they must
// be finite); unobserved ones become NaNs carrying their index into the pivot table
// (section 3.3: the equality constraints of the W-step are eliminated row by row, leaving
// one tridiagonal system per run of unobserved entries).  An observed value that is not finite is
// flagged and stored as index 0: the kernels that create launches before it reads the flag take the
// payload of any NaN as an index.  seg: the order (packed_g_at).
//
// Block (x, i): S = 2^ls segments of at most 16 columns of the rows (i, :, k), k = x KB .. + KB,
// KB = 256 / S, a thread per (segment, row): its entries are in flight at once, and the last
// observed column before the segment comes from the other segments' through LDS.
// 144 x 288 x 28: 11.4 us (186 with a thread per row).
__global__ void __launch_bounds__(256) k_pack_g(const float* __restrict__ g, const uint8_t* __restrict__ om,
                                                float* __restrict__ gp, int n2, int n3, int seg, int ls, int* flag) {
  constexpr int L = 16;
  __shared__ int last[256];
  const int KB = 256 >> ls, tid = threadIdx.x, s = tid >> (8 - ls), kk = tid & (KB - 1), k = blockIdx.x * KB + kk;
  const int kc = min(k, n3 - 1), len = (n2 + (1 << ls) - 1) >> ls, j0 = s * len, cnt = k < n3 ? min(len, n2 - j0) : 0;
  const size_t row = (size_t)blockIdx.y * n2 * n3;
  float v[L];
  uint8_t o[L];
#pragma unroll
  for (int u = 0; u < L; ++u) {
    const size_t at = row + (size_t)min(j0 + u, n2 - 1) * n3 + kc;
    v[u] = g[at];
    o[u] = om[at];
  }
  int prev = -1;   // the last observed column so far
#pragma unroll
  for (int u = 0; u < L; ++u)
    if (u < cnt && o[u]) prev = j0 + u;
  last[tid] = prev;
  __syncthreads();
  prev = -1;
  for (int t = kk; t < s * KB; t += KB) prev = max(prev, last[t]);
  // packed_g_at with one division: column j is column c of the slice kernel's segment q
  const int lf = seg ? n2 / seg : 0, rem = seg ? n2 % seg : 0, cut = rem * (lf + 1);
  const int jf = min(j0, n2 - 1);
  int q = 0, c = 0;
  if (seg) {
    q = jf < cut ? jf / (lf + 1) : rem + (jf - cut) / lf;
    c = jf < cut ? jf - q * (lf + 1) : jf - cut - (q - rem) * lf;
  }
#pragma unroll
  for (int u = 0; u < L; ++u) {
    if (u < cnt) {
      const int j = j0 + u;
      const size_t at = seg == 0 ? (size_t)j * n3 + k
                                 : (c < lf ? (size_t)(c * n3 + k) * seg + q : (size_t)lf * n3 * seg + (size_t)k * rem + q);
      if (++c == lf + (q < rem ? 1 : 0)) {
        c = 0;
        ++q;
      }
      if (o[u]) {
        const bool fin = isfinite(v[u]);
        if (!fin) atomicOr(flag, 1);
        gp[row + at] = fin ? v[u] : __uint_as_float(pack_unobserved(0));
        prev = j;
      } else {
        const uint32_t table = (j == n2 - 1 ? 2u : 0u) + (prev >= 0 ? 1u : 0u);
        gp[row + at] = __uint_as_float(pack_unobserved(table * (uint32_t)n2 + (uint32_t)(j - prev - 1)));
      }
    }
  }
}

void launch_pack_g(const Plan& p, const float* G, const uint8_t* omega) {
  int ls = 0;
  while (((p.n2 + (1 << ls) - 1) >> ls) > 16) ++ls;   // n2 <= 1024: ls <= 6
  const int KB = 256 >> ls;
  k_pack_g<<<dim3((p.n3 + KB - 1) / KB, p.n1), 256, 0, p.stream>>>(G, omega, p.gp, p.n2, p.n3, p.gseg, ls, p.flag);
}

// Reciprocal pivots of the W-step row systems (eq. (subquKKT)), in FP64 then rounded.
// Along a run of unobserved entries the system matrix is tridiagonal with off-diagonal
// -rho2 and diagonal (K_{mu rho2})_jj = 1 + mu + rho2 deg(j) (deg = 1 at the row ends,
// 2 inside).  Elimination without pivoting gives pivots alpha_t that depend only on the
// position t in the run, on whether the run starts at j = 0, and on whether j = n2 - 1.
//   wtab[0][t]: run starting at j = 0, interior j      wtab[1][t]: run after an observed entry
//   wtab[2][t]: as [0] but j = n2 - 1                   wtab[3][t]: as [1] but j = n2 - 1
// The H_rho1 = I + rho1 H^T H tables (Thomas coefficients along mode 1):
//   htab[0][i] = rho1 / alpha_{i-1} (0 for i = 0), htab[1][i] = 1/alpha_i,
//   htab[2][i] = rho1 / alpha_i.
// A chain of pivots needs one division per step, so each runs on one lane until two successive
// pivots are equal (then all further ones are), and the block forms the table from them.  T: float
// for the iteration, double for the adjoint.  144 x 288: 4.7 us (96 with every entry on one thread).
template <typename T>
__global__ void __launch_bounds__(256) k_tables(T* __restrict__ wtab, T* __restrict__ htab, int n1, int n2, double mu,
                                                double rho1, double rho2) {
  extern __shared__ double piv[];   // [n2] runs from column 0, [n2] runs after an observed entry, [n1] alpha
  __shared__ int last[3];           // the entry from which on a chain is constant
  const double dint = 1.0 + mu + 2.0 * rho2, dend = 1.0 + mu + rho2, r2 = rho2 * rho2;
  const double hint = 1.0 + 2.0 * rho1, hend = n1 == 1 ? 1.0 : 1.0 + rho1, h2 = rho1 * rho1;
  const int c = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0 && c < 3) {
    const int n = c < 2 ? n2 : n1;
    const double d = c < 2 ? dint : hint, off = c < 2 ? r2 : h2;
    double* chain = piv + c * n2;
    double p = c == 0 ? dend : (c == 1 ? dint : hend);
    chain[0] = p;
    int t = 1;
    for (; t < n; ++t) {
      const double q = d - off / p;
      chain[t] = q;
      if (q == p) break;
      p = q;
    }
    last[c] = t < n ? t : n - 1;
  }
  __syncthreads();
  auto pv = [&](int ch, int t) { return piv[ch * n2 + min(t, last[ch])]; };
  for (int t = threadIdx.x; t < n2; t += blockDim.x) {
    if (n2 == 1) {
      for (int q = 0; q < 4; ++q) wtab[q] = (T)(1.0 / (1.0 + mu));
    } else {
      wtab[0 * n2 + t] = (T)(1.0 / pv(0, t));
      wtab[1 * n2 + t] = (T)(1.0 / pv(1, t));
      wtab[2 * n2 + t] = (T)(1.0 / (t == 0 ? dend : dend - r2 / pv(0, t - 1)));
      wtab[3 * n2 + t] = (T)(1.0 / (t == 0 ? dend : dend - r2 / pv(1, t - 1)));
    }
  }
  for (int i = threadIdx.x; i < n1; i += blockDim.x) {
    const double prev = i > 0 ? pv(2, i - 1) : 0.0;
    const double alpha = i > 0 && i == n1 - 1 ? hend - h2 / prev : pv(2, i);
    htab[0 * n1 + i] = i == 0 ? (T)0 : (T)(rho1 / prev);
    htab[1 * n1 + i] = (T)(1.0 / alpha);
    htab[2 * n1 + i] = (T)(rho1 / alpha);
  }
}

template <typename T>
static void tables(const Plan& p, T* wtab, T* htab) {
  const size_t lds = (2 * (size_t)p.n2 + p.n1) * sizeof(double);
  if (lds > 65536)
    (void)hipFuncSetAttribute((const void*)k_tables<T>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  k_tables<T><<<1, 256, lds, p.stream>>>(wtab, htab, p.n1, p.n2, p.mu, p.rho1, p.rho2);
}
void launch_tables(const Plan& p) { tables(p, p.wtab, p.htab); }
void launch_tables64(const Plan& p, double* wtab, double* htab) { tables(p, wtab, htab); }

static inline unsigned blocks_for(long n, int bs) { return (unsigned)((n + bs - 1) / bs); }

// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11) keyed by the seed, counter = thread
// index; Box-Muller turns its four uniforms into four standard normals.
__device__ inline void philox4x32_10(uint32_t c[4], uint32_t k0, uint32_t k1) {
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * c[0];
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c[2];
    const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0;
    const uint32_t hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
    const uint32_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
    c[0] = n0; c[1] = lo1; c[2] = n2; c[3] = lo0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
}

__global__ void k_normal(float* __restrict__ out, long n, uint64_t seed) {
  const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t * 4 >= n) return;
  uint32_t c[4] = {(uint32_t)t, (uint32_t)(t >> 32), 0u, 0u};
  philox4x32_10(c, (uint32_t)seed, (uint32_t)(seed >> 32));
  for (int h = 0; h < 2; ++h) {
    const double u1 = ((double)c[2 * h] + 0.5) * (1.0 / 4294967296.0);
    const double u2 = ((double)c[2 * h + 1] + 0.5) * (1.0 / 4294967296.0);
    const double rad = sqrt(-2.0 * log(u1));
    double s, co;
    sincospi(2.0 * u2, &s, &co);
    if (t * 4 + 2 * h < n) out[t * 4 + 2 * h] = (float)(rad * co);
    if (t * 4 + 2 * h + 1 < n) out[t * 4 + 2 * h + 1] = (float)(rad * s);
  }
}

void launch_normal(const Plan& p, float* dst, size_t n, uint64_t seed) {
  k_normal<<<blocks_for(((long)n + 3) / 4, 256), 256, 0, p.stream>>>(dst, (long)n, seed);
}

__global__ void k_zero(uint32_t* __restrict__ d, long words) {
  const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < words) d[t] = 0u;
}

void launch_zero(const Plan& p, void* dst, size_t bytes) {
  const long words = (long)(bytes / 4);
  if (words > 0) k_zero<<<blocks_for(words, 256), 256, 0, p.stream>>>((uint32_t*)dst, words);
}

// f0 of eq. (TETP-optim): 1/2 fit + mu/2 ridge + rho2/2 (mode-2 differences) from the
// W-step rows, and rho1/2 ||H unfold(Z,1)||^2 = rho1/(2 n3) sum_b c_b tr(...) from the
// Fourier form eq. (fun-XYW).  Fixed-order FP64 sums.
__global__ void k_objective(const double* __restrict__ so, int n1, const double* __restrict__ bo, int nb,
                            double mu, double rho1, double rho2, int n3, double* out) {
  __shared__ double red[16];
  double fit = 0.0, ridge = 0.0, sm = 0.0, h = 0.0;
  for (int i = threadIdx.x; i < n1; i += blockDim.x) {
    fit += so[3 * i];
    ridge += so[3 * i + 1];
    sm += so[3 * i + 2];
  }
  for (int b = threadIdx.x; b < nb; b += blockDim.x) h += bo[b];
  fit = block_sum_d(fit, red);
  ridge = block_sum_d(ridge, red);
  sm = block_sum_d(sm, red);
  h = block_sum_d(h, red);
  if (threadIdx.x == 0) out[0] = 0.5 * fit + 0.5 * mu * ridge + 0.5 * rho2 * sm + 0.5 * rho1 * h / n3;
}

void launch_objective(const Plan& p) {
  k_objective<<<1, 256, 0, p.stream>>>(p.slice_obj, p.n1, p.bin_obj, p.nb, p.mu, p.rho1, p.rho2, p.n3, p.scal);
}

// Step 6 quantities between the snapshot and the current iterate:
// max |dX~|, max |dY~| (the maxima over stored frequencies equal those over all of them)
// and ||dW||_F from the stored frequencies by Parseval: ||dW||^2 = 1/n3 sum_b c_b ||dW~_b||^2.
// A non-finite difference counts as +inf in the maxima (fmax would drop a NaN) and stays NaN
// in the sum, so a non-finite iterate shows in the result.  Grid-stride loops over a grid
// that covers every compute unit; per-block partials, then one block combines them in a
// fixed order.
#define TERM_BLOCKS 1024
__global__ void __launch_bounds__(256) k_termination(const float2* __restrict__ x, const float2* __restrict__ xp, long nx,
                              const float2* __restrict__ y, const float2* __restrict__ yp, long ny,
                              const void* __restrict__ w, const void* __restrict__ wp, int mixed,
                              int n1, int nb, int n2, int n3, double* part) {
  __shared__ double red[16];
  double mx = 0.0, my = 0.0, sw = 0.0;
  const long stride = (long)gridDim.x * blockDim.x;
  const long t0 = (long)blockIdx.x * blockDim.x + threadIdx.x;
  for (long e = t0; e < nx; e += stride) {
    const double d = hypot((double)x[e].x - xp[e].x, (double)x[e].y - xp[e].y);
    mx = (d == d) ? fmax(mx, d) : INFINITY;
  }
  for (long e = t0; e < ny; e += stride) {
    const double d = hypot((double)y[e].x - yp[e].x, (double)y[e].y - yp[e].y);
    my = (d == d) ? fmax(my, d) : INFINITY;
  }
  const long nw = (long)n1 * nb * n2;
  for (long e = t0; e < nw; e += stride) {
    const int b = (int)((e / n2) % nb);
    float2 a, c;
    if (mixed) { a = unpack_bf16x2(((const uint32_t*)w)[e]); c = unpack_bf16x2(((const uint32_t*)wp)[e]); }
    else { a = ((const float2*)w)[e]; c = ((const float2*)wp)[e]; }
    const double dr = (double)a.x - c.x, di = (double)a.y - c.y;
    sw += bin_weight(b, n3) * (dr * dr + di * di);
  }
  mx = block_max_d(mx, red);
  my = block_max_d(my, red);
  sw = block_sum_d(sw, red);
  if (threadIdx.x == 0) {
    part[3 * blockIdx.x + 0] = mx;
    part[3 * blockIdx.x + 1] = my;
    part[3 * blockIdx.x + 2] = sw;
  }
}

__global__ void __launch_bounds__(256) k_termination_final(const double* __restrict__ part, int nblk, int n3, double* out) {
  __shared__ double red[16];
  double mx = 0.0, my = 0.0, sw = 0.0;
  for (int b = threadIdx.x; b < nblk; b += blockDim.x) {
    mx = fmax(mx, part[3 * b]);
    my = fmax(my, part[3 * b + 1]);
    sw += part[3 * b + 2];
  }
  mx = block_max_d(mx, red);
  my = block_max_d(my, red);
  sw = block_sum_d(sw, red);
  if (threadIdx.x == 0) {
    out[0] = mx;
    out[1] = my;
    out[2] = sqrt(sw / n3);
  }
}

size_t termination_work_doubles() { return 3 * TERM_BLOCKS; }

void launch_termination(const Plan& p) {
  const long nw = (long)p.n1 * p.nb * p.n2;
  int nblk = (int)((nw + 1023) / 1024);
  if (nblk > TERM_BLOCKS) nblk = TERM_BLOCKS;
  if (nblk < 1) nblk = 1;
  k_termination<<<nblk, 256, 0, p.stream>>>(p.xt, p.xt_prev, (long)p.nb * p.r * p.n1, p.yt, p.yt_prev,
                                            (long)p.nb * p.r * p.n2, p.wt, p.wt_prev, p.mixed, p.n1, p.nb,
                                            p.n2, p.n3, p.stat_work);
  k_termination_final<<<1, 256, 0, p.stream>>>(p.stat_work, nblk, p.n3, p.scal + 4);
}

// A checkpoint's regions in one launch, words as wide as a region's two addresses allow.  The blob's
// header is written, or checked: a blob of another problem is left alone.  529 x 96 x 112 in mixed
// precision, 13 MB: 9.3 us; a copy call per region took 10 launches and 40 us.
struct CopyArgs {
  CopyRegion r[COPY_REGIONS];
  uint32_t header[COPY_HEADER_WORDS];
  uint32_t* blob_header;
  int to_blob;
};
template <typename T>
__device__ __forceinline__ void copy_words(const unsigned char* src, unsigned char* dst, size_t bytes) {
  const size_t n = bytes / sizeof(T), step = (size_t)gridDim.x * blockDim.x;
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += 4 * step) {
    T v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = ((const T*)src)[min(e + u * step, n - 1)];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (e + u * step < n) ((T*)dst)[e + u * step] = v[u];
  }
}
__global__ void __launch_bounds__(256) k_copy_regions(CopyArgs a) {
  if (a.to_blob) {
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < COPY_HEADER_WORDS)
      a.blob_header[threadIdx.x] = a.header[threadIdx.x];
  } else {
    bool same = true;
#pragma unroll
    for (int w = 0; w < COPY_HEADER_CHECKED; ++w) same = same && a.blob_header[w] == a.header[w];
    if (!same) return;
  }
  const CopyRegion r = a.r[blockIdx.y];
  const uintptr_t al = (uintptr_t)r.src | (uintptr_t)r.dst | r.bytes;
  if ((al & 15) == 0) copy_words<uint4>(r.src, r.dst, r.bytes);
  else if ((al & 7) == 0) copy_words<uint2>(r.src, r.dst, r.bytes);
  else copy_words<uint32_t>(r.src, r.dst, r.bytes);
}
void launch_copy_regions(const Plan& p, const CopyRegion* r, int n, const void* header, void* blob, bool to_blob) {
  CopyArgs a;
  size_t most = 0;
  for (int k = 0; k < n; ++k) {
    a.r[k] = r[k];
    if (r[k].bytes > most) most = r[k].bytes;
  }
  a.blob_header = (uint32_t*)blob;
  a.to_blob = to_blob;
  std::memcpy(a.header, header, sizeof(a.header));
  const size_t blocks = (most + 16383) / 16384;
  k_copy_regions<<<dim3((unsigned)(blocks < 2048 ? blocks : 2048), n), 256, 0, p.stream>>>(a);
}

}  // namespace tctf
