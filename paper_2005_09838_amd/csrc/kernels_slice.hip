// Host side of the slice kernel (slice_kernel.h): its shapes, rules and launch.
#include "slice_kernel.h"

namespace tctf {

bool slice_supported(int n3) {
  switch (n3) {
#define TCTF_CASE(n) case n: return true;
    TUBE_DFT_SIZES(TCTF_CASE)
#undef TCTF_CASE
    default: return false;
  }
}

static int tube_ld(int n3, bool iter) {
  switch (n3) {
#define TCTF_CASE(n) case n: return iter ? slice_ld<n, true>() : slice_ld<n, false>();
    TUBE_DFT_SIZES(TCTF_CASE)
#undef TCTF_CASE
    default: return 1;
  }
}

static int tube_threads(int n3, bool iter) {
  switch (n3) {
#define TCTF_CASE(n) case n: return iter ? slice_tube_threads<n, true>() : slice_tube_threads<n, false>();
    TUBE_DFT_SIZES(TCTF_CASE)
#undef TCTF_CASE
    default: return 1;
  }
}

// A slice runs through the fused kernel when n3 is a generated length and a working set of rows one
// float past an odd stride, pivot table, two flag words per 32 entries and twiddles is within
// TCTF_SLICE_LDS_MAX: the rule is on the sizes alone, so a shape's arithmetic (FP32 transforms here,
// FP64 on the other path) does not change with this kernel's own LDS needs.  Those are less for most
// lengths and more where lanes share a tube and its row is padded (529 x 349 x 96: 160324 bytes, rule
// 153600), so that they fit a compute unit is checked for every size below.
static constexpr size_t slice_rule_bytes(int n2, int n3) {
  const size_t nwr = ((size_t)n2 + 31) / 32, ld = (n3 % 2 == 0) ? n3 + 3 : n3 + 2;
  const size_t floats = (size_t)n2 * ld + 4 * (size_t)n2 + 2 * (size_t)n3 * nwr + 1 + 2 * (size_t)(n3 + 1);
  return floats * sizeof(float) + 48 * sizeof(double) + 16;
}
bool slice_fused(int n2, int n3) { return slice_supported(n3) && slice_rule_bytes(n2, n3) <= TCTF_SLICE_LDS_MAX; }

// What the kernel's layout takes (k_slice): rows of ld floats, pivot table, twiddles where lanes
// share a tube, block sums.
static constexpr size_t slice_bytes(int n2, int n3, int ld, int threads) {
  const size_t floats = (size_t)n2 * (ld + 4) + 1 + (threads > 1 ? 2 * (size_t)(n3 + 1) : 0);
  return floats * sizeof(float) + 48 * sizeof(double) + 16;
}
static size_t slice_lds_bytes(int n2, int n3, bool iter) {
  return slice_bytes(n2, n3, tube_ld(n3, iter), tube_threads(n3, iter));
}

template <int N>
static constexpr bool slice_fits() {
  for (int n2 = 1; n2 <= TCTF_N2MAX; ++n2)
    if (slice_rule_bytes(n2, N) <= TCTF_SLICE_LDS_MAX &&
        (slice_bytes(n2, N, slice_ld<N, true>(), slice_tube_threads<N, true>()) > TCTF_LDS_BYTES ||
         slice_bytes(n2, N, slice_ld<N, false>(), slice_tube_threads<N, false>()) > TCTF_LDS_BYTES))
      return false;
  return true;
}
#define TCTF_CASE(n) static_assert(slice_fits<n>(), "a slice that the rule sends to the fused kernel does not fit its LDS");
TUBE_DFT_SIZES(TCTF_CASE)
#undef TCTF_CASE

int slice_default_path(int n2, int n3) {
  if (!slice_fused(n2, n3)) return SPATH_SPLIT;
  return tube_threads(n3, true) > 1 ? SPATH_COOP : SPATH_THREAD;
}

bool slice_path_valid(int path, int n2, int n3) { return path == SPATH_SPLIT || path == slice_default_path(n2, n3); }

bool slice_hosts_pinvy(const Plan& p) { return p.spath != SPATH_SPLIT; }

// Segments per row of the W-step: a power of two (the lanes of a row share a wavefront), the
// least that leaves at most 12 columns each (a longer segment means fewer scans per entry, but
// its values must stay in registers), and more where the rows would not fill one wavefront.
int slice_segments(int n2, int n3) {
  int s = 1;
  while (s < 64 && (n2 + s - 1) / s > 12) s <<= 1;
  while (2 * s * n3 <= 64 && n2 >= 8 * s) s <<= 1;
  return s;
}

// Threads per block: one per tube lane or W-step item, whichever is more, up to 640 while a
// compute unit holds one OD row (n1 <= 256) and up to 256 beyond, where the wavefronts of the
// other rows fill it and a smaller block lets three rows share it.  Kernel times in us with
// 256 / 448 / 640 / 1024 threads: 144 x 288 x 28 13.7 / 9.9 / 9.5 / 10.5, 144 x 96 x 112
// 18.4 / 15.7 / 15.2 / 16.4; 529 x 96 x 112 28.7 / 33.8 / 41.8 / 45.4, 529 x 288 x 28
// 20.8 / 21.9 / 27.4 / 29.7.
//
// In an iteration the blocks of the inverses have the same size and are the launch's longest, so
// past r = 8 (one entry per lane of a wavefront) short rows get 256 threads too, but 128, and those
// past r = 12 only, where thousands of rows would carry the idle wavefronts.  One iteration in us
// with 64 / 128 / 256 threads: 40 x 33 x 7, r = 32 140.8 / 115.3 / 102.8; 20 x 17 x 9, r = 12 36.2 /
// 34.2 / 32.9; 26 x 18 x 8, r = 16 by the eigen route 464 / 416 / 415; 4000 x 17 x 7, r = 16 104.1 /
// 101.8 / 106.4; 8192 x 12 x 4, r = 12 153.8 / 156.0 / 165.8; 20 x 17 x 9, r = 8 25.8 / 25.7 / 25.9.
static int slice_threads(const Plan& p, bool iter) {
  const int tubes = p.n2 * tube_threads(p.n3, iter), items = p.n3 * p.gseg;
  const int need = ((tubes > items ? tubes : items) + 63) / 64 * 64, most = p.n1 <= 256 ? 640 : 256;
  const int threads = need < most ? need : most;
  const int host = !iter || p.r <= 8 ? 64 : (p.n1 <= 2048 ? 256 : (p.r > 12 ? 128 : 64));
  return threads < host ? host : threads;
}

size_t slice_launch_lds_bytes(const Plan& p) {
  if (p.spath == SPATH_SPLIT) return 0;
  size_t lds = pinv_lds_bytes(p.r);
  for (int iter = 0; iter < 2; ++iter) {
    const size_t a = slice_lds_bytes(p.n2, p.n3, iter != 0);
    if (a > lds) lds = a;
  }
  return lds;
}

// The kernel of a tube length, segment length (at most 6, 9, 12 or 16 columns) and use.
typedef void (*SliceKernel)(SliceArgs);
template <int N>
static SliceKernel slice_kernel_n(int n2, int n3, bool iter) {
  const int s = slice_segments(n2, n3), len = (n2 + s - 1) / s;
  if (len <= 6) return iter ? k_slice<N, 6, true> : k_slice<N, 6, false>;
  if (len <= 9) return iter ? k_slice<N, 9, true> : k_slice<N, 9, false>;
  if (len <= 12) return iter ? k_slice<N, 12, true> : k_slice<N, 12, false>;
  if constexpr (N <= 40) return iter ? k_slice<N, 16, true> : k_slice<N, 16, false>;   // n2 > 768: no longer tube fits
  return nullptr;
}
static SliceKernel slice_kernel(int n2, int n3, bool iter) {
  switch (n3) {
#define TCTF_CASE(n) case n: return slice_kernel_n<n>(n2, n3, iter);
    TUBE_DFT_SIZES(TCTF_CASE)
#undef TCTF_CASE
    default: return nullptr;
  }
}

void slice_set_attr(int n2, int n3, size_t lds) {
  if (lds <= 65536) return;
  for (int iter = 0; iter < 2; ++iter)
    (void)hipFuncSetAttribute((const void*)slice_kernel(n2, n3, iter != 0), hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds);
}

void launch_slice(const Plan& p, int mode, float* w_out, float* z_out, int w_from_g) {
  if (p.spath == SPATH_SPLIT) {
    launch_slice_generic(p, mode, w_out, z_out, w_from_g);
    return;
  }
  SliceArgs a;
  a.npinv = mode == SLICE_ITER ? p.nb : 0;
  a.pa = pinvy_args(p);
  a.ctr = p.ctr;
  a.zt = p.zt;
  a.gp = p.gp;
  a.wtab = p.wtab;
  a.wt = p.wt;
  a.slice_obj = p.slice_obj;
  a.kkt = p.kkt;
  a.w_out = w_out;
  a.z_out = z_out;
  a.n1 = p.n1;
  a.n2 = p.n2;
  a.nb = p.nb;
  a.rho2 = (float)p.rho2;
  a.mu = p.mu;
  a.rho2d = p.rho2;
  a.mode = mode;
  a.mixed = p.mixed;
  a.w_from_g = w_from_g;
  a.nseg = p.gseg;
  slice_kernel(p.n2, p.n3, mode == SLICE_ITER)<<<p.n1 + a.npinv, slice_threads(p, mode == SLICE_ITER), slice_launch_lds_bytes(p),
                                                        p.stream>>>(a);
}

}  // namespace tctf
