// Kernel launchers of the TCTF2R gfx950 library (host-callable, stream-ordered).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "common.h"
#include "fft64_plan.h"

namespace tctf {

#define HINV_KMAX 12   // widest stencil of H_rho1^{-1} applied inside the X-update

// Device buffers and sizes of one completion (carved from the caller's workspace).
struct Plan {
  int n1, n2, n3, r, nb;       // nb = n3/2 + 1 stored frequencies
  int bcg;                     // complex columns per X~^* W~ block (16 or 32)
  int ny, ycw;                 // column blocks of the Y-step per frequency, columns per block
  int spath;                   // slice path: SPATH_COOP, SPATH_THREAD or SPATH_SPLIT
  double mu, rho1, rho2, eta;
  // H_rho1^{-1} as a stencil of half-width hk inside the X-update (k_agemm), hk = -1: the
  // X-update forms the right-hand side and k_hsolve solves (see hinv_stencil)
  int hk;
  double htap[2 * HINV_KMAX + 2];
  int mixed, force_eigen;
  hipStream_t stream;

  float* gp;        // observed values, unobserved entries NaN-coded (pivot index), at packed_g_at
  int gseg;         // its order: lanes per row of the fused slice kernel's W-step, 0 on the
                    // three-launch path
  void* wt;         // W~ [n1][nb][n2] float2 (FP32) or packed bf16x2 (mixed)
  float2* zt;       // Z~ [n1][nb][n2], from its product to the slice work; row groups' G_X (launch_bgemm)
  float2* xt;       // X~ [nb][r][n1]
  float2* yt;       // Y~ [nb][r][n2]
  float2* rhs;      // right-hand side of the H_rho1 solve [nb][r][n1]
  double2* bpart;   // X~^* W~ [nb][r][n2] (FP64)
  cd* gxm;          // G_X = X~^* H_rho1 X~ [nb][r][r]
  cd* dmat;         // (H X~)^* (H X~) [nb][r][r]
  cd* gxp;          // G_X^+ [nb][r][r]
  cd* qx;           // I - eta P_X [nb][r][r]
  int* qx_zero;     // [nb] 1 when I - eta P_X is exactly 0
  cd* gym;          // partial Y~ Y~^* over column blocks [nb][ny][r][r]
  cd* gyp;          // (Y~ Y~^*)^+ [nb][r][r]
  cd* qy;           // I - eta P_Y [nb][r][r]
  int* qy_zero;     // [nb] 1 when I - eta P_Y is exactly 0 (eta = 1, full rank)
  double* slice_obj;// [n1][3] fit, ridge and mode-2 difference sums of the last W-step
  double* bin_obj;  // [nb] c_b tr((H X~_b)^*(H X~_b) Y~_b Y~_b^*)
  float* wtab;      // [4][n2] reciprocal pivots of the W-step row systems
  float* htab;      // [3][n1] Thomas coefficients of H_rho1
  int* flag;        // non-finite detector
  uint32_t* ctr;    // iteration counter of the BF16 rounding bits (advanced by each X-step)
  // the three-launch slice path (tube lengths outside the generated set, or slices larger
  // than the fused kernel's LDS): spatial Z and W, partials of each OD row's three objective terms
  // (slice_generic_part_doubles), roots of unity
  float* zsp;       // [n1][n2][n3]
  float* wsp;       // [n1][n2][n3]
  double* rowpart;  // [n1][blocks per OD row][3]
  double2* twg;     // [n3] (cos, sin)(2 pi m / n3); NULL without that path
  Fft64Plan fft, fft_half;   // of tubes of n3, and of n3 / 2 where n3 is even
  // step 5 (rank adjustment)
  double* rsig;     // [nb][r] singular values of Z~_b, descending
  cd* rtx;          // [nb][r][r] factor rotations of X~ and Y~
  cd* rty;
  int* ranks;       // [nb] the rank vector r_b
  double* scal;     // [16] scalar results (objective, termination, stationarity)
  float2* xt_prev;  // snapshots for the termination test
  float2* yt_prev;
  void* wt_prev;
  double* stat_work;// [nb][8] stationarity partial sums (and termination partials)
  double* kkt;      // [n1][3] W-KKT residual maxima of the slices
};

size_t wt_elem_bytes(const Plan& p);

// setup
void launch_pack_g(const Plan& p, const float* G, const uint8_t* omega);
void launch_tables(const Plan& p);
void launch_tables64(const Plan& p, double* wtab, double* htab);   // the same tables in FP64
// FP64 tube transforms: P x Q tubes between a spectrum (bin b of tube (p, q) at b bs + p ps +
// q qs) and spatial tubes (entry k at p sp + q sq + k), times s; the inverse sums over all n3
// frequencies of the conjugate-symmetric spectrum.  out2 (or NULL): a second copy.
enum SpecKind { SPEC_F32 = 0, SPEC_F64 = 1, SPEC_BF16 = 2 };   // float2, double2, packed bf16 pairs
void launch_tube_inv(const Plan& p, int kind, const void* in, long bs, long ps, long qs, float* out, float* out2, long sp,
                     long sq, int P, int Q, double s);
void launch_tube_inv64(const Plan& p, int kind, const void* in, long bs, long ps, long qs, double* out, long sp, long sq,
                       int P, int Q, double s);
// rows (part NULL: none): out[p][3] = sums over c of part[p][c][3], for each of the P rows in the
// same launch; returns whether it did (direct sums have no block per row).
struct RowSums {
  const double* part;
  double* out;
  int nchunk;
};
bool launch_tube_fwd(const Plan& p, int kind, const float* in, void* out, long bs, long ps, long qs, long sp, long sq, int P,
                     int Q, double s, RowSums rows = RowSums{nullptr, nullptr, 0});
void launch_tube_fwd64(const Plan& p, const double* in, double2* out, long bs, long ps, long qs, long sp, long sq, int P,
                       int Q, double s);
void launch_roots(const Plan& p);   // p.twg
void launch_normal(const Plan& p, float* dst, size_t n, uint64_t seed);
void launch_zero(const Plan& p, void* dst, size_t bytes);
// n <= COPY_REGIONS copies between the context and a checkpoint blob in one launch; addresses and
// sizes are multiples of 4 bytes, on the context's device.  to_blob: the header goes to the blob;
// else nothing is copied unless the first COPY_HEADER_CHECKED words of the blob's are the same.
#define COPY_REGIONS 16
#define COPY_HEADER_WORDS 18
#define COPY_HEADER_CHECKED 7
struct CopyRegion {
  const unsigned char* src;
  unsigned char* dst;
  size_t bytes;
};
void launch_copy_regions(const Plan& p, const CopyRegion* r, int n, const void* header, void* blob, bool to_blob);

// iteration
enum SliceMode { SLICE_INIT = 0, SLICE_ITER = 1, SLICE_RESULT = 2, SLICE_KKT = 3 };
// How steps 3, 4 and 7 run: one fused kernel per OD row with several threads per tube
// (COOP) or one thread per tube (THREAD), as the tube length has it, or three launches through
// spatial buffers (SPLIT).
enum SlicePath { SPATH_COOP = 1, SPATH_THREAD = 2, SPATH_SPLIT = 3 };
int slice_default_path(int n2, int n3);
bool slice_path_valid(int path, int n2, int n3);
bool slice_supported(int n3);
bool slice_fused(int n2, int n3);          // the fused LDS slice kernel applies
size_t slice_generic_part_doubles(int n1, int n2, int n3);
void launch_slice_generic(const Plan& p, int mode, float* w_out, float* z_out, int w_from_g);
bool slice_hosts_pinvy(const Plan& p);   // the iteration's slice launch also forms G_Y^+
size_t slice_launch_lds_bytes(const Plan& p);
int slice_segments(int n2, int n3);              // lanes per row of the fused kernel's W-step
void launch_slice(const Plan& p, int mode, float* w_out, float* z_out, int w_from_g);
void launch_zgemm(const Plan& p, int with_pinv = 0);   // with_pinv: also G_Y^+ (pinvy_block)
// advance: next rounding-bit counter; scratch_out: with the stencil, X~ goes to the rhs
// buffer instead of X~ itself (a stage timing that leaves the state as it was)
void launch_agemm(const Plan& p, int raw_a = 0, int advance = 0, int scratch_out = 0);
// Half-width k and taps c lambda^d (d = 0 .. 2k + 1) of H_rho1^{-1} as a stencil, or -1
// where the stencil would be wider than HINV_KMAX, r > 16 or n1 < 2k + 2
int hinv_stencil(double rho1, int n1, int r, double* tap);
void launch_hsolve(const Plan& p);
void launch_bgemm(const Plan& p);   // X~^* W~; G_X, (H X~)^*(H X~), G_X^+ and I - eta P_X
bool bgemm_cols_valid(int r, int bcg);
void launch_ystep(const Plan& p, int init);
void ystep_split(int n2, int r, int nb, int* ny, int* cw);
size_t ystep_lds_bytes(int r, int cw);
void ystep_set_attr(size_t lds);
void launch_pinvy(const Plan& p, hipStream_t stream);
void pinvy_set_attr(int r);
void zgemm_set_attr(int r);
void launch_objective(const Plan& p);
void launch_termination(const Plan& p);
void launch_rank_init(const Plan& p);
void launch_rank_adjust(const Plan& p, double tol);
void rank_set_attr(int r);
size_t termination_work_doubles();   // partials of the step-6 reduction held in stat_work
void launch_stationarity(const Plan& p, int w_from_g);

// differentiation (reverse mode) of one iteration, FP64 (kernels_adjoint.hip)
// Complex matrix batch view: element (b, i, j) at b bs + i rs + j cs of float2 (f32 = 1) or
// double2 storage, conjugated on load when conj = 1.
struct CView {
  const void* p;
  long bs, rs, cs;
  int f32, conj;
};
struct AdjState {        // forward values of one iterate (inside a checkpoint blob)
  const float2* xt;      // X~ [nb][r][n1]
  const float2* yt;      // Y~ [nb][r][n2]
  const float2* wt;      // W~ [n1][nb][n2]
};
struct AdjWork {         // adjoint scratch carved from the caller's adjoint workspace
  double *w1s, *zbar;
  double2 *ztb, *wtb;
  double2 *x1b, *hx1, *a, *pp, *q, *pb, *qb, *ab, *dt;
  double2 *y1b, *bm, *bb, *rb;
  double2 *gy, *gyi, *gx, *gxi, *gyib, *gxib, *gyb, *gxb, *S, *T;
  double *htab, *wtab;   // pivot tables in FP64
  double *part, *wpart;
  int* flag;
};
size_t adjoint_work_bytes(const Plan& p);
void adjoint_carve(const Plan& p, void* ws, AdjWork* w);
void adjoint_set_attr(int r);
void launch_adjoint_step(const Plan& p, const AdjWork& w, const AdjState& in, const AdjState& out, double2* xt_bar,
                         double2* yt_bar, double* w_bar, double* theta);
void launch_adjoint_initial(const Plan& p, const double2* xt_bar, const double2* yt_bar, double* x0_bar,
                            double* y0_bar);
void launch_objective_gradient(const Plan& p, const AdjWork& w, double* x_grad, double* y_grad);

}  // namespace tctf
