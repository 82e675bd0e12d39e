// Internal: the context object behind the opaque chfsi_ctx handle and the
// helpers shared by the single-problem (context.hip) and batched (batch.hip)
// drivers.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>
#include <vector>

#include "../../include/chfsi.h"
#include "kernels.hpp"
#include "mesh.hpp"

namespace chfsi {

struct DevBuf {
  void *p = nullptr;
  size_t bytes = 0;
  hipError_t ensure(size_t want) {
    if (want <= bytes) return hipSuccess;
    if (p) {
      hipError_t e = hipFree(p);
      p = nullptr;
      bytes = 0;
      if (e != hipSuccess) return e;
    }
    hipError_t e = hipMalloc(&p, want);
    if (e == hipSuccess) bytes = want;
    else p = nullptr;
    return e;
  }
  void release() {
    if (p) (void)hipFree(p);
    p = nullptr;
    bytes = 0;
  }
  template <typename T> T *as() const { return reinterpret_cast<T *>(p); }
};


}  // namespace chfsi

struct chfsi_ctx {
  int device = 0;           // -1: host-only context (tables only, no device work)
  hipStream_t stream = nullptr;
  std::string err;
  chfsi::MeshTables mesh;
  bool has_mesh = false, has_pot = false;
  double vmax = 0, ub = 0;
  // device tables
  chfsi::DevBuf minv64, V64;
  chfsi::DevBuf vpart; // partial maxima of a potential given on the device
  chfsi::DevBuf ae64;  // 1D element matrices Ae and C of the Chebyshev step, (p+1)^2 each
  int tile_variant = -1;  // tile of the step kernel (-1: built-in choice)
  int rr_residual = 0;    // Ritz residuals: 0 cost model, 1 rotate HX, 2 apply Htilde again
  int jac_sweeps = 40;    // cap on Jacobi sweeps of the projected eigensolve
  // workspaces
  chfsi::DevBuf fbuf[2];      // the filter recursion's blocks
  chfsi::DevBuf occ_d;    // density: fr occupancy weights
  double kvec[3] = {0, 0, 0};
  double kin_k = 0;       // sum over directions of lambda_max of the 1D Bloch operators at kvec
  chfsi::DevBuf csel;     // complex Rayleigh-Ritz: selected Ritz values and the pairing status
  chfsi::DevBuf kgroup_d; // k-point group: its 3 nk wave vectors
  // Poisson: 1D band / mass tables (for the mesh they were built for), CG
  // workspace, point charges
  chfsi::DevBuf pois_kb, pois_m, pois_work, pois_q;
  int pois_n = 0, pois_p = 0;
  double pois_h = 0;
  int nk = 0;
  std::vector<double> kgroup;
  chfsi::DevBuf gram_part, Smat, dinv, Zmat, Wmat, jac_work, evals_d, resid_part, resid_d, flag, HX, diag0, minratio,
      rscratch;
  std::vector<double> host_scratch = std::vector<double>(16);
  // timing of the cell-product launches
  bool timing = false;
  std::vector<hipEvent_t> ev_pool;
  size_t ev_used = 0;
  int64_t cell_vecs = 0;
  bool verbose = false;   // CHFSI_VERBOSE: one progress line per solve pass on stderr
  // every device buffer the context owns
  template <typename F> void each_buf(F f) {
    chfsi::DevBuf *all[] = {&minv64, &V64, &vpart, &ae64, &fbuf[0],
                            &fbuf[1], &gram_part, &Smat, &dinv, &Zmat, &Wmat, &jac_work, &evals_d,
                            &resid_part, &resid_d, &flag, &HX, &diag0, &minratio, &rscratch, &occ_d, &kgroup_d, &pois_kb, &pois_m, &pois_work, &pois_q, &csel};
    for (chfsi::DevBuf *b : all) f(*b);
  }
};


namespace chfsi {

int fail(chfsi_ctx *c, int code, const std::string &msg);
int set_dev(chfsi_ctx *c);
int check_block(chfsi_ctx *c, const void *X, int64_t ld, int ncols);
int ensure_small(chfsi_ctx *c, int n);
// Workspace of one CholGS: device buffers for the overlap's split partials
// (part_elems doubles), S, the 32x32 diagonal inverses, Z and W (n x n each),
// the pivot diagnostics and the rotation's row panel (panel_elems doubles),
// and a host array of ceil(n/32) doubles for the pivot ratios.
struct CholWs {
  double *part = nullptr;
  size_t part_elems = 0;
  // complex blocks (interleaved re, im; ncols counts real columns): the raw
  // real Gram of the interleaved columns goes to G and its Hermitian
  // embedding to S (null for real blocks)
  double *G = nullptr;
  double *S = nullptr, *Z = nullptr, *W = nullptr, *dinv = nullptr, *diag0 = nullptr, *minratio = nullptr;
  int *flag = nullptr;
  double *panel = nullptr;
  size_t panel_elems = 0;
  double *host_ratio = nullptr;
};
int cholgs_core(chfsi_ctx *c, double *X, int64_t ld, int ncols, int mixed, double shift_rel, double *rmin,
                const CholWs &w);
// Looks up the device address of the allocation-free entry point's scratch
// array on `device` (current) once; 0 or an error status.
int noalloc_init(int device);
// the solve's CholGS (CholeskyQR2 / shifted Cholesky QR when needed); cplx:
// X is a complex block seen as interleaved reals (ld and nb count reals)
int orth_robust(chfsi_ctx *c, double *X, int64_t ld, int nb, int mixed, int *passes, bool cplx = false);
// Rayleigh-Ritz with HX in a caller buffer; evals/resid on the host
// Rayleigh-Ritz in three parts (a batch shares the middle one across problems)
int rr_project(chfsi_ctx *c, double *X, int64_t ld, int ncols, double *HX, int64_t ldh);
JacobiJob rr_eigen_job(chfsi_ctx *c, int ncols);
int rr_finish(chfsi_ctx *c, double *X, int64_t ld, int ncols, double *HX, int64_t ldh, double *evals,
              double *resid);
// Returns CHFSI_WARN_NOT_CONVERGED (with the results of the last Jacobi
// iterate) when the projected eigensolve ran out of sweeps.
int rr_impl(chfsi_ctx *c, double *X, int64_t ld, int ncols, double *HX, int64_t ldh, double *evals, double *resid,
            int *sweeps);
// A row-major block with row stride ld (of reals).
template <typename T>
inline ColBuf<T> row_major(const chfsi_ctx *c, T *p, int64_t ld) {
  return ColBuf<T>{p, ld, kron_group(c->mesh.p, sizeof(T))};
}
// Columns to a group of the library's own block of w columns (INT32_MAX:
// row-major): grouped where the tile kernel runs, also on the row-major block of
// stride ld that it alternates with, unless whole groups (one such block in FP64, two
// in FP32) take 16 MiB more than three blocks of w columns would: a column of a large
// mesh in FP32 would otherwise take 32 times its memory.  (Row-major is also the
// faster there, 32^3 cells of degree 5, FP32, 10 steps of 1 and 33 columns 4.1 -> 3.1
// and 9.2 -> 8.1 ms, but not on small meshes, 8^3 of degree 4 x 33 155 -> 170 us.)
inline int group_of(const chfsi_ctx *c, size_t elem, int w, int64_t ld = 1) {
  const int g = kron_group(c->mesh.p, elem);
  if (g == 0 || !kron_tiled(c->mesh.p, c->mesh.n, std::max<int64_t>(ld, 32), elem)) return INT32_MAX;
  const int64_t extra = (elem == 8 ? 1 : 2) * ((w + g - 1) / g * g) - 3 * w;   // columns
  return extra * c->mesh.n_dof * (int64_t)elem > (16 << 20) ? INT32_MAX : g;
}
// A w-column block of the library's own.
template <typename T>
inline ColBuf<T> work_block(const chfsi_ctx *c, T *p, int w, int64_t ld = 1) {
  const int g = group_of(c, sizeof(T), w, ld);
  if (g == INT32_MAX) return row_major<T>(c, p, w);
  return ColBuf<T>{p, g, c->mesh.n_dof * g};
}
// Device bytes of a block of the library's own of w columns or fewer.
size_t work_bytes(const chfsi_ctx *c, int w, size_t elem);
// Y = s1 (Htilde_k - shift) X + s2 Xp on complex blocks seen as 2 ncols real
// columns (Xp in Y's layout, or null).
int cheb_step_c(chfsi_ctx *c, const ColBuf<const double> &X, const double *Xp, const ColBuf<double> &Y, int ncols,
                double s1, double s2, double shift);
// Records the unconverged-eigensolve message and returns the warning.
int jacobi_warning(chfsi_ctx *c);
// Whether Rayleigh-Ritz obtains Htilde times the rotated columns by a fresh
// application (true) or by rotating HX (false), for ncols columns.
bool rr_reapply(const chfsi_ctx *c, int ncols);

}  // namespace chfsi

#define HIPCHK(ctx, call)                                                                         \
  do {                                                                                            \
    hipError_t e_ = (call);                                                                       \
    if (e_ != hipSuccess)                                                                         \
      return chfsi::fail(ctx, e_ == hipErrorOutOfMemory ? CHFSI_ERR_OOM : CHFSI_ERR_HIP,          \
                         std::string(#call) + ": " + hipGetErrorString(e_));                      \
  } while (0)
