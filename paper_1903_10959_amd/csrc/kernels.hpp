// Host-side launchers of the device kernels (internal interface of the library).
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>
#include <vector>

namespace chfsi {

// ---- Chebyshev step (kron.hip) ---------------------------------------------
// A block of columns: value (dof i, column j) is at
// p[(j / g) * cg + i * ld + j % g], g = kron_group columns to a group.  A
// row-major block has cg = g; a grouped one (the library's own buffers: ld =
// g, cg = n_dof * g) keeps a group's rows next to each other, which the tile
// kernel reads 4 to 15 % faster.
template <typename T>
struct ColBuf {
  T *p;
  int64_t ld, cg;
};
// Columns to a group for values of `elem` bytes (0: degree p has no tile
// kernel and its blocks are row-major).
int kron_group(int p, size_t elem);
// Whether row stride ld fits the tile kernel's 32-bit plane offsets (a block
// that does not must be row-major).
bool kron_tiled(int p, int n, int64_t ld, size_t elem);
// Y = s1 (Htilde - shift) X + s2 Xp in one launch.  Xp has Y's layout and may
// be Y (each value is read before it is written, by the thread that writes
// it); Y must not be X.  Xp null: no previous block (s2 = 0).
template <typename T>
struct KronArgs {
  ColBuf<const T> X;
  const T *Xp;
  ColBuf<T> Y;
  const double *V;     // [n_dof]
  const double *ae;    // 1D element matrices Ae and C, (p+1)^2 each
  int n_el, p, n, periodic, ncols;
  double s1, s2, shift;
  int variant = -1;    // tile: -1 built-in choice, 0 2 x 2 cells, 1 4 x 2 where available
  int bf16 = 0;        // float: X enters the products with the 1D matrices' off-diagonal entries rounded to BF16
  double k[3] = {0, 0, 0};   // complex: Bloch vector
};
int kron_launch(const KronArgs<double> &a, hipStream_t s);
int kron_launch(const KronArgs<float> &a, hipStream_t s);
// Complex blocks as interleaved (re, im) real columns (a.ncols even), a.k the
// Bloch vector of the -i k.G term (its |k|^2/2 is the caller's, in a.shift).
int kron_launch_complex(const KronArgs<double> &a, hipStream_t s);
// A group of nk k-points (kv: 3 nk values on the device, host_kv on the host)
// in one launch: block g at X + g xstride (Y + g ystride, real elements).
int kron_launch_kpts(const KronArgs<double> &a, int nk, const double *kv, const double *host_kv, int64_t xstride,
                     int64_t ystride, hipStream_t s);
// Cells per z chunk of a march by `tiles` tiles.
int kron_zlen(int n_el, int p, int64_t tiles);

// One problem of a batched filter sweep (device-resident descriptor).  Step k
// reads buf[k & 1] and updates buf[(k & 1) ^ 1].
template <typename T>
struct KronBatchProblem {
  ColBuf<T> buf[2];
  const double *V, *ae;
  const double *coef;  // [degree x 3]: s1, s2, shift per step
  int n_el, n, periodic, ncols, bf16;
};
// The tile variant a problem runs (its context's setting, or for -1 the
// built-in choice); with it, its tiles (-1: no tile kernel for the degree), its
// work items appended to `work`, and the launch of one step for a work list of
// one degree and variant (bf16: some of its problems round to BF16).
template <typename T>
int kron_batch_variant(int p, int variant, int n_el, int ncols);
template <typename T>
int64_t kron_batch_tiles(int p, int variant, int n_el, int ncols);
template <typename T>
int kron_batch_work(int p, int variant, int n_el, int ncols, int prob, int zlen, std::vector<int4> &work);
template <typename T>
int kron_batch_launch(int p, int variant, bool bf16, const KronBatchProblem<T> *probs, const int4 *work, int nwork,
                      int step, hipStream_t s);
// out = in, values converted; gin, gout: columns to a group of either side
// (any value >= ncols for a row-major block).
template <typename Tin, typename Tout>
void copy_cols_launch(const ColBuf<Tin> &in, int gin, const ColBuf<Tout> &out, int gout, int64_t nrows, int ncols,
                      hipStream_t s);
template <typename T>
void nonfinite_launch(const T *X, int64_t ld, int64_t nrows, int ncols, int *flag, hipStream_t s);

// ---- tall-skinny products (dense.hip) ---------------------------------------
// G = A^T B over nrows rows, lower-triangular tiles, split over rows; partial
// tiles go to `part` and are summed in a fixed order into G (n x n, row-major,
// lower triangle mirrored to upper).  mixed: 64x64 diagonal blocks in FP64, the
// rest with FP32 inputs/products.  The number of splits follows from the rows and
// columns; gram_part_elems bounds the partial buffer of any launch.
size_t gram_part_elems(int64_t nrows, int n);
void gram_launch(const double *A, int64_t lda, const double *B, int64_t ldb, int64_t nrows, int n, double *part,
                 double *G, int mixed, hipStream_t s);
// As gram_launch with a partial buffer of part_elems doubles (0: sized by
// gram_part_elems): fewer row splits when it holds less; -1 when it cannot
// hold one split of every tile.
int gram_launch_capped(const double *A, int64_t lda, const double *B, int64_t ldb, int64_t nrows, int n,
                       double *part, size_t part_elems, double *G, int mixed, hipStream_t s);
// As gram_launch, with the trailing block (rows and columns >= fr0, rounded
// down to a multiple of 64) in FP64 and everything else with FP32 inputs and
// products: the split projected Hamiltonian.
void gram_split_launch(const double *A, int64_t lda, const double *B, int64_t ldb, int64_t nrows, int n, double *part,
                       double *G, int fr0, hipStream_t s);
// X[r, 0:n] <- X[r, 0:n] W for all rows, in LDS up to 624 columns, beyond that
// chunk by chunk through `scratch`
// (scratch_elems doubles, at least 128 x n; rmul_scratch_elems gives the size
// used by the library).  W: n x n row-major.  upper: W upper triangular (zero
// blocks skipped).  mixed (requires upper): the 64-wide diagonal blocks of W in
// FP64, the rest with FP32 inputs and products.  Returns -1 on bad arguments.
size_t rmul_scratch_elems(int64_t nrows, int n);
int rmul_launch(double *X, int64_t ld, int64_t nrows, int n, const double *W, int upper, int mixed,
                double *scratch, size_t scratch_elems, hipStream_t s);
// X[r, out_col0 : out_col0+nout] <- X[r, 0:n] W[0:n, 0:nout] (W row stride ldw),
// for all rows, chunk by chunk through `scratch` (as above); a partial
// rotation when nout < n.  upper/mixed as above (upper requires nout = ldw = n).
int rmul_cols_launch(double *X, int64_t ld, int64_t nrows, int n, const double *W, int64_t ldw, int nout,
                     int out_col0, int upper, int mixed, double *scratch, size_t scratch_elems, hipStream_t s);
// C[r, 0:nout] = X[r, 0:n] W[0:n, 0:nout] for all rows, out of place (C must
// not overlap X); one launch.  Returns -1 when the grid would not fit.
int rmul_out_launch(const double *X, int64_t ld, int64_t nrows, int n, const double *W, int64_t ldw, int nout,
                    double *C, int64_t ldc, hipStream_t s);
// rho[j] = 2 minv[j]^2 (sum_{i<ncols} X[j,i]^2 + sum_{k<nfr} w[k] Xfr[j,k]^2),
// j < nrows; w on the device.
void density_launch(const double *X, int64_t ld, int ncols, const double *Xfr, int64_t ldfr, int nfr,
                    const double *w, const double *minv, int64_t nrows, double *rho, hipStream_t s);
// resid[j] = || HX[:,j] - lam[j] X[:,j] ||_2 ; part: [nchunk x n]
int resid_nchunk(int64_t nrows);
void resid_launch(const double *X, int64_t ldx, const double *HX, int64_t ldh, const double *lam, int64_t nrows,
                  int n, double *part, double *resid, hipStream_t s);

// ---- small dense FP64 kernels (small.hip) ---------------------------------
// In-place blocked Cholesky of the lower triangle of S (n x n row-major):
// S + shift_rel*max(diag S)*I = L L^T; dinv receives the inverses of the 32x32
// diagonal blocks of L; *flag = first failing pivot + 1 (0 if every pivot
// d_j > 1e-14 * diag_j); diag0 [n] scratch; minratio[ceil(n/32)] = per-block
// minimum of d_j / diag_j.
void potrf_launch(double *S, int n, double *dinv, int *flag, double *diag0, double *minratio, double shift_rel,
                  hipStream_t s);
// W = L^-T (upper triangular, n x n row-major) from L and dinv; Z scratch n x n.
void trtri_t_launch(const double *L, const double *dinv, int n, double *Z, double *W, hipStream_t s);
// Symmetric eigensolver (cyclic Jacobi, round-robin pairs, one launch per round).
// A: n x n symmetric (row-major, full), destroyed; work: see jacobi_work_elems.
// On exit: evals ascending (device, n), Q (n x n row-major, columns = vectors).
size_t jacobi_work_elems(int n);
// Many independent eigenproblems at once: every round launch covers all
// problems still iterating, one host synchronisation per sweep checks them
// all.  Job k: A (destroyed), work (jacobi_work_elems(n)), evals/Q as above.
// table: device scratch of jacobi_table_bytes(njobs); norms: device and
// host_norms: host, jacobi_norms_elems(njobs) doubles each (jacobi_eigh:
// host_scratch of jacobi_norms_elems(1)).
struct JacobiJob {
  double *A;
  int n;
  double *work, *evals, *Q;
};
size_t jacobi_table_bytes(int njobs);
size_t jacobi_norms_elems(int njobs);
// Returns -1 on a HIP error, else the number of jobs whose off-diagonal norm
// had not met tol when max_sweeps sweeps were done (their evals/Q hold the
// last iterate); converged (may be null) receives 1/0 per job.
int jacobi_eigh_batch(const JacobiJob *jobs, int njobs, double tol, int max_sweeps, void *table, double *norms,
                      double *host_norms, hipStream_t s, int *sweeps_done, int *converged);
int jacobi_eigh(double *A, int n, double *work, double *evals, double *Q, double tol, int max_sweeps,
                double *host_scratch, hipStream_t s, int *sweeps_done);
// ---- complex (Hermitian) subspace steps on interleaved blocks (complex.hip)
// A complex n x N block X seen as the real n x 2N block R of its interleaved
// (re, im) columns.  G = R^T B (real 2N x 2N, lower triangle used) of two such
// blocks gives the Hermitian N x N matrix M = X^H Y through
//   Re M_jk = G[2j][2k] + G[2j+1][2k+1],  Im M_jk = G[2j][2k+1] - G[2j+1][2k]
// (j > k; the diagonal is real and the upper triangle follows by symmetry).
// herm_embed_launch writes E (2N x 2N real symmetric) = emb(M), the real form
// with 2 x 2 blocks [[Re, Im], [-Im, Re]], in which right-multiplication of R
// by emb(W) is the complex product X W.
void herm_embed_launch(const double *G, int n2, double *E, hipStream_t s);
// From the eigenvectors V (n2 x n2 row-major, column i = pair i, ascending
// values ev) of an embedded Hermitian matrix, where every eigenvalue appears
// twice, picks N = n2/2 complex eigenvectors: candidates in ascending order
// are orthogonalised (twice) against the kept w and J w (J the pair rotation,
// (Jw)_2j = -w_2j+1, (Jw)_2j+1 = w_2j) and kept when a tenth of their norm
// survives.  Q (n2 x n2) = [w_0, J w_0, w_1, J w_1, ...] is the embedding of
// the complex eigenvector matrix; evals [N] and lam2 [n2] (each value twice)
// receive the kept values; *status = number kept.  One work-group; n2 <= 4096.
void herm_select_launch(const double *V, const double *ev, int n2, double *Q, double *evals, double *lam2,
                        int *status, hipStream_t s);

// part[k], k < npart: maxima of v over npart interleaved parts (-inf for an empty
// one, NaN where a value is not finite).
void max_finite_launch(const double *v, int64_t n, double *part, int npart, hipStream_t s);
// Zero the strictly upper triangle, helpers.
void fill_launch(double *X, int64_t n, double v, hipStream_t s);
void zero_int_launch(int *p, int n, hipStream_t s);

}  // namespace chfsi
