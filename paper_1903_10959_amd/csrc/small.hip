// Small dense FP64 kernels on N_b x N_b matrices (N_b up to a few thousand).
//
//  * potrf: blocked right-looking Cholesky S = L L^T (Sec. 3.4 Alg. 3 step 2;
//    the paper uses ScaLAPACK pXpotrf).  32x32 diagonal blocks are factored
//    by one wave, which also inverts them for the panel solve.
//  * trtri_t: W = L^-T (Alg. 3 step 3; the paper uses pXtrtri), block row by
//    block row from the diagonal-block inverses.
//  * jacobi: symmetric eigensolver for the projected Hamiltonian (Sec. 3.5
//    step ii).  Block-cyclic Jacobi: blocks of 32 indices paired in
//    round-robin (parallel) order; each pair's 64 x 64 submatrix gets a sweep
//    of plane rotations in LDS, and the accumulated 64 x 64 rotations are
//    applied to the whole matrix and to the eigenvectors as small dense
//    products.  Many independent eigenproblems share each launch (the
//    batched workload's projected Hamiltonians), with one convergence check
//    per sweep for all of them.
#include "common.hpp"
#include "kernels.hpp"

#include <cmath>
#include <utility>
#include <vector>

namespace chfsi {

static constexpr int NB = 32;

// Relative pivot below which the overlap counts as numerically singular.
static constexpr double PIVOT_FLOOR = 1e-14;

// 1 / sqrt(x) to about an ulp (x normal and positive): the hardware estimate
// (about 24 bits) and one third-order step.
__device__ __forceinline__ double rsqrt_full(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = __builtin_fma(-x * y, y, 1.0);
  return __builtin_fma(y * e, __builtin_fma(0.375, e, 0.5), y);
}

// Before the factorisation: diag0 = diag(S) (after an optional shift of
// shift_rel * max diag(S) added to the diagonal, the shifted Cholesky remedy).
__global__ __launch_bounds__(1024) void potrf_prep_kernel(double *S, int n, double shift_rel, double *diag0) {
  __shared__ double red[1024];
  double m = 0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) m = fmax(m, S[(int64_t)i * n + i]);
  red[threadIdx.x] = m;
  __syncthreads();
  for (int w = 512; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + w]);
    __syncthreads();
  }
  const double sh = shift_rel * red[0];
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    double d = S[(int64_t)i * n + i] + sh;
    S[(int64_t)i * n + i] = d;
    diag0[i] = d;
  }
}

// Factor one 32x32 diagonal block.  Pivot j is accepted when
// d_j > PIVOT_FLOOR * diag0_j; minratio[block] = min_j d_j / diag0_j
// (d_j / S_jj is the squared sine of the angle between column j and the span
// of the columns before it, the loss-of-orthogonality indicator).
// One wave, no barriers: lane i holds row i of the trailing block in registers,
// its first column always in a[0]: a pivot's update moves every entry one
// register down, so that the loop over the pivots is one short body (unrolled
// it is 100 KB of code, fetched for one use).  The finished columns go through
// LDS, from where the update and the inverse (lane c: column c, shifted the
// same way) read them as broadcasts.  The chain of 32 pivots bounds it, so
// a pivot is one reciprocal square root and no division: 38 us per block with
// 256 threads, three barriers, a root and a division per pivot; 27 us so.
__device__ __forceinline__ double lane_of(double x, int l) {
  const long long b = __builtin_bit_cast(long long, x);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)b, l);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), l);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
__global__ __launch_bounds__(64) void potrf_diag_kernel(double *S, int n, int k0, double *dinv, int *flag,
                                                        const double *diag0, double *minratio) {
  __shared__ double L[NB][2 * NB];                   // L[c][r]: column c of the factor; r >= NB stays zero
  __shared__ double ri[NB];                          // 1 / L[c][c]
  const int kw = min(NB, n - k0);
  const int lane = threadIdx.x, i = lane & (NB - 1); // the upper half repeats the lower
  for (int e = lane; e < NB * 2 * NB; e += 64) (&L[0][0])[e] = 0.0;
  double a[NB];
#pragma unroll
  for (int c = 0; c < NB; ++c) {
    const bool in = i < kw && c <= i;                // padding rows: the identity
    const double v = S[(int64_t)(k0 + (in ? i : 0)) * n + k0 + (in ? c : 0)];
    a[c] = in ? v : (i == c ? 1.0 : 0.0);
  }
  const double ref_i = i < kw ? diag0[k0 + i] : 1.0;
  double d_i = 1.0;                                  // pivot i
#pragma unroll 1
  for (int jj = 0; jj < NB; ++jj) {
    const double d = lane_of(a[0], jj), ref = lane_of(ref_i, jj);
    double inv = rsqrt_full(d);
    if (!(d > PIVOT_FLOOR * ref) || !(ref > 0.0) || !(inv - inv == 0.0)) inv = __builtin_nan("");
    if (i == jj) d_i = d;
    const double l = i < jj ? 0.0 : i == jj ? d * inv : a[0] * inv;
    if (lane < NB) L[jj][i] = l;
    if (lane == 0) ri[jj] = inv;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int c = 0; c + 1 < NB; ++c) a[c] = __builtin_fma(-l, L[jj][jj + 1 + c], a[c + 1]);
    a[NB - 1] = 0.0;
  }
  // the ratios, all pivots at once; the first failing one is reported
  double ratio = i < kw ? (ref_i > 0.0 ? d_i / ref_i : -1.0) : 1.0;
  const bool fails = i < kw && !(L[i][i] - L[i][i] == 0.0);
  const unsigned bad = (unsigned)__ballot(fails);
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) ratio = fmin(ratio, __shfl_xor(ratio, o, 64));
  if (lane == 0) {
    if (bad && *flag == 0) *flag = k0 + __ffs((int)bad);
    minratio[k0 / NB] = fmin(1.0, ratio);
  }
  for (int e = lane; e < NB * NB; e += 64) {
    const int r = e / NB, c = e % NB;
    if (r < kw && c <= r) S[(int64_t)(k0 + r) * n + k0 + c] = L[c][r];
  }
  // inverse: column i of it solves L z = e_i
#pragma unroll
  for (int r = 0; r < NB; ++r) a[r] = r == i ? 1.0 : 0.0;
  double *dz = dinv + (int64_t)(k0 / NB) * NB * NB;
#pragma unroll 1
  for (int r = 0; r < NB; ++r) {
    const double z = a[0] * ri[r];
    if (lane < NB) dz[r * NB + i] = (r < kw && i <= r) ? z : 0.0;
#pragma unroll
    for (int q = 0; q + 1 < NB; ++q) a[q] = __builtin_fma(-L[r][r + 1 + q], z, a[q + 1]);
    a[NB - 1] = 0.0;
  }
}

// L[i, k0:k0+kw] = S[i, k0:k0+kw] Z^T for rows i >= k0+kw (Z = inverse diagonal block)
__global__ __launch_bounds__(256) void potrf_panel_kernel(double *S, int n, int k0, const double *dinv) {
  __shared__ double z[NB][NB + 1];
  __shared__ double rows[64][NB + 1];
  const int kw = min(NB, n - k0);
  const int r0 = k0 + kw + blockIdx.x * 64;
  const int tid = threadIdx.x;
  const double *dz = dinv + (int64_t)(k0 / NB) * NB * NB;
  for (int idx = tid; idx < NB * NB; idx += blockDim.x) z[idx / NB][idx % NB] = dz[idx];
  for (int idx = tid; idx < 64 * NB; idx += blockDim.x) {
    int r = idx / NB, c = idx % NB;
    int i = r0 + r;
    rows[r][c] = (i < n && c < kw) ? S[(int64_t)i * n + k0 + c] : 0.0;
  }
  __syncthreads();
  const int r = tid >> 2;
  const int cbeg = (tid & 3) * 8;
  const int i = r0 + r;
  if (i >= n) return;
  for (int c = cbeg; c < cbeg + 8 && c < kw; ++c) {
    double s = 0;
    for (int t = 0; t <= c; ++t) s += rows[r][t] * z[c][t];
    S[(int64_t)i * n + k0 + c] = s;
  }
}

// S[i][j] -= sum_t L[i][k0+t] L[j][k0+t] on the trailing lower triangle
__global__ __launch_bounds__(256) void potrf_update_kernel(double *S, int n, int k0) {
  __shared__ double li[NB][NB + 1];
  __shared__ double lj[NB][NB + 1];
  const int kw = min(NB, n - k0);
  const int k1 = k0 + kw;
  int t = blockIdx.x;
  int ti = (int)((sqrt(8.0 * t + 1.0) - 1.0) * 0.5);
  while ((ti + 1) * (ti + 2) / 2 <= t) ++ti;
  while (ti * (ti + 1) / 2 > t) --ti;
  const int tj = t - ti * (ti + 1) / 2;
  const int i0 = k1 + ti * NB, j0 = k1 + tj * NB;
  const int tid = threadIdx.x;
  for (int idx = tid; idx < NB * NB; idx += blockDim.x) {
    int r = idx / NB, c = idx % NB;
    li[r][c] = (i0 + r < n && c < kw) ? S[(int64_t)(i0 + r) * n + k0 + c] : 0.0;
    lj[r][c] = (j0 + r < n && c < kw) ? S[(int64_t)(j0 + r) * n + k0 + c] : 0.0;
  }
  __syncthreads();
  for (int idx = tid; idx < NB * NB; idx += blockDim.x) {
    int r = idx / NB, c = idx % NB;
    int i = i0 + r, jj = j0 + c;
    if (i >= n || jj >= n || jj > i) continue;
    double s = 0;
    for (int q = 0; q < kw; ++q) s += li[r][q] * lj[c][q];
    S[(int64_t)i * n + jj] -= s;
  }
}

void potrf_launch(double *S, int n, double *dinv, int *flag, double *diag0, double *minratio, double shift_rel,
                  hipStream_t s) {
  hipLaunchKernelGGL(potrf_prep_kernel, dim3(1), dim3(1024), 0, s, S, n, shift_rel, diag0);
  for (int k0 = 0; k0 < n; k0 += NB) {
    hipLaunchKernelGGL(potrf_diag_kernel, dim3(1), dim3(64), 0, s, S, n, k0, dinv, flag, diag0, minratio);
    const int k1 = k0 + NB;
    if (k1 >= n) break;
    const int rest = n - k1;
    hipLaunchKernelGGL(potrf_panel_kernel, dim3((rest + 63) / 64), dim3(256), 0, s, S, n, k0, dinv);
    const int nt = (rest + NB - 1) / NB;
    hipLaunchKernelGGL(potrf_update_kernel, dim3(nt * (nt + 1) / 2), dim3(256), 0, s, S, n, k0);
  }
}

// ---------------------------------------------------------------------------
// W = L^-T.  Z = L^-1 is lower triangular with Z_ii = dinv_i and, for ib > jb,
// Z_{ib,jb} = -dinv_ib * sum_{kb=jb}^{ib-1} L_{ib,kb} Z_{kb,jb}.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void trtri_init_kernel(const double *dinv, int n, double *Z) {
  const int64_t total = (int64_t)n * n;
  for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    int i = (int)(idx / n), jj = (int)(idx % n);
    double v = 0;
    if (i / NB == jj / NB) v = dinv[(int64_t)(i / NB) * NB * NB + (i % NB) * NB + (jj % NB)];
    Z[idx] = v;
  }
}

__global__ __launch_bounds__(256) void trtri_row_kernel(const double *L, const double *dinv, int n, int ib,
                                                        double *Z) {
  __shared__ double lb[NB][NB + 1];
  __shared__ double zb[NB][NB + 1];
  __shared__ double tb[NB][NB + 1];
  const int jb = blockIdx.x;  // < ib
  const int tid = threadIdx.x;
  double acc[4] = {0, 0, 0, 0};
  for (int kb = jb; kb < ib; ++kb) {
    for (int idx = tid; idx < NB * NB; idx += blockDim.x) {
      int r = idx / NB, c = idx % NB;
      int i = ib * NB + r, k = kb * NB + c;
      lb[r][c] = (i < n && k < n) ? L[(int64_t)i * n + k] : 0.0;
      int kk = kb * NB + r, jj = jb * NB + c;
      zb[r][c] = (kk < n && jj < n) ? Z[(int64_t)kk * n + jj] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      int idx = tid + u * 256;
      int r = idx / NB, c = idx % NB;
      double s = 0;
      for (int q = 0; q < NB; ++q) s += lb[r][q] * zb[q][c];
      acc[u] += s;
    }
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    int idx = tid + u * 256;
    tb[idx / NB][idx % NB] = acc[u];
  }
  const double *di = dinv + (int64_t)ib * NB * NB;
  for (int idx = tid; idx < NB * NB; idx += blockDim.x) lb[idx / NB][idx % NB] = di[idx];
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    int idx = tid + u * 256;
    int r = idx / NB, c = idx % NB;
    double s = 0;
    for (int q = 0; q < NB; ++q) s += lb[r][q] * tb[q][c];
    int i = ib * NB + r, jj = jb * NB + c;
    if (i < n && jj < n) Z[(int64_t)i * n + jj] = -s;
  }
}

__global__ __launch_bounds__(256) void transpose_kernel(const double *Z, int n, double *W) {
  const int64_t total = (int64_t)n * n;
  for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    int i = (int)(idx / n), jj = (int)(idx % n);
    W[idx] = Z[(int64_t)jj * n + i];
  }
}

static unsigned grid_for(int64_t total) {
  int64_t b = (total + 255) / 256;
  if (b > 16384) b = 16384;
  if (b < 1) b = 1;
  return (unsigned)b;
}

void trtri_t_launch(const double *L, const double *dinv, int n, double *Z, double *W, hipStream_t s) {
  const int nb = (n + NB - 1) / NB;
  hipLaunchKernelGGL(trtri_init_kernel, dim3(grid_for((int64_t)n * n)), dim3(256), 0, s, dinv, n, Z);
  for (int ib = 1; ib < nb; ++ib)
    hipLaunchKernelGGL(trtri_row_kernel, dim3(ib), dim3(256), 0, s, L, dinv, n, ib, Z);
  hipLaunchKernelGGL(transpose_kernel, dim3(grid_for((int64_t)n * n)), dim3(256), 0, s, Z, n, W);
}

// ---------------------------------------------------------------------------
// Jacobi eigensolver
// ---------------------------------------------------------------------------
__device__ __forceinline__ int rr_index(int pos, int r, int np) {
  return pos == 0 ? 0 : 1 + (pos - 1 + r) % (np - 1);
}

// Block-cyclic Jacobi.  The indices are grouped in blocks of JB = 32; a
// block round pairs the blocks in round-robin order (as the scalar method
// pairs indices), and for every pair (I, J) of blocks
//   1. one work-group takes the 64 x 64 submatrix S = A[I u J, I u J] into
//      LDS and rotates it in parallel rounds of 32 disjoint plane rotations,
//      accumulating them in R (64 x 64, orthogonal);
//   2. A <- R^T A R tile by tile (every pair of pairs: one 64 x 64 triple
//      product), into the other buffer;
//   3. V <- V R in place, panel by panel.
// A sweep is one block round g = 0 that rotates the pairs inside each block
// (31 rounds of 16 pairs in I and 16 in J), then nbp - 1 block rounds g >= 1
// (block pairing g - 1) that rotate only the pairs across I and J (32 rounds
// (t, 32 + (t + ir) mod 32)): every index pair once per sweep, a cyclic
// ordering, in 3 nbp launches instead of n - 1.  (Sweeping all 64 indices in
// every block round re-rotates the pairs inside blocks nbp - 1 times per
// sweep; checked on the host, it needs about as many sweeps for twice the
// inner rounds.)
static constexpr int JB = 32, J2 = 64;
static constexpr int OFFP = 32;   // work-groups per problem in the off-norm

// One problem of a batched block-Jacobi round: A (n x n) double buffered
// (A[b]), V updated in place, R the current round's pair rotations
// (npairs x 64 x 64), the buffer holding A at the start of the sweep (par0),
// and the first work-group of this problem in each of the three launches.
struct JacProb {
  double *A[2], *V, *R;
  int n, nbp, par0;
  int64_t first_inner, first_tile, first_panel;
};

__device__ __forceinline__ int jac_find(const JacProb *__restrict__ probs, int nprob, int which, int idx) {
  int lo = 0, hi = nprob - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    const int64_t f = which == 0 ? probs[mid].first_inner : which == 1 ? probs[mid].first_tile : probs[mid].first_panel;
    if (f <= (int64_t)idx) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// global index of local index i (0..63) of block pair (I, J); >= n: padding
__device__ __forceinline__ int jac_gidx(int i, int I, int J) { return i < JB ? I * JB + i : J * JB + (i - JB); }

// Local pair t (0..31) of inner round ir: inside the blocks (within) or
// across them.
__device__ __forceinline__ void jac_pair(int t, int ir, bool within, int &p, int &q) {
  if (within) {
    const int h = t >> 4, u = t & 15;                // block half, pair in it
    p = JB * h + rr_index(u, ir, JB);
    q = JB * h + rr_index(JB - 1 - u, ir, JB);
  } else {
    p = t;
    q = JB + (t + ir) % JB;
  }
}

// Rotation (c, s), t = s / c, that zeroes apq, |angle| <= 45 degrees.  With
// d = aqq - app, h = 2 apq, r = sqrt(d^2 + h^2): c^2 = (1 + |d|/r) / 2, s =
// |h| / (2 r c), signs those of d/h (+ for d = 0).  Two reciprocal square roots
// on one chain instead of two divisions and two roots; d and h are scaled by a
// power of two so that the squares neither over- nor underflow.
__device__ __forceinline__ void jac_angle(double app, double aqq, double apq, double &c, double &s, double &t) {
  c = 1.0;
  s = 0.0;
  t = 0.0;
  double d = aqq - app, h = 2.0 * apq;
  const bool neg = d != 0.0 && ((d < 0.0) != (h < 0.0));
  d = fabs(d);
  h = fabs(h);
  const int e = __builtin_amdgcn_frexp_exp(fmax(d, h));
  d = ldexp(d, -e);
  h = ldexp(h, -e);
  const double y = rsqrt_full(__builtin_fma(d, d, h * h));
  const double u = __builtin_fma(0.5 * d, y, 0.5);
  const double yc = rsqrt_full(u);
  const double sa = 0.5 * h * y * yc, ta = sa * yc;
  if (fabs(apq) >= 1e-300) {
    c = u * yc;
    s = neg ? -sa : sa;
    t = neg ? -ta : ta;
  }
}

// 1. one sweep of the 64-index pair submatrix in LDS; R out
// g: block round of the sweep (0: pairs inside the blocks, pairing 0;
// g >= 1: pairs across the blocks, pairing g - 1).
// Four waves rotate S: thread (a0, b) = (t / 32, t % 32) updates the 2 x 2
// blocks (pair a0 + 8 k rows, pair b columns).  Each of them computes all 32
// rotations for itself (lane b: pair b), so that a round has one barrier after
// its reads and one after its writes and no rotation waits for another wave.
// Four more waves accumulate R, one round behind, off that chain.  A round is
// bound by its chain of latencies: 47 us per 32 rounds with sixteen waves that
// wait for one wave's rotations (two divisions, two roots); across two blocks
// 28-31 us so, inside them (33 rounds over 64 indices) 42 us.
template <bool within>
__global__ __launch_bounds__(512) void jacobi_inner_kernel(const JacProb *__restrict__ probs, int nprob, int g) {
  __shared__ double S[J2][J2 + 1];
  __shared__ double Rs[within ? J2 : 1][J2 + 1];
  __shared__ double cs[4][J2 / 2], sn[4][J2 / 2];    // a wave's own rotations
  __shared__ double cr[2][J2 / 2], sr[2][J2 / 2];    // ... of a round, for R
  const JacProb &P = probs[jac_find(probs, nprob, 0, blockIdx.x)];
  if (g >= P.nbp) return;                          // this problem's sweep is complete
  const int r = within ? 0 : g - 1;                // (within: g = 0)
  const int k = (int)(blockIdx.x - P.first_inner);
  const int n = P.n;
  const int I = rr_index(k, r, P.nbp), J = rr_index(P.nbp - 1 - k, r, P.nbp);
  const double *A = P.A[(P.par0 + g) & 1];
  {
    double v[8];
    const int j = threadIdx.x % J2, i0 = threadIdx.x / J2, gj = jac_gidx(j, I, J);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int gi = jac_gidx(i0 + 8 * q, I, J);
      v[q] = (gi < n && gj < n) ? A[(int64_t)gi * n + gj] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      S[i0 + 8 * q][j] = v[q];
      if (within) Rs[i0 + 8 * q][j] = i0 + 8 * q == j ? 1.0 : 0.0;
    }
  }
  __syncthreads();
  const int nround = within ? JB - 1 : JB;
  const bool on_s = threadIdx.x < 256;
  const int t = threadIdx.x & 255;
  const int w = t >> 6, a0 = t / (J2 / 2), b = t % (J2 / 2);
  double *Rg = P.R + (int64_t)k * J2 * J2;
  if (on_s) {
#pragma unroll 1
    for (int ir = 0; ir <= nround; ++ir) {
      if (ir == nround) {                            // (R's last round)
        __syncthreads();
        __syncthreads();
        break;
      }
      int pb, qb, pa[4], qa[4];
      jac_pair(b, ir, within, pb, qb);
      const double app = S[pb][pb], aqq = S[qb][qb], apq = S[pb][qb];
      double b00[4], b01[4], b10[4], b11[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        jac_pair(a0 + 8 * u, ir, within, pa[u], qa[u]);
        b00[u] = S[pa[u]][pb];
        b01[u] = S[pa[u]][qb];
        b10[u] = S[qa[u]][pb];
        b11[u] = S[qa[u]][qb];
      }
      __syncthreads();                               // every wave has read the pairs' entries
      double cb, sb, tb;
      jac_angle(app, aqq, apq, cb, sb, tb);
      if ((t & 32) == 0) {
        cs[w][b] = cb;
        sn[w][b] = sb;
        if (w == 0) {
          cr[ir & 1][b] = cb;
          sr[ir & 1][b] = sb;
        }
      }
      __builtin_amdgcn_wave_barrier();               // (cs, sn are read back by this wave only)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int a = a0 + 8 * u;
        const double ca = cs[w][a], sa = sn[w][a];
        const double r00 = ca * b00[u] - sa * b10[u], r01 = ca * b01[u] - sa * b11[u];
        const double r10 = sa * b00[u] + ca * b10[u], r11 = sa * b01[u] + ca * b11[u];
        const bool dia = a == b;
        S[pa[u]][pb] = dia ? b00[u] - tb * apq : cb * r00 - sb * r01;
        S[pa[u]][qb] = dia ? 0.0 : sb * r00 + cb * r01;
        S[qa[u]][pb] = dia ? 0.0 : cb * r10 - sb * r11;
        S[qa[u]][qb] = dia ? b11[u] + tb * apq : sb * r10 + cb * r11;
      }
      __syncthreads();
    }
    return;
  }
  // R <- R J, rows a0 + 8 h of pair b.  Across the blocks pair b is
  // (b, JB + (b + ir) % JB): column b of R stays with the threads of pair b,
  // and the second column passes each round to the lane of pair b - 1 in the
  // same 32-lane half.  So R lives in registers there, with one lane shift per
  // round; inside the blocks the pairing has no such shape and R stays in LDS
  // (each thread's entries are its own within a round).
  const int src = (t & 32) | ((b + 1) & 31);         // lane holding pair b + 1
  double rP[8], rQ[8];
#pragma unroll
  for (int h = 0; h < 8; ++h) {
    rP[h] = a0 + 8 * h == b ? 1.0 : 0.0;
    rQ[h] = a0 + 8 * h == JB + b ? 1.0 : 0.0;
  }
#pragma unroll 1
  for (int ir = 0; ir <= nround; ++ir) {
    __syncthreads();
    if (ir > 0) {
      const double cb = cr[(ir - 1) & 1][b], sb = sr[(ir - 1) & 1][b];
      if (within) {
        int pb, qb;
        jac_pair(b, ir - 1, within, pb, qb);
#pragma unroll
        for (int h = 0; h < 8; ++h) {
          const int row = a0 + 8 * h;
          const double rp = Rs[row][pb], rq = Rs[row][qb];
          Rs[row][pb] = cb * rp - sb * rq;
          Rs[row][qb] = sb * rp + cb * rq;
        }
      } else {
#pragma unroll
        for (int h = 0; h < 8; ++h) {
          const double rp = rP[h], rq = rQ[h];
          rP[h] = cb * rp - sb * rq;
          rQ[h] = sb * rp + cb * rq;
          rQ[h] = __shfl(rQ[h], src, 64);              // next round's second column
        }
      }
    }
    __syncthreads();
  }
  if (within) {
    for (int e = t; e < J2 * J2; e += 256) Rg[e] = Rs[e / J2][e % J2];
  } else {
    // after the shift of the last round this thread holds column JB + (b + nround) % JB
    const int qcol = JB + (b + nround) % JB;
#pragma unroll
    for (int h = 0; h < 8; ++h) {
      Rg[(a0 + 8 * h) * J2 + b] = rP[h];
      Rg[(a0 + 8 * h) * J2 + qcol] = rQ[h];
    }
  }
}

// C = op(X) Y for 64 x 64 LDS operands on FP64 MFMA (16x16x4): wave w of 4
// computes rows 16 w .. 16 w + 15 as four 16 x 16 tiles along the columns;
// c[b][q] is row 16 w + acc_row(kq, q), column 16 b + (lane & 15).
// TRANS: X used transposed.
template <bool TRANS>
__device__ __forceinline__ void jac_mm64(const double (*X)[J2 + 1], const double (*Y)[J2 + 1], v4d (&c)[4], int w,
                                         int lane) {
  const int j = lane & 15, kq = lane >> 4;
#pragma unroll
  for (int b = 0; b < 4; ++b) c[b] = v4d{0, 0, 0, 0};
#pragma unroll 4
  for (int kk = 0; kk < J2; kk += 4) {
    const int k = kk + kq;
    const double a = TRANS ? X[k][16 * w + j] : X[16 * w + j][k];   // A[16 w + j][k]
#pragma unroll
    for (int b = 0; b < 4; ++b) c[b] = mfma16x4(a, Y[k][16 * b + j], c[b]);
  }
}

// 2. A_next[P1 rows, P2 cols] = R_P1^T A[P1, P2] R_P2 for every pair of pairs
//    k1 <= k2, with the mirror tile A_next[P2, P1] its transpose
// Tiles are loaded whole into registers before the first LDS store (one
// latency instead of sixteen), and the eigenvectors' rotation shares the
// launch: n = 360 takes 12 us where two kernels took 22 + 14.
typedef double (*jac_mat)[J2 + 1];
__device__ __forceinline__ void jac_load_r(const double *__restrict__ Rg, double (&v)[16], int t) {
#pragma unroll
  for (int q = 0; q < 16; ++q) v[q] = Rg[t + 256 * q];
}
__device__ __forceinline__ void jac_put(jac_mat M, const double (&v)[16], int t) {
#pragma unroll
  for (int q = 0; q < 16; ++q) M[t / J2 + 4 * q][t % J2] = v[q];
}
__device__ __forceinline__ void jacobi_apply_a(const JacProb &P, int tile, int g, jac_mat T, jac_mat R1, jac_mat R2) {
  const int r = g == 0 ? 0 : g - 1;
  // A is symmetric, so the tile of pairs (k2, k1) is the transpose of that of
  // (k1, k2): only k1 <= k2 are computed, each written with its mirror
  // (tile = k2 (k2 + 1) / 2 + k1)
  int k2 = (int)((sqrtf(8.0f * tile + 1.0f) - 1.0f) * 0.5f);
  while (k2 * (k2 + 1) / 2 > tile) --k2;
  while ((k2 + 1) * (k2 + 2) / 2 <= tile) ++k2;
  const int k1 = tile - k2 * (k2 + 1) / 2;
  const int n = P.n;
  const int I1 = rr_index(k1, r, P.nbp), J1 = rr_index(P.nbp - 1 - k1, r, P.nbp);
  const int I2 = rr_index(k2, r, P.nbp), J2b = rr_index(P.nbp - 1 - k2, r, P.nbp);
  const double *A = P.A[(P.par0 + g) & 1];
  double *An = P.A[(P.par0 + g + 1) & 1];
  const int t = threadIdx.x;
  {
    double v[16], v1[16], v2[16];
    const int gj = jac_gidx(t % J2, I2, J2b);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int gi = jac_gidx(t / J2 + 4 * q, I1, J1);
      v[q] = (gi < n && gj < n) ? A[(int64_t)gi * n + gj] : 0.0;
    }
    jac_load_r(P.R + (int64_t)k1 * J2 * J2, v1, t);
    jac_load_r(P.R + (int64_t)k2 * J2 * J2, v2, t);
    jac_put(T, v, t);
    jac_put(R1, v1, t);
    jac_put(R2, v2, t);
  }
  __syncthreads();
  const int wv = t >> 6, lane = t & 63, jl = lane & 15, kq = lane >> 4;
  v4d c[4];
  jac_mm64<false>(T, R2, c, wv, lane);             // U = T R2
  __syncthreads();
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int q = 0; q < 4; ++q) T[16 * wv + acc_row<double>(kq, q)][16 * b + jl] = c[b][q];
  __syncthreads();
  jac_mm64<true>(R1, T, c, wv, lane);              // C = R1^T U
  __syncthreads();                                  // every wave has read U
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int q = 0; q < 4; ++q) T[16 * wv + acc_row<double>(kq, q)][16 * b + jl] = c[b][q];
  __syncthreads();
  // C to rows of pair k1 x columns of pair k2, C^T to the mirror tile
  for (int e = t; e < J2 * J2; e += 256) {
    const int i = e / J2, j = e % J2;
    const int gi = jac_gidx(i, I1, J1), gj = jac_gidx(j, I2, J2b);
    if (gi < n && gj < n) An[(int64_t)gi * n + gj] = T[i][j];
    if (k1 != k2) {
      const int hi = jac_gidx(i, I2, J2b), hj = jac_gidx(j, I1, J1);
      if (hi < n && hj < n) An[(int64_t)hi * n + hj] = T[j][i];
    }
  }
}

// 3. V[panel rows, P cols] <- V[panel rows, P cols] R_P, in place
__device__ __forceinline__ void jacobi_apply_v(const JacProb &P, int w, int g, jac_mat T, jac_mat Rl) {
  const int r = g == 0 ? 0 : g - 1;
  const int np2 = P.nbp / 2;
  const int panel = w / np2, k = w % np2;
  const int n = P.n;
  const int I = rr_index(k, r, P.nbp), J = rr_index(P.nbp - 1 - k, r, P.nbp);
  const int t = threadIdx.x;
  const int row0 = panel * J2;
  {
    double v[16], vr[16];
    const int gj = jac_gidx(t % J2, I, J);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int gr = row0 + t / J2 + 4 * q;
      v[q] = (gr < n && gj < n) ? P.V[(int64_t)gr * n + gj] : 0.0;
    }
    jac_load_r(P.R + (int64_t)k * J2 * J2, vr, t);
    jac_put(T, v, t);
    jac_put(Rl, vr, t);
  }
  __syncthreads();
  const int wv = t >> 6, lane = t & 63, jl = lane & 15, kq = lane >> 4;
  v4d c[4];
  jac_mm64<false>(T, Rl, c, wv, lane);
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int gr = row0 + 16 * wv + acc_row<double>(kq, q), gj = jac_gidx(16 * b + jl, I, J);
      if (gr < n && gj < n) P.V[(int64_t)gr * n + gj] = c[b][q];
    }
}

// Steps 2 and 3 do not depend on each other: one launch, the first n_tile
// work-groups update A, the others V.
__global__ __launch_bounds__(256) void jacobi_apply_kernel(const JacProb *__restrict__ probs, int nprob, int g,
                                                           int n_tile) {
  __shared__ double T[J2][J2 + 1], R1[J2][J2 + 1], R2[J2][J2 + 1];
  const bool on_a = (int)blockIdx.x < n_tile;
  const int idx = on_a ? (int)blockIdx.x : (int)blockIdx.x - n_tile;
  const JacProb &P = probs[jac_find(probs, nprob, on_a ? 1 : 2, idx)];
  if (g >= P.nbp) return;
  if (on_a) jacobi_apply_a(P, idx - (int)P.first_tile, g, T, R1, R2);
  else jacobi_apply_v(P, idx - (int)P.first_panel, g, T, R1);
}

// Squared off-diagonal and diagonal Frobenius norms of each problem's A, as
// OFFP partial sums per problem (work-group part takes rows part*4 + wave,
// stepping by 4 OFFP); the host adds the partials in a fixed order.
__global__ __launch_bounds__(256) void offnorm_kernel(const JacProb *__restrict__ probs, double *__restrict__ out) {
  __shared__ double so[256], sd[256];
  const int a = blockIdx.x / OFFP, part = blockIdx.x % OFFP;
  const JacProb &J = probs[a];
  const double *A = J.A[J.par0];
  const int n = J.n;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  double o = 0, d = 0;
  for (int i = part * 4 + wave; i < n; i += OFFP * 4) {
    const double *row = A + (int64_t)i * n;
    for (int j = lane; j < n; j += 64) {
      const double v = row[j];
      if (j == i) d += v * v;
      else o += v * v;
    }
  }
  so[threadIdx.x] = o;
  sd[threadIdx.x] = d;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      so[threadIdx.x] += so[threadIdx.x + w];
      sd[threadIdx.x] += sd[threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[2 * blockIdx.x] = so[0];
    out[2 * blockIdx.x + 1] = sd[0];
  }
}

__global__ __launch_bounds__(256) void eye_kernel(double *V, int n) {
  const int64_t total = (int64_t)n * n;
  for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x)
    V[idx] = (idx / n == idx % n) ? 1.0 : 0.0;
}

// evals ascending; Q[:, rank(i)] = V[:, i]; ties broken by index.  Work-group =
// 256 columns x SORT_ROWS rows; each ranks its columns itself (the diagonal
// through LDS, 256 values at a time).
static constexpr int SORT_ROWS = 32;
__global__ __launch_bounds__(256) void jacobi_sort_kernel(const double *A, const double *V, int n, double *evals,
                                                          double *Q) {
  __shared__ double d[256];
  const int i = blockIdx.x * 256 + threadIdx.x;
  const double di = i < n ? A[(int64_t)i * n + i] : 0.0;
  int rank = 0;
  for (int k0 = 0; k0 < n; k0 += 256) {
    __syncthreads();
    const int kk = k0 + threadIdx.x;
    if (kk < n) d[threadIdx.x] = A[(int64_t)kk * n + kk];
    __syncthreads();
    const int m = n - k0 < 256 ? n - k0 : 256;
    for (int k = 0; k < m; ++k)
      if (d[k] < di || (d[k] == di && k0 + k < i)) ++rank;
  }
  if (i >= n) return;
  const int r0 = blockIdx.y * SORT_ROWS, r1 = r0 + SORT_ROWS < n ? r0 + SORT_ROWS : n;
  if (blockIdx.y == 0) evals[rank] = di;
#pragma unroll 4
  for (int row = r0; row < r1; ++row) Q[(int64_t)row * n + rank] = V[(int64_t)row * n + i];
}

static int jac_nbp(int n) {
  const int nblk = (n + JB - 1) / JB;
  return nblk + (nblk & 1);
}

// work: A's second buffer (n^2), V (n^2), the pair rotations
// (nbp/2 x 64 x 64), a tail for the single-problem table (16 doubles) and
// norms (jacobi_norms_elems(1))
static constexpr int JTAIL = 16 + 2 * OFFP;
size_t jacobi_norms_elems(int njobs) { return (size_t)2 * OFFP * (njobs > 0 ? njobs : 1); }
size_t jacobi_work_elems(int n) {
  return (size_t)2 * n * n + (size_t)(jac_nbp(n) / 2) * J2 * J2 + JTAIL;
}
size_t jacobi_table_bytes(int njobs) { return (size_t)(njobs > 0 ? njobs : 1) * sizeof(JacProb); }

int jacobi_eigh_batch(const JacobiJob *jobs, int njobs, double tol, int max_sweeps, void *table, double *norms,
                      double *host_norms, hipStream_t s, int *sweeps_done, int *converged) {
  if (njobs <= 0) return 0;
  std::vector<JacProb> all(njobs);
  std::vector<int> active(njobs, 1);
  std::vector<double> prev_off(njobs, -1.0);
  for (int k = 0; k < njobs; ++k) {
    const JacobiJob &jb = jobs[k];
    const int n = jb.n;
    JacProb &J = all[k];
    J.A[0] = jb.A;
    J.A[1] = jb.work;
    J.V = jb.work + (size_t)n * n;
    J.R = jb.work + (size_t)2 * n * n;
    J.n = n;
    J.nbp = jac_nbp(n);
    J.par0 = 0;                                    // nbp is even: each sweep ends in the buffer it started in
    J.first_inner = J.first_tile = J.first_panel = 0;
    hipLaunchKernelGGL(eye_kernel, dim3(grid_for((int64_t)n * n)), dim3(256), 0, s, J.V, n);
    if (n <= 1) active[k] = 0;
  }
  JacProb *dtab = static_cast<JacProb *>(table);
  int sweep = 0;
  // the problems still iterating, as the table on the device lists them; it is
  // written again only when one of them is done (an even number of block
  // rounds leaves A in the buffer it started in)
  std::vector<JacProb> run;
  std::vector<int> ids;
  int rmax = 0;
  int64_t n_inner = 0, n_tile = 0, n_panel = 0;
  auto set_table = [&]() {
    run.clear();
    ids.clear();
    rmax = 0;
    n_inner = n_tile = n_panel = 0;
    for (int k = 0; k < njobs; ++k) {
      if (!active[k]) continue;
      JacProb &J = all[k];
      const int np2 = J.nbp / 2;
      J.first_inner = n_inner;
      J.first_tile = n_tile;
      J.first_panel = n_panel;
      n_inner += np2;
      n_tile += (int64_t)np2 * (np2 + 1) / 2;
      n_panel += (int64_t)((J.n + J2 - 1) / J2) * np2;
      rmax = std::max(rmax, J.nbp);                // block rounds g = 0 .. nbp - 1
      run.push_back(J);
      ids.push_back(k);
    }
    if (run.empty()) return true;
    return hipMemcpyAsync(dtab, run.data(), run.size() * sizeof(JacProb), hipMemcpyHostToDevice, s) == hipSuccess;
  };
  if (!set_table()) return -1;
  for (; !run.empty(); ++sweep) {
    // convergence of every active problem, one host synchronisation (also
    // after the last allowed sweep, so that its result is judged)
    const int nr = (int)run.size();
    hipLaunchKernelGGL(offnorm_kernel, dim3((unsigned)(nr * OFFP)), dim3(256), 0, s, dtab, norms);
    if (hipMemcpyAsync(host_norms, norms, (size_t)2 * OFFP * nr * sizeof(double), hipMemcpyDeviceToHost, s) !=
        hipSuccess)
      return -1;
    if (hipStreamSynchronize(s) != hipSuccess) return -1;
    bool changed = false, left = false;
    for (int a = 0; a < nr; ++a) {
      const int k = ids[a];
      double off = 0, dg = 0;
      for (int q = 0; q < OFFP; ++q) {
        off += host_norms[2 * (a * OFFP + q)];
        dg += host_norms[2 * (a * OFFP + q) + 1];
      }
      const double tot = off + dg;
      bool done = off <= tol * tol * tot;
      if (prev_off[k] >= 0 && off >= prev_off[k] && off <= 1e-20 * tot) done = true;  // stagnated at rounding
      prev_off[k] = off;
      if (done) active[k] = 0;
      (done ? changed : left) = true;
    }
    // (out of sweeps: the rest stay unconverged.  The stream has read the table's
    // last copy by now, and no other is started that would outlive `run`.)
    if (!left || sweep >= max_sweeps) break;
    if (changed && !set_table()) return -1;
    for (int g = 0; g < rmax; ++g) {
      if (g == 0)
        hipLaunchKernelGGL((jacobi_inner_kernel<true>), dim3((unsigned)n_inner), dim3(512), 0, s, dtab, (int)run.size(), g);
      else
        hipLaunchKernelGGL((jacobi_inner_kernel<false>), dim3((unsigned)n_inner), dim3(512), 0, s, dtab, (int)run.size(), g);
      hipLaunchKernelGGL(jacobi_apply_kernel, dim3((unsigned)(n_tile + n_panel)), dim3(256), 0, s, dtab,
                         (int)run.size(), g, (int)n_tile);
    }
  }
  for (int k = 0; k < njobs; ++k) {
    const JacProb &J = all[k];
    hipLaunchKernelGGL(jacobi_sort_kernel, dim3((J.n + 255) / 256, (J.n + SORT_ROWS - 1) / SORT_ROWS), dim3(256), 0, s,
                       J.A[J.par0], J.V, J.n, jobs[k].evals, jobs[k].Q);
  }
  if (sweeps_done) *sweeps_done = sweep;
  int unconv = 0;
  for (int k = 0; k < njobs; ++k) {
    if (converged) converged[k] = active[k] ? 0 : 1;
    unconv += active[k];
  }
  return unconv;
}

int jacobi_eigh(double *A, int n, double *work, double *evals, double *Q, double tol, int max_sweeps,
                double *host_scratch, hipStream_t s, int *sweeps_done) {
  // one problem through the batched driver: the table (one entry) and the
  // norm partials live in the tail of the work array; host_scratch holds at
  // least jacobi_norms_elems(1) doubles
  static_assert(sizeof(JacProb) <= 16 * sizeof(double), "one table entry fits the work tail");
  const JacobiJob job{A, n, work, evals, Q};
  double *tail = work + jacobi_work_elems(n) - JTAIL;
  return jacobi_eigh_batch(&job, 1, tol, max_sweeps, tail, tail + 16, host_scratch, s, sweeps_done, nullptr);
}

__global__ __launch_bounds__(256) void max_finite_kernel(const double *__restrict__ v, int64_t n,
                                                         double *__restrict__ part) {
  __shared__ double red[256];
  double m = -__builtin_inf();
  bool bad = false;
  for (int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const double x = v[i];
    bad |= !(x - x == 0.0);
    m = fmax(m, x);
  }
  red[threadIdx.x] = bad ? __builtin_inf() : m;     // (every kept value is finite: +inf stands for "not finite")
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0] == __builtin_inf() ? __builtin_nan("") : red[0];
}
void max_finite_launch(const double *v, int64_t n, double *part, int npart, hipStream_t s) {
  hipLaunchKernelGGL(max_finite_kernel, dim3((unsigned)npart), dim3(256), 0, s, v, n, part);
}

__global__ void fill_kernel(double *X, int64_t n, double v) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    X[i] = v;
}
void fill_launch(double *X, int64_t n, double v, hipStream_t s) {
  hipLaunchKernelGGL(fill_kernel, dim3(grid_for(n)), dim3(256), 0, s, X, n, v);
}

__global__ void zero_int_kernel(int *p, int n) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}
void zero_int_launch(int *p, int n, hipStream_t s) {
  hipLaunchKernelGGL(zero_int_kernel, dim3((n + 255) / 256), dim3(256), 0, s, p, n);
}

}  // namespace chfsi
