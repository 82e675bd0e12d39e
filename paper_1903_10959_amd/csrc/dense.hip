// Tall-skinny FP64 products of CholGS and Rayleigh-Ritz on MFMA.
//
//  * gram: G = A^T B, lower triangle only (Sec. 3.4 step 1, computing only the
//    lower-triangular part of the Hermitian overlap; Sec. 3.5 the projected
//    Hamiltonian the same way).  Mixed variant (eq. overlapmixedprec): FP64 on
//    the 64x64 diagonal blocks, FP32 inputs/products on the rest.
//  * rmul: X <- X W in place by row panels (Sec. 3.4 step 4, X L^-T; Sec. 3.5
//    subspace rotation X Q).  The paper's outer blocking over rows (B^d) keeps
//    only a panel of the output in extra memory: here the rows of a work-group
//    in LDS, or beyond 624 columns a chunk of rows multiplied into a scratch
//    panel and copied back.
//  * resid: column norms ||HX_j - lam_j X_j||.
//
// A grid of 4.04 rounds of resident work-groups takes as long as one of 5: the
// rotation's panel chunks are cut to whole rounds of them (CUs x work-groups per
// CU at the kernel's occupancy), the Gram splits to about four rounds of 512.
// Work-groups are dispatched to the 8 XCDs round-robin; the block index
// is remapped so that work-groups sharing operand rows (the tiles of one gram
// split, the column tiles of one rmul row tile) run on one XCD and share its
// L2.
#include "common.hpp"
#include "kernels.hpp"

#include <cmath>
#include <type_traits>

namespace chfsi {

static constexpr int GT = 128;  // output tile of the LDS gram kernel (4 waves x 64x64)

// Resident work-groups of `kern` (256 threads) on the current device.
template <typename K>
static int resident_slots(K kern) {
  int dev = 0, cus = 0, per = 0;
  (void)hipGetDevice(&dev);
  (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kern, 256, 0);
  return (cus > 0 ? cus : 1) * (per > 0 ? per : 1);
}

// Physical block index -> logical index such that the logical indices on one
// XCD (physical b = 8 i + x) are contiguous: XCD x holds [x*per + min(x, rem),
// ... + per + (x < rem)).
__device__ __forceinline__ int xcd_grouped_block() {
  const int g = (int)gridDim.x, b = (int)blockIdx.x;
  const int per = g >> 3, rem = g & 7, x = b & 7;
  return x * per + min(x, rem) + (b >> 3);
}

// lower-triangle tile enumeration t -> (ti, tj), ti >= tj
__device__ __forceinline__ void tri_tile(int t, int &ti, int &tj) {
  int i = (int)((sqrt(8.0 * t + 1.0) - 1.0) * 0.5);
  while ((i + 1) * (i + 2) / 2 <= t) ++i;
  while (i * (i + 1) / 2 > t) --i;
  ti = i;
  tj = t - i * (i + 1) / 2;
}

// acc += A[r0 : r1, ib + ...]^T B[r0 : r1, jb + ...], one wave's tile of F x F
// fragments, with products in CT.  Fragments are read straight from memory (16
// consecutive columns of four rows each), UN groups of four rows ahead in
// registers.  frag: the fragments to multiply (ALL: every one).  The last row of
// the matrix is read with its columns clamped to n; in the rows before it a
// fragment may run on into the next row, whose values only reach entries
// beyond n.
template <typename CT, int F, bool ALL, typename ACC>
__device__ __forceinline__ void gram_tile(const double *__restrict__ A, int64_t lda, const double *__restrict__ B,
                                          int64_t ldb, int64_t r0, int64_t r1, int64_t nrows, int n, int ib, int jb,
                                          unsigned frag, ACC (&acc)[F][F]) {
  constexpr int UN = F < 4 ? 4 : 2;
  const int lane = threadIdx.x & 63, j = lane & 15, kq = lane >> 4;
  auto multiply = [&](const double (&av)[F], const double (&bv)[F]) {
#pragma unroll
    for (int a = 0; a < F; ++a)
#pragma unroll
      for (int b = 0; b < F; ++b)
        if (ALL || (frag >> (a * F + b) & 1)) acc[a][b] = mfma16x4((CT)av[a], (CT)bv[b], acc[a][b]);
  };
  const int64_t rfast = r1 < nrows ? r1 : nrows - 1;
  const int nfast = rfast > r0 ? (int)((rfast - r0) / (4 * UN)) : 0;   // groups of 4 UN rows
  const double *pa = A + (r0 + kq) * lda + ib + j, *pb = B + (r0 + kq) * ldb + jb + j;
  if (nfast > 0) {
    double av[UN][F], bv[UN][F];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
#pragma unroll
      for (int a = 0; a < F; ++a) av[u][a] = pa[16 * a];
#pragma unroll
      for (int b = 0; b < F; ++b) bv[u][b] = pb[16 * b];
      pa += 4 * lda;
      pb += 4 * ldb;
    }
#pragma unroll 1
    for (int g = 1; g < nfast; ++g) {
      // keeps the work-group's waves, which share columns, within a few rows of
      // each other (every wave of it makes the same turns, or has ended)
      __builtin_amdgcn_s_barrier();
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        multiply(av[u], bv[u]);
#pragma unroll
        for (int a = 0; a < F; ++a) av[u][a] = pa[16 * a];
#pragma unroll
        for (int b = 0; b < F; ++b) bv[u][b] = pb[16 * b];
        pa += 4 * lda;
        pb += 4 * ldb;
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int u = 0; u < UN; ++u) multiply(av[u], bv[u]);
  }
#pragma unroll 1
  for (int64_t r = r0 + (int64_t)nfast * (4 * UN); r < r1; r += 4) {
    const bool rok = r + kq < r1;
    const int64_t row = rok ? r + kq : r1 - 1;
    double av[F], bv[F];
#pragma unroll
    for (int a = 0; a < F; ++a) {
      const int c = ib + 16 * a + j;
      const double v = A[row * lda + min(c, n - 1)];
      av[a] = rok ? v : 0.0;
    }
#pragma unroll
    for (int b = 0; b < F; ++b) {
      const int c = jb + 16 * b + j;
      const double v = B[row * ldb + min(c, n - 1)];
      bv[b] = rok ? v : 0.0;
    }
    multiply(av, bv);
  }
}

// G = A^T B over a split of the rows, lower triangle: one wave per 16F x 16F
// lower tile, NW tiles of one tile row (they share the columns of A in the CU's
// cache) to a work-group, no LDS.  An FP64 fragment product takes the matrix
// core 64 clocks against 2 / F loads, so that tiles can be small and little is
// computed beyond the triangle and the last column; the columns that tiles of
// one split share and the L2 no longer holds are the next bound (F = 2: slower
// than F = 3).  857,375 rows, against 128 x 128 tiles by four waves through LDS:
// n = 283, 2.74 -> 1.51 ms; n = 568, 7.4 -> 5.2 (53 TFLOP/s of what is asked, 73
// the card's matrix rate); n = 1,128, 21.7 -> 19.7; mixed 568, 7.1 -> 5.0.
// MIXED (the mixed overlap): FP64 in the diagonal tiles, FP32 inputs and
// products in the rest.
// Grid: nsplit x ceil(ntl / NW) work-groups, ntl lower tiles.
template <bool MIXED, int F, int NW>
__global__ __launch_bounds__(64 * NW, F == 3 ? 3 : 2) void gram_kernel(const double *__restrict__ A, int64_t lda,
                                                                       const double *__restrict__ B, int64_t ldb,
                                                                       int64_t nrows, int n, int ntl,
                                                                       int64_t rows_per_split,
                                                                       double *__restrict__ part) {
  constexpr int T = 16 * F;
  const int lane = threadIdx.x & 63, j = lane & 15, kq = lane >> 4;
  const int ngrid = (ntl + NW - 1) / NW;
  const int lid = xcd_grouped_block();
  const int split = lid / ngrid;
  const int t = __builtin_amdgcn_readfirstlane(NW * (lid - split * ngrid) + (int)(threadIdx.x >> 6));
  if (t >= ntl) return;
  int ti, tj;
  tri_tile(t, ti, tj);
  const int ib = ti * T, jb = tj * T;
  const int64_t r0 = (int64_t)split * rows_per_split;
  const int64_t r1 = r0 + rows_per_split < nrows ? r0 + rows_per_split : nrows;
  // the fragments with an entry that is read
  constexpr unsigned ALLF = (1u << (F * F)) - 1;
  unsigned frag = 0;
#pragma unroll
  for (int a = 0; a < F; ++a)
#pragma unroll
    for (int b = 0; b < F; ++b)
      if (ib + 16 * a < n && jb + 16 * b < n && ib + 16 * a >= jb + 16 * b) frag |= 1u << (a * F + b);
  frag = __builtin_amdgcn_readfirstlane(frag);
  double *out = part + ((int64_t)split * ntl + t) * (T * T);
  auto run = [&](auto ct) {
    typedef decltype(ct) CT;
    typename acc4<CT>::type acc[F][F];
#pragma unroll
    for (int a = 0; a < F; ++a)
#pragma unroll
      for (int b = 0; b < F; ++b) acc[a][b] = typename acc4<CT>::type{0, 0, 0, 0};
    if (frag == ALLF) gram_tile<CT, F, true>(A, lda, B, ldb, r0, r1, nrows, n, ib, jb, frag, acc);
    else gram_tile<CT, F, false>(A, lda, B, ldb, r0, r1, nrows, n, ib, jb, frag, acc);
#pragma unroll
    for (int a = 0; a < F; ++a)
#pragma unroll
      for (int b = 0; b < F; ++b)
#pragma unroll
        for (int q = 0; q < 4; ++q) out[(a * 16 + acc_row<CT>(kq, q)) * T + b * 16 + j] = (double)acc[a][b][q];
  };
  if (!MIXED || ti == tj) run(double{});
  else run(float{});
}

// The split projected Hamiltonian, whose FP32 part is bound by the columns read
// rather than the matrix cores: 128 x 128 tiles by four waves, so that a column
// read serves 128 others (857,375 x 1,128: 14.5 ms against 16.6 in wave tiles;
// 256: 1.31 against 1.70).
// One (split, lower tile) work-group: partial G tile over rows [r0, r1).  The
// contraction runs over chunks of 16 rows: the chunk's 128 columns of A and
// of B are loaded into registers one chunk ahead (16-byte loads when the
// leading dimensions are even), written to the other half of a
// double-buffered LDS area after the chunk's MFMAs, and published by one
// barrier per chunk.  Wave (wi, wj) owns the 64 x 64 quarter (wi, wj); on a
// diagonal tile the strictly upper quarter is never read and is skipped.
// FR false: every quarter outside the trailing block (rows and columns >=
// fr0, fr0 a multiple of 64) with FP32 inputs and products, the chunk staged in
// LDS already rounded to FP32.  FR true: the quarters inside it in FP64.
// Grid: nsplit x ntl work-groups.  FR false: ntl = all lower tiles.  FR true:
// the lower tiles of the trailing sub-triangle starting at tile row/column tf,
// part indexed within it.
template <int VEC, bool FR>
__global__ __launch_bounds__(256) void gram_split_kernel(const double *__restrict__ A, int64_t lda,
                                                   const double *__restrict__ B, int64_t ldb, int64_t nrows, int n,
                                                   int ntl, int tf, int64_t rows_per_split, int fr0,
                                                   double *__restrict__ part) {
  typedef double vec_t __attribute__((ext_vector_type(VEC)));
  typedef typename std::conditional<FR, double, float>::type CT;   // product type
  typedef typename acc4<CT>::type acc_t;
  typedef CT lds_vec_t __attribute__((ext_vector_type(VEC)));
  constexpr int KR = sizeof(CT) == 4 ? 32 : 16;   // rows per chunk (FP32 chunks: same LDS bytes)
  constexpr int PT = KR * GT / (256 * VEC);       // vectors per thread per operand
  // staged in the product type: FP32 modes round once, at the LDS store
  __shared__ __align__(16) CT As[2][KR][GT];
  __shared__ __align__(16) CT Bs[2][KR][GT];
  const int lid = xcd_grouped_block();
  const int split = lid / ntl;
  const int t = lid - split * ntl;                // part tile index
  int ti, tj;
  tri_tile(t, ti, tj);
  ti += tf;
  tj += tf;
  const int tid = threadIdx.x;
  const int wave = tid >> 6, lane = tid & 63;
  const int wi = wave >> 1, wj = wave & 1;
  const int j = lane & 15, kq = lane >> 4;
  auto quarter_active = [&](int qi, int qj) {
    // strictly upper quarters and quarters wholly past the last column are never read
    const bool inside = ti * GT + qi * 64 < n && tj * GT + qj * 64 < n;
    const bool lower = !(ti == tj && qi < qj);
    const bool in_fr = ti * GT + qi * 64 >= fr0 && tj * GT + qj * 64 >= fr0;
    return inside && lower && in_fr == FR;
  };
  if (!(quarter_active(0, 0) || quarter_active(1, 0) || quarter_active(0, 1) || quarter_active(1, 1)))
    return;                                        // whole work-group idle
  const bool active = quarter_active(wi, wj);
  const int64_t r0 = (int64_t)split * rows_per_split;
  int64_t r1 = r0 + rows_per_split;
  if (r1 > nrows) r1 = nrows;
  const int ib = ti * GT, jb = tj * GT;           // tile origin

  vec_t areg[PT], breg[PT];
  // slot v -> (row v / (GT/VEC), column vector v % (GT/VEC)); out-of-range
  // slots load a clamped in-bounds address and store zero
  auto load_chunk = [&](int64_t k0) {
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      const int v = tid + 256 * i;
      const int64_t row = min(k0 + v / (GT / VEC), r1 - 1);
      const int cv = (v % (GT / VEC)) * VEC;
      areg[i] = *reinterpret_cast<const vec_t *>(A + row * lda + min(ib + cv, n - VEC));
      breg[i] = *reinterpret_cast<const vec_t *>(B + row * ldb + min(jb + cv, n - VEC));
    }
  };
  auto store_chunk = [&](int buf, int64_t k0) {
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      const int v = tid + 256 * i;
      const int kr = v / (GT / VEC), cv = (v % (GT / VEC)) * VEC;
      const bool rok = k0 + kr < r1;
      lds_vec_t a, b;
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        a[e] = (rok && ib + cv + e < n) ? (CT)areg[i][e] : (CT)0;
        b[e] = (rok && jb + cv + e < n) ? (CT)breg[i][e] : (CT)0;
      }
      *reinterpret_cast<lds_vec_t *>(&As[buf][kr][cv]) = a;
      *reinterpret_cast<lds_vec_t *>(&Bs[buf][kr][cv]) = b;
    }
  };

  acc_t acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = acc_t{0, 0, 0, 0};
  const int64_t nk = (r1 - r0 + KR - 1) / KR;
  if (nk > 0) {
    load_chunk(r0);
    store_chunk(0, r0);
  }
  __syncthreads();
#pragma unroll 1
  for (int64_t kc = 0; kc < nk; ++kc) {
    const int buf = (int)(kc & 1);
    if (kc + 1 < nk) load_chunk(r0 + (kc + 1) * KR);
    if (active) {
#pragma unroll
      for (int ks = 0; ks < KR; ks += 4) {
        const int kk = ks + kq;
        CT av[4], bv[4];
#pragma unroll
        for (int a = 0; a < 4; ++a) av[a] = As[buf][kk][wi * 64 + a * 16 + j];
#pragma unroll
        for (int b = 0; b < 4; ++b) bv[b] = Bs[buf][kk][wj * 64 + b * 16 + j];
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int b = 0; b < 4; ++b) acc[a][b] = mfma16x4(av[a], bv[b], acc[a][b]);
      }
    }
    if (kc + 1 < nk) store_chunk(buf ^ 1, r0 + (kc + 1) * KR);
    __syncthreads();
  }
  if (!active) return;
  double *out = part + ((int64_t)split * ntl + t) * (GT * GT) + (wi * 64) * GT + wj * 64;
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        out[(a * 16 + acc_row<CT>(kq, q)) * GT + b * 16 + j] = (double)acc[a][b][q];
      }
}

// n <= 64: one 64 x 64 tile, so the tile kernel would leave three of its
// four waves idle.  Here the waves of a work-group share its rows instead,
// each takes every fourth group of four rows straight from memory into MFMA
// fragments (NA = ceil(n / 16) of them per operand, lower tiles only), and
// the four partial tiles are added in LDS in wave order.  13,824 and
// 24,389 rows of 32 columns: 6 us against 54.  Tall blocks gain as well: CholGS of
// 4.0M rows, this and the rotation by rows, n = 8 794 us against 2,392, n = 33 1,347
// against 3,802, n = 64 1,677 against 4,258.
template <int NA, bool SAME>
__global__ __launch_bounds__(256) void gram_small_kernel(const double *__restrict__ A, int64_t lda,
                                                         const double *__restrict__ B, int64_t ldb, int64_t nrows,
                                                         int n, int64_t rows_per_split, double *__restrict__ part) {
  constexpr int UN = 4;                              // row groups in flight
  __shared__ double red[16 * NA][16 * NA + 1];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int j = lane & 15, kq = lane >> 4;
  const int64_t r0 = (int64_t)blockIdx.x * rows_per_split;
  const int64_t r1 = r0 + rows_per_split < nrows ? r0 + rows_per_split : nrows;
  v4d acc[NA][NA];
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b <= a; ++b) acc[a][b] = v4d{0, 0, 0, 0};
  for (int64_t r = r0 + 4 * wave; r < r1; r += 16 * UN) {
    double av[UN][NA], bv[UN][NA];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int64_t row = r + 16 * u + kq;
#pragma unroll
      for (int a = 0; a < NA; ++a) {
        const bool ok = row < r1 && 16 * a + j < n;
        av[u][a] = ok ? A[row * lda + 16 * a + j] : 0.0;
        if (!SAME) bv[u][a] = ok ? B[row * ldb + 16 * a + j] : 0.0;
      }
    }
#pragma unroll
    for (int u = 0; u < UN; ++u)
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b <= a; ++b) acc[a][b] = mfma16x4(av[u][a], SAME ? av[u][b] : bv[u][b], acc[a][b]);
  }
  for (int w = 0; w < 4; ++w) {
    if (wave == w) {
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b <= a; ++b)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            double &d = red[16 * a + acc_row<double>(kq, q)][16 * b + j];
            d = w == 0 ? acc[a][b][q] : d + acc[a][b][q];
          }
    }
    __syncthreads();
  }
  double *out = part + (int64_t)blockIdx.x * (64 * 64);
  for (int e = threadIdx.x; e < 16 * NA * 16 * NA; e += 256) {
    const int i = e / (16 * NA), k = e % (16 * NA);
    if (k / 16 <= i / 16) out[i * 64 + k] = red[i][k];
  }
}

// G[i, j] = sum over splits of the partial gt x gt tiles, for i >= j in the
// region [r0, n) x [r0, n) (tiles numbered within the sub-triangle from tile
// row tf), mirrored to the upper triangle.  skip0 >= 0: leave out the entries
// with both i and j >= skip0 (written by another reduction).  A work-group
// adds 32 entries, each by eight threads that take every eighth split and are
// then added in order: one thread per entry left the chip waiting on the
// serial chain over the splits (6 tiles x 341 splits: 487 us; this: 38).
__global__ __launch_bounds__(256) void gram_reduce_kernel(const double *__restrict__ part, int nsplit, int ntl,
                                                          int gt, int n, int tf, int r0, int skip0,
                                                          double *__restrict__ G) {
  __shared__ double red[8][33];
  const int m = n - r0;
  const int64_t total = (int64_t)m * m;
  const int e = threadIdx.x & 31, sl = threadIdx.x >> 5;
  for (int64_t base = blockIdx.x * (int64_t)32; base < total; base += (int64_t)gridDim.x * 32) {
    const int64_t idx = base + e;
    const int i = r0 + (int)(idx / m), jj = r0 + (int)(idx - idx / m * m);
    const bool on = idx < total && jj <= i && !(skip0 >= 0 && jj >= skip0);
    double s = 0;
    if (on) {
      const int ti = i / gt - tf, tj = jj / gt - tf;
      const int t = ti * (ti + 1) / 2 + tj;
      const double *p = part + (int64_t)t * (gt * gt) + (i % gt) * gt + (jj % gt);
      const int64_t st = (int64_t)ntl * (gt * gt);
#pragma unroll 4
      for (int sp = sl; sp < nsplit; sp += 8) s += p[sp * st];
    }
    red[sl][e] = s;
    __syncthreads();
    if (sl == 0 && on) {
#pragma unroll
      for (int k = 1; k < 8; ++k) s += red[k][e];
      G[(int64_t)i * n + jj] = s;
      G[(int64_t)jj * n + i] = s;
    }
    __syncthreads();
  }
}

// Row splits: as many as fill four rounds of 512 work-groups with 128 x 128
// tiles, at least 256 rows each.  The count is that of 128-wide tiles whatever
// the kernel's are, so that the sums and the partial buffer do not depend on
// the tile chosen (48-wide tiles: 2.7 to 4 rounds of 768 work-groups).
static int gram_nsplit(int64_t nrows, int n) {
  const int64_t nt = (n + 127) / 128, ntl = nt * (nt + 1) / 2;
  int64_t want = 2048 / ntl;
  const int64_t maxs = (nrows + 255) / 256;
  if (want > maxs) want = maxs;
  if (want < 1) want = 1;
  return (int)want;
}

// Enough for a launch over the full triangle or over any trailing sub-triangle.
size_t gram_part_elems(int64_t nrows, int n) {
  size_t best = 0;
  for (int64_t m = 1; m <= (n + 127) / 128; ++m) {
    const size_t e = (size_t)gram_nsplit(nrows, (int)(m * 128)) * (m * (m + 1) / 2);
    if (e > best) best = e;
  }
  return best * 128 * 128;
}

static int64_t gram_rows_per_split(int64_t nrows, int nsplit) {
  int64_t rps = (nrows + nsplit - 1) / nsplit;
  return (rps + 15) / 16 * 16;
}

static void gram_reduce(const double *part, int nsplit, int ntl, int n, double *G, hipStream_t s, int gt, int tf = 0,
                        int r0 = 0, int skip0 = -1) {
  const int64_t m = n - r0;
  int64_t blocks = (m * m + 31) / 32;
  if (blocks > 65536) blocks = 65536;
  if (blocks < 1) return;
  hipLaunchKernelGGL(gram_reduce_kernel, dim3((unsigned)blocks), dim3(256), 0, s, part, nsplit, ntl, gt, n, tf, r0,
                     skip0, G);
}

// n <= 64 (mixed or not: the 64-wide diagonal block is FP64 either way).
// Splits of at least 128 rows, at most one per CU: never more than the partial
// tiles of the 128-tile kernel take.
static void gram_small(const double *A, int64_t lda, const double *B, int64_t ldb, int64_t nrows, int n, double *part,
                       size_t max_split, double *G, hipStream_t s) {
  int64_t nsplit = (nrows + 127) / 128;
  if (nsplit > 256) nsplit = 256;
  if (nsplit < 1) nsplit = 1;
  if (max_split > 0 && nsplit > (int64_t)max_split) nsplit = (int64_t)max_split;
  const int64_t rps = gram_rows_per_split(nrows, (int)nsplit);
  nsplit = (nrows + rps - 1) / rps;
  const dim3 g((unsigned)nsplit), b(256);
  const bool same = A == B && lda == ldb;
#define GRAM_SMALL(NA)                                                                                             \
  case NA:                                                                                                         \
    if (same) hipLaunchKernelGGL((gram_small_kernel<NA, true>), g, b, 0, s, A, lda, B, ldb, nrows, n, rps, part);  \
    else hipLaunchKernelGGL((gram_small_kernel<NA, false>), g, b, 0, s, A, lda, B, ldb, nrows, n, rps, part);      \
    break;
  switch ((n + 15) / 16) {
    GRAM_SMALL(1) GRAM_SMALL(2) GRAM_SMALL(3) GRAM_SMALL(4)
  }
#undef GRAM_SMALL
  gram_reduce(part, (int)nsplit, 1, n, G, s, 64);
}

static bool gram_v16(const double *A, int64_t lda, const double *B, int64_t ldb, int n) {
  return lda % 2 == 0 && ldb % 2 == 0 && n % 2 == 0 && ((uintptr_t)A % 16) == 0 && ((uintptr_t)B % 16) == 0;
}

template <bool FR>
static void gram_split_part(bool v16, int nsplit, const double *A, int64_t lda, const double *B, int64_t ldb,
                            int64_t nrows, int n, int ntl, int tf, int fr0, double *part, hipStream_t s) {
  const dim3 grid((unsigned)(nsplit * ntl));
  const int64_t rps = gram_rows_per_split(nrows, nsplit);
  if (v16)
    hipLaunchKernelGGL((gram_split_kernel<2, FR>), grid, dim3(256), 0, s, A, lda, B, ldb, nrows, n, ntl, tf, rps, fr0,
                       part);
  else
    hipLaunchKernelGGL((gram_split_kernel<1, FR>), grid, dim3(256), 0, s, A, lda, B, ldb, nrows, n, ntl, tf, rps, fr0,
                       part);
}

template <bool MIXED, int F, int NW>
static int gram_tiles(const double *A, int64_t lda, const double *B, int64_t ldb, int64_t nrows, int n,
                      double *part, size_t part_elems, double *G, hipStream_t s) {
  constexpr int T = 16 * F;
  const int nt = (n + T - 1) / T, ntl = nt * (nt + 1) / 2, nwg = (ntl + NW - 1) / NW;
  int64_t nsplit = gram_nsplit(nrows, n);
  const int64_t fit = (int64_t)((part_elems > 0 ? part_elems : gram_part_elems(nrows, n)) / ((size_t)ntl * T * T));
  if (fit < 1) return -1;
  if (nsplit > fit) nsplit = fit;
  const int64_t rps = gram_rows_per_split(nrows, (int)nsplit);
  nsplit = (nrows + rps - 1) / rps;
  hipLaunchKernelGGL((gram_kernel<MIXED, F, NW>), dim3((unsigned)(nsplit * nwg)), dim3(64 * NW), 0, s, A, lda, B, ldb, nrows, n,
                     ntl, rps, part);
  gram_reduce(part, (int)nsplit, ntl, n, G, s, T);
  return 0;
}

void gram_launch(const double *A, int64_t lda, const double *B, int64_t ldb, int64_t nrows, int n, double *part,
                 double *G, int mixed, hipStream_t s) {
  gram_launch_capped(A, lda, B, ldb, nrows, n, part, 0, G, mixed, s);
}

int gram_launch_capped(const double *A, int64_t lda, const double *B, int64_t ldb, int64_t nrows, int n,
                       double *part, size_t part_elems, double *G, int mixed, hipStream_t s) {
  if (n <= 64) {
    if (part_elems > 0 && part_elems < 64 * 64) return -1;
    gram_small(A, lda, B, ldb, nrows, n, part, part_elems / (64 * 64), G, s);
    return 0;
  }
  if (mixed) return gram_tiles<true, 4, 8>(A, lda, B, ldb, nrows, n, part, part_elems, G, s);
  // 48-wide tiles by fours or 64-wide ones by eights: up to 800 columns by the
  // fragments they compute, the idle waves of the last work-group included
  // (857,375 rows: n = 568, 720 against 768, 5.2 and 6.3 ms; n = 640, 972 against
  // 896, 6.7 and 6.2), beyond that the wide ones, which read less (n = 1,128: 22.0
  // and 19.7 ms)
  const int nt3 = (n + 47) / 48, nt4 = (n + 63) / 64;
  const int wg3 = (nt3 * (nt3 + 1) / 2 + 3) / 4, wg4 = (nt4 * (nt4 + 1) / 2 + 7) / 8;
  if (n > 800 || wg4 * 8 * 16 < wg3 * 4 * 9) return gram_tiles<false, 4, 8>(A, lda, B, ldb, nrows, n, part, part_elems, G, s);
  return gram_tiles<false, 3, 4>(A, lda, B, ldb, nrows, n, part, part_elems, G, s);
}

void gram_split_launch(const double *A, int64_t lda, const double *B, int64_t ldb, int64_t nrows, int n, double *part,
                       double *G, int fr0, hipStream_t s) {
  fr0 = fr0 / 64 * 64;
  if (fr0 == 0) {
    gram_launch(A, lda, B, ldb, nrows, n, part, G, 0, s);
    return;
  }
  const bool v16 = gram_v16(A, lda, B, ldb, n);
  // the trailing block in FP64, on a grid over its own sub-triangle of tiles
  // (so that the few tiles it touches get every row split), reduced first
  const int nt = (n + GT - 1) / GT, tf = fr0 / GT, m = nt - tf, ntl4 = m * (m + 1) / 2;
  const int nsplit4 = gram_nsplit(nrows, m * GT);
  gram_split_part<true>(v16, nsplit4, A, lda, B, ldb, nrows, n, ntl4, tf, fr0, part, s);
  gram_reduce(part, nsplit4, ntl4, n, G, s, GT, tf, fr0);
  // everything else with FP32 inputs and products; part is reused in order
  const int ntl = nt * (nt + 1) / 2, nsplit = gram_nsplit(nrows, n);
  gram_split_part<false>(v16, nsplit, A, lda, B, ldb, nrows, n, ntl, 0, fr0, part, s);
  gram_reduce(part, nsplit, ntl, n, G, s, GT, 0, 0, fr0);
}

// ---------------------------------------------------------------------------
// Right multiplication X <- X W.  Rows are processed in chunks: an LDS-tiled
// MFMA GEMM writes C = X_chunk W into a scratch chunk, a coalesced copy puts
// it back (the paper's outer blocking over rows, which needs only a chunk of
// extra memory).  Work-group tile 128 x 128 (4 waves x 64 x 64); the
// contraction runs over chunks of 16: the X chunk (128 rows x 16, stored
// transposed so a fragment read is 16 consecutive words) and the W chunk
// (16 x 128) are loaded into registers one chunk ahead (16-byte loads when
// the leading dimensions are even), written to the other half of a
// double-buffered LDS area after the chunk's MFMAs, and published by one
// barrier per chunk.  upper: W upper triangular, so output column tile
// [n0, n0+128) only needs k < n0 + 128.  mixed (upper only): k in the
// 64-wide diagonal block of a wave's columns in FP64, smaller k in FP32.
// ---------------------------------------------------------------------------
static constexpr int MT = 128, NTL = 128, KC = 16;

// C[r, 0:nout] = X[row0 + r, 0:n] W[0:n, 0:nout] (W row stride ldw)
template <bool MIXED, int VEC>
__global__ __launch_bounds__(256) void rmul_gemm_kernel(const double *__restrict__ X, int64_t ld, int64_t row0,
                                                        int64_t nrows, int n, const double *__restrict__ W,
                                                        int64_t ldw, int nout, int upper, double *__restrict__ C,
                                                        int64_t ldc) {
  typedef double vec_t __attribute__((ext_vector_type(VEC)));
  constexpr int APT = KC * MT / (256 * VEC);     // X vectors per thread per chunk
  constexpr int WPT = KC * NTL / (256 * VEC);    // W vectors per thread per chunk
  __shared__ __align__(16) double As[2][KC][MT];   // As[k][row]
  __shared__ __align__(16) double Ws[2][KC][NTL];  // Ws[k][col]
  const int nt = (nout + NTL - 1) / NTL;
  const int lid = xcd_grouped_block();
  const int mt = lid / nt;
  const int ntile = lid - mt * nt;
  const int64_t r0 = row0 + (int64_t)mt * MT;    // first X row of this tile
  const int64_t rlast = row0 + nrows - 1;         // last valid row
  const int n0 = ntile * NTL;
  const int tid = threadIdx.x;
  const int wave = tid >> 6, lane = tid & 63;
  const int wi = wave >> 1, wj = wave & 1;
  const int j = lane & 15, kq = lane >> 4;
  const int kend = upper ? min(n, n0 + NTL) : n;
  const int c0 = n0 + wj * 64;                   // first column of this wave
  const bool live = c0 < nout;                   // a wave wholly past nout skips its MFMAs
  const int kdiag = MIXED ? (c0 / 64) * 64 : 0;  // mixed: k >= kdiag is the FP64 diagonal block

  // staging slots: X vector v -> (row v % MT, k-vector v / MT); W vector v ->
  // (k-row v / (NTL/VEC), column vector v % (NTL/VEC)).  Out-of-range slots
  // load a clamped in-bounds address and store zero.
  vec_t areg[APT], wreg[WPT];
  auto load_chunk = [&](int k0) {
#pragma unroll
    for (int i = 0; i < APT; ++i) {
      const int v = tid + 256 * i;
      const int64_t row = min(r0 + v % MT, rlast);
      const int k = min(k0 + (v / MT) * VEC, n - VEC);
      areg[i] = *reinterpret_cast<const vec_t *>(X + row * ld + k);
    }
#pragma unroll
    for (int i = 0; i < WPT; ++i) {
      const int v = tid + 256 * i;
      const int k = min(k0 + v / (NTL / VEC), n - 1);
      const int col = min(n0 + (v % (NTL / VEC)) * VEC, nout - VEC);
      wreg[i] = *reinterpret_cast<const vec_t *>(W + (int64_t)k * ldw + col);
    }
  };
  auto store_chunk = [&](int buf, int k0) {
#pragma unroll
    for (int i = 0; i < APT; ++i) {
      const int v = tid + 256 * i;
      const int r = v % MT, kv = (v / MT) * VEC;
      const bool rok = r0 + r <= rlast;
#pragma unroll
      for (int e = 0; e < VEC; ++e) As[buf][kv + e][r] = (rok && k0 + kv + e < n) ? areg[i][e] : 0.0;
    }
#pragma unroll
    for (int i = 0; i < WPT; ++i) {
      const int v = tid + 256 * i;
      const int kr = v / (NTL / VEC), cv = (v % (NTL / VEC)) * VEC;
      vec_t w = wreg[i];
      const bool kok = k0 + kr < kend;
#pragma unroll
      for (int e = 0; e < VEC; ++e) w[e] = (kok && n0 + cv + e < nout) ? w[e] : 0.0;
      *reinterpret_cast<vec_t *>(&Ws[buf][kr][cv]) = w;
    }
  };

  // one pipeline step: prefetch chunk kc + 1, multiply chunk kc, publish
  // chunk kc + 1.  F32: FP32 inputs and products into acc32.
  const int nk = (kend + KC - 1) / KC;
  auto step = [&](int kc, auto f32, auto &accs) {
    const int buf = kc & 1;
    if (kc + 1 < nk) load_chunk((kc + 1) * KC);
#pragma unroll
    for (int ks = 0; ks < KC && live; ks += 4) {
      const int kk = ks + kq;
      double av[4], bv[4];
#pragma unroll
      for (int a = 0; a < 4; ++a) av[a] = As[buf][kk][wi * 64 + a * 16 + j];
#pragma unroll
      for (int b = 0; b < 4; ++b) bv[b] = Ws[buf][kk][wj * 64 + b * 16 + j];
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          if constexpr (decltype(f32)::value)
            accs[a][b] = mfma16x4((float)av[a], (float)bv[b], accs[a][b]);
          else
            accs[a][b] = mfma16x4(av[a], bv[b], accs[a][b]);
        }
    }
    if (kc + 1 < nk) store_chunk(buf ^ 1, (kc + 1) * KC);
    __syncthreads();
  };

  load_chunk(0);
  store_chunk(0, 0);
  __syncthreads();
  v4d acc[4][4];
  int kc = 0;
  if constexpr (MIXED) {
    // chunks left of the wave's diagonal block in FP32 (kdiag is a multiple
    // of 64, so chunks never straddle it), then the FP64 accumulators start
    // from the converted FP32 sums
    const int nk32 = min(kdiag / KC, nk);
    v4f acc32[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) acc32[a][b] = v4f{0, 0, 0, 0};
#pragma unroll 1
    for (; kc < nk32; ++kc) step(kc, std::true_type{}, acc32);
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) acc[a][b] = f32acc_to_f64_layout(acc32[a][b], lane);
  } else {
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) acc[a][b] = v4d{0, 0, 0, 0};
  }
#pragma unroll 1
  for (; kc < nk; ++kc) step(kc, std::false_type{}, acc);
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int64_t rr = (int64_t)mt * MT + wi * 64 + a * 16 + acc_row<double>(kq, q);  // chunk-local row
        const int col = c0 + b * 16 + j;
        if (rr < nrows && col < nout) C[rr * ldc + col] = acc[a][b][q];
      }
}

// X <- X W by whole rows, without the panel: a work-group copies RB rows into LDS
// (18 loads in flight per thread), and its waves then take blocks of 16 NA rows
// x 16 columns of the result, the longest sums first when W is triangular, and
// write them over the rows just read, which no other work-group needs.  X
// fragments come from LDS; W, which all work-groups share in the L2, is read
// straight into fragments 16 rows ahead.  The waves draw the next block from a
// counter, so that SIMDs with the shorter ones do more of them.  A triangular
// product computes no more than it needs but for 16 columns, and the panel's
// write, read and copy are gone: 857,375 rows, n = 32, 223 -> 152 us; n = 283,
// 3.77 -> 2.27 ms (full W 4.74 -> 3.60); n = 568, 8.92 -> 6.64 ms.  Bound by the
// matrix cores at n > 100 (two thirds busy), by the rows' traffic below.  64
// rows to a block (NA = 4, half the reads of W): 2 to 10 % slower.
// CAP: doubles of LDS; S = ceil16(n) + 2 is the row stride there (2 mod 4: the
// 32 lanes of half a fragment read different banks).
template <bool MIXED, int CAP, int NW, int NA>
__global__ __launch_bounds__(64 * NW, NW == 16 ? 4 : 2) void rmul_rows_kernel(double *X, int64_t ld, int64_t nrows, int n,
                                                                               const double *__restrict__ W,
                                                                               int64_t ldw, int upper, int RB) {
  constexpr int UN = 4, RU = 16 * NA;
  __shared__ double Xs[CAP];
  __shared__ int next;
  if (threadIdx.x == 0) next = NW;
  const int n16 = (n + 15) / 16 * 16, S = n16 + 2;
  const int lane = threadIdx.x & 63, j = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t row0 = (int64_t)blockIdx.x * RB;
  // rows r = wave, wave + NW, ... in chunks of 64 columns, LB chunks in flight
  constexpr int LB = 18;
  const int nch = (n16 + 63) / 64, items = RB / NW * nch;
  for (int i0 = 0; i0 < items; i0 += LB) {
    double v[LB];
#pragma unroll
    for (int u = 0; u < LB; ++u) {
      const int i = min(i0 + u, items - 1), r = wave + i / nch * NW, k = i % nch * 64 + lane;
      v[u] = X[(row0 + r < nrows ? row0 + r : nrows - 1) * ld + min(k, n - 1)];
    }
#pragma unroll
    for (int u = 0; u < LB; ++u) {
      const int i = i0 + u, r = wave + i / nch * NW, k = i % nch * 64 + lane;
      if (i < items && k < n16) Xs[r * S + k] = row0 + r < nrows && k < n ? v[u] : 0.0;
    }
  }
  __syncthreads();
  const int ncb = (n + 15) / 16, units = ncb * (RB / RU);
  for (int o = wave; o < units;) {
    const int rg = o % (RB / RU), cb = ncb - 1 - o / (RB / RU);
    int taken = 0;                                 // the unit after this one
    if (lane == 0) taken = atomicAdd(&next, 1);
    o = __builtin_amdgcn_readfirstlane(taken);
    if (row0 + RU * rg >= nrows) continue;
    const int c0 = 16 * cb;
    const int kend = upper ? min(n, c0 + 16) : n, ngr = (kend + 15) / 16;
    const double *xs = Xs + (RU * rg + j) * S + kq;
    const int col = min(c0 + j, n - 1);
    double w[UN];
    auto load = [&](int g, int u) {                // rows of group g, all below n
      const double *p = W + (int64_t)(16 * g + 4 * u + kq) * ldw;
      w[u] = p[col];
    };
    auto load_last = [&](int g, int u) {
      const double *p = W + (int64_t)min(16 * g + 4 * u + kq, n - 1) * ldw;
      w[u] = p[col];
    };
    auto multiply = [&](int g, int u, auto &acc) {
      const int k = 16 * g + 4 * u;
#pragma unroll
      for (int a = 0; a < NA; ++a) {
        const double x = xs[16 * a * S + k];
        if constexpr (sizeof(acc[0]) == sizeof(v4f)) acc[a] = mfma16x4((float)x, (float)w[u], acc[a]);
        else acc[a] = mfma16x4(x, w[u], acc[a]);
      }
    };
    // groups [g0, g1), the rows of group g0 in w; afterwards those of g1 if g1 < ngr
    auto groups = [&](int g0, int g1, auto &acc) {
      int g = g0;
#pragma unroll 1
      for (; g < g1 && g + 2 < ngr; ++g)
#pragma unroll
        for (int u = 0; u < UN; ++u) {
          multiply(g, u, acc);
          load(g + 1, u);
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll 1
      for (; g < g1; ++g)
#pragma unroll
        for (int u = 0; u < UN; ++u) {
          multiply(g, u, acc);
          if (g + 1 < ngr) load_last(g + 1, u);
        }
    };
#pragma unroll
    for (int u = 0; u < UN; ++u) load_last(0, u);
    v4d acc[NA];
#pragma unroll
    for (int a = 0; a < NA; ++a) acc[a] = v4d{0, 0, 0, 0};
    int g0 = 0;
    if constexpr (MIXED) {
      g0 = min(c0 / 64 * 4, ngr);
      v4f acc32[NA];
#pragma unroll
      for (int a = 0; a < NA; ++a) acc32[a] = v4f{0, 0, 0, 0};
      groups(0, g0, acc32);
#pragma unroll
      for (int a = 0; a < NA; ++a) acc[a] = f32acc_to_f64_layout(acc32[a], lane);
    }
    groups(g0, ngr, acc);
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int64_t row = row0 + RU * rg + 16 * a + acc_row<double>(kq, q);
        const int c = c0 + j;
        if (row < nrows && c < n) X[row * ld + c] = acc[a][q];
      }
  }
}

__global__ __launch_bounds__(256) void copy_back_kernel(const double *__restrict__ C, int64_t ldc, double *X,
                                                        int64_t ld, int64_t row0, int64_t nrows, int n,
                                                        int col0) {
  const int64_t total = nrows * (int64_t)n;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = t / n;
    const int c = (int)(t - r * n);
    X[(row0 + r) * ld + col0 + c] = C[r * ldc + c];
  }
}

size_t rmul_scratch_elems(int64_t nrows, int n) {
  // at most 1 GiB, and no more than the whole product needs
  const int64_t cap = (int64_t)1 << 27;
  const int64_t all = (nrows + MT - 1) / MT * MT * (int64_t)(n > 0 ? n : 1);
  int64_t e = all < cap ? all : cap;
  if (e < (int64_t)MT * n) e = (int64_t)MT * n;
  return (size_t)e;
}

// Columns up to which 32 rows fit in LDS.
static constexpr int ROWS_MAXN = 624;

template <bool MIXED>
static void rmul_rows_launch(double *X, int64_t ld, int64_t nrows, int n, const double *W, int64_t ldw, int upper,
                             hipStream_t s) {
  const int S = (n + 15) / 16 * 16 + 2;
  auto go = [&](auto kern, int threads, int RB) {
    hipLaunchKernelGGL(kern, dim3((unsigned)((nrows + RB - 1) / RB)), dim3(threads), 0, s, X, ld, nrows, n, W, ldw, upper,
                       RB);
  };
  // four work-groups to a CU up to 144 columns, two up to 304, then one
  if (S <= 34) go(rmul_rows_kernel<MIXED, 5100, 4, 2>, 256, 128);
  else if (S <= 78) go(rmul_rows_kernel<MIXED, 5100, 4, 2>, 256, 64);
  else if (S <= 158) go(rmul_rows_kernel<MIXED, 5100, 4, 2>, 256, 32);
  else if (S <= 316) go(rmul_rows_kernel<MIXED, 10200, 8, 2>, 512, 32);
  else go(rmul_rows_kernel<MIXED, 20400, 16, 2>, 1024, 32);
}

int rmul_cols_launch(double *X, int64_t ld, int64_t nrows, int n, const double *W, int64_t ldw, int nout,
                     int out_col0, int upper, int mixed, double *scratch, size_t scratch_elems, hipStream_t s) {
  if (mixed && !upper) return -1;
  if (upper && (nout != n || ldw != n)) return -1;
  if (n <= 0 || nout <= 0 || nrows <= 0) return 0;
  if (scratch_elems < (size_t)MT * nout) return -1;
  // whole rows in LDS while they fit; a product of fewer columns than X has
  // too few blocks for a work-group's waves there (857,375 x 283 -> 35 columns:
  // 1.65 ms against 1.05 in tiles)
  if (n <= ROWS_MAXN && nout == n && out_col0 == 0) {
    if (mixed) rmul_rows_launch<true>(X, ld, nrows, n, W, ldw, upper, s);
    else rmul_rows_launch<false>(X, ld, nrows, n, W, ldw, upper, s);
    return 0;
  }
  const int nt = (nout + NTL - 1) / NTL;
  // row tiles per launch: as many as the scratch panel holds, rounded down to
  // whole rounds of resident work-groups when there is more than one round
  const int64_t mts_all = (nrows + MT - 1) / MT;
  int64_t mts_chunk = (int64_t)(scratch_elems / nout) / MT;
  if (mts_chunk < mts_all) {
    const int64_t slots = mixed ? resident_slots(rmul_gemm_kernel<true, 2>) : resident_slots(rmul_gemm_kernel<false, 2>);
    const int64_t rounds = mts_chunk * nt / slots;
    if (rounds >= 1) mts_chunk = rounds * slots / nt;
  } else {
    mts_chunk = mts_all;
  }
  if (mts_chunk < 1) mts_chunk = 1;
  const int64_t chunk = mts_chunk * MT;
  // 16-byte operand loads need even leading dimensions and 16-byte aligned bases
  const bool v16 = ld % 2 == 0 && n % 2 == 0 && ldw % 2 == 0 && nout % 2 == 0 && ((uintptr_t)X % 16) == 0 &&
                   ((uintptr_t)W % 16) == 0;
  for (int64_t r = 0; r < nrows; r += chunk) {
    const int64_t rows = (nrows - r < chunk) ? nrows - r : chunk;
    const int64_t mts = (rows + MT - 1) / MT;
    const dim3 grid((unsigned)(mts * nt)), block(256);
    const int64_t ldc = nout;
    if (mixed) {
      if (v16) hipLaunchKernelGGL((rmul_gemm_kernel<true, 2>), grid, block, 0, s, X, ld, r, rows, n, W, ldw, nout, upper, scratch, ldc);
      else hipLaunchKernelGGL((rmul_gemm_kernel<true, 1>), grid, block, 0, s, X, ld, r, rows, n, W, ldw, nout, upper, scratch, ldc);
    } else {
      if (v16) hipLaunchKernelGGL((rmul_gemm_kernel<false, 2>), grid, block, 0, s, X, ld, r, rows, n, W, ldw, nout, upper, scratch, ldc);
      else hipLaunchKernelGGL((rmul_gemm_kernel<false, 1>), grid, block, 0, s, X, ld, r, rows, n, W, ldw, nout, upper, scratch, ldc);
    }
    int64_t total = rows * nout;
    int64_t blocks = (total + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(copy_back_kernel, dim3((unsigned)blocks), dim3(256), 0, s, scratch, ldc, X, ld, r, rows, nout,
                       out_col0);
  }
  return 0;
}

int rmul_launch(double *X, int64_t ld, int64_t nrows, int n, const double *W, int upper, int mixed,
                double *scratch, size_t scratch_elems, hipStream_t s) {
  return rmul_cols_launch(X, ld, nrows, n, W, n, n, 0, upper, mixed, scratch, scratch_elems, s);
}

int rmul_out_launch(const double *X, int64_t ld, int64_t nrows, int n, const double *W, int64_t ldw, int nout,
                    double *C, int64_t ldc, hipStream_t s) {
  if (n <= 0 || nout <= 0 || nrows <= 0) return 0;
  const bool v16 = ld % 2 == 0 && n % 2 == 0 && ldw % 2 == 0 && nout % 2 == 0 && ((uintptr_t)X % 16) == 0 &&
                   ((uintptr_t)W % 16) == 0;
  const int nt = (nout + NTL - 1) / NTL;
  const int64_t mts = (nrows + MT - 1) / MT;
  if (mts * nt > INT32_MAX) return -1;
  const dim3 grid((unsigned)(mts * nt)), block(256);
  if (v16) hipLaunchKernelGGL((rmul_gemm_kernel<false, 2>), grid, block, 0, s, X, ld, 0, nrows, n, W, ldw, nout, 0, C, ldc);
  else hipLaunchKernelGGL((rmul_gemm_kernel<false, 1>), grid, block, 0, s, X, ld, 0, nrows, n, W, ldw, nout, 0, C, ldc);
  return 0;
}

// ---------------------------------------------------------------------------
// Nodal electron density (Alg. 5, eq. elecDensSP with the collocated GLL
// rule): rho_j = 2 minv_j^2 (sum_i X[j,i]^2 + sum_k w_k Xfr[j,k]^2), w_k =
// f(eps_k, mu) - 1.  One wave per DoF row (a row is contiguous in the
// DoF-major layout, so a wave's loads are coalesced), lanes over columns with
// 16-byte loads where the layout allows, a fixed shuffle tree for the sum.
// HBM-bound: 8 (ncols + nfr) + 16 bytes per DoF.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

template <bool V2, bool F2>
__global__ __launch_bounds__(256) void density_kernel(const double *__restrict__ X, int64_t ld, int ncols,
                                                      const double *__restrict__ Xfr, int64_t ldfr, int nfr,
                                                      const double *__restrict__ w, const double *__restrict__ minv,
                                                      int64_t nrows, double *__restrict__ rho) {
  typedef double d2 __attribute__((ext_vector_type(2)));
  const int lane = threadIdx.x & 63;
  const int64_t wid = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int64_t stride = (int64_t)gridDim.x * 4;
  for (int64_t row = wid; row < nrows; row += stride) {
    const double *xr = X + row * ld;
    double s0 = 0, s1 = 0;
    if (V2) {
      // two 16-byte loads per lane per step (a deeper unroll measured slower)
      int c = 2 * lane;
      for (; c + 128 < ncols; c += 256) {
        const d2 a = *reinterpret_cast<const d2 *>(xr + c);
        const d2 b = *reinterpret_cast<const d2 *>(xr + c + 128);
        s0 += a[0] * a[0] + a[1] * a[1];
        s1 += b[0] * b[0] + b[1] * b[1];
      }
      if (c < ncols) {
        const d2 a = *reinterpret_cast<const d2 *>(xr + c);
        s0 += a[0] * a[0] + a[1] * a[1];
      }
    } else {
      for (int c = lane; c < ncols; c += 64) {
        const double v = xr[c];
        s0 += v * v;
      }
    }
    const double *fr = Xfr + row * ldfr;
    if (F2) {
      for (int c = 2 * lane; c < nfr; c += 128) {
        const d2 v = *reinterpret_cast<const d2 *>(fr + c);
        const d2 wk = *reinterpret_cast<const d2 *>(w + c);
        s1 += wk[0] * (v[0] * v[0]) + wk[1] * (v[1] * v[1]);
      }
    } else {
      for (int c = lane; c < nfr; c += 64) {
        const double v = fr[c];
        s1 += w[c] * (v * v);
      }
    }
    const double tot = wave_sum(s0 + s1);
    if (lane == 0) {
      const double m = minv[row];
      rho[row] = 2.0 * (m * m) * tot;
    }
  }
}

void density_launch(const double *X, int64_t ld, int ncols, const double *Xfr, int64_t ldfr, int nfr,
                    const double *w, const double *minv, int64_t nrows, double *rho, hipStream_t s) {
  if (nrows <= 0) return;
  int64_t blocks = (nrows + 3) / 4;
  if (blocks > 8192) blocks = 8192;
  const dim3 g((unsigned)blocks), b(256);
  const bool v2 = ld % 2 == 0 && ncols % 2 == 0 && ((uintptr_t)X % 16) == 0;
  const bool f2 = nfr > 0 && ldfr % 2 == 0 && nfr % 2 == 0 && ((uintptr_t)Xfr % 16) == 0 && ((uintptr_t)w % 16) == 0;
  if (v2 && f2) hipLaunchKernelGGL((density_kernel<true, true>), g, b, 0, s, X, ld, ncols, Xfr, ldfr, nfr, w, minv, nrows, rho);
  else if (v2) hipLaunchKernelGGL((density_kernel<true, false>), g, b, 0, s, X, ld, ncols, Xfr, ldfr, nfr, w, minv, nrows, rho);
  else if (f2) hipLaunchKernelGGL((density_kernel<false, true>), g, b, 0, s, X, ld, ncols, Xfr, ldfr, nfr, w, minv, nrows, rho);
  else hipLaunchKernelGGL((density_kernel<false, false>), g, b, 0, s, X, ld, ncols, Xfr, ldfr, nfr, w, minv, nrows, rho);
}

// ---------------------------------------------------------------------------
// Residual column norms
// ---------------------------------------------------------------------------
// Work-group = a chunk of rows x CW columns, 256 / CW threads to a column, four
// rows in flight each, added in LDS in order.  Partial sums are stored column
// by column, part[c * nchunk + chunk], so that one wave adds a column's with
// coalesced loads.  (One thread per column and 1024 rows each took 304 us for
// 32 columns of some 20,000 rows, where eight threads now share a column: 7 us;
// 283 columns of 493,039 rows 1,020 against 571 us, memory-bound now.)
template <int CW>
__global__ __launch_bounds__(256) void resid_part_kernel(const double *__restrict__ X, int64_t ldx,
                                                         const double *__restrict__ HX, int64_t ldh,
                                                         const double *__restrict__ lam, int64_t nrows, int n,
                                                         int64_t rows_per, int nchunk, double *__restrict__ part) {
  constexpr int RL = 256 / CW;
  __shared__ double red[256];
  const int cl = threadIdx.x % CW, rl = threadIdx.x / CW;
  const int c = blockIdx.y * CW + cl;
  const int64_t r0 = (int64_t)blockIdx.x * rows_per;
  const int64_t r1 = r0 + rows_per < nrows ? r0 + rows_per : nrows;
  double acc = 0;
  if (c < n) {
    const double l = lam[c];
#pragma unroll 4
    for (int64_t r = r0 + rl; r < r1; r += RL) {
      const double d = HX[r * ldh + c] - l * X[r * ldx + c];
      acc += d * d;
    }
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  if (rl == 0 && c < n) {
#pragma unroll
    for (int k = 1; k < RL; ++k) acc += red[k * CW + cl];
    part[(int64_t)c * nchunk + blockIdx.x] = acc;
  }
}

// one wave per column
__global__ __launch_bounds__(256) void resid_reduce_kernel(const double *__restrict__ part, int nchunk, int n,
                                                           double *__restrict__ out) {
  const int c = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (c >= n) return;
  double s = 0;
  for (int k = lane; k < nchunk; k += 64) s += part[(int64_t)c * nchunk + k];
  s = wave_sum(s);
  if (lane == 0) out[c] = sqrt(s);
}

int resid_nchunk(int64_t nrows) {
  int64_t c = (nrows + 255) / 256;
  if (c > 2048) c = 2048;
  if (c < 1) c = 1;
  return (int)c;
}

void resid_launch(const double *X, int64_t ldx, const double *HX, int64_t ldh, const double *lam, int64_t nrows,
                  int n, double *part, double *resid, hipStream_t s) {
  const int nchunk = resid_nchunk(nrows);
  const int64_t rows_per = (nrows + nchunk - 1) / nchunk;
  if (n <= 32)
    hipLaunchKernelGGL((resid_part_kernel<32>), dim3(nchunk), dim3(256), 0, s, X, ldx, HX, ldh, lam, nrows, n, rows_per,
                       nchunk, part);
  else if (n > 512)                                // whole lines of a row at a time: 4,019,679 x 1,128 12.3 against 13.1 ms
    hipLaunchKernelGGL((resid_part_kernel<256>), dim3(nchunk, (n + 255) / 256), dim3(256), 0, s, X, ldx, HX, ldh, lam,
                       nrows, n, rows_per, nchunk, part);
  else
    hipLaunchKernelGGL((resid_part_kernel<64>), dim3(nchunk, (n + 63) / 64), dim3(256), 0, s, X, ldx, HX, ldh, lam, nrows,
                       n, rows_per, nchunk, part);
  hipLaunchKernelGGL(resid_reduce_kernel, dim3((n + 3) / 4), dim3(256), 0, s, part, nchunk, n, resid);
}

}  // namespace chfsi
