// Electrostatics: the discrete Poisson problem (Sec. 2.4 eq.
// phiTotDiscreteSolve) with homogeneous Dirichlet conditions, solved by the
// Jacobi-preconditioned conjugate-gradient method the paper uses for it
// (Sec. 3.2, matrix-free operator).
//
//   A phi = f,  A = 1/(4 pi) int grad N_i . grad N_j,  f = M rho + point charges.
//
// On the uniform Cartesian GLL mesh the assembled stiffness is the Kronecker
// sum k (+) k (+) k weighted by the diagonal 1D masses:
//   (A x)(I,J,K) = s [ m_J m_K sum_I' k(I,I') x(I',J,K) + m_I m_K sum_J' k(J,J') x(I,J',K)
//                    + m_I m_J sum_K' k(K,K') x(I,J,K') ],   s = 1/(4 pi),
// k the assembled 1D Laplacian stiffness (band half-width p), m the 1D GLL
// mass.  This is the matrix-free operator in its assembled form, applied cell by
// cell in one pass over x and y (16 bytes per DoF).
//
// One CG iteration is three launches: the product fused with the partial
// p.q; z -= alpha q / diag(A) with the partials of r.z and r.r; x += alpha p and
// the new direction p = z + beta p.  The two global sums each iteration needs
// are formed where they are used: every work-group of the update sums the
// product's partials (alpha = r.z / p.q), every work-group of the direction
// pass sums the update's (beta = r.z' / r.z and the stop test r.r <=
// tol^2 f.f), each in the same fixed order, so all work-groups hold the same
// bits.  Work-group 0 keeps the results for later launches: r.z alternates
// between two slots by iteration parity, so no work-group reads the slot its
// own launch writes; the stop count, which every work-group of the same
// launch also reads, can only change from "never" to this iteration's number
// plus one, and both values let iteration it run.  The residual is kept as z =
// r / diag(A), which the direction pass reads as it is; diag(A) itself is
// recomputed in the update, from 1D values, and an iteration moves ten arrays
// of n_dof values and the partials (24^3 cells of degree 6, which the last-level cache holds:
// 20 + 15 + 19 us and 2 us between launches; 32 + 19 + 27 and 4 before, with the band
// stencil, a third of the lanes idle in rows of 143, and r / diag(A) formed in
// both vector passes).  The
// iteration that meets the tolerance records its number; launches of later
// iterations return at once, so the host launches iterations in groups and
// reads that number between groups.  (Forming p inside the product, where
// the stencil reads it, saves the direction pass but reads two arrays at
// every halo point: measured 2.3x slower per product.  Summing partials in
// the last work-group of each grid instead, every work-group's device-scope
// release writes back its L2: slower still.)
#include "common.hpp"
#include "ctx.hpp"
#include "kernels.hpp"

#include <algorithm>
#include <cmath>
#include <map>
#include <vector>

namespace chfsi {

static constexpr int PB = 256;              // threads per work-group
static constexpr int PR = 1024;             // threads of the single-work-group reductions
static constexpr int MAXG = 2048;           // element-wise grids: at most this many work-groups (grid-stride)
// scalars: r.z of the last two iterations (slot by parity), r.r, f.f, the
// stop threshold tol^2 f.f, the number of iterations done when the tolerance
// was met (kNever until then), alpha of the last update
enum { S_RZ = 0, S_RR = 2, S_FF, S_STOP, S_STOPAT, S_ALPHA, S_NSCAL };
static constexpr double kNever = 9.0e15;

// Sum over the work-group in a fixed order (butterfly within each wave, then
// the wave sums in wave order), so every work-group that sums the same
// values gets the same bits.
template <int NT = PB>
__device__ __forceinline__ double block_sum(double v, double *sh) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) s += sh[w];
  __syncthreads();
  return s;
}

// The centrosymmetric table T(k, l) = (2 / h) K1(k, l) / m(k) of a cell, m the
// assembled 1D mass (a vertex's on both ends): row k of A's 1D part divided by
// the mass, so that a node's sum over the three directions is multiplied by
// s m_I m_J m_K once.
template <int P> struct CellTable {
  static constexpr int N = ((P + 1) * (P + 1) + 1) / 2;
  double t[N];
  __device__ __forceinline__ double operator()(int k, int l) const {
    const int i = k * (P + 1) + l, r = (P + 1) * (P + 1) - 1 - i;
    return t[i < r ? i : r];
  }
};

// y = A x by cells.  A wave takes 64 consecutive I and half of the P rows J of
// one cell (all of them up to P = 3), and marches over the planes K of its cell
// layers.  The y- and z-direction sums of a cell are its small dense table times
// the values in registers (8 products per node where a band row has 2 P + 1),
// the sums of a layer's P + 1 planes are held until the layer is complete, and
// what they owe the next layer's first plane is carried on.  The x-direction
// band goes through LDS, a strip per wave: no barriers.  Planes are loaded one
// ahead, as buffers whose range ends with the plane: what lies outside the mesh
// reads as zero (no branch, no address arithmetic per plane) and is not written.
// It is bound by instructions, not by memory: 24^3 cells of degree 6, 32 -> 20
// us per product (a whole cell per wave: 26, too few waves to hide the chains).  DOT: part[work-group] = its share of x . y.
// Grid: ceil(n / 64) ceil(n_el / cells per work-group) ceil(n_el / zl)
// work-groups (1D, XCD-grouped).
static constexpr unsigned OFF_OUT = 0x80000000u;   // beyond any plane
template <int P> struct StencilSplit {
  static constexpr int H = P < 4 ? 1 : 2;          // waves per cell
  static constexpr int RM = (P + H - 1) / H;       // rows of the first
  static constexpr int CELLS = 4 / H;              // cells per work-group, along y
};

// the wave's rows [R0, R1) of cell cy, layers [L0, L1); returns its share of x . y
template <int P, int R0, int R1, bool DOT>
__device__ __forceinline__ double stencil_march(const double *__restrict__ x, double *__restrict__ y,
                                                const double *__restrict__ kbs, const double *__restrict__ m,
                                                const CellTable<P> &T, int n, int n_el, double s, int I0, int cy, int L0,
                                                int L1, double *st) {
  constexpr int R = R1 - R0, BW = 2 * P + 1, WX = 64 + 2 * P, HL = (2 * P * R + 63) / 64;
  constexpr bool LOW = R0 == 0;                    // the vertex row also belongs to the cell before
  typedef unsigned u2_t __attribute__((ext_vector_type(2)));
  const int lane = threadIdx.x & 63;
  const int I = I0 + lane;
  const bool ilive = I < n, live = cy < n_el;
  const unsigned pbytes = (unsigned)n * (unsigned)n * 8u;
  // offsets in a plane: the cell's rows, the rows of the cell before
  auto row_off = [&](int i, int node) {
    return live && i >= 0 && i < n && node >= 1 && node <= n ? (unsigned)(i + n * (node - 1)) * 8u : OFF_OUT;
  };
  unsigned oo[P + 1], ol[P], ox[HL];
  int ex[HL];                                      // strip slots of the x-direction halo (-1: none)
#pragma unroll
  for (int r = 0; r <= P; ++r) oo[r] = row_off(I, cy * P + r);
#pragma unroll
  for (int r = 0; r < P; ++r) ol[r] = row_off(I, (cy - 1) * P + r);
#pragma unroll
  for (int u = 0; u < HL; ++u) {
    const int e = lane + 64 * u, r = e / (2 * P), c = e % (2 * P);
    const int slot = c < P ? c : 64 + c;
    ex[u] = e < 2 * P * R ? r * WX + slot : -1;
    ox[u] = e < 2 * P * R ? row_off(I0 - P + slot, cy * P + R0 + r) : OFF_OUT;
  }
  double kx[BW];
#pragma unroll
  for (int d = 0; d < BW; ++d) kx[d] = ilive ? kbs[(int64_t)I * BW + d] : 0.0;
  const double wI = ilive ? s * m[I] : 0.0;
  auto plane_of = [&](const double *v, int node) {  // the plane of a node, empty outside the mesh
    const bool in = node >= 1 && node <= n;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<double *>(v + (int64_t)(in ? node - 1 : 0) * n * n), 0,
                                             in ? (int)pbytes : 0, 0x00020000);
  };
  auto ld = [&](__amdgpu_buffer_rsrc_t r, unsigned off) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0));
  };
  double acc[P + 1][R];
#pragma unroll
  for (int r = 0; r < R; ++r) acc[P][r] = 0;
  double vn[P + 1], ln[P], xn[HL];                 // the plane ahead
  auto fetch = [&](int node) {
    const auto rp = plane_of(x, node);
#pragma unroll
    for (int r = 0; r <= P; ++r) vn[r] = ld(rp, oo[r]);
    if constexpr (LOW) {
#pragma unroll
      for (int r = 0; r < P; ++r) ln[r] = ld(rp, ol[r]);
    }
#pragma unroll
    for (int u = 0; u < HL; ++u) xn[u] = ld(rp, ox[u]);
  };
  fetch(L0 * P);
  // what the layer before owes the first plane
  if (L0 > 0) {
    double pv[P][R];
#pragma unroll
    for (int k = 0; k < P; ++k) {
      const auto rp = plane_of(x, (L0 - 1) * P + k);
#pragma unroll
      for (int r = 0; r < R; ++r) pv[k][r] = ld(rp, oo[R0 + r]);
    }
#pragma unroll
    for (int k = 0; k < P; ++k)
#pragma unroll
      for (int r = 0; r < R; ++r) acc[P][r] = __builtin_fma(T(P, k), pv[k][r], acc[P][r]);
  }
#pragma unroll
  for (int r = 0; r < R; ++r) asm volatile("" : "+v"(acc[P][r]));
  double dot = 0;
#pragma unroll 1
  for (int L = L0; L < L1; ++L) {
#pragma unroll
    for (int k = 0; k < P; ++k) {
      double v[P + 1], ty[R];
#pragma unroll
      for (int r = 0; r <= P; ++r) v[r] = vn[r];
#pragma unroll
      for (int r = 0; r < R; ++r) st[r * WX + P + lane] = v[R0 + r];
      if constexpr (LOW) {
        ty[0] = T(0, 0) * v[0];                    // the cell before: its last row is this vertex row
#pragma unroll
        for (int d = 0; d < P; ++d) ty[0] = __builtin_fma(T(P, d), ln[d], ty[0]);
      }
#pragma unroll
      for (int u = 0; u < HL; ++u)
        if (ex[u] >= 0) st[ex[u]] = xn[u];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      fetch(L * P + k + 1);
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int d = 0; d <= P; ++d)
          ty[r] = d == 0 && !(LOW && r == 0) ? T(R0 + r, d) * v[d] : __builtin_fma(T(R0 + r, d), v[d], ty[r]);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        double tx = kx[P] * v[R0 + r];
#pragma unroll
        for (int d = 0; d < BW; ++d)
          if (d != P) tx = __builtin_fma(kx[d], st[r * WX + lane + d], tx);
        const double t = tx + ty[r], vr = v[R0 + r];
        if (k == 0) {
          acc[0][r] = __builtin_fma(2.0 * T(0, 0), vr, acc[P][r] + t);
#pragma unroll
          for (int l = 1; l <= P; ++l) acc[l][r] = T(l, 0) * vr;
        } else {
#pragma unroll
          for (int l = 0; l <= P; ++l) acc[l][r] = __builtin_fma(T(l, k), vr, l == k ? acc[l][r] + t : acc[l][r]);
        }
      }
      // the sums are formed here, not put off to their use at the layer's end
      // (which would keep every operand until then)
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int l = 0; l <= P; ++l) asm volatile("" : "+v"(acc[l][r]));
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_sched_barrier(0);
    }
    // the layer's planes are complete with the first plane of the next, in vn
#pragma unroll
    for (int k = 0; k < P; ++k) {
      const int node = L * P + k;
      const auto ry = plane_of(y, node), rp = plane_of(x, node);
      const double wK = node >= 1 ? wI * m[node - 1] : 0.0;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int jn = cy * P + R0 + r;
        const double wJ = live && jn >= 1 ? m[jn - 1] : 0.0;
        const double q = wK * wJ * __builtin_fma(T(k, P), vn[R0 + r], acc[k][r]);
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2_t, q), ry, (int)oo[R0 + r], 0, 0);
        if constexpr (DOT) dot = __builtin_fma(ld(rp, oo[R0 + r]), q, dot);
      }
    }
  }
  return dot;
}

template <int P, bool DOT>
__global__ __launch_bounds__(PB, 2) void poisson_stencil_kernel(const double *__restrict__ x, double *__restrict__ y,
                                                                const double *__restrict__ kbs,
                                                                const double *__restrict__ m, CellTable<P> T, int n,
                                                                int n_el, int zl, double s,
                                                                const double *__restrict__ scal, int it,
                                                                double *__restrict__ part) {
  typedef StencilSplit<P> SP;
  __shared__ double sh[PB / 64];
  __shared__ double strip[4][SP::RM][64 + 2 * P];
  if (DOT && it >= scal[S_STOPAT]) return;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // XCD-grouped block order: the hardware deals consecutive work-groups to the
  // 8 XCDs in turn; the logical index below is contiguous per XCD
  const int g = (int)gridDim.x, b = (int)blockIdx.x;
  const int lid = (b & 7) * (g >> 3) + min(b & 7, g & 7) + (b >> 3);
  const int gx = (n + 63) / 64, gy = (n_el + SP::CELLS - 1) / SP::CELLS;
  const int I0 = lid % gx * 64, cy = lid / gx % gy * SP::CELLS + w / SP::H, L0 = lid / (gx * gy) * zl;
  const int L1 = min(L0 + zl, n_el);
  double dot;
  if (SP::H == 1 || (w & 1) == 0)
    dot = stencil_march<P, 0, SP::RM, DOT>(x, y, kbs, m, T, n, n_el, s, I0, cy, L0, L1, &strip[w][0][0]);
  else
    dot = stencil_march<P, SP::RM % P, P, DOT>(x, y, kbs, m, T, n, n_el, s, I0, cy, L0, L1, &strip[w][0][0]);
  if constexpr (DOT) {
    const double bsum = block_sum(dot, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = bsum;
  }
}

// The two vector passes run over the values in memory order, VU per thread 256
// apart: every lane works whatever n is.  The loads of the partials a pass sums
// are issued first, then all of its values', so the global sum is formed while
// they are in flight.  Every work-group reads every partial, so their number is
// bounded: beyond MAXG blocks of values (4.2M) a work-group takes several (MORE), as
// many as the others (us per iteration, one block each against so: 9.9M values 190
// against 170, 59.8M 2,396 against 1,215; up to 4.2M the loop costs 2 to 3 %, 57.2
// against 55.6 at 2.9M, and is left out).
constexpr int VU = 8, VBLOCK = PB * VU;
constexpr int PU = 4;   // partials per thread loaded ahead (the rest, if any, after)
static dim3 vec_grid(int64_t nd) {
  const int64_t blocks = (nd + VBLOCK - 1) / VBLOCK, each = (blocks + MAXG - 1) / MAXG;
  return dim3((unsigned)((blocks + each - 1) / each));
}
// (I, J, K) of a value, and of the one 256 further on
struct NodePos {
  int I, J, K;
  __device__ __forceinline__ NodePos(int64_t base, int off, int n) {
    const int64_t row = base / n;                  // wave-uniform
    const int i = (int)(base - row * n) + off, j = i / n;
    I = i - j * n;
    K = (int)(row / n);
    J = (int)(row - (int64_t)K * n) + j;
    wrap(n);
  }
  __device__ __forceinline__ void wrap(int n) {
    if (J >= n) {
      const int k = J / n;
      K += k;
      J -= k * n;
    }
  }
  __device__ __forceinline__ void advance(int n, int dI, int dJ) {
    I += dI;
    J += dJ;
    if (I >= n) {
      I -= n;
      ++J;
    }
    wrap(n);
  }
};
// diag(A) at (I, J, K): s m_I m_J m_K (a_I + a_J + a_K), a = k_II / m_I after m
__device__ __forceinline__ double diag_at(const double *m, int n, double s, int I, int J, int K) {
  const double *a = m + n;
  return s * m[I] * m[J] * m[K] * (a[I] + a[J] + a[K]);
}
// Sum of a[0 .. na) in a fixed order, in two steps: parts_load issues the
// thread's first PU loads, parts_sum adds them, then the rest, then sums over
// the work-group.
__device__ __forceinline__ void parts_load(const double *__restrict__ a, int na, double (&v)[PU]) {
#pragma unroll
  for (int u = 0; u < PU; ++u) {
    const int i = (int)threadIdx.x + u * PB;
    v[u] = i < na ? a[i] : 0.0;
  }
}
__device__ __forceinline__ double parts_sum(const double *__restrict__ a, int na, const double (&v)[PU],
                                            double *sh) {
  double t = 0;
#pragma unroll
  for (int u = 0; u < PU; ++u) t += v[u];
  for (int i = (int)threadIdx.x + PU * PB; i < na; i += PB) t += a[i];
  return block_sum(t, sh);
}

// Iteration it: alpha = r.z / p.q from the product's partials (work-group 0
// keeps it for the direction pass); z -= alpha q / diag(A), the residual r =
// diag(A) z not being stored; partials of r.z and r.r.
template <bool MORE>
__global__ __launch_bounds__(PB) void poisson_update_kernel(double *__restrict__ z, const double *__restrict__ q,
                                                            const double *__restrict__ m, int n, int64_t nd, double s,
                                                            double *__restrict__ scal, int it,
                                                            const double *__restrict__ part_pq, int npq,
                                                            double *__restrict__ part_rz, double *__restrict__ part_rr) {
  extern __shared__ double mt[];                   // m and a
  __shared__ double sh[PB / 64];
  if (it >= scal[S_STOPAT]) return;
  double pp[PU];
  parts_load(part_pq, npq, pp);
  for (int i = (int)threadIdx.x; i < 2 * n; i += PB) mt[i] = m[i];
  double zv[VU], qv[VU];
  auto load = [&](int64_t base) {
    const int left = nd - base < VBLOCK ? (int)(nd - base) : VBLOCK;
    const double *zb = z + base, *qb = q + base;
#pragma unroll
    for (int u = 0; u < VU; ++u) {
      const int e = (int)threadIdx.x + PB * u;
      zv[u] = e < left ? zb[e] : 0.0;
      qv[u] = e < left ? qb[e] : 0.0;
    }
  };
  int64_t base = (int64_t)blockIdx.x * VBLOCK;
  load(base);
  NodePos at(base, (int)threadIdx.x, n);
  const int dJ = PB / n, dI = PB - dJ * n;
  const double pq = parts_sum(part_pq, npq, pp, sh);
  const double alpha = pq != 0 ? scal[S_RZ + (it & 1)] / pq : 0.0;
  if (blockIdx.x == 0 && threadIdx.x == 0) scal[S_ALPHA] = alpha;
  double rz = 0, rr = 0;
  for (;;) {
    const int left = nd - base < VBLOCK ? (int)(nd - base) : VBLOCK;
    double *zb = z + base;
#pragma unroll
    for (int u = 0; u < VU; ++u) {
      const int e = (int)threadIdx.x + PB * u;
      if (e < left) {
        const double d = diag_at(mt, n, s, at.I, at.J, at.K);
        // 1 / d to an ulp: the hardware estimate and two Newton steps
        double y = __builtin_amdgcn_rcp(d);
        y = fma(fma(-d, y, 1.0), y, y);
        y = fma(fma(-d, y, 1.0), y, y);
        const double v = zv[u] - alpha * (qv[u] * y), r = d * v;
        zb[e] = v;
        rz += r * v;
        rr += r * r;
      }
      at.advance(n, dI, dJ);
    }
    if (!MORE) break;
    base += (int64_t)gridDim.x * VBLOCK;
    if (base >= nd) break;
    load(base);
    at = NodePos(base, (int)threadIdx.x, n);
  }
  const double a = block_sum(rz, sh);
  const double b = block_sum(rr, sh);
  if (threadIdx.x == 0) {
    part_rz[blockIdx.x] = a;
    part_rr[blockIdx.x] = b;
  }
}

// Iteration it: r.z' and r.r from the update's partials; x += alpha p (the
// update's alpha); unless r.r meets the tolerance, p = z + beta p, beta = r.z' /
// r.z.  Work-group 0 keeps r.z' (the other parity slot), r.r, and the iteration
// count once the tolerance is met.
template <bool MORE>
__global__ __launch_bounds__(PB) void poisson_dir_kernel(double *__restrict__ x, double *__restrict__ pv,
                                                         const double *__restrict__ z, int64_t nd,
                                                         double *__restrict__ scal, int it,
                                                         const double *__restrict__ part_rz,
                                                         const double *__restrict__ part_rr, int nparts) {
  __shared__ double sh[PB / 64];
  if (it >= scal[S_STOPAT]) return;
  double pz[PU], pr[PU];
  parts_load(part_rz, nparts, pz);
  parts_load(part_rr, nparts, pr);
  const double alpha = scal[S_ALPHA], rz_old = scal[S_RZ + (it & 1)], stop = scal[S_STOP];
  double pw[VU], zw[VU];
  auto load_and_add = [&](int64_t base) {            // p and z of a block; x += alpha p
    const int left = nd - base < VBLOCK ? (int)(nd - base) : VBLOCK;
    double *xb = x + base, *pb = pv + base;
    const double *zb = z + base;
    double xw[VU];
#pragma unroll
    for (int u = 0; u < VU; ++u) {
      const int e = (int)threadIdx.x + PB * u;
      pw[u] = e < left ? pb[e] : 0.0;
      xw[u] = e < left ? xb[e] : 0.0;
      zw[u] = e < left ? zb[e] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < VU; ++u) {
      const int e = (int)threadIdx.x + PB * u;
      if (e < left) xb[e] = fma(alpha, pw[u], xw[u]);
    }
  };
  int64_t base = (int64_t)blockIdx.x * VBLOCK;
  load_and_add(base);
  const double rz = parts_sum(part_rz, nparts, pz, sh);
  const double rr = parts_sum(part_rr, nparts, pr, sh);
  const bool last = rr <= stop;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    scal[S_RZ + ((it + 1) & 1)] = rz;
    scal[S_RR] = rr;
    if (last) scal[S_STOPAT] = it + 1;
  }
  if (!MORE && last) return;
  const double beta = rz_old != 0 ? rz / rz_old : 0.0;
  for (;;) {
    if (!MORE || !last) {
      const int left = nd - base < VBLOCK ? (int)(nd - base) : VBLOCK;
      double *pb = pv + base;
#pragma unroll
      for (int u = 0; u < VU; ++u) {
        const int e = (int)threadIdx.x + PB * u;
        if (e < left) pb[e] = fma(beta, pw[u], zw[u]);
      }
    }
    if (!MORE) break;
    base += (int64_t)gridDim.x * VBLOCK;
    if (base >= nd) break;
    load_and_add(base);
  }
}

// Setup: r = f - A x (q = A x given), z = p = r / diag(A); partials of r.z, r.r
// and f.f.
__global__ __launch_bounds__(PB) void poisson_init_kernel(const double *__restrict__ f, const double *__restrict__ q,
                                                          double *__restrict__ z, double *__restrict__ pv,
                                                          const double *__restrict__ m, int n, double s,
                                                          double *__restrict__ part_rz, double *__restrict__ part_rr,
                                                          double *__restrict__ part_ff) {
  __shared__ double sh[PB];
  const int64_t nd = (int64_t)n * n * n;
  double rz = 0, rr = 0, ff = 0;
  for (int64_t idx = (int64_t)blockIdx.x * PB + threadIdx.x; idx < nd; idx += (int64_t)gridDim.x * PB) {
    const double fv = f[idx];
    const double rv = fv - q[idx];
    const int I = (int)(idx % n), J = (int)((idx / n) % n), K = (int)(idx / ((int64_t)n * n));
    const double zv = rv / diag_at(m, n, s, I, J, K);
    z[idx] = zv;
    pv[idx] = zv;
    rz += rv * zv;
    rr += rv * rv;
    ff += fv * fv;
  }
  const double a = block_sum(rz, sh);
  const double b = block_sum(rr, sh);
  const double c = block_sum(ff, sh);
  if (threadIdx.x == 0) {
    part_rz[blockIdx.x] = a;
    part_rr[blockIdx.x] = b;
    part_ff[blockIdx.x] = c;
  }
}

// f = M rho, M = 1 / minv^2
__global__ __launch_bounds__(PB) void poisson_rhs_kernel(const double *__restrict__ rho,
                                                         const double *__restrict__ minv, double *__restrict__ f,
                                                         int64_t nd) {
  for (int64_t idx = (int64_t)blockIdx.x * PB + threadIdx.x; idx < nd; idx += (int64_t)gridDim.x * PB)
    f[idx] = rho[idx] / (minv[idx] * minv[idx]);
}

// point charges on their nodes (distinct dofs)
__global__ __launch_bounds__(PB) void poisson_charges_kernel(double *__restrict__ f, const int64_t *__restrict__ dofs,
                                                             const double *__restrict__ q, int nq) {
  const int i = blockIdx.x * PB + threadIdx.x;
  if (i < nq) f[dofs[i]] += q[i];
}

// Setup sums in a fixed order: r.z (the slot of iteration 0), r.r, f.f; the
// stop threshold tol^2 f.f and the stop count (0 when the initial guess
// already meets the tolerance).
__global__ __launch_bounds__(PR) void poisson_setup_reduce_kernel(const double *__restrict__ a,
                                                                  const double *__restrict__ b,
                                                                  const double *__restrict__ c, int nparts,
                                                                  double tol2, double *__restrict__ scal) {
  __shared__ double sh[PR];
  double sa = 0, sb = 0, sc = 0;
  for (int i = threadIdx.x; i < nparts; i += PR) {
    sa += a[i];
    sb += b[i];
    sc += c[i];
  }
  sa = block_sum<PR>(sa, sh);
  sb = block_sum<PR>(sb, sh);
  sc = block_sum<PR>(sc, sh);
  if (threadIdx.x == 0) {
    scal[S_RZ] = sa;
    scal[S_RZ + 1] = 0.0;
    scal[S_RR] = sb;
    scal[S_FF] = sc;
    scal[S_STOP] = tol2 * sc;
    scal[S_ALPHA] = 0.0;
    scal[S_STOPAT] = sb <= tol2 * sc ? 0.0 : kNever;
  }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
// 1D Laplacian stiffness (band, half-width p, each row over its mass) and GLL mass
// on the interior nodes.  A band entry of two nodes of one element is that
// element's; an element end's diagonal is twice its half.
static void poisson_tables(const MeshTables &M, std::vector<double> &kb, std::vector<double> &m1) {
  const int p = M.p, q = M.q, n = M.n, bw = 2 * p + 1;
  kb.assign((size_t)n * bw, 0.0);
  m1.resize(2 * (size_t)n);                        // the mass, then the band's diagonal over it
  for (int i = 0; i < n; ++i) {
    const int e = (i + 1) / p, a = (i + 1) % p;    // node a of element e
    m1[i] = M.m1[a];
    auto put = [&](int row, int b, int node) {     // entry (row, b) of an element, b at grid node `node`
      const int j = node - 1;
      if (j >= 0 && j < n) kb[(size_t)i * bw + (j - i) + p] += M.km[(size_t)row * q + b];
    };
    for (int b = 0; b <= p; ++b) {
      put(a, b, e * p + b);
      if (a == 0) put(p, b, (e - 1) * p + b);
    }
    m1[n + i] = kb[(size_t)i * bw + p];
  }
}

static int poisson_ready(chfsi_ctx *c) {
  if (!c) return CHFSI_ERR_ARG;
  if (c->device < 0) return fail(c, CHFSI_ERR_STATE, "host-only context: no device work");
  if (!c->has_mesh) return fail(c, CHFSI_ERR_STATE, "poisson: set_mesh first");
  if (c->mesh.periodic)
    return fail(c, CHFSI_ERR_STATE, "poisson: the periodic cell needs a neutral charge (not supported)");
  if (int r = set_dev(c)) return r;
  const MeshTables &M = c->mesh;
  if (c->pois_n != M.n || c->pois_p != M.p || c->pois_h != M.h) {
    std::vector<double> kb, m1;
    poisson_tables(M, kb, m1);
    HIPCHK(c, c->pois_kb.ensure(kb.size() * sizeof(double)));
    HIPCHK(c, c->pois_m.ensure(m1.size() * sizeof(double)));
    HIPCHK(c, hipMemcpyAsync(c->pois_kb.p, kb.data(), kb.size() * sizeof(double), hipMemcpyHostToDevice, c->stream));
    HIPCHK(c, hipMemcpyAsync(c->pois_m.p, m1.data(), m1.size() * sizeof(double), hipMemcpyHostToDevice, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    c->pois_n = M.n;
    c->pois_p = M.p;
    c->pois_h = M.h;
  }
  return 0;
}

static const double kInv4Pi = 0.079577471545947667884;   // 1 / (4 pi)

// Work-groups of the stencil at zl cell layers each.  Two layers save the reads
// of the one before (24^3 cells of degree 6: 19.6 against 21.1 us; 32^3 of degree
// 5: 19.4 against 21.4) where that leaves 400 work-groups, the 256 CUs' worth and
// some (20^3 of degree 7, 300: 28.3 against 27.0; 12^3 of degree 6: 12.1 against
// 8.0).
static int64_t stencil_groups(int n, int n_el, int p, int zl) {
  const int cells = p < 4 ? StencilSplit<1>::CELLS : StencilSplit<4>::CELLS;
  return (int64_t)((n + 63) / 64) * ((n_el + cells - 1) / cells) * ((n_el + zl - 1) / zl);
}
static int stencil_zl(int n, int n_el, int p) { return stencil_groups(n, n_el, p, 2) >= 400 ? 2 : 1; }
static dim3 apply_grid(const MeshTables &M) {
  return dim3((unsigned)stencil_groups(M.n, M.n_el, M.p, stencil_zl(M.n, M.n_el, M.p)));
}

// y = A x; with part (and scal, it): the partials of x . y for iteration it
// (skipped once the solve has stopped).  -1 for an unsupported degree.
template <int P>
static void poisson_stencil_go(const MeshTables &M, const double *x, double *y, const double *kbs, const double *m,
                               const double *scal, int it, double *part, hipStream_t s) {
  CellTable<P> T;
  for (int i = 0; i < CellTable<P>::N; ++i) T.t[i] = M.km[i];
  const dim3 g = apply_grid(M), b(PB);
  const int zl = stencil_zl(M.n, M.n_el, M.p);
  if (part)
    hipLaunchKernelGGL((poisson_stencil_kernel<P, true>), g, b, 0, s, x, y, kbs, m, T, M.n, M.n_el, zl, kInv4Pi, scal,
                       it, part);
  else
    hipLaunchKernelGGL((poisson_stencil_kernel<P, false>), g, b, 0, s, x, y, kbs, m, T, M.n, M.n_el, zl, kInv4Pi,
                       nullptr, 0, nullptr);
}
static int poisson_stencil_launch(const MeshTables &M, const double *x, double *y, const double *kbs, const double *m,
                                  const double *scal, int it, double *part, hipStream_t s) {
  switch (M.p) {
    case 1: poisson_stencil_go<1>(M, x, y, kbs, m, scal, it, part, s); return 0;
    case 2: poisson_stencil_go<2>(M, x, y, kbs, m, scal, it, part, s); return 0;
    case 3: poisson_stencil_go<3>(M, x, y, kbs, m, scal, it, part, s); return 0;
    case 4: poisson_stencil_go<4>(M, x, y, kbs, m, scal, it, part, s); return 0;
    case 5: poisson_stencil_go<5>(M, x, y, kbs, m, scal, it, part, s); return 0;
    case 6: poisson_stencil_go<6>(M, x, y, kbs, m, scal, it, part, s); return 0;
    case 7: poisson_stencil_go<7>(M, x, y, kbs, m, scal, it, part, s); return 0;
    default: return -1;
  }
}

}  // namespace chfsi

using namespace chfsi;

extern "C" int chfsi_poisson_apply(chfsi_ctx *c, const double *x, double *y) {
  if (int r = poisson_ready(c)) return r;
  if (!x || !y || x == y) return fail(c, CHFSI_ERR_ARG, "poisson_apply: x and y must be separate device arrays");
  if (poisson_stencil_launch(c->mesh, x, y, c->pois_kb.as<double>(), c->pois_m.as<double>(), nullptr, 0, nullptr,
                             c->stream))
    return fail(c, CHFSI_ERR_ARG, "poisson_apply: degree p must be in 1..7");
  HIPCHK(c, hipGetLastError());
  return 0;
}

extern "C" int chfsi_poisson_solve(chfsi_ctx *c, const double *rho, int ncharges, const int64_t *charge_dofs,
                                   const double *charges, double *phi, double tol, int max_iter, int *iters,
                                   double *rel_resid) {
  if (int r = poisson_ready(c)) return r;
  const MeshTables &M = c->mesh;
  const int64_t nd = M.n_dof;
  if (!rho || !phi || !(tol > 0) || max_iter < 0 || ncharges < 0 || (ncharges > 0 && (!charge_dofs || !charges)))
    return fail(c, CHFSI_ERR_ARG, "poisson_solve: bad arguments");
  if (M.p < 1 || M.p > 7) return fail(c, CHFSI_ERR_ARG, "poisson_solve: degree p must be in 1..7");
  // point charges: combined per node on the host, so the device adds each once
  std::map<int64_t, double> qmap;
  for (int i = 0; i < ncharges; ++i) {
    if (charge_dofs[i] < 0 || charge_dofs[i] >= nd || !std::isfinite(charges[i]))
      return fail(c, CHFSI_ERR_ARG, "poisson_solve: charge dof out of range or non-finite charge");
    qmap[charge_dofs[i]] += charges[i];
  }
  const int64_t nb = std::min<int64_t>((nd + PB - 1) / PB, MAXG);   // element-wise grids (grid-stride)
  const int64_t nv = vec_grid(nd).x;                 // the two vector passes
  const bool more = nv * VBLOCK < nd;
  const dim3 ga = apply_grid(M);
  const int64_t na = (int64_t)ga.x * ga.y * ga.z;  // product grid
  const int64_t npart = std::max(std::max(nb, na), nv);
  // workspace: f, z, p, q (nd each), partials (3 npart), scalars
  HIPCHK(c, c->pois_work.ensure((size_t)(4 * nd + 3 * npart + S_NSCAL) * sizeof(double)));
  double *f = c->pois_work.as<double>(), *z = f + nd, *pv = z + nd, *q = pv + nd;
  double *pa = q + nd, *pb = pa + npart, *pc = pb + npart, *scal = pc + npart;
  const double *kbs = c->pois_kb.as<double>(), *m = c->pois_m.as<double>();
  const dim3 grid((unsigned)nb), block(PB);
  hipStream_t s = c->stream;
  hipLaunchKernelGGL(poisson_rhs_kernel, grid, block, 0, s, rho, c->minv64.as<double>(), f, nd);
  if (!qmap.empty()) {
    std::vector<int64_t> qd;
    std::vector<double> qv;
    for (auto &e : qmap) {
      qd.push_back(e.first);
      qv.push_back(e.second);
    }
    HIPCHK(c, c->pois_q.ensure(qd.size() * (sizeof(int64_t) + sizeof(double))));
    int64_t *dq = c->pois_q.as<int64_t>();
    double *vq = reinterpret_cast<double *>(dq + qd.size());
    HIPCHK(c, hipMemcpyAsync(dq, qd.data(), qd.size() * sizeof(int64_t), hipMemcpyHostToDevice, s));
    HIPCHK(c, hipMemcpyAsync(vq, qv.data(), qv.size() * sizeof(double), hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(poisson_charges_kernel, dim3((unsigned)((qd.size() + PB - 1) / PB)), block, 0, s, f, dq, vq,
                       (int)qd.size());
    HIPCHK(c, hipStreamSynchronize(s));            // the host staging vectors go out of scope
  }
  poisson_stencil_launch(M, phi, q, kbs, m, nullptr, 0, nullptr, s);
  hipLaunchKernelGGL(poisson_init_kernel, grid, block, 0, s, f, q, z, pv, m, M.n, kInv4Pi, pa, pb, pc);
  hipLaunchKernelGGL(poisson_setup_reduce_kernel, dim3(1), dim3(PR), 0, s, pa, pb, pc, (int)nb, tol * tol, scal);
  // iterations in groups; the device records the iteration that met the
  // tolerance, the host reads it between groups (a group started after the
  // stop costs only its empty launches).  A group is a quarter of what has run,
  // at least 8 and at most 32: a wait for the host costs about a third of an
  // iteration, launches past the stop as much each (24^3 cells of degree 6, 972
  // iterations: groups of 8 57.7 ms, of 32 54.1; 4^3 of degree 3, 70: 1.51, 1.59).
  double hs[S_NSCAL];
  int launched = 0;
  while (launched < max_iter) {
    const int k = std::min(std::min(std::max(launched / 4, 8), 32), max_iter - launched);
    for (int i = 0; i < k; ++i, ++launched) {
      poisson_stencil_launch(M, pv, q, kbs, m, scal, launched, pc, s);
      hipLaunchKernelGGL(more ? poisson_update_kernel<true> : poisson_update_kernel<false>, dim3((unsigned)nv), block,
                         2 * M.n * sizeof(double), s, z, q, m, M.n, nd, kInv4Pi, scal, launched, pc, (int)na, pa, pb);
      hipLaunchKernelGGL(more ? poisson_dir_kernel<true> : poisson_dir_kernel<false>, dim3((unsigned)nv), block, 0, s, phi,
                         pv, z, nd, scal, launched, pa, pb, (int)nv);
    }
    HIPCHK(c, hipMemcpyAsync(hs, scal, sizeof(hs), hipMemcpyDeviceToHost, s));
    HIPCHK(c, hipStreamSynchronize(s));
    if (hs[S_STOPAT] <= launched) break;
  }
  HIPCHK(c, hipMemcpyAsync(hs, scal, sizeof(hs), hipMemcpyDeviceToHost, s));
  HIPCHK(c, hipStreamSynchronize(s));
  const int it = hs[S_STOPAT] < launched ? (int)hs[S_STOPAT] : launched;
  // the true residual of the returned phi
  poisson_stencil_launch(M, phi, q, kbs, m, nullptr, 0, nullptr, s);
  hipLaunchKernelGGL(poisson_init_kernel, grid, block, 0, s, f, q, z, pv, m, M.n, kInv4Pi, pa, pb, pc);
  hipLaunchKernelGGL(poisson_setup_reduce_kernel, dim3(1), dim3(PR), 0, s, pa, pb, pc, (int)nb, tol * tol, scal);
  HIPCHK(c, hipMemcpyAsync(hs, scal, sizeof(hs), hipMemcpyDeviceToHost, s));
  HIPCHK(c, hipStreamSynchronize(s));
  HIPCHK(c, hipGetLastError());
  if (iters) *iters = it;
  const double ff = hs[S_FF];
  const double res = ff > 0 ? std::sqrt(hs[S_RR] / ff) : 0.0;
  if (rel_resid) *rel_resid = res;
  return res <= tol ? 0 : CHFSI_WARN_NOT_CONVERGED;
}
