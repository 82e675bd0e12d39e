// Chebyshev-step kernels: Y = s1 (Htilde - shift) X + s2 Xprev.
//
// Paper, Sec. 3.3 (practical implementation of Chebyshev filtering) stores
// the cell Hamiltonian and multiplies it densely with the cell's
// wavefunctions.  On the uniform mesh with the diagonal GLL mass (Sec. 2.4,
// eq. hep) the assembled operator is a Kronecker sum,
//   Htilde = A (x) I (x) I + I (x) A (x) I + I (x) I (x) A + diag(V),
// A the 1D operator in the mass-scaled basis: inside an element a row couples
// to the element's p + 1 nodes, an element end to both elements' 2 p + 1.  So
// a value of Htilde X costs about 3 (p + 2) multiply-adds instead of the
// (p + 1)^6 / p^3 of the dense cell products (p = 5: 21 against 373), and the
// step is bound by the memory traffic of X, Xprev and Y instead of by the
// matrix cores.  One launch per step: every output is written once, by one
// thread, in a fixed order (no colours, no atomics), and its arithmetic does
// not depend on the tiling.
//
// The element matrix Ae [p+1][p+1] (A restricted to one element; the two ends
// carry half of the assembled diagonal) is symmetric and centrosymmetric
// (Ae[i][j] = Ae[p-i][p-j]), so a dozen values serve all three directions;
// they sit in scalar registers.  The Bloch operator adds -i k_d C per
// direction (Sec. 2.1 eq. ksproblemPer), C the element's first-derivative
// matrix, antisymmetric in both senses.
#include "common.hpp"
#include "kernels.hpp"

#include <algorithm>
#include <type_traits>
#include <vector>

namespace chfsi {

// A value that is the same in every lane, moved to scalar registers (behind the
// empty asm it is not known to be: a readfirstlane of a uniform value is dropped
// and the value stays in vector registers).
__device__ __forceinline__ int uniform_bits(int b) {
  asm("" : "+v"(b));
  return __builtin_amdgcn_readfirstlane(b);
}
__device__ __forceinline__ float uniform(float x) {
  return __builtin_bit_cast(float, uniform_bits(__builtin_bit_cast(int, x)));
}
__device__ __forceinline__ double uniform(double x) {
  const long long b = __builtin_bit_cast(long long, x);
  const unsigned lo = (unsigned)uniform_bits((int)b), hi = (unsigned)uniform_bits((int)(b >> 32));
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
template <typename T>
__device__ __forceinline__ T fma_t(T a, T b, T c) {
  return __builtin_elementwise_fma(a, b, c);
}
// The neighbour lane's value (0 <-> 1, 2 <-> 3, ...): re <-> im of a complex column.
__device__ __forceinline__ double swap_pair(double x) {
  const long long b = __builtin_bit_cast(long long, x);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)b, 0xB1, 0xf, 0xf, true);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0xB1, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ float swap_pair(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0xB1, 0xf, 0xf, true));
}

// First index of the class of (i, j) under transposition and reversal.
__host__ __device__ constexpr int canon(int P, int i, int j) {
  const int n = P + 1;
  int best = i * n + j;
  const int alt[3] = {j * n + i, (P - i) * n + (P - j), (P - j) * n + (P - i)};
  for (int k = 0; k < 3; ++k)
    if (alt[k] < best) best = alt[k];
  return best;
}
// Sign of C[i][j] against C at canon(i, j) for the first-derivative element
// matrix: antisymmetric, and antisymmetric under reversal.
__host__ __device__ constexpr int canon_sign(int P, int i, int j) {
  const int n = P + 1, c = canon(P, i, j);
  return (c == i * n + j || c == (P - j) * n + (P - i)) ? 1 : -1;
}

// Global access through buffer resources: 32-bit lane offsets from a scalar
// base, and accesses beyond the given size read zero and write nothing, so
// nodes that do not exist (Dirichlet boundary, cells beyond the mesh, columns
// beyond the block) need no branch: their offset is OFF_NONE.
static constexpr unsigned OFF_NONE = 0x80000000u;   // plane sizes stay below it (checked on the host)
typedef unsigned u2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_of(const void *p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
}
template <typename T>
__device__ __forceinline__ T buf_load(__amdgpu_buffer_rsrc_t r, unsigned off, unsigned soff) {
  if constexpr (sizeof(T) == 8)
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, (int)soff, 0));
  else
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, (int)soff, 0));
}
template <typename T>
__device__ __forceinline__ void buf_store(__amdgpu_buffer_rsrc_t r, unsigned off, unsigned soff, T v) {
  if constexpr (sizeof(T) == 8)
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2_t, v), r, (int)off, (int)soff, 0);
  else
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, (int)off, (int)soff, 0);
}

// Work-group barrier for LDS that leaves global loads and stores in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// One problem as the kernels see it (columns are real values; a complex
// column is two of them).
template <typename T>
struct KronProb {
  const T *X, *Xp;
  T *Y;
  int64_t ldx, ldy;   // row strides; Xp has Y's layout
  int64_t cgx, cgy;   // elements from one group of CL columns to the next (tile kernel)
  // coefficients stay in double until they are complete (s1 times an entry of
  // Ae, s1 times a whole diagonal entry), also for float blocks
  const double *V;    // [n_dof]
  const double *ae;   // Ae [(P+1)^2], then the first-derivative matrix C [(P+1)^2]
  int n_el, n, periodic, ncols;
  double s1, s2, shift;
  int bf16;           // (BF tiles) round the values that enter the products to BF16
  double k[3];        // complex: Bloch vector
};

// DoF index along a line of local node `a` of element e (e may lie one beyond
// either end), or -1 where there is no unknown.
__device__ __forceinline__ int line_dof(int e, int a, int P, int n_el, bool periodic) {
  if (periodic) {
    if (e < 0) e += n_el;
    if (e > n_el || (e == n_el && a > 0)) return -1;
    if (e == n_el) return 0;
    return e * P + a;
  }
  if (e < 0 || e >= n_el) return -1;
  return e * P + a - 1;                              // -1 for the boundary node
}

// ---------------------------------------------------------------------------
// Tile kernel (degrees 3..7).
//
// A work-group owns CX x CY cells in (x, y) for CL columns and marches along
// z through nz cells, plane by plane.  The 64 lanes of a wave hold the same
// local node of different cells and columns, so that every coefficient is a
// scalar; wave row (h, b) owns the nodes a in part h of 0..P-1, at b, of its
// cells (NS parts).  Per plane:
//   * the plane's own nodes and its halo (P nodes to the left and below, one
//     to the right and above) go to LDS; the next plane's loads are then
//     issued and land while this plane is multiplied;
//   * x: a node line is read once for all its outputs; y: P + 1 values per
//     output (element end: 2 P + 1);
//   * z: the P + 1 rows of the z-element are accumulators in registers, each
//     plane adds to all of them, and the finished planes are stored when the
//     next element's first plane arrives;
//   * the whole diagonal (the three directions', V and the shift, which
//     cancel in part) is summed in double, once per node, and applied as one
//     coefficient.
// The scheduling barriers keep the LDS reads of one output row from being
// hoisted over the others': without them the register need grows past two
// work-groups' share (measured, FP64 p = 5: 209 against 168 registers).  A
// launch that leaves every CU at most one work-group goes without them (LONE).
//
// BF tiles (float) can round the values that the 1D element matrices multiply to
// BF16.  The diagonal, where the potential and the shift are, multiplies the
// value itself, which the thread keeps until the coefficient is known: in
// registers, at p = 7 in LDS (16^3 cells x 128 columns 790 us per step; kept in
// registers, 42 of which spill, 870).
// ---------------------------------------------------------------------------
template <typename T_, int P_, int CL_, int CX_, int CY_, int NS_, bool CPLX_ = false, bool LONE_ = false,
          bool BF_ = false>
struct KronTile {
  typedef T_ T;
  static constexpr int P = P_, CL = CL_, CX = CX_, CY = CY_, NS = NS_;
  static constexpr bool CPLX = CPLX_;
  static constexpr bool LONE = LONE_;                // one work-group per CU: registers to spare
  static constexpr bool BF = BF_;                    // products may take their values rounded to BF16
  static constexpr bool XD_LDS = BF && P == 7;       // (BF) the diagonal's values wait in LDS
  static_assert(!BF || std::is_same<T, float>::value, "BF16 rounding of FP32 blocks");
  static constexpr int NA = (P + NS - 1) / NS;       // nodes of a line per part
  static constexpr int L = CL * CX * CY;             // lanes of one wave row
  static constexpr int NT = NS * P * L;              // threads
  // Row of nodes in LDS: the left halo element, CX elements, one end node.
  // For even P every element is padded by one node: the two elements of a
  // half wave are then an odd number of 128-byte nodes apart (all 64 banks).
  static constexpr int EW = (P % 2 == 0) ? P + 1 : P;
  static constexpr int W = (CX + 1) * EW + 1;
  static constexpr int H = (CY + 1) * P + 1;
  static constexpr int NODE = CL * (int)sizeof(T);   // bytes of one node
  static constexpr int NN = P * P * CX * CY;         // nodes of a plane
  // halo runs: P CY rows (a run of P nodes on the left and one on the right)
  // and P CX columns (P below and one above); one run per CL lanes of a part,
  // its P + 1 nodes split over the parts (HK nodes each)
  static constexpr int NRUN = P * (CX + CY);
  static constexpr int HK = (P + 1 + NS - 1) / NS;
  static_assert(NRUN * CL <= P * L, "a run per node group");
  static_assert(CX % 2 == 0 && CY % 2 == 0, "tiles start at even cells: a halo element is never the mesh's first");
  static_assert(NN <= NT, "one V value per thread");
  static_assert(L % 64 == 0 && NT <= 1024, "wave rows");
};

template <typename C>
__device__ __forceinline__ void kron_tile(const KronProb<typename C::T> &pr, int tx, int ty, int z0, int nz, int cg) {
  typedef typename C::T T;
  constexpr int P = C::P, CL = C::CL, CX = C::CX, CY = C::CY, NA = C::NA, HK = C::HK;
  constexpr bool CPLX = C::CPLX;
  __shared__ __align__(16) char lds[C::W * C::H * C::NODE];
  __shared__ T dlds[C::NN];          // this plane's diagonal coefficients
  __shared__ double dxy[C::NN];      // the x and y parts of the diagonal less the shift
  __shared__ T xdl[C::XD_LDS ? NA * C::NT : 1];      // a thread's own values, NT apart
  const int t = threadIdx.x;
  const int row = __builtin_amdgcn_readfirstlane(t / C::L);    // wave row
  const int part = C::NS == 1 ? 0 : row / P, b = row - part * P;
  const int li = t - row * C::L;
  const int cl = li % CL, cell = li / CL;
  const int cx = cell % CX, cy = cell / CX;
  const int n = pr.n, n_el = pr.n_el;
  const bool per = pr.periodic != 0;
  const bool col_ok = cg * CL + cl < pr.ncols;
  const unsigned colb = (unsigned)(cl * (int)sizeof(T));
  const T *const X = pr.X + cg * pr.cgx, *const Xp = pr.Xp ? pr.Xp + cg * pr.cgy : nullptr;
  T *const Y = pr.Y + cg * pr.cgy;
  const int ex0 = tx * CX, ey0 = ty * CY, ex = ex0 + cx, ey = ey0 + cy;

  // ---- coefficients, scaled by s1 ----
  T ae[(P + 1) * (P + 1)], yr[P + 1];
  T ce[CPLX ? (P + 1) * (P + 1) : 1], yc[CPLX ? P + 1 : 1];
  const double *ct = pr.ae + (P + 1) * (P + 1);
#pragma unroll
  for (int i = 0; i <= P; ++i)
#pragma unroll
    for (int j = 0; j <= P; ++j)
      if (canon(P, i, j) == i * (P + 1) + j) {
        ae[i * (P + 1) + j] = uniform((T)(pr.s1 * pr.ae[i * (P + 1) + j]));
        if (CPLX) ce[i * (P + 1) + j] = uniform((T)(pr.s1 * ct[i * (P + 1) + j]));
      }
#pragma unroll
  for (int j = 0; j <= P; ++j) {
    yr[j] = uniform(j == b ? T(0) : (T)(pr.s1 * pr.ae[b * (P + 1) + j]));   // (the diagonal is applied apart)
    if (CPLX) yc[j] = uniform((T)(pr.s1 * ct[b * (P + 1) + j]));
  }
  auto A = [&](int i, int j) -> T { return ae[canon(P, i, j)]; };
  auto Cc = [&](int i, int j) -> T { return canon_sign(P, i, j) > 0 ? ce[canon(P, i, j)] : -ce[canon(P, i, j)]; };
  const T s2 = uniform((T)pr.s2);
  auto diag1 = [&](int i) { return i == 0 ? 2.0 * pr.ae[0] : pr.ae[i * (P + 1) + i]; };   // of the assembled 1D operator
  // -i k g: re += k g_im, im -= k g_re, with re and im in neighbouring lanes
  const T sgn = (cl & 1) ? T(-1) : T(1);
  auto mul_ik = [&](int dir, T g) -> T { return (sgn * (T)pr.k[dir]) * swap_pair(g); };

  // ---- own nodes: offsets in a plane, OFF_NONE where there is nothing ----
  const int iy = line_dof(ey, b, P, n_el, per);
  const int ix1 = line_dof(ex, 1, P, n_el, per), ix0 = line_dof(ex, 0, P, n_el, per);
  const bool v1 = col_ok && iy >= 0 && ix1 >= 0;                 // nodes a = 1 .. P-1 (offset of a = 1)
  const bool v0 = col_ok && iy >= 0 && ix0 >= 0;                 // node a = 0
  const bool inside = ex < n_el && ey < n_el;                    // (a wrapped node beyond the mesh is read only)
  const unsigned ldxb = (unsigned)(pr.ldx * (int)sizeof(T)), ldyb = (unsigned)(pr.ldy * (int)sizeof(T));
  const unsigned d0 = (unsigned)(iy * n + ix0), d1 = (unsigned)(iy * n + ix1);
  const unsigned ox0 = v0 ? d0 * ldxb + colb : OFF_NONE, ox1 = v1 ? d1 * ldxb + colb : OFF_NONE;
  const unsigned oy0 = v0 && inside ? d0 * ldyb + colb : OFF_NONE, oy1 = v1 && inside ? d1 * ldyb + colb : OFF_NONE;
  // V of the tile's nodes goes through LDS: thread t < NN loads that of node
  // a = t % P of (row b, cell) t / P
  unsigned ov = OFF_NONE;
  if (t < C::NN) {
    const int va = t % P, vc = t / P % (CX * CY), vb = t / P / (CX * CY);
    const int vx = line_dof(ex0 + vc % CX, va, P, n_el, per), vy = line_dof(ey0 + vc / CX, vb, P, n_el, per);
    if (vx >= 0 && vy >= 0) ov = (unsigned)(vy * n + vx) * 8u;
    dxy[t] = diag1(va) + diag1(vb) - pr.shift;                   // (read by this thread only)
  }
  const T *own_d = dlds + (b * CX * CY + cell) * P;

  // ---- halo run of this node group: nodes 0 .. P-1 and, apart, the end node ----
  const int run = (t - part * P * C::L) / CL;
  unsigned h_off, h_end, h_step;
  int h_lds, h_lend, h_lstep;
  {
    const bool isx = run < P * CY;
    const int q = isx ? run : run - P * CY;                      // row (x) or column (y) of the tile
    const int qe = q / P, qa = q % P;
    const int f0 = isx ? ex0 : ey0, fc = isx ? CX : CY;
    const int fix = line_dof((isx ? ey0 : ex0) + qe, qa, P, n_el, per);
    const int fl = line_dof(f0 - 1, 0, P, n_el, per), fe = line_dof(f0 + fc, 0, P, n_el, per);
    const bool on = run < C::NRUN && fix >= 0 && col_ok;
    const int su = isx ? 1 : n, sf = isx ? n : 1;                // DoF strides along the run and across
    const int k0 = part * HK;                                    // this part's first node
    h_step = (unsigned)su * ldxb;
    h_off = on && fl >= 0 ? (unsigned)(fix * sf + (fl + k0) * su) * ldxb + colb : OFF_NONE;
    h_end = on && fe >= 0 ? (unsigned)(fix * sf + fe * su) * ldxb + colb : OFF_NONE;
    const int lx = isx ? 0 : (qe + 1) * C::EW + qa, ly = isx ? P + q : 0;
    h_lstep = (isx ? 1 : C::W) * C::NODE;
    h_lds = (ly * C::W + lx) * C::NODE + cl * (int)sizeof(T) + k0 * h_lstep;
    h_lend = (isx ? (ly * C::W + (CX + 1) * C::EW) : ((P + CY * P) * C::W + lx)) * C::NODE + cl * (int)sizeof(T);
  }
  // this thread's cell in LDS, at its left-lower halo corner: local node (i, j)
  // of the cell, i, j = -P .. P, is at cbase + node_at(i, j)
  const int cbase = (cy * P * C::W + cx * C::EW) * C::NODE + cl * (int)sizeof(T);
  auto node_at = [&](int i, int j) {
    const int lx = i < 0 ? i + P : (i < P ? i + C::EW : 2 * C::EW);
    return ((j + P) * C::W + lx) * C::NODE;
  };
  const int row_lds = cbase + b * C::W * C::NODE;
  auto lds_at = [&](int off) -> T & { return *reinterpret_cast<T *>(lds + off); };

  auto rnd = [&](T x) -> T {
    if constexpr (C::BF) return pr.bf16 ? (float)(__bf16)x : x;
    else return x;
  };

  // ---- planes ----
  // Plane kd of a block (kd: DoF index along z, uniform): a buffer resource;
  // of no bytes, so reading zero and writing nothing, where it does not exist.
  const unsigned nd2 = (unsigned)(n * n);
  const unsigned nbx = nd2 * ldxb, nby = nd2 * ldyb, nbp = Xp ? nby : 0u, nbv = nd2 * 8u;
  auto plane = [&](const void *base, unsigned bytes, int kd) {
    return buf_of(reinterpret_cast<const char *>(base) + (uint64_t)bytes * (unsigned)(kd < 0 ? 0 : kd), kd < 0 ? 0u : bytes);
  };

  auto row_fence = [] {
    if constexpr (!C::LONE) __builtin_amdgcn_sched_barrier(0);
  };

  // The march, for the nodes of part PART (its waves run their own copy; all
  // copies pass the same barriers).
  auto march = [&](auto part_c) {
    constexpr int PART = decltype(part_c)::value;
    constexpr int A0 = PART * NA, NO = P - A0 < NA ? P - A0 : NA;          // own nodes A0 .. A0 + NO - 1
    constexpr int K0 = PART * HK, NK = P + 1 - K0 < HK ? P + 1 - K0 : HK;  // run nodes K0 .. K0 + NK - 1; node P is the end
    T xo[NO], xh[NK], xp[NO];
    double vv;
    auto load_own = [&](int kd, T(&o)[NO]) {
      const __amdgpu_buffer_rsrc_t rx = plane(X, nbx, kd);
#pragma unroll
      for (int a = 0; a < NO; ++a)
        o[a] = A0 + a == 0 ? buf_load<T>(rx, ox0, 0) : buf_load<T>(rx, ox1, (A0 + a - 1) * ldxb);
    };
    auto load_rest = [&](int kd) {
      const __amdgpu_buffer_rsrc_t rx = plane(X, nbx, kd);
      unsigned o = h_off;
      asm("" : "+v"(o));                             // (recomputed per plane: keeping every offset costs registers)
#pragma unroll
      for (int k = 0; k < NK; ++k) {
        xh[k] = buf_load<T>(rx, K0 + k == P ? h_end : o, 0);
        o += h_step;
      }
      vv = buf_load<double>(plane(pr.V, nbv, kd), ov, 0);
      const __amdgpu_buffer_rsrc_t rp = plane(Xp, nbp, kd);
#pragma unroll
      for (int a = 0; a < NO; ++a)
        xp[a] = A0 + a == 0 ? buf_load<T>(rp, oy0, 0) : buf_load<T>(rp, oy1, (A0 + a - 1) * ldyb);
    };

    // acc[r][a]: row r (local plane) of the current z-element
    T acc[P + 1][NO];
    // products of one plane (local plane c of the element) into accumulator
    // row r != c; xk = -i k_z x (complex)
    auto zrow = [&](int r, int c, const T *x, const T *xk) {
      if (r == c) return;
#pragma unroll
      for (int a = 0; a < NO; ++a) {
        acc[r][a] = fma_t(A(r, c), x[a], acc[r][a]);
        if (CPLX) acc[r][a] = fma_t(Cc(r, c), xk[a], acc[r][a]);
      }
    };
    auto set_xk = [&](const T *x, T *xk) {
      if (CPLX)
#pragma unroll
        for (int a = 0; a < NO; ++a) xk[a] = mul_ik(2, x[a]);
    };
    auto flush = [&](int zc) {                       // planes 0 .. P-1 of element zc (>= z0) are complete
#pragma unroll
      for (int c = 0; c < P; ++c) {
        const __amdgpu_buffer_rsrc_t ry = plane(Y, nby, zc < z0 ? -1 : line_dof(zc, c, P, n_el, per));
#pragma unroll
        for (int a = 0; a < NO; ++a) {
          if (A0 + a == 0) buf_store(ry, oy0, 0, acc[c][a]);
          else buf_store(ry, oy1, (A0 + a - 1) * ldyb, acc[c][a]);
        }
      }
    };

    // the element below: its planes' contributions to this chunk's first plane
#pragma unroll
    for (int a = 0; a < NO; ++a) acc[P][a] = 0;
    {
      T xb[P][NO], xk[NO];
#pragma unroll
      for (int c = 0; c < P; ++c) load_own(line_dof(z0 - 1, c, P, n_el, per), xb[c]);
      load_own(line_dof(z0, 0, P, n_el, per), xo);
      load_rest(line_dof(z0, 0, P, n_el, per));
#pragma unroll
      for (int c = 0; c < P; ++c) {
#pragma unroll
        for (int a = 0; a < NO; ++a) xb[c][a] = rnd(xb[c][a]);
        set_xk(xb[c], xk);
        zrow(P, c, xb[c], xk);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < P; ++r)
#pragma unroll
      for (int a = 0; a < NO; ++a) acc[r][a] = 0;    // (no element before z0 to finish)

#pragma unroll 1
    for (int zc = z0; zc < z0 + nz; ++zc) {
#pragma unroll
      for (int c = 0; c < P; ++c) {
        // plane c of this element to LDS
        T x[NO], dg[NO], xd[NO];                     // xd: what the diagonal multiplies
#pragma unroll
        for (int a = 0; a < NO; ++a) {
          if constexpr (C::XD_LDS) xdl[a * C::NT + t] = xo[a];
          else xd[a] = xo[a];
          x[a] = rnd(xo[a]);
        }
#pragma unroll
        for (int a = 0; a < NO; ++a) lds_at(row_lds + node_at(A0 + a, 0)) = x[a];
        int hl = h_lds;
        asm("" : "+v"(hl));
        if (C::NRUN * CL == P * C::L || run < C::NRUN) {
#pragma unroll
          for (int k = 0; k < NK; ++k) {
            lds_at(K0 + k == P ? h_lend : hl) = rnd(xh[k]);
            hl += h_lstep;
          }
        }
        int td = t;
        asm("" : "+v"(td));                        // (the sum is not kept per plane)
        if (t < C::NN) dlds[t] = (T)(pr.s1 * (vv + (dxy[td] + diag1(c))));
#pragma unroll
        for (int a = 0; a < NO; ++a) dg[a] = s2 * xp[a];
        if (c == 0) {
          // the element below is complete with this plane
          T xk[NO];
          set_xk(x, xk);
#pragma unroll
          for (int r = 0; r <= P; ++r) zrow(r, P, x, xk);
        }
        __builtin_amdgcn_sched_barrier(0);
        // next plane's loads
        const int kn = c + 1 < P ? line_dof(zc, c + 1, P, n_el, per) : line_dof(zc + 1, 0, P, n_el, per);
        load_own(kn, xo);
        load_rest(c + 1 < P || zc + 1 < z0 + nz ? kn : -1);
        __builtin_amdgcn_sched_barrier(0);
        if (c == 0) {
          flush(zc - 1);
#pragma unroll
          for (int a = 0; a < NO; ++a) acc[0][a] = acc[P][a];
#pragma unroll
          for (int r = 1; r <= P; ++r)
#pragma unroll
            for (int a = 0; a < NO; ++a) acc[r][a] = 0;
        }
#pragma unroll
        for (int a = 0; a < NO; ++a) acc[c][a] += dg[a];
        lds_barrier();
        // x: the node line of this cell, for its first node also the left neighbour's
        {
          T gx[NO], xs[P + 1];                       // gx: complex, first-derivative sums
          if (A0 == 0) {
#pragma unroll
            for (int m = 0; m < P; ++m) xs[m] = lds_at(row_lds + node_at(m - P, 0));
            gx[0] = 0;
#pragma unroll
            for (int m = 0; m < P; ++m) {
              acc[c][0] = fma_t(A(P, m), xs[m], acc[c][0]);
              if (CPLX) gx[0] = fma_t(Cc(P, m), xs[m], gx[0]);
            }
            row_fence();
          }
#pragma unroll
          for (int m = 0; m <= P; ++m) xs[m] = lds_at(row_lds + node_at(m, 0));
#pragma unroll
          for (int a = 0; a < NO; ++a) {
            if (A0 + a > 0) gx[a] = 0;
#pragma unroll
            for (int m = 0; m <= P; ++m) {
              if (m == A0 + a) continue;
              acc[c][a] = fma_t(A(A0 + a, m), xs[m], acc[c][a]);
              if (CPLX) gx[a] = fma_t(Cc(A0 + a, m), xs[m], gx[a]);
            }
            if (CPLX) {
              acc[c][a] += mul_ik(0, gx[a]);
              row_fence();
            }
          }
          row_fence();
          // the diagonal, and z
          T xk[NO];
          set_xk(xs + A0, xk);
#pragma unroll
          for (int a = 0; a < NO; ++a) {
            if constexpr (C::XD_LDS) xd[a] = xdl[a * C::NT + t];
            acc[c][a] = fma_t(own_d[A0 + a], C::BF ? xd[a] : xs[A0 + a], acc[c][a]);
          }
#pragma unroll
          for (int r = 0; r <= P; ++r) zrow(r, c, xs + A0, xk);
        }
        row_fence();
        // y: this element, and for its first node the element below it
        // (Ae[P][m] = Ae[0][P - m], C[P][m] = -C[0][P - m])
#pragma unroll
        for (int a = 0; a < NO; ++a) {
          T g = 0;
#pragma unroll
          for (int m = 0; m <= P; ++m) {
            const T v = lds_at(cbase + node_at(A0 + a, m));
            acc[c][a] = fma_t(yr[m], v, acc[c][a]);
            if (CPLX) g = fma_t(yc[m], v, g);        // (C's diagonal is stored as zero)
          }
          if (CPLX) acc[c][a] += mul_ik(1, g);
          row_fence();
        }
        if (b == 0) {
#pragma unroll
          for (int a = 0; a < NO; ++a) {
            T g = 0;
#pragma unroll
            for (int m = 0; m < P; ++m) {
              const T v = lds_at(cbase + node_at(A0 + a, m - P));
              acc[c][a] = fma_t(yr[P - m], v, acc[c][a]);
              if (CPLX) g = fma_t(-yc[P - m], v, g);
            }
            if (CPLX) acc[c][a] += mul_ik(1, g);
            row_fence();
          }
        }
        lds_barrier();
      }
    }
    T x[NO], xk[NO];
#pragma unroll
    for (int a = 0; a < NO; ++a) x[a] = rnd(xo[a]);
    set_xk(x, xk);
#pragma unroll
    for (int r = 0; r < P; ++r) zrow(r, P, x, xk);
    flush(z0 + nz - 1);
  };
  if constexpr (C::NS == 1) {
    march(std::integral_constant<int, 0>());
  } else {
    static_assert(C::NS == 2, "one or two parts");
    if (part == 0) march(std::integral_constant<int, 0>());
    else march(std::integral_constant<int, 1>());
  }
}

struct KronGrid {
  int ntx, nty, nzc, ncg, zlen;      // tiles in x and y, z chunks, column groups, cells per chunk
};

// Work-groups are dealt round-robin to the 8 XCDs: give each XCD a contiguous
// run of the list, so that tiles that share halo lines share an L2.
__device__ __forceinline__ int xcd_order(int bid, int nwg) {
  const int q = nwg / 8, r = nwg % 8;
  const int x = bid % 8, i = bid / 8;
  return x < r ? x * (q + 1) + i : r * (q + 1) + (x - r) * q + i;
}

template <typename C, int WAVES>
__global__ __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(WAVES))) void kron_kernel(
    KronProb<typename C::T> pr, KronGrid gr) {
  int w = xcd_order(blockIdx.x, gridDim.x);
  const int tx = w % gr.ntx;
  w /= gr.ntx;
  const int ty = w % gr.nty;
  w /= gr.nty;
  const int zc = w % gr.nzc, cg = w / gr.nzc;
  const int z0 = zc * gr.zlen;
  const int nz = pr.n_el - z0 < gr.zlen ? pr.n_el - z0 : gr.zlen;
  kron_tile<C>(pr, tx, ty, z0, nz, cg);
}

// Batched: work item (problem, tx | ty << 16, z0 | nz << 16, column group);
// the step's buffer roles (in, out = previous) are the same for every problem,
// its coefficients come from the problem's table (s1, s2, shift per step).
template <typename C, int WAVES>
__global__ __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(WAVES))) void kron_batch_kernel(
    const KronBatchProblem<typename C::T> *__restrict__ probs, const int4 *__restrict__ work, int step) {
  typedef typename C::T T;
  const int4 w = work[xcd_order(blockIdx.x, gridDim.x)];
  const KronBatchProblem<T> &B = probs[w.x];
  const int in = step & 1, out = in ^ 1;
  KronProb<T> p;
  p.X = B.buf[in].p;
  p.ldx = B.buf[in].ld;
  p.cgx = B.buf[in].cg;
  p.Y = B.buf[out].p;
  p.ldy = B.buf[out].ld;
  p.cgy = B.buf[out].cg;
  p.Xp = step > 0 ? p.Y : nullptr;
  p.V = B.V;
  p.ae = B.ae;
  p.n_el = B.n_el;
  p.n = B.n;
  p.periodic = B.periodic;
  p.ncols = B.ncols;
  const double *coef = B.coef + 3 * step;
  p.s1 = coef[0];
  p.s2 = coef[1];
  p.shift = coef[2];
  p.bf16 = B.bf16;
  kron_tile<C>(p, w.y & 0xffff, w.y >> 16, w.z & 0xffff, w.z >> 16, w.w);
}

// A group of k-points on one mesh: k-point g's block, Bloch vector and
// |k|^2/2 shift by index, the mesh tables shared.
template <typename C, int WAVES>
__global__ __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(WAVES))) void kron_kpts_kernel(
    KronProb<typename C::T> pr, KronGrid gr, const double *__restrict__ kv, int64_t xstride, int64_t ystride) {
  int w = xcd_order(blockIdx.x, gridDim.x);
  const int tx = w % gr.ntx;
  w /= gr.ntx;
  const int ty = w % gr.nty;
  w /= gr.nty;
  const int zc = w % gr.nzc;
  w /= gr.nzc;
  const int cg = w % gr.ncg, g = w / gr.ncg;
  const int z0 = zc * gr.zlen;
  const int nz = pr.n_el - z0 < gr.zlen ? pr.n_el - z0 : gr.zlen;
  pr.X += g * xstride;
  pr.Y += g * ystride;
  double k2 = 0;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    pr.k[d] = kv[3 * g + d];
    k2 += pr.k[d] * pr.k[d];
  }
  pr.shift = -0.5 * k2;
  kron_tile<C>(pr, tx, ty, z0, nz, cg);
}

// ---------------------------------------------------------------------------
// General kernel: any degree, size and row stride (row-major blocks).  One
// thread per value of Y, lanes along the columns; the 3 (p + 2) values it
// gathers come from the caches.  Used for degrees 8..12 and where a plane of
// the block exceeds the tile kernel's 32-bit offsets.  The coefficients, s1 times
// an entry, wait in LDS.
//
// FP > 0: the degree, for blocks of more than 32 columns.  A wave's lanes are 64
// columns of one node, whose index arithmetic is then scalar, and an element's
// p + 1 values are all in flight at once: the latency of gathers one or two at a
// time is what bounds the other form.  Columns come in groups of 64, the group
// outermost, so that the planes a z line reaches stay in the last-level cache.
// 16^3 cells x 128 columns, us per step, FP64 and FP32: p = 8 4,950 and 4,030, p =
// 10 11,000 and 8,230 (with the degree at run time 7,270, 6,930, 18,260, 14,410;
// dense cell products 13,390, 6,960, 35,030, 17,890).
// ---------------------------------------------------------------------------
static constexpr int GEN_Q = 13;                     // nodes of an element's line, at most (p <= 12)
template <typename T, bool CPLX, int FP>
__global__ __launch_bounds__(256) void kron_general_kernel(KronProb<T> pr, int P_, int lanes_) {
  static_assert(!(CPLX && FP > 0) && FP < GEN_Q, "complex blocks stop at degree 7");
  const int P = FP > 0 ? FP : P_, lanes = FP > 0 ? 64 : lanes_;
  const int n = pr.n, n_el = pr.n_el, q = P + 1;
  const bool per = pr.periodic != 0;
  __shared__ T cf[GEN_Q * GEN_Q], cc[CPLX ? GEN_Q * GEN_Q : 1];
  __shared__ double cd[GEN_Q];                       // Ae's diagonal
  for (int t = threadIdx.x; t < q * q; t += 256) {
    cf[t] = (T)(pr.s1 * pr.ae[t]);
    if (CPLX) cc[t] = (T)(pr.s1 * pr.ae[q * q + t]);
    if (t % (q + 1) == 0) cd[t / (q + 1)] = pr.ae[t];
  }
  __syncthreads();
  const int rows = 256 / lanes, lane = (int)threadIdx.x % lanes;
  int row0 = (int)threadIdx.x / lanes;
  if (FP > 0) row0 = __builtin_amdgcn_readfirstlane(row0);
  const int ncg = (pr.ncols + lanes - 1) / lanes;
  const int64_t nd = (int64_t)n * n * n;
  const int64_t nrow = (nd + rows - 1) / rows, nblk = nrow * ncg;
  auto rnd = [&](T x) -> T {
    if constexpr (std::is_same<T, float>::value) return pr.bf16 ? (float)(__bf16)x : x;
    else return x;
  };
  for (int64_t w = blockIdx.x; w < nblk; w += gridDim.x) {
    const int64_t cg = w / nrow, d = (w - cg * nrow) * rows + row0;
    const int col = (int)cg * lanes + lane;
    if (d >= nd || col >= pr.ncols) continue;
    const int r = (int)(d / n), id[3] = {(int)(d - (int64_t)r * n), r % n, r / n};
    const T *const own = pr.X + d * pr.ldx;
    T y = 0;
    double dg = pr.V[d] - pr.shift;
    int64_t st = pr.ldx;                             // from one node of the line to the next
#pragma unroll
    for (int dir = 0; dir < 3; ++dir) {
      const int I = id[dir] + (per ? 0 : 1), e = I / P, a = I - e * P;
      const T *const x0 = own - id[dir] * st;        // node 0 of the line
      T g = 0;
      // elements that hold the node: its own, and for an element end the one before
      for (int half = 0; half < (a == 0 ? 2 : 1); ++half) {
        const int row = half ? P : a, ee = e - half < 0 ? n_el - 1 : e - half;   // (before the first: periodic)
        dg += cd[row];
        // node m of the element is xe + m st, for m0 <= m <= m1 (Dirichlet ends
        // left out); the last one of a periodic line is its first
        const int m0 = !per && ee == 0 ? 1 : 0, m1 = per || ee + 1 < n_el ? P : P - 1;
        const bool wrap = per && ee + 1 == n_el;
        const T *const xe = x0 + (int64_t)(ee * P - (per ? 0 : 1)) * st;
        const T *const ca = cf + row * q, *const cb = cc + (CPLX ? row * q : 0);
        if constexpr (FP > 0) {
          T v[FP + 1];
#pragma unroll
          for (int m = 0; m <= FP; ++m) {
            const T *x = m == FP && wrap ? x0 : xe + m * st;
            if (m < m0 || m > m1) x = own;           // (not used)
            v[m] = x[col];
          }
#pragma unroll
          for (int m = 0; m <= FP; ++m)
            if (m >= m0 && m <= m1 && m != row) y = fma_t(ca[m], rnd(v[m]), y);
        } else {
          auto add = [&](int m, const T *x) {
            y = fma_t(ca[m], rnd(x[col]), y);
            if (CPLX) g = fma_t(cb[m], x[col ^ 1], g);
          };
          const T *x = xe + m0 * st;
#pragma unroll 4
          for (int m = m0; m < row; ++m, x += st) add(m, x);
          x += st;
#pragma unroll 4
          for (int m = row + 1; m < P; ++m, x += st) add(m, x);
          if (row < P && m1 == P) add(P, wrap ? x0 : x);
        }
      }
      if (CPLX) y = fma_t((T)((col & 1) ? -pr.k[dir] : pr.k[dir]), g, y);
      st *= n;
    }
    y = fma_t((T)(pr.s1 * dg), own[col], y);         // (the value itself, as in the tile kernel)
    if (pr.Xp) y = fma_t((T)pr.s2, pr.Xp[d * pr.ldy + col], y);
    pr.Y[d * pr.ldy + col] = y;
  }
}

// ---- host side -------------------------------------------------------------

// Tile per degree: V = 0 is 2 x 2 cells, V = 1 is 4 x 2 (half the halo per
// value, so less to fetch again from beyond the L2) where two SIMDs' registers
// hold it; the built-in choice is what measured faster, us per step:
//   FP64 p = 5, 32^3 cells x 128 columns: 4 x 2 2765, 2 x 2 3144;
//   FP64 p = 4, 36^3 x 128: 4 x 2 2039, 2 x 2 2080;
//   FP64 p = 6, 24^3 x 128: nodes of a line in two parts 2280 (twelve waves
//   of 127 registers), one part 2325; p = 7, 20^3 x 128: two parts 3297, one
//   part 3165 (two parts spill at the 128 registers of fourteen waves);
//   FP32, 32 columns per node: p = 6, 24^3 x 128 1090 (16 lanes of two
//   columns each: 1270).
template <typename T, int P, int V, bool CPLX, bool BF = false>
struct TileOf {
  static constexpr bool f64 = sizeof(T) == 8;
  static constexpr int CL = f64 ? 16 : 32;
  static constexpr int CX = (V == 1 && f64 && !CPLX && P >= 3 && P <= 5) ? 4 : 2;
  static constexpr int NS = (f64 && (CPLX ? (P == 5 || P == 6) : P == 6)) ? 2 : 1;
  static constexpr int WAVES = !f64 ? 4 : CPLX ? (P == 7 ? 2 : 3) : P <= 3 ? 4 : P == 4 ? (CX == 4 ? 3 : 4)
                               : P == 5 ? 3 : P == 6 ? 4 : 2;
  typedef KronTile<T, P, CL, CX, 2, NS, CPLX, false, BF> type;
  // The same tile for launches of at most one work-group per CU, whose time is
  // its waves' chains: no scheduling barriers, and in FP64 the nodes of a line in
  // two parts, twice the waves.  us per step, lone against not: FP64 p = 4, 4^3
  // cells x 24 columns 8.25, 9.05; p = 5, 5^3 x 32 13.95, 15.3; FP32 p = 4 8.04,
  // 8.79; p = 6, 5^3 x 32 19.9, 21.0.  (FP64 p = 6, already in two parts, 21.7
  // against 21.3, p = 7 53 against 36: spills.)
  static constexpr bool HAS_LONE = !CPLX && CX == 2 && P >= 3 && P <= (f64 ? 5 : 6);
  typedef typename std::conditional<HAS_LONE, KronTile<T, P, CL, 2, 2, f64 ? 2 : 1, false, true, BF>, type>::type lone;
  static constexpr int LONE_WAVES = (lone::NT + 255) / 256;
};
// (a mesh whose 4 x 2 tiles, one cell deep, do not fill the CUs takes 2 x 2:
// p = 4, 4^3 cells x 24 columns 9.1 against 12.1 us)
static constexpr int CUS = 256;
static int tile_variant(int p, bool f64, int variant, int n_el, int ncols) {
  if (variant >= 0) return variant;
  if (!f64 || p < 3 || p > 5) return 0;
  const int64_t cells = (int64_t)((n_el + 3) / 4) * ((n_el + 1) / 2) * n_el;
  return cells * ((ncols + 15) / 16) >= CUS ? 1 : 0;
}

// Calls f.template run<TileOf<...>>() for degree p (1..7) and variant v; -1 otherwise.
template <typename T, bool CPLX, bool BF = false, typename F>
static int with_tile(int p, int v, F &&f) {
  switch (p) {
#define KRON_CASE(N)                                                   \
  case N:                                                              \
    if constexpr (TileOf<T, N, 1, CPLX, BF>::CX == 4)                  \
      if (v != 0) return f.template run<TileOf<T, N, 1, CPLX, BF>>(), 0; \
    return f.template run<TileOf<T, N, 0, CPLX, BF>>(), 0;
    KRON_CASE(1) KRON_CASE(2) KRON_CASE(3) KRON_CASE(4) KRON_CASE(5) KRON_CASE(6) KRON_CASE(7)
#undef KRON_CASE
    default: return -1;
  }
}

// z chunks of a march through n_el cells by `tiles` tiles.  Time follows
// rounds of one work-group per CU times planes per chunk (a second resident
// work-group shares the CU's bandwidth, it does not add to it), plus about
// two planes' time per chunk for the element below that it reads again.
// Measured, FP64 p = 5, 8^3 cells x 128 columns (64 tiles), us per step: 1
// chunk 113, 2 62, 4 39, 8 46; p = 7, 11^3 x 77 (180 tiles): 535, 560, 488
// and (11 chunks) 495.
int kron_zlen(int n_el, int p, int64_t tiles) {
  int best = n_el;
  int64_t best_t = -1;
  for (int zlen = n_el; zlen >= 1; --zlen) {
    const int nzc = (n_el + zlen - 1) / zlen;
    const int64_t rounds = (tiles * nzc + CUS - 1) / CUS;
    const int64_t t = rounds * ((int64_t)zlen * p + 2);
    if (best_t < 0 || t < best_t) {
      best = zlen;
      best_t = t;
    }
  }
  return best;
}

template <typename T>
static KronProb<T> prob_of(const KronArgs<T> &a) {
  KronProb<T> p;
  p.X = a.X.p;
  p.ldx = a.X.ld;
  p.cgx = a.X.cg;
  p.Xp = a.Xp;
  p.Y = a.Y.p;
  p.ldy = a.Y.ld;
  p.cgy = a.Y.cg;
  p.V = a.V;
  p.ae = a.ae;
  p.n_el = a.n_el;
  p.n = a.n;
  p.periodic = a.periodic;
  p.ncols = a.ncols;
  p.s1 = a.s1;
  p.s2 = a.s2;
  p.shift = a.shift;
  p.bf16 = a.bf16;
  for (int d = 0; d < 3; ++d) p.k[d] = a.k[d];
  return p;
}

int kron_group(int p, size_t elem) { return p > 7 ? 0 : elem == 8 ? 16 : 32; }
bool kron_tiled(int p, int n, int64_t ld, size_t elem) {
  return p <= 7 && (int64_t)n * n < (int64_t)OFF_NONE / (int64_t)elem / ld;
}

template <typename C>
static KronGrid grid_of(int n_el, int ncols, int64_t blocks) {
  KronGrid g;
  g.ntx = (n_el + C::CX - 1) / C::CX;
  g.nty = (n_el + C::CY - 1) / C::CY;
  g.ncg = (ncols + C::CL - 1) / C::CL;
  g.zlen = kron_zlen(n_el, C::P, (int64_t)g.ntx * g.nty * g.ncg * blocks);
  g.nzc = (n_el + g.zlen - 1) / g.zlen;
  return g;
}

template <typename T>
struct LaunchOp {
  KronProb<T> pr;
  hipStream_t s;
  int status = 0;
  template <typename TO> void run() {
    typedef typename TO::type C;
    const KronGrid g = grid_of<C>(pr.n_el, pr.ncols, 1);
    const int64_t nwg = (int64_t)g.ntx * g.nty * g.nzc * g.ncg;
    if (nwg > INT32_MAX) {
      status = -1;
      return;
    }
    if constexpr (TO::HAS_LONE)
      if (nwg <= CUS) {
        typedef typename TO::lone L;
        hipLaunchKernelGGL((kron_kernel<L, TO::LONE_WAVES>), dim3((unsigned)nwg), dim3(L::NT), 0, s, pr, g);
        return;
      }
    hipLaunchKernelGGL((kron_kernel<C, TO::WAVES>), dim3((unsigned)nwg), dim3(C::NT), 0, s, pr, g);
  }
};

template <typename T, bool CPLX>
static int launch(const KronArgs<T> &a, hipStream_t s) {
  const KronProb<T> pr = prob_of(a);
  if (a.ncols < 1 || a.n < 1) return -1;
  if (kron_tiled(a.p, a.n, std::max(a.X.ld, a.Y.ld), sizeof(T))) {
    LaunchOp<T> op{pr, s};
    const int v = CPLX ? 0 : tile_variant(a.p, sizeof(T) == 8, a.variant, a.n_el, a.ncols);
    if constexpr (std::is_same<T, float>::value)
      if (a.bf16) return with_tile<T, CPLX, true>(a.p, v, op) ? -1 : op.status;
    return with_tile<T, CPLX>(a.p, v, op) ? -1 : op.status;
  }
  // the general kernel reads row-major blocks
  const int cg = kron_group(a.p, sizeof(T));
  if ((a.ncols > cg && cg > 0) && (a.X.cg != cg || a.Y.cg != cg)) return -1;
  int lanes = CPLX ? 2 : 1;
  while (lanes < 64 && lanes < a.ncols) lanes *= 2;
  const int64_t nd = (int64_t)pr.n * pr.n * pr.n;
  const int64_t blocks = (nd + 256 / lanes - 1) / (256 / lanes) * ((pr.ncols + lanes - 1) / lanes);
  const dim3 g((unsigned)std::min<int64_t>(blocks, 1 << 24));
  auto go = [&](auto kern) { hipLaunchKernelGGL(kern, g, dim3(256), 0, s, pr, a.p, lanes); };
  if constexpr (!CPLX)
    if (lanes == 64) switch (a.p) {
        case 8: return go(kron_general_kernel<T, false, 8>), 0;
        case 9: return go(kron_general_kernel<T, false, 9>), 0;
        case 10: return go(kron_general_kernel<T, false, 10>), 0;
        case 11: return go(kron_general_kernel<T, false, 11>), 0;
        case 12: return go(kron_general_kernel<T, false, 12>), 0;
      }
  go(kron_general_kernel<T, CPLX, 0>);
  return 0;
}
int kron_launch(const KronArgs<double> &a, hipStream_t s) { return launch<double, false>(a, s); }
int kron_launch(const KronArgs<float> &a, hipStream_t s) { return launch<float, false>(a, s); }
int kron_launch_complex(const KronArgs<double> &a, hipStream_t s) {
  return a.ncols % 2 ? -1 : launch<double, true>(a, s);
}

struct KptsOp {
  KronProb<double> pr;
  int nk;
  const double *kv;
  int64_t xs, ys;
  hipStream_t s;
  int status = 0;
  template <typename TO> void run() {
    typedef typename TO::type C;
    const KronGrid g = grid_of<C>(pr.n_el, pr.ncols, nk);
    const int64_t nwg = (int64_t)g.ntx * g.nty * g.nzc * g.ncg * nk;
    if (nwg > INT32_MAX) {
      status = -1;
      return;
    }
    hipLaunchKernelGGL((kron_kpts_kernel<C, TO::WAVES>), dim3((unsigned)nwg), dim3(C::NT), 0, s, pr, g, kv, xs, ys);
  }
};
int kron_launch_kpts(const KronArgs<double> &a, int nk, const double *kv, const double *host_kv, int64_t xstride,
                     int64_t ystride, hipStream_t s) {
  if (a.ncols % 2 || nk < 1) return -1;
  if (kron_tiled(a.p, a.n, std::max(a.X.ld, a.Y.ld), 8)) {
    KptsOp op{prob_of(a), nk, kv, xstride, ystride, s};
    return with_tile<double, true>(a.p, 0, op) ? -1 : op.status;
  }
  for (int g = 0; g < nk; ++g) {                     // planes beyond the tile kernel's offsets: one k-point at a time
    KronArgs<double> b = a;
    b.X.p += g * xstride;
    b.Y.p += g * ystride;
    double k2 = 0;
    for (int d = 0; d < 3; ++d) {
      b.k[d] = host_kv[3 * g + d];
      k2 += b.k[d] * b.k[d];
    }
    b.shift = -0.5 * k2;
    if (int r = kron_launch_complex(b, s)) return r;
  }
  return 0;
}

struct BatchWorkOp {
  int n_el, ncols, prob, zlen;
  std::vector<int4> &work;
  template <typename TO> void run() {
    typedef typename TO::type C;
    const KronGrid g = grid_of<C>(n_el, ncols, 1);
    for (int cg = 0; cg < g.ncg; ++cg)
      for (int z0 = 0; z0 < n_el; z0 += zlen)
        for (int ty = 0; ty < g.nty; ++ty)
          for (int tx = 0; tx < g.ntx; ++tx)
            work.push_back(make_int4(prob, tx | ty << 16, z0 | std::min(zlen, n_el - z0) << 16, cg));
  }
};
struct BatchTilesOp {
  int n_el, ncols;
  int64_t tiles = 0;
  template <typename TO> void run() {
    const KronGrid g = grid_of<typename TO::type>(n_el, ncols, 1);
    tiles = (int64_t)g.ntx * g.nty * g.ncg;
  }
};
template <typename T>
int kron_batch_variant(int p, int variant, int n_el, int ncols) {
  return tile_variant(p, sizeof(T) == 8, variant, n_el, ncols);
}
template <typename T>
int64_t kron_batch_tiles(int p, int variant, int n_el, int ncols) {
  BatchTilesOp op{n_el, ncols};
  return with_tile<T, false>(p, variant, op) ? -1 : op.tiles;
}
template <typename T>
int kron_batch_work(int p, int variant, int n_el, int ncols, int prob, int zlen, std::vector<int4> &work) {
  BatchWorkOp op{n_el, ncols, prob, zlen, work};
  return with_tile<T, false>(p, variant, op);
}
template <typename T>
struct BatchLaunchOp {
  const KronBatchProblem<T> *probs;
  const int4 *work;
  int nwork, step;
  hipStream_t s;
  template <typename TO> void run() {
    if constexpr (TO::HAS_LONE)
      if (nwork <= CUS) {
        typedef typename TO::lone L;
        hipLaunchKernelGGL((kron_batch_kernel<L, TO::LONE_WAVES>), dim3((unsigned)nwork), dim3(L::NT), 0, s, probs, work,
                           step);
        return;
      }
    hipLaunchKernelGGL((kron_batch_kernel<typename TO::type, TO::WAVES>), dim3((unsigned)nwork), dim3(TO::type::NT), 0, s,
                       probs, work, step);
  }
};
template <typename T>
int kron_batch_launch(int p, int variant, bool bf16, const KronBatchProblem<T> *probs, const int4 *work, int nwork,
                      int step, hipStream_t s) {
  if (nwork <= 0) return 0;
  BatchLaunchOp<T> op{probs, work, nwork, step, s};
  if constexpr (std::is_same<T, float>::value)
    if (bf16) return with_tile<T, false, true>(p, variant, op);
  return with_tile<T, false>(p, variant, op);
}
#define KRON_BATCH(T)                                                                                        \
  template int kron_batch_variant<T>(int, int, int, int);                                                    \
  template int64_t kron_batch_tiles<T>(int, int, int, int);                                                  \
  template int kron_batch_work<T>(int, int, int, int, int, int, std::vector<int4> &);                        \
  template int kron_batch_launch<T>(int, int, bool, const KronBatchProblem<T> *, const int4 *, int, int, hipStream_t);
KRON_BATCH(double)
KRON_BATCH(float)
#undef KRON_BATCH

// ---------------------------------------------------------------------------
// Precision conversion and column-block copies
// ---------------------------------------------------------------------------
// out(i, j) = in(i, j) for two blocks of any layout (row-major, or grouped by
// columns): lanes along the columns of a group of the grouped side.
template <typename Tin, typename Tout>
__global__ __launch_bounds__(256) void copy_cols_kernel(ColBuf<const Tin> in, int gin, ColBuf<Tout> out, int gout,
                                                        int64_t nrows, int ncols) {
  const int64_t total = nrows * (int64_t)ncols;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = t / ncols;
    const int j = (int)(t - i * ncols);
    const int gi = j / gin, go = j / gout;
    out.p[go * out.cg + i * out.ld + (j - go * gout)] = (Tout)in.p[gi * in.cg + i * in.ld + (j - gi * gin)];
  }
}

template <typename Tin, typename Tout>
void copy_cols_launch(const ColBuf<Tin> &in, int gin, const ColBuf<Tout> &out, int gout, int64_t nrows, int ncols,
                      hipStream_t s) {
  int64_t total = nrows * ncols;
  int64_t blocks = (total + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (blocks == 0) return;
  const ColBuf<const Tin> cin{in.p, in.ld, in.cg};
  hipLaunchKernelGGL((copy_cols_kernel<Tin, Tout>), dim3((unsigned)blocks), dim3(256), 0, s, cin, gin, out, gout, nrows,
                     ncols);
}
template void copy_cols_launch<double, double>(const ColBuf<double> &, int, const ColBuf<double> &, int, int64_t, int,
                                               hipStream_t);
template void copy_cols_launch<double, float>(const ColBuf<double> &, int, const ColBuf<float> &, int, int64_t, int,
                                              hipStream_t);
template void copy_cols_launch<float, double>(const ColBuf<float> &, int, const ColBuf<double> &, int, int64_t, int,
                                              hipStream_t);

// Sets *flag = 1 if any of the nrows x ncols values is NaN or Inf.
template <typename T>
__global__ __launch_bounds__(256) void nonfinite_kernel(const T *__restrict__ X, int64_t ld, int64_t nrows,
                                                        int ncols, int *flag) {
  const int64_t total = nrows * (int64_t)ncols;
  bool bad = false;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total;
       t += (int64_t)gridDim.x * blockDim.x) {
    int64_t i = t / ncols;
    int j = (int)(t - i * ncols);
    T v = X[i * ld + j];
    if (!(v - v == T(0))) bad = true;
  }
  if (bad) *flag = 1;
}

template <typename T>
void nonfinite_launch(const T *X, int64_t ld, int64_t nrows, int ncols, int *flag, hipStream_t s) {
  int64_t total = nrows * ncols;
  int64_t blocks = (total + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  if (blocks == 0) return;
  hipLaunchKernelGGL((nonfinite_kernel<T>), dim3((unsigned)blocks), dim3(256), 0, s, X, ld, nrows, ncols, flag);
}
template void nonfinite_launch<double>(const double *, int64_t, int64_t, int, int *, hipStream_t);

}  // namespace chfsi
