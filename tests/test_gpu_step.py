"""The Chebyshev-step kernels at the edges of their tiles, against the oracle's
Kronecker-sum operator: meshes that fill and under-fill the 2 x 2 and 4 x 2 cell
tiles, column counts around the 16- and 32-column groups, every degree, odd and
even filter degrees (the result ends in either buffer), a row stride beyond the
tile kernel's 32-bit plane offsets, and the complex operator."""
import ctypes

import numpy as np
import pytest

from oracle import chfsi as och
from oracle import kpoint
import workload
from gpu_util import make_ctx, oracle_apply, to_gpu, to_host

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return np.max(np.abs(a - b)) / max(np.max(np.abs(b)), 1e-300)


@pytest.mark.parametrize("p", [1, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("n_el,ncols", [(1, 3), (2, 16), (3, 17), (5, 33), (6, 1)])
def test_apply_at_tile_edges(n_el, p, ncols):
    """FP64 to rounding and FP32 at single-precision level, the same bits from
    either tile (each value is summed in one fixed order)."""
    if n_el * p < 2:
        pytest.skip("no interior node")
    L = 2.0 * n_el
    c, V = make_ctx(L, n_el, p, V=np.random.default_rng(n_el * 10 + p).uniform(-3, 1, (n_el * p - 1) ** 3))
    X = workload.start_block(c.n_dof, ncols, 500 + p)
    Yo = oracle_apply(L, n_el, p, V)(X)
    got = {}
    for v in (-1, 0, 1):
        c.set_tile_variant(v)
        Xg = to_gpu(X, ncols + 3)
        got[v] = to_host(c.apply(Xg))
        assert _rel(got[v], Yo) < 1e-13
        assert _rel(to_host(c.apply(Xg, prec="fp32")), Yo) < 2e-6
    np.testing.assert_array_equal(got[0], got[1])
    np.testing.assert_array_equal(got[0], got[-1])
    c.close()


@pytest.mark.parametrize("p", [3, 5, 6, 7, 9])
@pytest.mark.parametrize("degree", [1, 2, 5, 6])
def test_filter_odd_and_even_degrees(p, degree):
    """The filtered block against the oracle's recursion, in blocks of 18 columns
    (the last ragged) of rows 5 values apart from the next."""
    L, n_el, ncols = 6.0, 3, 41
    c, V = make_ctx(L, n_el, p, wells=workload.draw_wells(2, L, 90 + p, (1.0, 2.0), (0.4, 0.5)))
    X = workload.start_block(c.n_dof, ncols, 600 + p)
    b = c.upper_bound
    Zo = och.cheb_filter_scaled(oracle_apply(L, n_el, p, V), X, degree, 3.0, b, -1.0)
    Xg = to_gpu(X, ncols + 5)
    c.chebyshev_filter(Xg, degree, 3.0, b, -1.0, block_width=18)
    assert _rel(to_host(Xg), Zo) < 1e-11
    Xg = to_gpu(X, ncols + 5)
    c.chebyshev_filter(Xg, degree, 3.0, b, -1.0, prec="fp32", block_width=18)
    assert _rel(to_host(Xg), Zo) < 1e-4
    c.close()


def test_row_stride_beyond_the_tile_offsets():
    """A plane of the block spans more than 2 GiB: the general kernel, also in
    the filter, whose own buffer is then row-major too."""
    import torch
    n_el, p, ncols, L = 2, 3, 5, 4.0
    c, V = make_ctx(L, n_el, p, wells=workload.draw_wells(1, L, 5, (1.0, 2.0), (0.3, 0.4)))
    ld = 11_000_000                                    # 25 nodes per plane: 2.2 GB
    X = workload.start_block(c.n_dof, ncols, 7)
    Xs = torch.empty(c.n_dof * ld, dtype=torch.float64, device="cuda:0").as_strided((c.n_dof, ncols), (ld, 1))
    Xs.copy_(torch.from_numpy(X))
    Ys = torch.empty(c.n_dof * ld, dtype=torch.float64, device="cuda:0").as_strided((c.n_dof, ncols), (ld, 1))
    ap = oracle_apply(L, n_el, p, V)
    st = c._lib.chfsi_apply(c._h, ctypes.c_void_p(Xs.data_ptr()), ctypes.c_void_p(Ys.data_ptr()), ld, ncols, 0)
    assert st == 0
    assert _rel(to_host(Ys), ap(X)) < 1e-13
    b = c.upper_bound
    c.chebyshev_filter(Xs, 5, 3.0, b, -1.0)
    assert _rel(to_host(Xs), och.cheb_filter_scaled(ap, X, 5, 3.0, b, -1.0)) < 1e-11
    del Xs, Ys
    torch.cuda.empty_cache()
    c.close()


@pytest.mark.parametrize("p", [1, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("n_el,ncols", [(2, 3), (4, 8), (6, 17)])
def test_bloch_operator_every_degree(n_el, p, ncols):
    """Htilde_k X and the k-point group's, against the oracle's Bloch operator."""
    import torch
    import paper_1903_10959_amd as P
    L = 2.0 * n_el
    ks = np.array([[0.13, -0.4, 0.07], [0.0, 0.21, -0.3]])
    c = P.Context(0).set_mesh(L, n_el, p, periodic=True)
    V = np.random.default_rng(p).uniform(-2, 1, c.n_dof)
    c.set_potential(V)
    g = np.random.default_rng(40 + p)
    X = g.standard_normal((2, c.n_dof, ncols)) + 1j * g.standard_normal((2, c.n_dof, ncols))
    Yo = [kpoint.apply_kron_k(*[kpoint.operator_1d_periodic(L, n_el, p, kd) for kd in k], V, x) for k, x in zip(ks, X)]
    Xg = torch.from_numpy(X).cuda()
    Y = c.set_kpoints(ks).apply_complex_kpoints(Xg).cpu().numpy()
    for i in range(2):
        assert _rel(Y[i], Yo[i]) < 1e-13
        c.set_kpoint(ks[i])
        np.testing.assert_array_equal(c.apply_complex(Xg[i]).cpu().numpy(), Y[i])
    c.close()
