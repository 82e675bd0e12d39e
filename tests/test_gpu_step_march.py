"""The step kernels over several cells of one march: the carry from one element to the
next, the planes stored in between, a last chunk shorter than the others, the
previous block overwritten in place.  Meshes are taken so that chunks of more than
one cell with a ragged last one run both in launches of at most one work-group per
CU and beyond, in every degree, precision and tile (the rule that cuts the chunks is
repeated here to check that).  A few columns of each block against the oracle, all of
them between the tiles."""
import numpy as np
import pytest

from oracle import chfsi as och
from oracle import kpoint
import workload
from gpu_util import make_ctx, oracle_apply, to_gpu, to_host

pytestmark = pytest.mark.gpu

CUS = 256
REAL = [(7, 65), (11, 97), (11, 130), (13, 65)]      # cells per edge, columns
BLOCH = [(8, 33), (8, 65), (14, 24)]                 # complex columns


def _zlen(n_el, p, tiles):
    best, best_t = n_el, None
    for z in range(n_el, 0, -1):
        t = -(-tiles * -(-n_el // z) // CUS) * (z * p + 2)
        if best_t is None or t < best_t:
            best, best_t = z, t
    return best


def _launch(n_el, p, ncols, group, cx):
    """(cells per chunk, work-groups) of a launch with cx x 2 cell tiles."""
    tiles = -(-n_el // cx) * -(-n_el // 2) * -(-ncols // group)
    z = _zlen(n_el, p, tiles)
    return z, tiles * -(-n_el // z)


def _rel(a, b):
    return np.max(np.abs(a - b)) / np.max(np.abs(b))


@pytest.mark.parametrize("p", [1, 2, 3, 4, 5, 6, 7])
def test_the_sizes_cover_the_marches(p):
    def kinds(launches):
        got = set()
        for n_el, (z, nwg) in launches:
            if z > 1:
                got.add("small" if nwg <= CUS else "large")
                if n_el % z:
                    got.add("ragged")
        return got
    for group, cx in [(16, 2), (32, 2)] + ([(16, 4)] if 3 <= p <= 5 else []):
        assert kinds((n, _launch(n, p, nc, group, cx)) for n, nc in REAL) == {"small", "large", "ragged"}
    assert kinds((n, _launch(n, p, 2 * nc, 16, 2)) for n, nc in BLOCH) >= {"large", "ragged"}


@pytest.mark.parametrize("p", [1, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("n_el,ncols", REAL)
def test_marches_of_several_cells(n_el, ncols, p):
    L = 2.0 * n_el
    nd = (n_el * p - 1) ** 3
    V = np.random.default_rng(n_el + p).uniform(-3, 1, nd)
    c, _ = make_ctx(L, n_el, p, V=V)
    X = workload.start_block(nd, ncols, 880 + p)
    ap = oracle_apply(L, n_el, p, V)
    pick = sorted({0, 15, 16, 31, 32, ncols - 1})
    Y = ap(X[:, pick])
    b = c.upper_bound
    Xg, got, filtered = to_gpu(X), {}, {}
    for v in (-1, 0, 1):
        c.set_tile_variant(v)
        got[v] = to_host(c.apply(Xg))
        for degree in (4, 5):
            Z = Xg.clone()
            c.chebyshev_filter(Z, degree, 0.4 * b, b, -1.0, block_width=ncols)
            filtered[v, degree] = to_host(Z)
        np.testing.assert_array_equal(got[v], got[-1])
        for degree in (4, 5):
            np.testing.assert_array_equal(filtered[v, degree], filtered[-1, degree])
    assert _rel(got[-1][:, pick], Y) < 1e-13
    assert _rel(to_host(c.apply(Xg, prec="fp32"))[:, pick], Y) < 2e-6
    for degree in (4, 5):
        Z = och.cheb_filter_scaled(ap, X[:, pick], degree, 0.4 * b, b, -1.0)
        assert _rel(filtered[-1, degree][:, pick], Z) < 1e-11
        F = Xg.clone()
        c.chebyshev_filter(F, degree, 0.4 * b, b, -1.0, prec="fp32", block_width=ncols)
        assert _rel(to_host(F)[:, pick], Z) < 1e-4
    c.close()


@pytest.mark.parametrize("p", [1, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("n_el,ncols", BLOCH)
def test_bloch_marches_of_several_cells(n_el, ncols, p):
    import torch
    import paper_1903_10959_amd as P
    L, k = 2.0 * n_el, (0.13, -0.4, 0.07)
    c = P.Context(0).set_mesh(L, n_el, p, periodic=True)
    V = np.random.default_rng(p).uniform(-2, 1, c.n_dof)
    c.set_potential(V).set_kpoint(k)
    g = np.random.default_rng(60 + p)
    X = g.standard_normal((c.n_dof, ncols)) + 1j * g.standard_normal((c.n_dof, ncols))
    pick = sorted({0, 7, 8, ncols - 1})
    As = [kpoint.operator_1d_periodic(L, n_el, p, kd) for kd in k]
    ap = lambda Z: kpoint.apply_kron_k(*As, V, Z)
    Xg = torch.from_numpy(X).cuda()
    assert _rel(c.apply_complex(Xg).cpu().numpy()[:, pick], ap(X[:, pick])) < 1e-13
    b = c.upper_bound_k
    for degree in (4, 5):
        Z = Xg.clone()
        c.chebyshev_filter_complex(Z, degree, 0.4 * b, b, -1.0, block_width=ncols)
        assert _rel(Z.cpu().numpy()[:, pick], och.cheb_filter_scaled(ap, X[:, pick], degree, 0.4 * b, b, -1.0)) < 1e-11
    c.close()
