"""The general step kernel (degrees 8..12): blocks on both sides of 32 columns (a
wave of several nodes; of 64 columns of one), whole and ragged groups of 64, lines
of one, two and three elements with Dirichlet ends and wrapped ones, against the
oracle's Kronecker operator; the filter's recursion in both precisions."""
import numpy as np
import pytest

from oracle import chfsi as och
from oracle import fem, kpoint
import workload
from gpu_util import oracle_apply, to_gpu, to_host

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return np.max(np.abs(a - b)) / np.max(np.abs(b))


@pytest.mark.parametrize("p", [8, 9, 10, 11, 12])
@pytest.mark.parametrize("n_el,ncols,periodic", [(1, 3, False), (1, 64, False), (2, 33, False), (3, 32, False),
                                                 (2, 130, False), (2, 31, True), (2, 65, True)])
def test_apply_and_filter(p, n_el, ncols, periodic):
    import paper_1903_10959_amd as P
    L = 2.0 * n_el
    c = P.Context(0).set_mesh(L, n_el, p, periodic=periodic)
    V = np.random.default_rng(p).uniform(-3, 1, c.n_dof)
    c.set_potential(V)
    if periodic:
        A = np.real(kpoint.operator_1d_periodic(L, n_el, p, 0.0))
        ap = lambda X: fem.apply_kron(A, V, X)
    else:
        ap = oracle_apply(L, n_el, p, V)
    X = workload.start_block(c.n_dof, ncols, 700 + p)
    Y = ap(X)
    Xg = to_gpu(X, ncols + 3)
    assert _rel(to_host(c.apply(Xg)), Y) < 1e-13
    assert _rel(to_host(c.apply(Xg, prec="fp32")), Y) < 2e-6
    b = c.upper_bound
    for degree in (4, 5):
        Z = och.cheb_filter_scaled(ap, X, degree, 3.0, b, -1.0)
        for prec, tol in (("fp64", 1e-11), ("fp32", 1e-4)):
            Xg = to_gpu(X, ncols + 3)
            c.chebyshev_filter(Xg, degree, 3.0, b, -1.0, prec=prec)
            assert _rel(to_host(Xg), Z) < tol
    c.close()
