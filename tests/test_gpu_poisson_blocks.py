"""Poisson solves of more values than the vector passes have work-groups for in one
block each (4.2M): the iterates of two or three blocks to a work-group, the last
ones with fewer and ragged, and the bound on the partial sums that every work-group
reads."""
import numpy as np
import pytest

import paper_1903_10959_amd as P
from oracle import fem, poisson

pytestmark = pytest.mark.gpu


class _KronPoisson:
    """A = M^1/2 (A1 (+) A1 (+) A1) M^1/2 / (2 pi), A1 the oracle's 1D operator."""

    def __init__(self, L, n_el, p):
        self.A1 = fem.operator_1d(L, n_el, p)
        m = fem.mass_1d(L, n_el, p)
        self.M = np.kron(m, np.kron(m, m))
        self.zero = np.zeros(self.M.size)

    def __matmul__(self, x):
        s = np.sqrt(self.M)
        return s * fem.apply_kron(self.A1, self.zero, (s * x)[:, None])[:, 0] / (2 * np.pi)

    def diagonal(self):
        a = np.diag(self.A1)
        return self.M * (a[:, None, None] + a[None, :, None] + a[None, None, :]).reshape(-1) / (2 * np.pi)


@pytest.mark.parametrize("n_el,p", [(43, 4), (60, 3), (55, 4)])   # 171^3, 179^3 and 219^3
def test_iterates_and_workspace_beyond_one_block_per_work_group(n_el, p):
    import torch
    L, cap = 0.5 * n_el, 5
    c = P.Context(0).set_mesh(L, n_el, p)
    nd, n = c.n_dof, n_el * p - 1
    before = c.device_bytes()
    rho = np.random.default_rng(n_el).uniform(-1, 0, nd)
    out = c.poisson_solve(torch.from_numpy(rho).to("cuda:0"), charges=[(nd // 3, -2.0)], tol=1e-14, max_iter=cap)
    assert not out["converged"] and out["iters"] == cap
    A = _KronPoisson(L, n_el, p)
    f = poisson.load_vector(A.M, rho, [nd // 3], [-2.0])
    x_o, it_o, _ = poisson.jacobi_pcg(A, f, tol=1e-14, max_iter=cap)
    phi = out["phi"].cpu().numpy()
    assert np.max(np.abs(phi - x_o)) < 1e-11 * np.max(np.abs(x_o))
    np.testing.assert_allclose(out["rel_resid"], np.linalg.norm(f - A @ phi) / np.linalg.norm(f), rtol=1e-8)
    # four vectors, three times the most partials, the 1D tables, the charge
    tables = n * (2 * p + 1) * 8 + 2 * n * 8
    stencil = -(-n // 64) * -(-n_el // 2) * -(-n_el // 2)
    assert c.device_bytes() - before <= 4 * nd * 8 + 3 * 8 * max(2048, stencil) + tables + 4096
    c.close()
