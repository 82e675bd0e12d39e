"""The cell-wise Poisson product at the edges of its tiles, against the oracle's
matrix: every degree, meshes of one cell, of fewer cells than a work-group takes
and of a last one by itself, rows that end within the first, at and just beyond
a wave's 64 nodes, and meshes large enough for two cell layers per work-group
with an odd number of layers."""
import numpy as np
import pytest

import paper_1903_10959_amd as P
from oracle import poisson

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_el,p", [(1, 2), (1, 7), (2, 2), (3, 1), (5, 2), (7, 3), (65, 1), (66, 1), (13, 5), (11, 6),
                                    (9, 7), (41, 2)])
def test_product_and_solve_at_tile_edges(n_el, p):
    """The product to the roundoff of its sums; the solve to its tolerance, in the
    oracle's number of iterations (the same recurrences, summed in other orders:
    within one)."""
    L = 0.8 * n_el
    c = P.Context(0).set_mesh(L, n_el, p)
    import torch
    A, M = poisson.poisson_matrix(L, n_el, p)
    rng = np.random.default_rng(10 * n_el + p)
    x = rng.standard_normal(c.n_dof)
    y = c.poisson_apply(torch.from_numpy(x).to("cuda:0")).cpu().numpy()
    yo = A @ x
    assert np.max(np.abs(y - yo)) < 1e-13 * np.max(np.abs(yo))
    if c.n_dof > 50000:                              # the oracle solves these in seconds
        return
    rho = rng.uniform(-1, 0, c.n_dof)
    out = c.poisson_solve(torch.from_numpy(rho).to("cuda:0"), tol=1e-9)
    f = poisson.load_vector(M, rho, [], [])
    x_o, it_o, _ = poisson.jacobi_pcg(A, f, tol=1e-9)
    assert out["converged"] and abs(out["iters"] - it_o) <= 1
    r = np.linalg.norm(f - A @ out["phi"].cpu().numpy()) / np.linalg.norm(f)
    assert r <= 2e-9
    c.close()
