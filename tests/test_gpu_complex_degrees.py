"""The complex operator stops at degree 7: every complex step on a periodic mesh
of a higher degree is refused and leaves its block as it was."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [8, 12])
def test_complex_steps_are_refused_above_degree_7(p):
    import torch
    import paper_1903_10959_amd as P
    c = P.Context(0).set_mesh(6.0, 2, p, periodic=True)
    c.set_potential(np.zeros(c.n_dof))
    X0 = torch.randn(c.n_dof, 3, dtype=torch.complex128, device="cuda:0")
    X = X0.clone()
    for call in (lambda: c.apply_complex(X), lambda: c.chebyshev_filter_complex(X, 4, 3.0, 200.0, -1.0),
                 lambda: c.rayleigh_ritz_complex(X), lambda: c.set_kpoint((0.1, 0.0, 0.0)),
                 lambda: c.set_kpoints(np.zeros((2, 3)))):
        with pytest.raises(P.ChfsiError) as ei:
            call()
        assert ei.value.status == -1
    assert torch.equal(X, X0)
    c.close()
