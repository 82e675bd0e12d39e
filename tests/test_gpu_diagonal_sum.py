"""The operator's diagonal, read off as one step applied to the identity: the three
directions' entries, the potential and a shift that cancels most of them are added
with no rounding but those of the potential's addition and of the result."""
import ctypes as C
from decimal import Decimal

import numpy as np
import pytest

from gpu_util import make_ctx
from test_tables_precision import _gll

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [1, 2, 3, 4, 5, 6, 7, 8, 9])
def test_diagonal_is_rounded_once_besides_the_potential(p):
    import torch
    n_el, L = (3, 7.1) if p < 6 else (2, 5.3)
    n = n_el * p - 1
    nd = n ** 3
    V = np.random.default_rng(p).uniform(-2, -1, nd)
    c, _ = make_ctx(L, n_el, p, V=V)
    w, D = _gll(p)
    h = Decimal(L / n_el)
    # A's diagonal at node a of an element, 1/2 (2/h) K1[a][a] / ((h/2) w[a]): at an
    # element's end both halves of it over both halves of the mass
    d = [2 * sum(w[i] * D[i][a] ** 2 for i in range(p + 1)) / (h * h * w[a]) for a in range(p)]
    line = [d[(i + 1) % p] for i in range(n)]
    X = torch.eye(nd, dtype=torch.float64, device="cuda:0")
    Y = torch.empty_like(X)
    for shift in (0.5 * c.upper_bound, 1.5 * float(max(d)), float(d[0]) - 0.3):
        st = c._lib.chfsi_cheb_step(c._h, C.c_void_p(X.data_ptr()), C.c_void_p(0), C.c_void_p(Y.data_ptr()), nd, nd,
                                    C.c_double(1.0), C.c_double(0.0), C.c_double(shift))
        assert st == 0
        got = torch.diagonal(Y).cpu().numpy().reshape(n, n, n)
        u = Decimal(2.0 ** -53)
        for k in range(n):
            for j in range(n):
                for i in range(n):
                    v = Decimal(V[i + n * (j + n * k)])
                    ref = line[i] + line[j] + line[k] - Decimal(shift) + v
                    tol = u * (abs(ref) + abs(v)) * Decimal("1.001") + u * max(d) * Decimal(2.0 ** -44)
                    assert abs(Decimal(got[k, j, i]) - ref) <= tol, (i, j, k)
    c.close()
