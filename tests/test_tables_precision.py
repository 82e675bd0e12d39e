"""The 1D tables behind the operators are correctly rounded, not only consistent:
entries of the exported cell matrix against 50-digit decimal arithmetic.  (Host
tables, no device calls.)"""
from decimal import Decimal, getcontext

import numpy as np
import pytest

getcontext().prec = 50


def _legendre(k, x):
    a, b = Decimal(1), x
    if k == 0:
        return a
    for i in range(1, k):
        a, b = b, ((2 * i + 1) * x * b - i * a) / (i + 1)
    return b


def _gll(p):
    """Nodes (bisection on P_{p+1} - P_{p-1}, whose sign changes once between the
    rounded neighbours of the library's nodes), weights and derivative matrix."""
    from oracle import fem
    x0 = fem.gll(p)[0]
    f = lambda x: _legendre(p + 1, x) - _legendre(p - 1, x)
    x = [Decimal(-1)]
    for k in range(1, p):
        lo, hi = Decimal(float(x0[k])) - Decimal("1e-12"), Decimal(float(x0[k])) + Decimal("1e-12")
        s = f(lo) > 0
        assert (f(hi) > 0) != s
        for _ in range(130):
            mid = (lo + hi) / 2
            if (f(mid) > 0) == s:
                lo = mid
            else:
                hi = mid
        x.append(mid)
    x.append(Decimal(1))
    lp = [_legendre(p, v) for v in x]
    w = [2 / (p * (p + 1) * v * v) for v in lp]
    D = [[lp[i] / (lp[j] * (x[i] - x[j])) if i != j else Decimal(0) for j in range(p + 1)] for i in range(p + 1)]
    D[0][0], D[p][p] = Decimal(-p * (p + 1)) / 4, Decimal(p * (p + 1)) / 4
    return w, D


@pytest.mark.parametrize("p", range(1, 13))
def test_cell_matrix_entries_are_exact_to_the_rounding_of_their_factors(p):
    """A coupling along x inside a cell is 1/2 (h/2) K1 w w: three rounded table
    entries and four products, at most 7 half units of rounding (2^-53 each)."""
    import paper_1903_10959_amd as P
    c = P.Context(device=-1).set_mesh(4.0, 2, p)     # h/4 = 0.5, exact
    K = c.cell_matrix()
    c.close()
    w, D = _gll(p)
    q = p + 1
    worst = 0
    for a in range(q):
        for b in range(q):
            if a == b:
                continue
            k1 = sum(w[i] * D[i][a] * D[i][b] for i in range(q))
            for t in (0, p // 2):
                ref = Decimal("0.5") * k1 * w[t] * w[p]
                got = Decimal(float(K[a + q * t + q * q * p, b + q * t + q * q * p]))
                worst = max(worst, abs(got - ref) / abs(ref))
    assert worst <= Decimal(7 * 2.0 ** -53), float(worst)
