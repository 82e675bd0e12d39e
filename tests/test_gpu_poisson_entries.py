"""Entries of the Poisson operator, read off as products with unit vectors, are exact
to the rounding of their factors: a coupling along one line is 1/(4 pi), three masses
and a table entry, each rounded, in four products, at most nine half units (2^-53
each)."""
from decimal import Decimal, getcontext

import numpy as np
import pytest

from oracle import fem

pytestmark = pytest.mark.gpu
getcontext().prec = 50
PI = Decimal("3.14159265358979323846264338327950288419716939937511")


def _legendre(k, x):
    a, b = Decimal(1), x
    if k == 0:
        return a
    for i in range(1, k):
        a, b = b, ((2 * i + 1) * x * b - i * a) / (i + 1)
    return b


def _gll(p):
    """Weights and derivative matrix; the nodes by bisection on P_{p+1} - P_{p-1}."""
    f = lambda x: _legendre(p + 1, x) - _legendre(p - 1, x)
    x = [Decimal(-1)]
    for x0 in fem.gll(p)[0][1:p]:
        lo, hi = Decimal(float(x0)) - Decimal("1e-12"), Decimal(float(x0)) + Decimal("1e-12")
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


@pytest.mark.parametrize("p", [1, 2, 3, 4, 5, 6, 7])
def test_couplings_along_lines(p):
    import torch
    import paper_1903_10959_amd as P
    n_el, L = 3, 6.0                                 # h = 2
    c = P.Context(0).set_mesh(L, n_el, p)
    n = n_el * p - 1
    w, D = _gll(p)
    q = p + 1
    K1 = [[sum(w[i] * D[i][a] * D[i][b] for i in range(q)) for b in range(q)] for a in range(q)]
    n1 = n_el * p + 1
    K = [[Decimal(0)] * n1 for _ in range(n1)]
    m = [Decimal(0)] * n1
    for e in range(n_el):
        for a in range(q):
            m[e * p + a] += w[a]
            for b in range(q):
                K[e * p + a][e * p + b] += K1[a][b]
    worst = Decimal(0)
    j, k = n // 2, n - 1
    for i in range(n):
        for axis in range(3):                        # the unit vector at i on a line along each axis
            pos = [j, j, k]
            pos[axis] = i
            x = torch.zeros(c.n_dof, dtype=torch.float64, device="cuda:0")
            x[pos[0] + n * (pos[1] + n * pos[2])] = 1.0
            y = c.poisson_apply(x).cpu().numpy().reshape(n, n, n)
            for r in range(n):
                if r == i or abs(r - i) > p:
                    continue
                at = list(pos)
                at[axis] = r
                others = [at[d] for d in range(3) if d != axis]
                ref = K[r + 1][i + 1] * m[others[0] + 1] * m[others[1] + 1] / (4 * PI)
                got = Decimal(float(y[at[2], at[1], at[0]]))
                if ref == 0:
                    assert got == 0
                else:
                    worst = max(worst, abs(got - ref) / abs(ref))
    assert worst <= Decimal(9 * 2.0 ** -53), float(worst)
    c.close()
