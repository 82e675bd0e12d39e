"""The filter's recursion factors are correctly rounded: the filtered block equals,
bit for bit, the one of the recursion driven step by step through chfsi_cheb_step
with factors from 40-digit arithmetic (a step's values do not depend on the layout
of its blocks)."""
import ctypes as C
from decimal import Decimal, getcontext

import numpy as np
import pytest

import workload
from gpu_util import make_ctx, to_gpu, to_host

pytestmark = pytest.mark.gpu
getcontext().prec = 40


def _factors(a, b, a0, degree):
    a, b, a0 = Decimal(a), Decimal(b), Decimal(a0)
    c, e = (a + b) / 2, (b - a) / 2
    xi0 = (a0 - c) / e
    rho, out = Decimal(0), []
    for k in range(degree):
        nxt = 1 / (xi0 if k == 0 else 2 * xi0 - rho)
        out.append((float((1 if k == 0 else 2) * nxt / e), float(-nxt * rho), float(c)))
        rho = nxt
    return out


@pytest.mark.parametrize("p,degree,a,a0", [(3, 20, 3.1, -1.7), (5, 30, 4.3, -0.9), (6, 21, 2.7, -2.3), (9, 15, 3.3, -1.1)])
def test_filter_equals_the_recursion_with_exact_factors(p, degree, a, a0):
    import torch
    n_el, L, ncols = 3, 7.3, 20
    c, _ = make_ctx(L, n_el, p, wells=workload.draw_wells(3, L, 40 + p, (1.0, 2.0), (0.4, 0.5)))
    X = to_gpu(workload.start_block(c.n_dof, ncols, 860 + p))
    b = c.upper_bound
    cur, prev = X.clone(), None
    for s1, s2, sh in _factors(a, b, a0, degree):
        out = torch.empty_like(cur)
        st = c._lib.chfsi_cheb_step(c._h, C.c_void_p(cur.data_ptr()), C.c_void_p(prev.data_ptr() if prev is not None else 0),
                                    C.c_void_p(out.data_ptr()), ncols, ncols, C.c_double(s1), C.c_double(s2), C.c_double(sh))
        assert st == 0
        prev, cur = cur, out
    c.chebyshev_filter(X, degree, a, b, a0)
    np.testing.assert_array_equal(to_host(X), to_host(cur))
    c.close()
