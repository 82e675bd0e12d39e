"""BF16 products round what the off-diagonal entries multiply and nothing else:
the potential and the shift act on the FP32 values."""
import numpy as np
import pytest

from oracle import fem
import workload
from gpu_util import make_ctx, oracle_apply, to_gpu, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [1, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("n_el,ncols", [(3, 17), (9, 70)])      # launches below and above one work-group per CU
def test_deep_potential_keeps_fp32_accuracy(n_el, p, ncols):
    """|error| <= 2^-8 sum_off |A||x| (BF16 rounding) + g 2^-24 sum |A||x| (FP32
    coefficients, inputs and g - 4 sums), under a potential a thousand times the
    off-diagonal entries: rounding the diagonal's value would exceed it."""
    L = 4.0 * n_el
    A = fem.operator_1d(L, n_el, p)
    off = np.abs(A) - np.diag(np.abs(np.diag(A)))
    nd = A.shape[0] ** 3
    V = -1000.0 * np.abs(off).sum(1).max() * (1.0 + np.random.default_rng(p).random(nd))
    c, _ = make_ctx(L, n_el, p, V=V)
    X = workload.start_block(nd, ncols, 800 + p)
    Y = oracle_apply(L, n_el, p, V)(X)
    noff = fem.apply_kron(off, np.zeros(nd), np.abs(X))
    dg = np.abs(np.diag(A))
    kin = (dg[:, None, None] + dg[None, :, None] + dg[None, None, :]).reshape(-1)
    ndia = (kin + np.abs(V))[:, None] * np.abs(X)
    tol = 2.0 ** -8 * noff + (3 * (2 * p + 2) + 4) * 2.0 ** -24 * (noff + ndia)
    for v in (-1, 0):
        c.set_tile_variant(v)
        err = np.abs(to_host(c.apply(to_gpu(X), prec="bf16")) - Y)
        assert np.all(err <= tol), np.max(err / tol)
    c.close()
