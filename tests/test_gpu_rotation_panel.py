"""Rotations of more than 624 columns over more rows than one scratch panel holds:
216,000 x 640 values are 1.03 panels of 2^27, so a second, ragged chunk of rows runs,
for the triangular factor (FP64 and mixed) and for the full one."""
import numpy as np
import pytest

from oracle import chfsi as och
import workload
from gpu_util import make_ctx, oracle_apply, to_gpu, to_host

pytestmark = pytest.mark.gpu


def test_cholgs_and_rayleigh_ritz_over_two_row_chunks():
    n_el, p, ncols = 61, 1, 640
    L = 0.6 * n_el
    nd = (n_el * p - 1) ** 3
    assert nd * ncols > 1 << 27 and nd % 128
    V = np.random.default_rng(4).uniform(-3, 1, nd)
    c, _ = make_ctx(L, n_el, p, V=V)
    X = workload.start_block(nd, ncols, 32)
    kappa = np.linalg.cond(X[:: 50])                 # (a random block's is that of its parts)
    Xo = och.cholgs(X)
    Xg = to_gpu(X)
    c.orthonormalize(Xg)
    got = to_host(Xg)
    assert np.max(np.abs(got - Xo)) < 1e-13 * kappa ** 2
    Xm = to_gpu(X)
    c.orthonormalize(Xm, mixed=True)
    assert np.max(np.abs(to_host(Xm) - Xo)) < 4e-7 * kappa ** 2
    del Xm
    H = oracle_apply(L, n_el, p, V)
    D = np.linalg.eigvalsh(got.T @ H(got))
    ev, rs = c.rayleigh_ritz(Xg)
    scale = c.upper_bound
    assert np.max(np.abs(ev - D)) < 1e-13 * scale * kappa ** 2
    Y = to_host(Xg)
    Q = got.T @ Y                                    # the rotation: Y = X Q, row by row
    assert np.max(np.abs(Q.T @ Q - np.eye(ncols))) < 1e-12
    assert np.max(np.abs(got @ Q - Y)) < 1e-13 * np.sqrt(ncols)
    res = np.linalg.norm(H(Y) - Y * ev[None, :], axis=0)
    assert np.max(np.abs(rs - res)) < 1e-13 * scale * np.sqrt(ncols)
    c.close()
