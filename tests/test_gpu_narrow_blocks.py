"""The library's blocks for a few columns of a large mesh take no more than three
blocks of that many columns (and 16 MiB), not whole groups of 16 or 32, and give the
bits of the same columns in a wide block."""
import numpy as np
import pytest

import workload
from gpu_util import make_ctx, to_gpu, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [2, 5, 7])
@pytest.mark.parametrize("w", [1, 9, 10, 11, 17, 21, 22, 32, 33, 42, 43])
def test_memory_and_bits_of_narrow_blocks(p, w):
    n_el, L = 66 // p, 12.0
    wells = workload.draw_wells(3, L, 3, (1.0, 2.0), (0.4, 0.5))
    X = workload.start_block((n_el * p - 1) ** 3, 96, 870 + p)
    for prec, elem in (("fp64", 8), ("fp32", 4), ("bf16", 4)):
        c, _ = make_ctx(L, n_el, p, wells=wells)
        held, b = c.device_bytes(), c.upper_bound
        A = to_gpu(X[:, :w], w + 1)
        c.chebyshev_filter(A, 5, 3.0, b, -1.0, prec=prec)
        assert c.device_bytes() - held <= 3 * c.n_dof * w * elem + (16 << 20) + 4096
        B = to_gpu(X)                                # one block of 96 columns, whole groups
        c.chebyshev_filter(B, 5, 3.0, b, -1.0, prec=prec)
        np.testing.assert_array_equal(to_host(A), to_host(B)[:, :w])
        if prec != "fp64":
            Y = to_host(c.apply(to_gpu(X[:, :w]), prec=prec))
            np.testing.assert_array_equal(Y, to_host(c.apply(to_gpu(X), prec=prec))[:, :w])
        c.close()
