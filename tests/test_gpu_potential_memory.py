"""A potential announced as the device's but lying elsewhere: pinned host memory is
copied (another device's memory takes the same way), memory that the runtime does
not know is refused; no kernel of this device reads either."""
import ctypes as C

import numpy as np
import pytest

import workload
from gpu_util import make_ctx, to_gpu, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_el,p", [(1, 2), (5, 4)])
def test_potential_outside_the_device(n_el, p):
    import torch
    nd = (n_el * p - 1) ** 3
    V = np.random.default_rng(11).uniform(-9, -1, nd)
    c, _ = make_ctx(3.0, n_el, p, V=V)
    X = workload.start_block(nd, 3, 12)
    ub, Y = c.upper_bound, to_host(c.apply(to_gpu(X)))

    def set_as_device(t):
        return c._lib.chfsi_set_potential(c._h, C.c_void_p(t.data_ptr()), nd, 1)

    def unchanged():
        assert c.upper_bound == ub
        np.testing.assert_array_equal(to_host(c.apply(to_gpu(X))), Y)

    pinned = torch.empty(nd, dtype=torch.float64, pin_memory=True)
    pinned.copy_(torch.from_numpy(V))
    c.set_potential(np.zeros(nd))
    assert set_as_device(pinned) == 0
    unchanged()
    pinned[nd // 2] = float("nan")
    assert set_as_device(pinned) == -1
    unchanged()
    assert set_as_device(torch.zeros(nd, dtype=torch.float64)) == -4
    unchanged()
    c.close()
