"""A batch of projected eigenproblems of which one is done at the very check at which
the others run out of sweeps: the done one's pairs are right, the others are
reported unconverged, and the next eigensolve of the same session starts clean."""
import numpy as np
import pytest

from oracle import chfsi as och
import workload
from gpu_util import make_ctx, oracle_apply, to_gpu

pytestmark = pytest.mark.gpu


def test_last_check_with_one_problem_done_and_the_others_out_of_sweeps():
    import paper_1903_10959_amd as P
    L, n_el, p = 6.0, 3, 4
    wells = workload.draw_wells(3, L, 33, (1.0, 2.0), (0.4, 0.5))
    sizes = (2, 100, 130)                            # two columns: one rotation
    ctxs, blocks, exact = [], [], []
    for i, nb in enumerate(sizes):
        c, V = make_ctx(L, n_el, p, wells=wells)
        c.set_jacobi_sweeps(1)
        X = workload.start_block(c.n_dof, nb, 340 + i)
        exact.append(och.rayleigh_ritz(oracle_apply(L, n_el, p, V), och.cholgs(X))[2])
        ctxs.append(c)
        blocks.append(X)
    sess = P.BatchSession(0)
    for sweeps in (1, 40):
        for c in ctxs:
            c.set_jacobi_sweeps(sweeps)
        ids = [sess.add(c, to_gpu(X), X.shape[1], 4, 1e9, max_iter=0) for c, X in zip(ctxs, blocks)]
        out = sess.run()
        for i, (pid, D) in enumerate(zip(ids, exact)):
            done = sweeps > 1 or i == 0
            assert out[pid]["converged"] == done
            if done:
                np.testing.assert_allclose(out[pid]["evals"], D, rtol=0, atol=1e-12 * np.max(np.abs(D)))
            else:
                assert np.all(np.isfinite(out[pid]["evals"]))
    sess.close()
    for c in ctxs:
        c.close()
