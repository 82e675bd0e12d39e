"""What a batch member is admitted by: the two blocks its recursion alternates and HX,
with the workspaces that do not grow with the mesh.  (Host arithmetic, no device
calls; the device's side is compared with it where a GPU is.)"""
import pytest


@pytest.mark.parametrize("n_el,p,nb", [(20, 7, 288), (32, 5, 320), (16, 6, 1024)])
def test_batch_footprint_counts_two_recursion_blocks(n_el, p, nb):
    import paper_1903_10959_amd as P
    nd = (n_el * p - 1) ** 3
    block = nd * nb * 8
    # rotation panel 1 GiB, Gram partials 2,048 tiles of 128 KiB, a dozen nb x nb matrices
    small = (1 << 30) + (2048 << 17) + 12 * nb * nb * 8 + (64 << 20)
    fb = P.batch_footprint_bytes(n_el, p, nb)
    assert 3 * block < fb <= 3 * block + 16 * nd + small
