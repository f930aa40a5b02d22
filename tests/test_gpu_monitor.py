"""Block weights, ring integrals and the cell speed at the edges of their tiles: blocks of 1 to 256 cells
(several per tile, one, and parts of one), boxes of one tile, one more and one less along each axis."""
import numpy as np
import pytest
import torch

import paper_1601_00035_amd as nslgf
import workloads
from oracle import blocks, diagnostics, ifherk

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("nb", [1, 3, 8, 11, 16, 17, 33, 256])
@pytest.mark.parametrize("shape", [(19, 35, 33), (34, 16, 18)])
def test_block_weights_every_size(nb, shape):
    u = workloads.random_field((3,) + shape, 5)
    for n_buf in (0, 2):
        mu_r, nu_r = blocks.weights(u, 0.3, nb, n_buf)
        for dtype, tol in ((torch.float64, 1e-12), (torch.float32, 1e-5)):
            mu, nu = nslgf.block_weights(torch.from_numpy(u).to(DEV, dtype), 0.3, nb, n_buf)
            assert mu.shape == mu_r.shape and nu.shape == nu_r.shape
            assert np.abs(mu - mu_r).max() < tol * mu_r.max(), (n_buf, dtype)
            assert np.abs(nu - nu_r).max() < tol * nu_r.max(), (n_buf, dtype)


@pytest.mark.parametrize("shape", [(24, 15, 31), (25, 16, 32), (26, 31, 63), (3, 4, 5)])
def test_integrals_and_speed_tile_edges(shape):
    u = workloads.random_field((3,) + shape, 6)
    dx, origin = 0.1, (-1.3, 0.4, 0.2)
    t = torch.from_numpy(u).to(DEV)
    for n_buf in (0, 1):
        ref = diagnostics.of_velocity(u, dx, origin, n_buf)
        got = nslgf.flow_diagnostics(t, dx, origin, n_buf)
        w2 = np.sqrt(2 * ref["E"] * dx ** 3 * np.prod(shape))  # scale of the sums (terms of both signs)
        assert np.abs(np.array(got["I"]) - np.array(ref["I"])).max() < 1e-12 * w2 * 10
        for k, s in (("K", np.abs(u).max() * w2 * 10), ("E", ref["E"]), ("J", np.abs(u).max() * w2 * 10)):
            assert abs(got[k] - ref[k]) < 1e-12 * s, (k, n_buf)
    assert abs(nslgf.max_cell_speed(t) - ifherk.cell_speed_max(u)) < 1e-14 * ifherk.cell_speed_max(u)
