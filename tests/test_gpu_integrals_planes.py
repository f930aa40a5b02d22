"""The ring integrals where a workgroup walks few planes (small boxes): plane counts around the split's four planes and
its 256 workgroups, against the oracle (tolerances as for the tiles' edges: 1e-12 of the sums' scale)."""
import numpy as np
import pytest
import torch

import paper_1601_00035_amd as nslgf
import workloads
from oracle import diagnostics

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("shape", [(1, 6, 9), (4, 15, 31), (5, 16, 32), (9, 33, 70), (23, 61, 40), (49, 31, 93),
                                   (66, 16, 250)])
def test_integrals_few_planes(shape):
    u = workloads.random_field((3,) + shape, 8)
    dx, origin = 0.1, (-1.3, 0.4, 0.2)
    t = torch.from_numpy(u).to(DEV)
    for n_buf in (0, 1):
        ref = diagnostics.of_velocity(u, dx, origin, n_buf)
        got = nslgf.flow_diagnostics(t, dx, origin, n_buf)
        w2 = np.sqrt(2 * ref["E"] * dx ** 3 * np.prod(shape))  # scale of the sums (terms of both signs)
        far = np.abs(np.array(shape) * dx).sum() + 2  # (largest coordinate)
        assert np.abs(np.array(got["I"]) - np.array(ref["I"])).max() <= 1e-12 * w2 * 10 * far
        for k, s in (("K", np.abs(u).max() * w2 * 10 * far), ("E", ref["E"]), ("J", np.abs(u).max() * w2 * 10)):
            assert abs(got[k] - ref[k]) <= 1e-12 * s, (k, n_buf)
