"""The tiled x-y pass of the integrating factor (small launches) at the edges of its tiles: rows of 63, 64,
65, 128 and 129 points, 31 to 33 and 65 rows, odd widths; against the oracle, and bit for bit against the
walking pass, which the same fields take when more components fill the chip; and the passes of wide radii
(FP64, 13 to 24 points)."""
import numpy as np
import pytest
import torch

import paper_1601_00035_amd as nslgf
import workloads
from oracle import intfac

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("ny,nx", [(31, 63), (32, 64), (33, 65), (65, 20), (5, 129), (34, 3)])
@pytest.mark.parametrize("alpha", [1e-7, 0.02, 0.2])
def test_tile_edges_against_oracle(ny, nx, alpha):
    h = workloads.random_field((1, 3, ny, nx), ny + nx)
    ref = intfac.apply(h[0], alpha)
    for dtype, tol in ((torch.float64, 1e-13), (torch.float32, 1e-6)):
        out = nslgf.if_apply(torch.from_numpy(h).to(DEV, dtype), alpha).double().cpu().numpy()[0]
        assert np.abs(out - ref).max() < tol * np.abs(ref).max(), (dtype, alpha)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("ny,nx", [(33, 65), (40, 64), (63, 130)])
def test_tile_equals_walk(dtype, ny, nx):
    g = torch.Generator().manual_seed(5)
    h = torch.randn((6, 220, ny, nx), generator=g, dtype=torch.float64).to(DEV, dtype)
    for alpha in (0.004, 0.02, 0.1):
        both = nslgf.if_apply(h, alpha)
        for q in (0, 5):
            assert torch.equal(nslgf.if_apply(h[q:q + 1].contiguous(), alpha)[0], both[q]), (alpha, q)


@pytest.mark.parametrize("alpha", [0.25, 0.55, 1.35])
@pytest.mark.parametrize("shape", [(5, 37, 7), (33, 6, 65), (3, 4, 130)])
def test_wide_radii_against_oracle(shape, alpha):
    """Radii of 13 to 24 points (FP64), wider than the box along some axis, odd rows, the ends of the z pass's
    32-point segments."""
    h = workloads.random_field((2,) + shape, 11)
    ref = np.stack([intfac.apply(h[q], alpha) for q in range(2)])
    out = nslgf.if_apply(torch.from_numpy(h).to(DEV), alpha).cpu().numpy()
    assert np.abs(out - ref).max() < 1e-13 * np.abs(ref).max()
