"""The weight gradient on rows of at most 8 voxels, where the two halves of a wave take neighbouring rows: odd and even
row counts, fewer rows than a step's 8 and more, chunks of several planes, rows filled up to 8; against the oracle
(tolerance: FP32 sums of at most 8192 products of BF16 values, relative to the norm, below sqrt(n) eps = 1e-5)."""
import numpy as np
import pytest
import torch

import paper_1601_00035_amd.surrogate as S
from oracle import conv3d as C
from test_gpu_surrogate import DEV, rand_bf16, rel, to_bf16_bits

pytestmark = pytest.mark.gpu


def _run(x, gy, cin, cout):
    D, H, W = x.shape[:3]
    work = torch.full((S.lib().sur_bwd_weight_work_bytes(D, H, W, cin, cout) // 4 + 1,), float("nan"), device=DEV)
    gw = torch.full((27 * cout * cin + 8,), float("nan"), dtype=torch.float32, device=DEV)
    S.call("sur_conv3d_bwd_weight", to_bf16_bits(gy), to_bf16_bits(x), gw, work, D, H, W, cin, cout)
    assert torch.isnan(gw[-8:]).all()
    return gw[:-8].double().cpu().numpy().reshape(27, cout, cin)


@pytest.mark.parametrize("dims,cin,cout", [((8, 8, 8), 96, 128), ((64, 8, 8), 32, 64), ((4, 1, 8), 16, 32),
                                           ((32, 3, 8), 32, 32), ((4, 9, 8), 64, 32), ((12, 17, 8), 32, 32),
                                           ((4, 40, 8), 32, 32), ((1, 128, 8), 16, 32), ((4, 4, 4), 96, 128),
                                           ((16, 10, 6), 32, 32), ((32, 15, 1), 32, 32), ((5, 32, 7), 16, 32)])
def test_narrow_rows(dims, cin, cout):
    x, gy = rand_bf16(dims + (cin,), 3), rand_bf16(dims + (cout,), 5)
    ref = C.conv_bwd_weight(gy, x)
    assert rel(_run(x, gy, cin, cout).reshape(ref.shape), ref) < 1e-5


@pytest.mark.parametrize("H", [7, 8])
@pytest.mark.parametrize("W", [5, 8])
def test_infinity_in_the_last_row(H, W):
    """An infinite input in a plane's last row and voxel reaches the taps that pair it with a voxel of the volume, and
    no row beyond the volume makes it NaN in the others."""
    D, cin, cout = 32, 32, 32
    x, gy = rand_bf16((D, H, W, cin), 3), rand_bf16((D, H, W, cout), 5)
    x[3, H - 1, W - 1, 0] = np.inf
    gy[gy == 0] = 1.0
    bad = ~np.isfinite(_run(x, gy, cin, cout))
    want = np.zeros_like(bad)
    for t in range(27):  # partner v - off
        dz, dy, dx = t // 9 - 1, t // 3 % 3 - 1, t % 3 - 1
        want[t, :, 0] = 0 <= 3 - dz < D and 0 <= H - 1 - dy < H and 0 <= W - 1 - dx < W
    assert np.array_equal(bad, want)
