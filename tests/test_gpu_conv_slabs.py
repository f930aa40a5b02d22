"""The convolutions on volumes of few planes, which take two planes a workgroup: one to ten planes, rows and columns
that end inside a block, one and several channel slices, against the oracle (tolerance: FP32
sums of at most 27 * 128 products of BF16 values, relative to the norm, below sqrt(n) eps = 1e-5)."""
import numpy as np
import pytest
import torch

import paper_1601_00035_amd.surrogate as S
from oracle import conv3d as C
from test_gpu_surrogate import DEV, rand_bf16, rel, to_bf16_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,cin,cout", [((1, 143, 96), 32, 32), ((2, 33, 128), 16, 96), ((2, 64, 70), 48, 128),
                                           ((6, 64, 72), 32, 32), ((5, 32, 90), 64, 64), ((9, 32, 41), 16, 64),
                                           ((10, 48, 16), 16, 128)])
def test_slabs(dims, cin, cout):
    D, H, W = dims
    nv = D * H * W
    assert nv % 32 == 0
    x, w, gy = rand_bf16((D, H, W, cin), 3), rand_bf16((27, cout, cin), 4, 0.1), rand_bf16((D, H, W, cout), 5)
    xb, wb, gb = to_bf16_bits(x), to_bf16_bits(w), to_bf16_bits(gy)
    for relu in (0, 1):
        y = torch.full((nv * cout + 8,), float("nan"), dtype=torch.float32, device=DEV)
        S.call("sur_conv3d_fwd", xb, wb, y, D, H, W, cin, cout, relu)
        ref = C.conv_fwd(x, w)
        if relu:
            ref = np.maximum(ref, 0)
        got = y.double().cpu().numpy()
        assert np.isnan(got[-8:]).all()
        assert rel(got[:-8].reshape(ref.shape), ref) < 1e-5
    if cin % 32 == 0:
        wt = S.bf16_empty(w.size, DEV)
        S.call("sur_weight_transpose", wb, wt, cin, cout)
        gx = torch.full((nv * cin,), float("nan"), dtype=torch.float32, device=DEV)
        S.call("sur_conv3d_bwd_data", gb, wt, gx, D, H, W, cin, cout)
        refx = C.conv_bwd_data(gy, w)
        assert rel(gx.double().cpu().numpy().reshape(refx.shape), refx) < 1e-5
