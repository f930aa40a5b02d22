"""The BF16 cast over the widths that take different tiles with the blocked copy (64 channels where they divide the
width, else 32), and, without it, counts of values around a workgroup's 2048: bit for bit the separate casts, NaN
and infinities too."""
import pytest
import torch

import paper_1601_00035_amd.surrogate as S

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("nv,c", [(8, 64), (72, 64), (64, 128), (136, 192), (16, 72), (32, 64), (40, 56), (8, 1024),
                                  (1040, 64), (2056, 40)])
@pytest.mark.parametrize("use_act", [False, True])
def test_cast_widths(nv, c, use_act):
    g = torch.Generator(device=DEV).manual_seed(nv + c)
    src = torch.randn(nv * c, generator=g, device=DEV)
    src[::17], src[5::31] = float("inf"), float("nan")
    act = torch.randn(nv * c, generator=g, device=DEV)
    act[::13], act[1::19] = float("nan"), 0.0
    ref, ref_b, ref_k = src.clone(), S.bf16_empty(nv * c, DEV), S.bf16_empty(nv * c, DEV)
    if use_act:
        S.call("sur_relu_bwd", act, ref, nv * c)
    S.call("sur_cast_bf16", ref, ref_b, nv * c)
    S.call("sur_to_blocked8", ref_b, ref_k, nv, c)
    for blocked in (True, False):
        y, yk = (torch.full((nv * c + 8,), 77, dtype=torch.int16, device=DEV) for _ in range(2))
        S.call("sur_cast_bf16_ex", src, act if use_act else None, y, yk if blocked else None, nv, c)
        assert torch.equal(y[:-8], ref_b.view(torch.int16))
        assert torch.equal(yk[:-8], ref_k.view(torch.int16) if blocked else torch.full_like(yk[:-8], 77))
        assert (y[-8:] == 77).all() and (yk[-8:] == 77).all()
