"""Where the block weights' results lie on their way to the host: in pinned memory of the handle where they are
few, in device memory where they are many (blocks of one or two cells on a large box), with the same values."""
import ctypes

import numpy as np
import pytest
import torch

import paper_1601_00035_amd as nslgf

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info(0)[0]


def test_many_block_weights_do_not_stay_in_pinned_memory():
    n = 160
    g = torch.Generator().manual_seed(0)
    u = torch.randn((3, n, n, n), generator=g, dtype=torch.float64).to(DEV)
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    nslgf.block_weights(u, 0.1, 16, 2)  # (kernels loaded)
    L = nslgf.lib()
    h = ctypes.c_void_p()
    assert L.nslgf_create(ctypes.byref(h), 0) == 0
    out = {}
    try:
        start = _free()
        for nb in (16, 8, 2, 1):
            m = n // nb
            mu, nu = np.zeros((m, m, m)), np.zeros((m, m, m))
            assert L.block_weights(h, u.data_ptr(), n, n, n, nb, 2, ctypes.c_double(0.1), 0, mu.ctypes.data,
                                   nu.ctypes.data, stream) == 0
            out[nb] = (mu, nu)
            used = start - _free()
            if 2 * mu.nbytes <= 4 << 20:
                assert used < 4 << 20, (nb, used)
            else:
                assert used >= 2 * mu.nbytes, (nb, used)
    finally:
        L.nslgf_destroy(h)
    assert _free() >= start - (4 << 20)  # given back
    # the weights of larger blocks are the maxima of the smaller ones in them
    for nb in (16, 8, 2):
        m = n // nb
        for coarse, fine in zip(out[nb], out[1]):
            assert np.array_equal(coarse, fine.reshape(m, nb, m, nb, m, nb).max(axis=(1, 3, 5)))
