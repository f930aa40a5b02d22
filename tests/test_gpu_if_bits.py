"""The two forms of the fused x-y integrating-factor pass (the walk and the tiles) give the same bits for every
input they form: plain, combined and projected.  Which one a step takes depends on how many problems share a launch
and on the rows per workgroup, so a batch of many equal boxes must equal single steps, and every row choice of
the tuner the default, at boxes whose tiles are wider than a wave less the halo (64 columns) and narrower."""
import json

import pytest
import torch

import paper_1601_00035_amd as nslgf

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _field(shape, seed, dtype):
    g = torch.Generator().manual_seed(seed)
    return (0.1 * torch.randn((3,) + shape, generator=g, dtype=torch.float64)).to(DEV, dtype)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("scheme", ["A", "C"])
def test_many_equal_boxes_step_as_single_ones(dtype, scheme):
    """32 boxes of 64^3 walk where a single one takes tiles; two steps, the second on the captured graph."""
    single, batch = [], []
    for seed in range(32):
        u = _field((64, 64, 64), seed, dtype)
        single.append(nslgf.HerkState(u.clone(), 0.1, 0.01, 200.0, scheme, n_buf=2))
        batch.append(nslgf.HerkState(u, 0.1, 0.01, 200.0, scheme, n_buf=2))
    for step in range(2):
        for st in single:
            st.step()
        nslgf.herk_step_batched(batch)
        assert nslgf.batch_info()[0] == 1  # one group: every launch is shared
        for i, (a, b) in enumerate(zip(single, batch)):
            assert torch.equal(a.u, b.u) and torch.equal(a.d, b.d), (step, i)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("box,padded", [((120, 116, 118), 256), ((70, 127, 126), 256)])
def test_row_choices_step_alike(tmp_path, dtype, box, padded):
    """32 rows per workgroup walk at these boxes (nx, ny, nz), 64 and more take tiles."""
    nx, ny, nz = box
    px = 160 if nx == 70 else padded
    entry = {"nx": nx, "ny": ny, "nz": nz, "dtype": "f64" if dtype == torch.float64 else "f32", "Px": px, "Py": padded,
             "Pz": padded, "vy": -1, "vz": -1, "launch": 1, "if_seg": 16, "cell_shape": 0}
    path = tmp_path / "t.json"
    u0 = _field((nz, ny, nx), nx, dtype)

    def run(rows, launch=1):
        path.write_text(json.dumps({"format": "nslgf-tuning-1", "entries": [dict(entry, if_rows=rows, launch=launch)]}))
        nslgf.tuning_load(str(path))
        st = nslgf.HerkState(u0.clone(), 0.1, 0.01, 200.0, "C", n_buf=2)
        st.step()
        return st.u, st.d, st.work[:12 * nx * ny * nz * u0.element_size()]  # q, w1, w2, r

    try:
        ref = run(32)
        for rows in (64, 128, 256):
            for a, b in zip(run(rows), ref):
                assert torch.equal(a, b), rows
    finally:
        run(32, launch=0)  # back to the defaults on the process's handle


@pytest.mark.parametrize("alpha", [1e-9, 1e-6, 1e-4, 0.01, 0.2])
def test_radii_from_one_point_walk_as_they_tile(alpha):
    """Radii 1 to 12 (FP64): one component takes tiles, six walk."""
    g = torch.Generator().manual_seed(3)
    h = torch.randn((6, 230, 35, 70), generator=g, dtype=torch.float64).to(DEV)
    both = nslgf.if_apply(h, alpha)
    assert torch.equal(nslgf.if_apply(h[4:5].contiguous(), alpha)[0], both[4])
