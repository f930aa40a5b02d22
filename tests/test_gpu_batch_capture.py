"""When a batch is captured: by the second of two calls in a row on it, and not again while it alternates with
another one."""
import pytest
import torch

import paper_1601_00035_amd as nslgf

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _states(sizes, seed):
    out = []
    for i, n in enumerate(sizes):
        g = torch.Generator().manual_seed(seed + i)
        u = (0.1 * torch.randn((3, n, n, n), generator=g, dtype=torch.float64)).to(DEV)
        out.append(nslgf.HerkState(u, 0.1, 0.01, 300.0, "A", n_buf=2))
    return out


@pytest.mark.parametrize("order,captures", [("aababababa", 1), ("abababab", 0), ("aabbabab", 2), ("aaabaabaa", 1)])
def test_captures_of_alternating_batches(order, captures):
    """order: the batch of each call."""
    sizes = {"a": (16, 20), "b": (24,)}
    batched = {k: _states(v, ord(k)) for k, v in sizes.items()}
    single = {k: _states(v, ord(k)) for k, v in sizes.items()}
    nslgf.herk_step_batched(_states((12,), 7))  # (nothing of what follows was stepped last)
    for k in "ab":
        for st in _states(sizes[k], 0):
            st.step()  # (plans exist)
    nslgf.profile_enable(True)
    try:
        for k in order:
            nslgf.herk_step_batched(batched[k])
        torch.cuda.synchronize()
        count = nslgf.profile_read().get("batch_capture", (0, 0.0))[0]
    finally:
        nslgf.profile_enable(False)
    for k in order:
        for st in single[k]:
            st.step()
    for k in "ab":
        for x, y in zip(batched[k], single[k]):
            assert torch.equal(x.u, y.u) and torch.equal(x.d, y.d)
    assert count == captures
