"""When a batch is captured: by the second of two calls in a row on it, and not again while it alternates with
another one."""
import pytest
import torch

import paper_1601_00035_amd as nslgf

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _states(sizes, seed, dt=0.01):
    out = []
    for i, n in enumerate(sizes):
        g = torch.Generator().manual_seed(seed + i)
        u = (0.1 * torch.randn((3, n, n, n), generator=g, dtype=torch.float64)).to(DEV)
        out.append(nslgf.HerkState(u, 0.1, dt, 300.0, "A", n_buf=2))
    return out


@pytest.mark.parametrize("order,captures", [("aababababa", 1), ("abababab", 0), ("aabbabab", 2), ("aaabaabaa", 1)])
def test_captures_of_alternating_batches(order, captures):
    """order: the batch of each call."""
    sizes = {"a": (16, 20), "b": (24,)}
    batched = {k: _states(v, ord(k)) for k, v in sizes.items()}
    single = {k: _states(v, ord(k)) for k, v in sizes.items()}
    nslgf.set_batch_mode(nslgf.BATCH_PER_PROBLEM)  # (drops the graph that an earlier batch left, whose states may
    nslgf.set_batch_mode(nslgf.BATCH_PASSES)       # have had these ones' memory and parameters)
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


def test_new_batch_is_refused_in_a_callers_capture():
    """A batch without a graph of its own would put the upload of its argument table, from memory that later
    calls write over, into the caller's graph.  It is refused; nothing is stepped, and the caller's capture and
    the handle go on."""
    a, ref = _states((16, 20), 1, 0.011), _states((16, 20), 1, 0.011)  # (a dt of their own: no graph serves them)
    for st in _states((16, 20), 0):
        st.step()  # (plans exist)
    x = torch.zeros(4, device=DEV)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        with pytest.raises(nslgf.NslgfError) as e:
            nslgf.herk_step_batched(a)
        x.add_(1.0)
    assert e.value.code == -5 and a[0].t == 0.0
    graph.replay()
    for i in range(6):  # (more calls than the handle has argument tables)
        nslgf.herk_step_batched(a if i % 2 == 0 else _states((16, 20), 9 + i, 0.01 + 0.002 * i))
        graph.replay()
    for _ in range(3):
        for st in ref:
            st.step()
    torch.cuda.synchronize()
    assert x.tolist() == [7.0] * 4
    for p, q in zip(a, ref):
        assert torch.equal(p.u, q.u) and torch.equal(p.d, q.d)
