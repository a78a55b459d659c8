"""What a batch call enqueues: the nodes of a graph that captures it."""
import ctypes

import numpy as np
import pytest

from oracle import oracle as O
from paper_2110_12952_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

B3S23 = W.rule_mask("B3/S23")


@pytest.fixture(scope="module")
def N():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2110_12952_amd import nbbfrac
    nbbfrac.lib()
    return nbbfrac


def nodes(fn):
    """Nodes of the graph that captures fn(stream) (never launched)."""
    hip = ctypes.CDLL("libamdhip64.so")
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph, n = ctypes.c_void_p(), ctypes.c_size_t()
    assert hip.hipStreamBeginCapture(ctypes.c_void_p(stream.cuda_stream), 2) == 0
    try:
        fn(stream)
    finally:
        assert hip.hipStreamEndCapture(ctypes.c_void_p(stream.cuda_stream), ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    return n.value


def make(N, specs, **kw):
    frs = [N.Fractal(W.FRACTALS[n].s, W.FRACTALS[n].offsets, r) for n, r in specs]
    batch = N.Batch(frs, **kw)
    a, b = batch.new_arena(), batch.new_arena()
    for i, f in enumerate(frs):
        f.init_compact(i, 0.45, out=batch.state(a, i))
    return frs, batch, a, b


@pytest.mark.parametrize("counts,launches", [([1], 1), ([3], 3), ([0], 0)])
def test_step_counts_upload_only_for_launches_that_read_them(N, counts, launches):
    # a few generations of a group take one launch each, which carry no counts
    frs, batch, a, b = make(N, [("triangle", 11)], resident=False)
    assert batch.step_info().matrix == 1
    assert nodes(lambda s: batch.step_each(a, b, counts, stream=s)) == launches
    held = nodes(lambda s: batch.step_each(a, b, [40], stream=s))
    assert 3 <= held < 20  # the counts, launches of several generations, the last one
    batch.step_each(a, b, counts)
    o = O.Fractal(2, W.TRIANGLE.offsets, 11)
    np.testing.assert_array_equal(batch.state(b if counts[0] & 1 else a, 0).cpu().numpy(),
                                  o.compact_steps(o.init_compact(0, 0.45), B3S23, counts[0]))
