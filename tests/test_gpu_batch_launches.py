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


SETS = [("triangle", 5), ("carpet", 3), ("hfractal", 3), ("chandelier", 5)]


def test_short_calls_on_many_fractals_take_one_launch(N):
    # small instances of four fractals: one LDS launch while the generations
    # are few, a held launch for each fractal where that pays
    frs, batch, a, b = make(N, SETS * 3)
    s = batch.step_info()
    assert s.held_whole == 12 and s.lds_resident == 0 and batch.info().groups == 0
    for steps in (1, 2, 4):
        assert nodes(lambda st: batch.step(a, b, steps, stream=st)) == 1
    assert nodes(lambda st: batch.step(a, b, 200, stream=st)) == 4
    assert nodes(lambda st: batch.step_each(a, b, [1] * 12, stream=st)) == 2  # with the counts
    frs, batch, a, b = make(N, SETS[:1] * 12)  # one fractal: one launch in either form
    assert nodes(lambda st: batch.step(a, b, 1, stream=st)) == 1


# held sets of several fractals; beside them what only the LDS launch takes
# (small squares and a 12-cell block), instances of groups, per-cell ones
REST = [("grid4_12", 2), ("fullsquare", 2)]
GROUPS = [("triangle", 12), ("carpet", 6), ("hfractal", 7), ("chandelier", 9), ("vicsek", 8)]


@pytest.mark.parametrize("kinds", [SETS, SETS + REST, SETS + GROUPS[:1], SETS + REST + GROUPS[:2], SETS + REST + GROUPS,
                                   SETS[:1] + REST + GROUPS, SETS + ["direct"], SETS + REST + GROUPS[:2] + ["direct"]])
def test_every_route_against_oracle(N, kinds):
    specs = [k for k in kinds if k != "direct"]
    frs = [N.Fractal(W.FRACTALS[n].s, W.FRACTALS[n].offsets, r) for n, r in specs]
    if "direct" in kinds:
        frs.append(N.Fractal(2, W.TRIANGLE.offsets, 6))
        frs[-1].configure(N.STRATEGY_DIRECT)
    batch = N.Batch(frs, resident=True)
    orcs = [O.Fractal(f.s, f.offsets, f.r) for f in frs]
    a, b = batch.new_arena(), batch.new_arena()
    st0 = [o.init_compact(90 + i, 0.45) for i, o in enumerate(orcs)]
    for steps in (1, 3, 8, 20, 70):
        for each in (False, True):
            a.fill_(7)
            b.fill_(7)
            for i, st in enumerate(st0):
                batch.state(a, i).copy_(torch.from_numpy(st))
            counts = [max(0, steps - (i % 3)) if each else steps for i in range(len(frs))]
            if each:
                batch.step_each(a, b, counts)
            else:
                batch.step(a, b, steps)
            ha, hb = a.cpu().numpy(), b.cpu().numpy()
            for i, (o, st, off) in enumerate(zip(orcs, st0, batch.offsets)):
                got = (hb if counts[i] & 1 else ha)[off:off + len(st)]
                np.testing.assert_array_equal(got, o.compact_steps(st, B3S23, counts[i]),
                                              err_msg=f"{frs[i].k},{frs[i].r} {counts[i]} generations")


@pytest.mark.parametrize("steps", [4097, 4098, 8193, 12291])
def test_resident_instances_leave_the_other_arena(N, steps):
    # more generations than one held launch takes, in one, two and four launches
    frs, batch, a, b = make(N, [("triangle", 3), ("triangle", 5), ("triangle", 4)])
    assert batch.step_info().held_whole == 3
    orcs = [O.Fractal(f.s, f.offsets, f.r) for f in frs]
    a0 = a.clone()
    for counts in ([steps] * 3, [steps, steps - 1, 5]):
        a.copy_(a0)
        b.fill_(9)
        batch.step_each(a, b, counts) if len(set(counts)) > 1 else batch.step(a, b, steps)
        for i, o in enumerate(orcs):
            sa, sb, st = (batch.state(t, i).cpu().numpy() for t in (a, b, a0))
            got, other = (sb, sa) if counts[i] & 1 else (sa, sb)
            np.testing.assert_array_equal(got, o.compact_steps(st, B3S23, counts[i]), err_msg=f"{i} {counts}")
            np.testing.assert_array_equal(other, st if counts[i] & 1 else np.full_like(st, 9), err_msg=f"{i} {counts}")
