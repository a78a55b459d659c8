"""The vector forms of the tiled step asked for by name: TILED takes the
matrix-core form wherever that applies, at every tile level, so edge records,
byte scatter, the instances stepped in LDS and the packed step's own kernel
run on most fractals only for a descriptor configured to TILED_EDGE or
TILED_BOX.  Expected values come from oracle/ (large states: the default
form); inputs are seeded and synthetic.
"""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2110_12952_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

B3S23 = W.rule_mask("B3/S23")
RULES = ["B3/S23", "B36/S23", "B1357/S02468", "B35/S0123456", "vN:B2/S12"]
SMALL = [("triangle", r) for r in (2, 3, 5, 8)] + [("carpet", r) for r in (1, 2, 3, 4)] + \
        [("hfractal", r) for r in (1, 2, 4)] + [("chandelier", r) for r in (2, 5)] + \
        [("fullsquare", 5), ("vicsek", 4), ("xfractal", 3), ("cantordust", 3), ("cantor", 6), ("grid4_12", 3)]


@pytest.fixture(scope="module")
def N():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2110_12952_amd import nbbfrac
    nbbfrac.lib()
    return nbbfrac


def to_form(N, f, form, m):
    """Configure f to the form at level m; False where it does not apply."""
    try:
        f.configure({"edge": N.STRATEGY_TILED_EDGE, "box": N.STRATEGY_TILED_BOX}[form], m)
    except N.NbbError:
        return False
    s = f.step_info()
    assert (s.form, s.tile_level) == ({"edge": N.FORM_EDGE_RECORDS, "box": N.FORM_BYTE_SCATTER}[form], m)
    return True


def any_form(N, f, m):
    """Edge records at level m, or byte scatter where they do not apply."""
    assert to_form(N, f, "edge", m) or to_form(N, f, "box", m)


@pytest.mark.parametrize("name,r", SMALL)
def test_edge_records_at_every_level(N, name, r):
    fd = W.FRACTALS[name]
    o, g = O.Fractal(fd.s, fd.offsets, r), N.Fractal(fd.s, fd.offsets, r)
    st0 = o.init_compact(77 + r, 0.45)
    for m in range(1, r + 1):
        if not to_form(N, g, "edge", m):
            continue
        for rule in RULES:
            rm = W.rule_mask(rule)
            for steps in (1, 2, 7):
                a = torch.from_numpy(st0).cuda()
                res = g.step_compact(a, torch.full_like(a, 0xAB), steps, rm).cpu().numpy()
                np.testing.assert_array_equal(res, o.compact_steps(st0, rm, steps),
                                              err_msg=f"{name} r={r} m={m} {rule} steps={steps}")


@pytest.mark.parametrize("seed", range(8))
def test_edge_records_random_fractals(N, seed):
    fd = W.random_fractal(200 + seed)
    r = 1
    while fd.k ** (r + 1) <= 300000 and r < 12:
        r += 1
    o, g = O.Fractal(fd.s, fd.offsets, r), N.Fractal(fd.s, fd.offsets, r)
    st0 = o.init_compact(seed, 0.5)
    want = o.compact_steps(st0, B3S23, 5)
    for m in range(1, r + 1):
        if to_form(N, g, "edge", m):
            a = torch.from_numpy(st0).cuda()
            np.testing.assert_array_equal(g.step_compact(a, torch.empty_like(a), 5).cpu().numpy(), want,
                                          err_msg=f"{fd} r={r} m={m}")


@pytest.mark.parametrize("name,r,steps", [("triangle", 12, 300), ("carpet", 6, 200), ("hfractal", 7, 200),
                                          ("chandelier", 9, 200), ("grid4_12", 5, 150)])
def test_long_runs(N, name, r, steps):
    fd = W.FRACTALS[name]
    o, g = O.Fractal(fd.s, fd.offsets, r), N.Fractal(fd.s, fd.offsets, r)
    m = g.info().tile_level
    st0 = o.init_compact(4242 + r, 0.4)
    want = o.compact_steps(st0, B3S23, steps)
    for form in ("edge", "box"):
        assert to_form(N, g, form, m)
        a = torch.from_numpy(st0).cuda()
        np.testing.assert_array_equal(g.step_compact(a, torch.empty_like(a), steps).cpu().numpy(), want,
                                      err_msg=f"{name} r={r} {form}")


@pytest.mark.parametrize("name,r,steps", [("triangle", 16, 30), ("carpet", 9, 10), ("hfractal", 10, 10), ("triangle", 20, 2)])
def test_large_states_equal_the_default_form(N, name, r, steps):
    fd = W.FRACTALS[name]
    g = N.Fractal(fd.s, fd.offsets, r)
    m = g.info().tile_level
    assert g.step_info().form == N.FORM_MATRIX
    a = g.init_compact(31, 0.4)
    b = torch.empty_like(a)
    want = g.step_compact(a, b, steps)
    c = torch.empty_like(a) if want is a else a
    d = b if want is a else torch.empty_like(a)
    for form in ("edge", "box"):
        assert to_form(N, g, form, m)
        g.init_compact(31, 0.4, out=c)
        assert torch.equal(g.step_compact(c, d, steps), want), form


BATCH = [("triangle", 12, 6), ("carpet", 5, 2), ("hfractal", 6, 3), ("triangle", 9, 6), ("triangle", 7, 6),
         ("carpet", 4, 2), ("hfractal", 5, 3), ("chandelier", 7, 3), ("chandelier", 5, 3), ("triangle", 3, 3),
         ("vicsek", 4, 2), ("hfractal", 4, 3), ("grid4_12", 3, 2)]


@pytest.mark.parametrize("resident", [True, False])
@pytest.mark.parametrize("rule", ["B3/S23", "B1357/S02468", "vN:B13/S13"])
def test_batches(N, rule, resident):
    # group launches of both vector forms, and the small instances in LDS;
    # whole batches and decreasing step counts; guard bytes
    rm = W.rule_mask(rule)
    frs, offs, top = [], [], 0
    for name, r, m in BATCH:
        fd = W.FRACTALS[name]
        f = N.Fractal(fd.s, fd.offsets, r)
        any_form(N, f, m)
        frs.append(f)
        offs.append(top)
        top += (f.cells + 15) // 16 * 16 + 32
    batch = N.Batch(frs, offs, resident=resident)
    s = batch.step_info()
    assert s.matrix == 0 and s.held_whole == 0 and s.edge_records > 0
    assert (s.lds_resident > 6) if resident else (s.lds_resident == 0 and s.byte_scatter > 0)
    orcs = [O.Fractal(f.s, f.offsets, f.r) for f in frs]
    st0 = [o.init_compact(50 + i, 0.4) for i, o in enumerate(orcs)]
    arena = np.full(top, 0x11, np.uint8)
    for off, st in zip(offs, st0):
        arena[off:off + len(st)] = st
    for counts in ([6] * len(frs), [max(0, 15 - i) for i in range(len(frs))]):
        a = torch.from_numpy(arena).cuda()
        b = torch.full_like(a, 0x11)
        if len(set(counts)) == 1:
            batch.step(a, b, counts[0], rm)
        else:
            batch.step_each(a, b, counts, rm)
        ha, hb = a.cpu().numpy(), b.cpu().numpy()
        for i, (off, st, o) in enumerate(zip(offs, st0, orcs)):
            got = (hb if counts[i] & 1 else ha)[off:off + len(st)]
            np.testing.assert_array_equal(got, o.compact_steps(st, rm, counts[i]), err_msg=f"{BATCH[i]} {counts[i]}")
            ha[off:off + len(st)] = 0x11
            hb[off:off + len(st)] = 0x11
        assert (ha == 0x11).all() and (hb == 0x11).all()


@pytest.mark.parametrize("form", ["edge", "box"])
@pytest.mark.parametrize("name,r,m", [("triangle", 9, 4), ("carpet", 4, 3), ("hfractal", 5, 3), ("chandelier", 6, 4),
                                      ("grid4_12", 3, 2), ("cantor", 8, 5)])
def test_writes_stay_inside(N, name, r, m, form):
    # byte and packed states inside larger allocations
    fd = W.FRACTALS[name]
    o, g = O.Fractal(fd.s, fd.offsets, r), N.Fractal(fd.s, fd.offsets, r)
    if not to_form(N, g, form, m):
        pytest.skip("the form does not apply")
    st0 = o.init_compact(9, 0.45)
    for rule in ("B3/S23", "B1357/S02468"):
        want = o.compact_steps(st0, W.rule_mask(rule), 5)
        for packed in (False, True):
            n = g.packed_bytes() if packed else g.cells
            bufs = [torch.full((n + 8192,), 0x6B, dtype=torch.uint8, device="cuda") for _ in range(2)]
            a, b = (t[4096:4096 + n] for t in bufs)
            src = torch.from_numpy(st0).cuda()
            if packed:
                g.pack(src, out=a)
                res = g.unpack(g.step_packed(a, b, 5, W.rule_mask(rule)))
            else:
                a.copy_(src)
                res = g.step_compact(a, b, 5, W.rule_mask(rule))
            np.testing.assert_array_equal(res.cpu().numpy(), want, err_msg=f"{name} {form} packed={packed}")
            for t in bufs:
                h = t.cpu().numpy()
                assert (h[:4096] == 0x6B).all() and (h[4096 + n:] == 0x6B).all()


@pytest.mark.parametrize("resident", [None, True, False])
def test_captured_graphs(N, resident):
    # a single state (None) and a batch with and without LDS instances,
    # replayed with eager work between the replays
    specs = BATCH if resident is not None else [("triangle", 8, 5)]
    frs = []
    for name, r, m in specs:
        f = N.Fractal(W.FRACTALS[name].s, W.FRACTALS[name].offsets, r)
        any_form(N, f, m)
        frs.append(f)
    orcs = [O.Fractal(f.s, f.offsets, f.r) for f in frs]
    batch = None if resident is None else N.Batch(frs, resident=resident)
    offs, length = (batch.offsets, batch.new_arena().numel()) if batch else ([0], frs[0].cells)
    a0 = torch.zeros(length, dtype=torch.uint8, device="cuda")
    for i, (f, off) in enumerate(zip(frs, offs)):
        f.init_compact(i, 0.45, out=a0[off:off + f.cells])
    a, b = a0.clone(), torch.empty_like(a0)
    step = (lambda: batch.step(a, b, 4)) if batch else (lambda: frs[0].step_compact(a, b, 4))
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()  # outside the capture
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    want = [o.compact_steps(o.init_compact(i, 0.45), B3S23, 4) for i, o in enumerate(orcs)]
    for rep in range(3):
        a.copy_(a0)
        graph.replay()
        b.clone().add_(1)
        torch.cuda.synchronize()
        h = a.cpu().numpy()
        for i, (f, off) in enumerate(zip(frs, offs)):
            np.testing.assert_array_equal(h[off:off + f.cells], want[i], err_msg=f"replay {rep} {specs[i]}")
