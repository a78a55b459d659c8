"""The compact step on the matrix cores (the default plan's form wherever a
block level has 16 to 64 cells) against the CPU oracle, whole states, bit by
bit: blocks of 16, 25, 27, 32, 36, 49 and 64 cells, every number of lanes per
block, tiles of one block up to several groups per wavefront, groups with
lanes left over, every rule form."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2110_12952_amd import workloads as W

torch = pytest.importorskip("torch")
gpu = pytest.mark.gpu

# (fractal, r): the smallest states the form takes, one tile, few and many
# tiles; the levels change with r
STATES = [("triangle", r) for r in (3, 4, 5, 7, 8, 9, 10, 11, 12, 13)] + \
         [("carpet", r) for r in (2, 3, 4, 5, 6)] + [("hfractal", r) for r in (2, 3, 4, 5, 6, 7)] + \
         [("chandelier", r) for r in (3, 4, 7, 8, 9)] + [("fullsquare", r) for r in (3, 5, 8, 9)] + \
         [("vicsek", r) for r in (2, 3, 6, 7, 8)] + [("xfractal", r) for r in (2, 5, 7)] + \
         [("cantordust", 7), ("cantor", 6), ("cantor", 14), ("grid4_12", 3)]
RULES = ["B3/S23", "B36/S23", "B1357/S02468", "B35/S0123456", "vN:B2/S12", "vN:B13/S024"]


@pytest.fixture(scope="module")
def N():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2110_12952_amd import nbbfrac
    nbbfrac.lib()
    return nbbfrac


def check(N, fd, r, rules, seed=5):
    o, g = O.Fractal(fd.s, fd.offsets, r), N.Fractal(fd.s, fd.offsets, r)
    st0 = o.init_compact(seed, 0.45)
    for rule in rules:
        rm = W.rule_mask(rule)
        for steps in (1, 2):
            a = torch.from_numpy(st0).cuda()
            b = torch.full_like(a, 0xEE)
            res = g.step_compact(a, b, steps, rm).cpu().numpy()
            want = o.compact_steps(st0, rm, steps)
            np.testing.assert_array_equal(res, want, err_msg=f"{fd.name} r={r} {rule} steps={steps}")


@gpu
@pytest.mark.parametrize("name,r", STATES)
def test_default_step_against_oracle(N, name, r):
    check(N, W.FRACTALS[name], r, RULES)


@gpu
@pytest.mark.parametrize("seed", range(24))
def test_random_fractals_against_oracle(N, seed):
    fd = W.random_fractal(seed + 100)
    r = 1
    while fd.k > 1 and fd.k ** (r + 1) <= 200_000 and fd.s ** (r + 1) < 4000:
        r += 1
    check(N, fd, r, RULES[:3] + RULES[4:5], seed)


@gpu
@pytest.mark.parametrize("s,offsets,r", [(3, ((0, 0), (2, 0)), 17), (4, ((0, 0), (1, 1)), 15), (4, ((2, 1), (2, 2)), 14)])
def test_sparse_fractals_at_large_levels(N, s, offsets, r):
    # few cells in a box of up to 2^30 a side: the plans hold the blocks alone
    check(N, W.FractalDef("sparse", s, offsets), r, RULES[:1] + RULES[4:5])


@gpu
def test_full_rule_words(N):
    # births and survivals at eight neighbours (the bit-extract form) on the
    # fractals that have such cells
    for name, r in (("fullsquare", 6), ("carpet", 4), ("grid4_12", 3)):
        fd = W.FRACTALS[name]
        o, g = O.Fractal(fd.s, fd.offsets, r), N.Fractal(fd.s, fd.offsets, r)
        st0 = o.init_compact(3, 0.9)
        for rule in (1 << 8, 1 << 24, 0x01FF01FF, 0x00AA0155):
            a = torch.from_numpy(st0).cuda()
            res = g.step_compact(a, torch.empty_like(a), 3, rule).cpu().numpy()
            np.testing.assert_array_equal(res, o.compact_steps(st0, rule, 3), err_msg=f"{name} {rule:#x}")


@gpu
@pytest.mark.parametrize("name,levels", [("triangle", (3, 4, 7, 9, 10, 11)), ("carpet", (2, 3, 4, 5)),
                                         ("hfractal", (2, 3, 4, 6)), ("chandelier", (3, 4, 6, 8)),
                                         ("vicsek", (2, 3, 5, 7)), ("fullsquare", (3, 4, 7))])
def test_batch_of_many_levels(N, name, levels):
    # instances above, at and below the launch's tile level in one group, with
    # live bytes between them that no step may read as cells or change; whole
    # batches and decreasing step counts
    fd = W.FRACTALS[name]
    rs = [levels[(5 * i) % len(levels)] for i in range(2 * len(levels))]
    frs = [N.Fractal(fd.s, fd.offsets, r) for r in rs]
    for f in frs:
        f.configure(N.STRATEGY_TILED, min(levels))  # one group of the batch
    offs, top = [], 0
    for f in frs:
        offs.append(top)
        top = (top + f.cells + 15) // 16 * 16 + 48
    batch = N.Batch(frs, offsets=offs, resident=False)
    assert batch.info().groups == 1
    orcs = [O.Fractal(fd.s, fd.offsets, r) for r in rs]
    st0 = [o.init_compact(17 + i, 0.4) for i, o in enumerate(orcs)]
    arena = np.ones(top + 64, np.uint8)
    for off, st in zip(offs, st0):
        arena[off:off + len(st)] = st
    for rule in ("B3/S23", "B1357/S02468", "vN:B2/S12"):
        rm = W.rule_mask(rule)
        for counts in ([2] * len(rs), [max(1, 6 - i // 2) for i in range(len(rs))]):
            a = torch.from_numpy(arena).cuda()
            b = torch.full_like(a, 1)
            if len(set(counts)) == 1:
                batch.step(a, b, counts[0], rm)
            else:
                batch.step_each(a, b, counts, rm)
            ha, hb = a.cpu().numpy(), b.cpu().numpy()
            for i, (off, st, o) in enumerate(zip(offs, st0, orcs)):
                got = (hb if counts[i] & 1 else ha)[off:off + len(st)]
                np.testing.assert_array_equal(got, o.compact_steps(st, rm, counts[i]),
                                              err_msg=f"{name} r={rs[i]} {rule} steps={counts[i]}")
                ha[off:off + len(st)] = 1
                hb[off:off + len(st)] = 1
            assert (ha == 1).all() and (hb == 1).all()


# Levels of one batch whose own plans have different blocks: 16 and 64 cells
# (k = 4), 16, 32 and 64 (k = 2); an instance may be a quarter of a block
BLOCK_LEVELS = [("chandelier", (2, 3, 4, 6)), ("cantor", (4, 5, 6, 8)), ("cantor", (4, 5)), ("cantordust", (2, 3, 5))]


@gpu
@pytest.mark.parametrize("name,levels", BLOCK_LEVELS)
def test_batch_of_many_block_levels(N, name, levels):
    test_batch_of_many_levels(N, name, levels)


HELD = [("triangle", r) for r in (3, 5, 7, 9, 10, 12)] + [("carpet", r) for r in (2, 3, 4, 5, 6)] + \
       [("hfractal", r) for r in (2, 3, 4, 5, 6)] + [("chandelier", r) for r in (3, 5, 7, 8, 9)] + \
       [("fullsquare", r) for r in (3, 6, 8)] + [("vicsek", r) for r in (2, 4, 6, 7)] + \
       [("xfractal", 6), ("cantordust", 6), ("cantor", 9)]


@gpu
@pytest.mark.parametrize("name,r", HELD)
def test_several_generations_per_call_against_oracle(N, name, r):
    # step counts around the generations a launch takes (8, 9, 16, 18, ...), of
    # both parities: the result and the generation before it in the other
    # buffer, for the default plan and for TEMPORAL's automatic one
    fd = W.FRACTALS[name]
    o, g, t = (O.Fractal(fd.s, fd.offsets, r), N.Fractal(fd.s, fd.offsets, r), N.Fractal(fd.s, fd.offsets, r))
    t.configure_temporal()
    st0 = o.init_compact(21, 0.45)
    for rule in ("B3/S23", "B1357/S02468", "vN:B2/S12"):
        rm = W.rule_mask(rule)
        states = [st0]
        for _ in range(41):
            states.append(o.compact_steps(states[-1], rm, 1))
        for steps in (2, 3, 4, 5, 9, 10, 18, 19, 28, 41):
            a = torch.from_numpy(st0).cuda()
            b = torch.full_like(a, 0xEE)
            res = g.step_compact(a, b, steps, rm)
            assert (res is b) == bool(steps & 1)
            other = a if res is b else b
            np.testing.assert_array_equal(res.cpu().numpy(), states[steps], err_msg=f"{name} r={r} {rule} {steps}")
            np.testing.assert_array_equal(other.cpu().numpy(), states[steps - 1],
                                          err_msg=f"{name} r={r} {rule} {steps}: the generation before")
            a = torch.from_numpy(st0).cuda()
            res = t.step_compact(a, torch.full_like(a, 0xEE), steps, rm)
            np.testing.assert_array_equal(res.cpu().numpy(), states[steps], err_msg=f"temporal {name} {rule} {steps}")


@gpu
@pytest.mark.parametrize("resident", [True, False])
@pytest.mark.parametrize("name,levels", [("triangle", (3, 6, 8, 9, 11)), ("carpet", (2, 4, 5, 6)),
                                         ("hfractal", (2, 4, 5)), ("chandelier", (3, 5, 7, 9)),
                                         ("vicsek", (2, 4, 6))])
def test_batch_several_generations(N, name, levels, resident):
    # whole batches and per-instance counts that take several launches of
    # several generations; guard bytes between the instances
    fd = W.FRACTALS[name]
    rs = [levels[(3 * i) % len(levels)] for i in range(2 * len(levels))]
    frs = [N.Fractal(fd.s, fd.offsets, r) for r in rs]
    for f in frs:
        f.configure(N.STRATEGY_TILED, min(levels))
    offs, top = [], 0
    for f in frs:
        offs.append(top)
        top = (top + f.cells + 15) // 16 * 16 + 32
    batch = N.Batch(frs, offsets=offs, resident=resident)
    orcs = [O.Fractal(fd.s, fd.offsets, r) for r in rs]
    st0 = [o.init_compact(31 + i, 0.4) for i, o in enumerate(orcs)]
    arena = np.ones(top + 64, np.uint8)
    for off, st in zip(offs, st0):
        arena[off:off + len(st)] = st
    for rule in ("B3/S23", "B1357/S02468"):
        rm = W.rule_mask(rule)
        for counts in ([11] * len(rs), [20] * len(rs), [max(0, 37 - 5 * i) for i in range(len(rs))]):
            a = torch.from_numpy(arena).cuda()
            b = torch.full_like(a, 1)
            if len(set(counts)) == 1:
                batch.step(a, b, counts[0], rm)
            else:
                batch.step_each(a, b, counts, rm)
            ha, hb = a.cpu().numpy(), b.cpu().numpy()
            for i, (off, st, o) in enumerate(zip(offs, st0, orcs)):
                got = (hb if counts[i] & 1 else ha)[off:off + len(st)]
                np.testing.assert_array_equal(got, o.compact_steps(st, rm, counts[i]),
                                              err_msg=f"{name} r={rs[i]} {rule} steps={counts[i]}")
                other = (ha if counts[i] & 1 else hb)[off:off + len(st)]
                if not resident and counts[i]:  # the generation before, in the other arena
                    np.testing.assert_array_equal(other, o.compact_steps(st, rm, counts[i] - 1),
                                                  err_msg=f"{name} r={rs[i]} {rule} steps={counts[i]}: before")
                elif resident and batch.info().groups == 0:  # stepped whole: untouched
                    np.testing.assert_array_equal(other, st if counts[i] & 1 else np.ones_like(st))
                ha[off:off + len(st)] = 1
                hb[off:off + len(st)] = 1
            assert (ha == 1).all() and (hb == 1).all()


@gpu
@pytest.mark.parametrize("resident", [True, False])
@pytest.mark.parametrize("name,levels", BLOCK_LEVELS)
def test_batch_of_many_block_levels_several_generations(N, name, levels, resident):
    test_batch_several_generations(N, name, levels, resident)


def bits(state):
    words = np.zeros((len(state) + 31) // 32 * 32, np.uint8)
    words[:len(state)] = state
    return np.packbits(words, bitorder="little")


@gpu
@pytest.mark.parametrize("name,r", HELD)
def test_packed_generations_against_oracle(N, name, r):
    # the bit-packed state in the held form: every bit of the result and of
    # the generation before it, bits past the last cell unchanged
    fd = W.FRACTALS[name]
    o, g = O.Fractal(fd.s, fd.offsets, r), N.Fractal(fd.s, fd.offsets, r)
    st0 = o.init_compact(77, 0.45)
    past = np.zeros(g.packed_bytes() * 8, np.uint8)
    past[len(st0):] = 1
    past = np.packbits(past, bitorder="little")
    for rule in ("B3/S23", "B1357/S02468"):
        rm = W.rule_mask(rule)
        states = [st0]
        for _ in range(20):
            states.append(o.compact_steps(states[-1], rm, 1))
        for steps in (1, 2, 3, 10, 19, 20):
            a = torch.from_numpy(bits(st0)).cuda()
            b = torch.full_like(a, 0xFF)
            res = g.step_packed(a, b, steps, rm)
            other = a if res is b else b
            for t, n in ((res, steps), (other, steps - 1)):
                want = bits(states[n]) | (past if t is b else 0)
                np.testing.assert_array_equal(t.cpu().numpy(), want, err_msg=f"{name} r={r} {rule} {steps} gen {n}")


@gpu
@pytest.mark.parametrize("count", [1, 3, 4099, 2_100_003])
@pytest.mark.parametrize("off", [0, 1, 3])
def test_maps_at_any_alignment(N, count, off):
    fd = W.TRIANGLE
    o, g = O.Fractal(fd.s, fd.offsets, 12), N.Fractal(fd.s, fd.offsets, 12)
    idx = W.random_indices(1, count, 3 ** 12 + 9)
    t = torch.zeros(count + 4, dtype=torch.int32, device="cuda")
    t[off:off + count] = torch.from_numpy(idx.astype(np.int32)).cuda()
    outs = [torch.full((count + 8,), 7, dtype=torch.int32, device="cuda") for _ in range(3)]
    x, y, back = (v[off:off + count] for v in outs)
    g.lam(t[off:off + count], out=(x, y))
    inside = idx < 3 ** 12
    wx, wy = (np.where(inside, v.astype(np.int64), -1) for v in o.lam_many(np.where(inside, idx, 0).astype(np.uint32)))
    np.testing.assert_array_equal(x.cpu().numpy(), wx)
    np.testing.assert_array_equal(y.cpu().numpy(), wy)
    g.nu(x, y, out=back)
    np.testing.assert_array_equal(back.cpu().numpy().view(np.uint32), np.where(idx < 3 ** 12, idx, 0xFFFFFFFF))
    for v in outs:
        h = v.cpu().numpy()
        assert (h[:off] == 7).all() and (h[off + count:] == 7).all()


@gpu
def test_step_info_names_what_runs(N):
    fd = W.TRIANGLE
    f = N.Fractal(fd.s, fd.offsets, 10)
    level = f.info().tile_level
    d = f.step_info()
    assert d.form == N.FORM_MATRIX and d.tiles == 3 ** (10 - d.tile_level) and d.tile_side == 2 ** d.tile_level
    assert d.held_generations > 1 and d.held_tiles == 3 ** (10 - d.held_level) and 0 < d.lds_bytes <= 65536
    for strategy, form in ((N.STRATEGY_TILED_EDGE, N.FORM_EDGE_RECORDS), (N.STRATEGY_TILED_BOX, N.FORM_BYTE_SCATTER),
                           (N.STRATEGY_TILED_WAVE, N.FORM_BYTE_SCATTER)):
        m = 5 if strategy == N.STRATEGY_TILED_WAVE else level
        f.configure(strategy, m)
        s, v = f.step_info(), f.info()
        assert (s.form, s.tile_level, s.tiles, s.lds_bytes) == (form, m, v.tiles, v.lds_bytes)
        assert s.held_generations == 0 and s.whole_generations == 0
    f.configure(N.STRATEGY_DIRECT)
    s = f.step_info()
    assert (s.form, s.tile_level, s.held_generations) == (N.FORM_DIRECT, 0, 0)
    f.configure_temporal(4, 8)
    s = f.step_info()
    assert (s.form, s.tile_level, s.held_generations) == (N.FORM_TEMPORAL, 4, 8)
    f.configure_temporal()
    s = f.step_info()
    assert (s.form, s.tile_level, s.held_generations) == (N.FORM_MATRIX, d.held_level, d.held_generations)
    f.configure(N.STRATEGY_TILED, 4)  # the tile plan's level: the matrix form keeps its own
    s = f.step_info()
    assert f.info().tile_level == 4
    assert all(getattr(s, n) == getattr(d, n) for n, _ in s._fields_)
    g = N.Fractal(2, ((0, 0), (1, 1)), 3)  # 8 cells: no block of 16
    assert g.step_info().form in (N.FORM_EDGE_RECORDS, N.FORM_BYTE_SCATTER)
    whole = N.Fractal(fd.s, fd.offsets, 7).step_info()
    assert whole.whole_generations > 0


@gpu
def test_batch_step_info_names_what_runs(N):
    tri = [N.Fractal(2, W.TRIANGLE.offsets, r) for r in (11, 7)]
    car = [N.Fractal(3, W.CARPET.offsets, r) for r in (6, 3)]
    car[0].configure(N.STRATEGY_TILED_BOX, 3)
    direct = N.Fractal(2, W.TRIANGLE.offsets, 5)
    direct.configure(N.STRATEGY_DIRECT)
    frs = tri + car + [direct]
    s = N.Batch(frs, resident=False).step_info()
    assert (s.matrix, s.edge_records, s.byte_scatter, s.direct, s.held_whole, s.lds_resident) == (3, 0, 1, 1, 0, 0)
    assert s.tiles >= 8 ** 3 + 3  # the box plan's own, at least one of every other
    s = N.Batch(frs, resident=True).step_info()
    assert (s.matrix, s.byte_scatter, s.direct, s.held_whole, s.lds_resident) == (1, 1, 1, 2, 0)
