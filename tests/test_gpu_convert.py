"""Box <-> compact conversion by strips of tiles, bit-exact against the oracle: fractals
with tiles of 16, 25, 27 and 32 columns, cell counts that are no multiple of
four, boxes narrower and wider than a strip, wider pitches, compact states at
any address, boxes on both sides of the rule that picks this form, boxes full
of other values before, guard bytes around every output."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2110_12952_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

FRACTALS = {name: (fd.s, tuple(fd.offsets)) for name, fd in W.FRACTALS.items()}
# lambda(0) away from the corner, k no multiple of 4
FRACTALS["corner3"] = (3, ((2, 2), (0, 0), (1, 0), (0, 2), (2, 1), (1, 2), (2, 0)))
FRACTALS["cross5"] = (5, ((2, 2), (0, 0), (1, 1), (3, 3), (4, 4), (0, 4), (1, 3), (3, 1), (4, 0), (2, 0), (0, 2)))


@pytest.mark.parametrize("name,r,extra,off", [
    ("carpet", 3, 0, 0), ("carpet", 4, 0, 1), ("carpet", 5, 16, 2), ("carpet", 7, 0, 3), ("fullsquare", 4, 0, 0),
    ("fullsquare", 9, 48, 1), ("fullsquare", 12, 0, 0), ("triangle", 4, 0, 1), ("triangle", 5, 400, 1), ("triangle", 11, 16, 3),
    ("hfractal", 6, 0, 1), ("hfractal", 7, 0, 0), ("vicsek", 5, 32, 3), ("chandelier", 5, 0, 1), ("grid4_12", 3, 0, 2), ("corner3", 5, 0, 1),
    ("corner3", 7, 16, 0), ("cross5", 2, 0, 1), ("cross5", 4, 0, 3)])
def test_strips(name, r, extra, off):
    from paper_2110_12952_amd import nbbfrac as N
    s, offsets = FRACTALS[name]
    o, g = O.Fractal(s, offsets, r), N.Fractal(s, offsets, r)
    st = o.init_compact(8, 0.5)
    pad = torch.full((g.cells + 64,), 9, dtype=torch.uint8, device="cuda")
    comp = pad[16 + off:16 + off + g.cells]
    comp.copy_(torch.from_numpy(st))
    pitch = g.pitch + extra
    whole = torch.full((g.n * pitch + 256,), 7, dtype=torch.uint8, device="cuda")
    box = whole[128:128 + g.n * pitch].view(g.n, pitch)
    g.expand(comp, out=box)
    got = whole.cpu().numpy()
    assert (got[:128] == 7).all() and (got[128 + g.n * pitch:] == 7).all()
    got = got[128:128 + g.n * pitch].reshape(g.n, pitch)
    np.testing.assert_array_equal(got[:, :g.n], o.expand(st))
    assert not got[:, g.n:].any()
    comp.fill_(5)
    g.gather(box, out=comp)
    back = pad.cpu().numpy()
    np.testing.assert_array_equal(back[16 + off:16 + off + g.cells], st)
    assert (back[:16 + off] == 9).all() and (back[16 + off + g.cells:] == 9).all()


@pytest.mark.parametrize("name,r", [("triangle", 16), ("triangle", 20), ("carpet", 7), ("carpet", 10), ("hfractal", 9),
                                    ("grid4_12", 8), ("chandelier", 10), ("cross5", 9), ("fullsquare", 15), ("cantor", 19)])
@pytest.mark.parametrize("count", [4097, 300_003])
def test_nu_divisions(name, r, count):
    """Coordinates at the edges of every level's copies, inside and outside the
    box, and cells of the fractal."""
    from paper_2110_12952_amd import nbbfrac as N
    s, offsets = FRACTALS[name]
    o, g = O.Fractal(s, offsets, r), N.Fractal(s, offsets, r)
    rng = np.random.default_rng(3)
    n = s ** r

    def axis():
        v = rng.integers(-2, n + 2, count)
        step = s ** rng.integers(0, r + 1, count)
        edge = rng.integers(0, 2, count).astype(bool)
        v = np.where(edge, v // step * step + rng.integers(-1, 2, count), v)
        return np.clip(v, -3, 2 ** 31 - 1).astype(np.int32)

    x, y = axis(), axis()
    inside = rng.integers(0, o.cells, count // 2, dtype=np.uint64).astype(np.uint32)
    x[:count // 2], y[:count // 2] = o.lam_many(inside)
    want = o.nu_many(x, y)
    got = g.nu(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()).cpu().numpy().view(np.uint32)
    np.testing.assert_array_equal(got, np.asarray(want).astype(np.int64).astype(np.uint32))
    np.testing.assert_array_equal(got[:count // 2], inside)
