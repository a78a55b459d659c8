"""Performance cases: the calls that programs using this library spend their time in.

Each listed case is one use of the public entry points at a size taken from
the repository's workloads (paper_2110_12952_amd/workloads.py), its benchmark
or its tests:

  compact  generations on the compact state (Fractal.step_compact), the
           library's main path, with the descriptor's default plan
  temporal the same with several generations per launch
           (Fractal.configure_temporal), for instances too small to fill the GPU
  packed   generations on the bit-packed state (Fractal.step_packed)
  batch    many instances stepped together (Batch.step)
  served   many small instances with step counts of their own
           (Batch.step_each), what the request loop runs per round
  maps     lambda on random compact indices, nu on random points
  box      the bounding-box method: compact state expanded, stepped on the
           box, gathered back
"""
import math

import numpy as np
import torch

from paper_2110_12952_amd import nbbfrac as N
from paper_2110_12952_amd import workloads as W

# Largest cell count of a drawn case of each kind (its listed cases reach it).
# (kind, fractal) pairs draw among the levels whose cells lie in the range.
RANGES = {
    "compact": (2_000, 290_000_000, ("triangle", "carpet", "hfractal", "chandelier", "grid4_12", "vicsek",
                                     "fullsquare", "xfractal")),
    "temporal": (2_000, 200_000, ("triangle", "carpet", "hfractal", "chandelier")),
    "packed": (500_000, 140_000_000, ("triangle", "carpet", "hfractal", "chandelier", "vicsek")),
    "box": (20_000, 17_000_000, ("triangle", "carpet", "hfractal", "chandelier")),
}
RULES = ("B3/S23", "B36/S23", "vN:B13/S13", "B1357/S02468")
BOX_SIDE_MAX = 20_000   # n of a drawn box case
EXACT_CELLS = 300_000   # cells up to which the 64-bit reference of a state is quick


def listed():
    return [
        # One small automaton stepped a few generations at a time (an
        # interactive program): latency and launches.
        {"name": "compact_triangle_r7", "kind": "compact", "fractal": "triangle", "r": 7, "steps": 2,
         "rule": "B3/S23", "p": 0.5},
        # The small workload of the benchmark: 59,049 cells, 100 generations in one call.
        {"name": "compact_triangle_r10", "kind": "compact", "fractal": "triangle", "r": 10, "steps": 100,
         "rule": "B3/S23", "p": 0.5},
        # The same for a program that asks for several generations per launch.
        {"name": "temporal_triangle_r10", "kind": "temporal", "fractal": "triangle", "r": 10, "steps": 100,
         "rule": "B3/S23", "p": 0.5},
        # The paper's case study at the headline size.
        {"name": "compact_triangle_r16", "kind": "compact", "fractal": "triangle", "r": 16, "steps": 20,
         "rule": "B3/S23", "p": 0.3},
        # The two workloads that do not fit the caches.
        {"name": "compact_carpet_r9", "kind": "compact", "fractal": "carpet", "r": 9, "steps": 10,
         "rule": "B3/S23", "p": 0.5},
        {"name": "compact_hfractal_r10", "kind": "compact", "fractal": "hfractal", "r": 10, "steps": 10,
         "rule": "B3/S23", "p": 0.5},
        # A fractal of the user's own (growth 3, five replicas) under another
        # rule and the four-cell neighbourhood.
        {"name": "compact_vicsek_r10_vn", "kind": "compact", "fractal": "vicsek", "r": 10, "steps": 10,
         "rule": "vN:B13/S13", "p": 0.4},
        # The batched workload: 512 instances of four fractals and many levels.
        {"name": "batch_512", "kind": "batch", "count": 512, "draw_seed": 2110, "steps": 20, "rule": "B3/S23"},
        # A round of small requests, each with a step count of its own.
        {"name": "served_60", "kind": "served", "count": 60, "draw_seed": 5, "max_steps": 64, "rule": "B3/S23"},
        # The two maps on an odd number of random points.
        {"name": "maps_triangle_r16", "kind": "maps", "fractal": "triangle", "r": 16, "count": 20_000_003},
        # A state held at one bit per cell.
        {"name": "packed_hfractal_r9", "kind": "packed", "fractal": "hfractal", "r": 9, "steps": 10,
         "rule": "B3/S23", "p": 0.5},
        # The comparison method on the box of the carpet (n = 6,561).
        {"name": "box_carpet_r8", "kind": "box", "fractal": "carpet", "r": 8, "steps": 4, "rule": "B3/S23",
         "p": 0.5},
    ]


def _levels(name, lo, hi):
    fd = W.FRACTALS[name]
    return [r for r in range(1, 24) if lo <= fd.k ** r <= hi]


def draw(rng):
    kind = rng.choice(("compact", "compact", "compact", "temporal", "batch", "served", "maps", "packed", "box"))
    if kind == "batch":
        return {"kind": kind, "count": rng.randrange(20, 400), "draw_seed": rng.randrange(1 << 20),
                "steps": rng.randrange(2, 20), "rule": "B3/S23"}
    if kind == "served":
        return {"kind": kind, "count": rng.randrange(10, 60), "draw_seed": rng.randrange(1 << 20),
                "max_steps": rng.randrange(8, 64), "rule": "B3/S23"}
    if kind == "maps":
        name = rng.choice(("triangle", "carpet", "hfractal", "chandelier"))
        r = rng.choice(_levels(name, 50_000, 290_000_000))
        return {"kind": kind, "fractal": name, "r": r, "count": int(round(10 ** rng.uniform(3.5, 7.3)))}
    lo, hi, names = RANGES[kind]
    name = rng.choice(names)
    levels = _levels(name, lo, hi)
    if kind == "box":
        levels = [r for r in levels if W.FRACTALS[name].s ** r <= BOX_SIDE_MAX]
    r = rng.choice(levels)
    most = {"compact": 10, "temporal": 100, "packed": 10, "box": 4}[kind]
    return {"kind": kind, "fractal": name, "r": r, "steps": rng.randrange(1, most + 1), "rule": rng.choice(RULES),
            "p": round(rng.uniform(0.2, 0.6), 3)}


def _bits(seed, count, p):
    """count cells, each alive with probability p, on the GPU."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    out = torch.empty(count, dtype=torch.uint8, device="cuda")
    for lo in range(0, count, 1 << 26):
        hi = min(lo + (1 << 26), count)
        out[lo:hi] = torch.rand(hi - lo, generator=g, device="cuda") < p
    return out


def _points(case, seed):
    fd = W.FRACTALS[case["fractal"]]
    cells, n = fd.k ** case["r"], fd.s ** case["r"]
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    ints = [torch.randint(0, hi, (case["count"],), generator=g, device="cuda", dtype=torch.int32)
            for hi in (cells, n, n)]
    return ints


def _instances(case):
    """(fractal, r, p, steps) of every instance of a batch or a served round."""
    if case["kind"] == "batch":
        wl = W.BatchWorkload("batch", case["count"], case["steps"], case["draw_seed"],
                             tuple(W.BATCH_LEVELS.items()))
        return [(it.fractal, it.r, it.p, case["steps"]) for it in wl.items()]
    rng = np.random.default_rng(case["draw_seed"])
    levels = {"triangle": (7, 10), "carpet": (4, 6), "hfractal": (4, 6), "chandelier": (5, 8)}
    names = sorted(levels)
    out = []
    for _ in range(case["count"]):
        name = names[int(rng.integers(len(names)))]
        lo, hi = levels[name]
        r = int(rng.integers(lo, hi + 1))
        steps = int(round(math.exp(rng.uniform(0.0, math.log(case["max_steps"])))))
        out.append((W.FRACTALS[name], r, 0.5, steps))
    # by decreasing step count, as the request loop orders a round
    return sorted(out, key=lambda it: -it[3])


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case}
    if kind in ("batch", "served"):
        items = _instances(case)
        frs = N.shared_descriptors([(fd.s, fd.offsets, r) for fd, r, _, _ in items])
        batch = N.Batch(frs)
        a, b = batch.new_arena(), batch.new_arena()
        a[:] = _bits(seed, a.numel(), 0.4)
        for off, cells, end in zip(batch.offsets, batch.cells, batch.offsets[1:] + [a.numel()]):
            a[off + cells:end] = 0
        st.update(batch=batch, a=a, b=b, steps=[s for _, _, _, s in items], rule=W.rule_mask(case["rule"]))
        return st
    fd = W.FRACTALS[case["fractal"]]
    f = N.Fractal(fd.s, fd.offsets, case["r"])
    st["f"] = f
    if kind == "maps":
        st["idx"], st["x"], st["y"] = _points(case, seed)
        return st
    st["rule"] = W.rule_mask(case["rule"])
    a = _bits(seed, f.cells, case["p"])
    if kind == "temporal":
        f.configure_temporal()
    if kind == "packed":
        a = f.pack(a)
        st.update(a=a, b=torch.zeros_like(a))
    elif kind == "box":
        st.update(a=a, box_a=f.new_bbox(), box_b=f.new_bbox(), out=f.new_compact())
    else:
        st.update(a=a, b=torch.zeros_like(a))
    return st


def run(st):
    case, kind = st["case"], st["case"]["kind"]
    if kind == "batch":
        return st["batch"].step(st["a"], st["b"], case["steps"], st["rule"])
    if kind == "served":
        st["batch"].step_each(st["a"], st["b"], st["steps"], st["rule"])
        # an instance's result is in b where its step count is odd, else in a
        return [st["batch"].state(st["b"] if s & 1 else st["a"], i) for i, s in enumerate(st["steps"])]
    f = st["f"]
    if kind == "maps":
        return list(f.lam(st["idx"])) + [f.nu(st["x"], st["y"])]
    if kind == "packed":
        return f.step_packed(st["a"], st["b"], case["steps"], st["rule"])
    if kind == "box":
        f.expand(st["a"], out=st["box_a"])
        box = f.step_bbox(st["box_a"], st["box_b"], case["steps"], st["rule"])
        return [box, f.gather(box, out=st["out"])]
    return f.step_compact(st["a"], st["b"], case["steps"], st["rule"])


def work(case):
    """Bytes: each input read once and each output written once per
    generation; operations: eight neighbour additions and the rule per cell."""
    kind = case["kind"]
    if kind in ("batch", "served"):
        cells = sum(fd.k ** r * s for fd, r, _, s in _instances(case))
        return {"bytes": 2 * cells, "flops": 9 * cells}
    fd = W.FRACTALS[case["fractal"]]
    cells, n = fd.k ** case["r"], fd.s ** case["r"]
    if kind == "maps":
        c, r = case["count"], case["r"]
        return {"bytes": 24 * c, "flops": 8 * r * c}
    if kind == "packed":
        return {"bytes": max(1, cells // 4 * case["steps"]), "flops": 9 * cells * case["steps"]}
    if kind == "box":
        # the box written by the expansion, read and written per generation; the compact state read and written
        return {"bytes": n * n * (1 + 2 * case["steps"]) + 3 * cells, "flops": 9 * n * n * case["steps"]}
    if kind == "temporal" or cells <= EXACT_CELLS:
        # the state read once and written once: such an instance fits one CU's or the chip's local memories
        return {"bytes": 2 * cells, "flops": 9 * cells * case["steps"]}
    return {"bytes": 2 * cells * case["steps"], "flops": 9 * cells * case["steps"]}


def _lambda64(fd, r, idx):
    x, y = np.zeros_like(idx), np.zeros_like(idx)
    o = np.array(fd.offsets, dtype=np.int64)
    rest, scale = idx.copy(), 1
    for _ in range(r):
        d = rest % fd.k
        rest //= fd.k
        x += o[d, 0] * scale
        y += o[d, 1] * scale
        scale *= fd.s
    return x, y


def _nu64(fd, r, x, y):
    """Compact index of (x, y), -1 outside the fractal."""
    hl = np.full(fd.s * fd.s, -1, np.int64)
    for j, (ox, oy) in enumerate(fd.offsets):
        hl[ox + fd.s * oy] = j
    n = fd.s ** r
    ok = (x >= 0) & (y >= 0) & (x < n) & (y < n)
    xx, yy = np.where(ok, x, 0), np.where(ok, y, 0)
    idx, scale = np.zeros_like(xx), 1
    for _ in range(r):
        h = hl[xx % fd.s + fd.s * (yy % fd.s)]
        ok &= h >= 0
        idx += h * scale
        xx, yy = xx // fd.s, yy // fd.s
        scale *= fd.k
    return np.where(ok, idx, -1)


def _generations64(fd, r, state, steps, rule):
    """Generations of the automaton on the compact state (int64, 0 or 1)."""
    cells = fd.k ** r
    x, y = _lambda64(fd, r, np.arange(cells, dtype=np.int64))
    near = [(dx, dy) for dy in (-1, 0, 1) for dx in (-1, 0, 1) if (dx, dy) != (0, 0)]
    if rule & W.VON_NEUMANN:
        near = [d for d in near if 0 in d]
    nbr = [_nu64(fd, r, x + dx, y + dy) for dx, dy in near]
    nbr = [np.where(v < 0, cells, v) for v in nbr]
    born = np.array([(rule >> c) & 1 for c in range(9)], np.int64)
    surv = np.array([(rule >> (16 + c)) & 1 for c in range(9)], np.int64)
    for _ in range(steps):
        padded = np.append(state, 0)
        count = sum(padded[v] for v in nbr)
        state = np.where(state == 1, surv[count], born[count])
    return state


def exact(case, seed):
    kind = case["kind"]
    if kind in ("batch", "served"):
        return None
    fd, r = W.FRACTALS[case["fractal"]], case["r"]
    cells, n = fd.k ** r, fd.s ** r
    if kind == "maps":
        idx, x, y = (t.cpu().numpy().astype(np.int64) for t in _points(case, seed))
        if case["count"] > 2_000_000:
            return None
        lx, ly = _lambda64(fd, r, idx)
        return [torch.from_numpy(v) for v in (lx, ly, _nu64(fd, r, x, y))]
    if cells > EXACT_CELLS:
        return None
    a = _bits(seed, cells, case["p"]).cpu().numpy().astype(np.int64)
    s = _generations64(fd, r, a, case["steps"], W.rule_mask(case["rule"]))
    if kind == "packed":
        bits = np.zeros((cells + 31) // 32 * 32, np.uint8)
        bits[:cells] = s
        return torch.from_numpy(np.packbits(bits, bitorder="little").astype(np.int64))
    if kind == "box":
        if n > 4096:
            return [None, torch.from_numpy(s)]
        box = np.zeros((n, (n + 15) // 16 * 16), np.int64)
        x, y = _lambda64(fd, r, np.arange(cells, dtype=np.int64))
        box[y, x] = s
        return [torch.from_numpy(box), torch.from_numpy(s)]
    return torch.from_numpy(s)
