"""The counting kernel's computed bins, replayed on the CPU.

Where the edges of every axis are uniform the kernel forms a pair's bin from the
hardware reciprocal square root (fcfc_plan_computed) and bins it again in FP64
only near an edge.  Its FP32 arithmetic is emulated here operation by operation,
with the hardware functions at both ends of their error bound: positions in the
frame of a tile of up to 32 cells, the tolerances widened for the tile's span
(or leaf-local positions and their lattice, for trees), the displacement, the
squares, x = v rsq(v) scale + offset and the distance of x to the next integer.
Every pair that it places without the recheck has to be in the oracle's bin, and
every pair that it drops has to be out of range.
"""
import numpy as np
import pytest

import oracle
from paper_2301_12557_amd import fcfc, synth
from test_bands_cpu import F32, F64, _cells, _exact_values, _geometries, _knife_pairs, _pairs, _rsq, fma32

SHELL = ([400.0, -10.0, -560.0], [2010.0, 1760.0, 560.0])
PAIRS = 600_000


def _cases():
    lin = synth.linear_edges
    base = [g for g in _geometries() if "log" not in g[0]]
    return base + [
        ("s from above zero", "s", "z", 1000.0, lin(30, 150, 24), None, 20_000, None),
        ("s narrow bins", "s", "z", 1000.0, lin(0, 60, 4000), None, 200_000, None),
        ("s far offset", "s", "z", 1000.0, lin(100, 101, 10), None, 200_000, None),
        ("smu one mu bin", "smu", "z", 1000.0, lin(0, 100, 20), synth.mu_edges(1), 200_000, None),
        ("smu many mu bins", "smu", "z", 1000.0, lin(0, 100, 10), synth.mu_edges(1000), 200_000, None),
        ("spi z from above zero", "spi", "z", 1000.0, lin(5, 45, 8), lin(10, 50, 10), 200_000, None),
        ("spi mid narrow", "spi", "mid", 0.0, lin(0, 60, 120), lin(0, 60, 120), 300_000, SHELL),
        ("spi mid short pi", "spi", "mid", 0.0, lin(0, 200, 20), lin(0, 4, 4), 300_000, SHELL),
        ("smu mid from above zero", "smu", "mid", 0.0, lin(20, 150, 13), synth.mu_edges(50), 300_000, SHELL),
    ]


def _grid_frame(A, B, num, box, cst, rng):
    """Displacement and the widening of the tolerances, in the frame of a tile whose
    first cell lies 0 to 31 cells before the A point's."""
    cA, oA = _cells(A, num, box)
    cB, oB = _cells(B, num, box)
    a, b = (A - oA).astype(F32), (B - oB).astype(F32)
    dc = cB - cA
    if box > 0:
        n = np.array([num["nx"], num["ny"], num["nz"]])
        dc = dc - n * np.round(dc / n).astype(np.int64)
    side = F32(num["side32"])
    s = rng.integers(0, 32, len(A))
    fa = a[:, 0] + s.astype(F32) * side
    fb = b[:, 0] + (s + dc[:, 0]).astype(F32) * side
    dx = fb - fa
    dy = b[:, 1] - (a[:, 1] - dc[:, 1].astype(F32) * side)
    dz = b[:, 2] - (a[:, 2] - dc[:, 2].astype(F32) * side)
    # the narrowest span such a tile can have: its first point at the end of its cell, or anywhere in it
    first = np.minimum(fa, side) * np.where(rng.random(len(A)) < 0.5, 1.0, rng.random(len(A))).astype(F32)
    eh = (F32(16) * side + F32(6) * (fa - first) + F32(4.1) * F32(cst["reach"])) * F32(cst["e_unit"])
    return np.stack([dx, dy, dz], 1), np.maximum(F32(1), eh)


def _tree_frame(A, B, num, extent, rng):
    """Displacement of leaf-local coordinates: origins on a lattice, up to the largest
    local coordinate away."""
    q = 2.0 ** (int(np.frexp(extent)[1]) - 22)
    top = num["side"] - 2 * q

    def org(x):
        return np.floor((x - rng.random(x.shape) * top) / q)

    ja, jb = org(A), org(B)
    a, b = (A - ja * q).astype(F32), (B - jb * q).astype(F32)
    d = (b + (jb - ja).astype(F32) * F32(q)) - a
    return d, np.ones(len(A), dtype=F32)


def _decide(kind, los, n1, n2, cst, d, A, widen, deltas):
    """Flat bin, -1 (out of range) or -2 (binned again in FP64), and x and the tolerance per axis."""
    with np.errstate(divide="ignore", invalid="ignore"):
        dx, dy, dz = d[:, 0], d[:, 1], d[:, 2]
        d2 = fma32(dz, dz, fma32(dy, dy, dx * dx))
        if los == "mid":
            l = F32(2) * A.astype(F32) + d
            dot = fma32(dz, l[:, 2], fma32(dy, l[:, 1], dx * l[:, 0]))
            rl = _rsq(fma32(l[:, 2], l[:, 2], fma32(l[:, 1], l[:, 1], l[:, 0] * l[:, 0])), deltas[1])
        t1, t2 = F32(cst["tol1"]) * widen, F32(cst["tol2"]) * widen
        near2 = np.zeros(len(d), dtype=bool)
        in2 = np.ones(len(d), dtype=bool)
        b2 = np.zeros(len(d), dtype=np.int64)
        v1, seen = d2, {}
        if kind == "smu":
            mu = F32(cst["mu_n"])
            proj = np.abs(dot) * (rl * mu) if los == "mid" else np.abs(dz) * mu
            rs = _rsq(d2, deltas[0])
            mun = proj * rs
            b2 = np.nan_to_num(np.trunc(mun), nan=0.0).astype(np.int64)
            cr = np.clip(np.rint(mun), F32(1), F32(max(n2 - 1, 1))).astype(F32) if n2 > 1 else \
                np.clip(np.rint(mun), F32(0), F32(1))
            tol = fma32(F32(cst["mu_tolA"]) * widen, rs, F32(cst["mu_tolC"]) * widen)
            near2 = ~(np.abs(mun - cr) >= tol)
            seen["mu"] = (mun, tol)
        elif kind == "spi":
            if los == "mid":
                p = np.abs(dot) * rl
                v1 = np.maximum(fma32(-p, p, d2), F32(0))
            else:
                p = np.abs(dz)
                v1 = fma32(dy, dy, dx * dx)
            x2 = fma32(p, np.full_like(p, cst["scale2"]), np.full_like(p, cst["offset2"]))
            b2 = np.floor(x2).astype(np.int64)
            near2 = ~(np.abs(x2 - np.rint(x2)) >= t2)
            if cst["zero2"] and los == "z":
                near2 &= ~(x2 < F32(1) - t2)
            in2 = (b2 >= 0) & (b2 < n2)
            seen["pi"] = (x2, t2)
        rs = _rsq(v1, deltas[0])
        x1 = fma32(v1 * rs, np.full_like(v1, cst["scale1"]), np.full_like(v1, cst["offset1"]))
        if cst["tol1_abs"]:
            t1 = fma32(F32(cst["tol1_abs"]) * widen, rs, t1)
        near1 = ~(np.abs(x1 - np.rint(x1)) >= t1)
        seen["s"] = (x1, t1)
        b1 = np.nan_to_num(np.floor(x1), nan=-1.0).astype(np.int64)
        out = np.where((b1 >= 0) & (b1 < n1) & in2, b1 * n2 + b2, -1)
        return np.where(near1 | near2, -2, out), seen


def _check(g, tree, seed):
    name, kind, los, box, e1, e2, n_hint, bounds = g
    p = fcfc.Plan(kind, e1, e2, los=los, box=0.0 if tree else box, n_hint=n_hint, **({"tree_leaf": 128} if tree else {}))
    if bounds is not None:
        p.set_bounds(*bounds)
    elif tree:
        p.set_bounds((0.0,) * 3, (box,) * 3)
    num, cst = p.numerics(), p.computed()
    p.close()
    assert cst["uniform"] == 1
    n1, n2 = len(e1) - 1, 1 if kind == "s" else len(e2) - 1
    rng = np.random.default_rng(seed)
    bbox = tuple(np.asarray(b) for b in bounds) if bounds else None
    parts = [_pairs(g, PAIRS, rng, bbox)]
    if not bounds:
        parts.append(_knife_pairs(g, rng))
    A, B = (np.concatenate([q[i] for q in parts]) for i in (0, 1))
    if tree and not bounds:  # an open box: no pairs across a face
        keep = np.all(np.abs(A - B) < 0.5 * box, axis=1)
        A, B = A[keep], B[keep]
    ref = oracle.classify_pairs(A, B, kind=kind, edges1=e1, edges2=e2, los=los, box=0.0 if tree else box)
    if tree:
        extent = float(np.max(np.subtract(bounds[1], bounds[0]))) if bounds else box
        d, widen = _tree_frame(A, B, num, extent, rng)
    else:
        d, widen = _grid_frame(A, B, num, box, cst, rng)
    ex = _exact_values(kind, los, 0.0 if tree else box, n2, A, B)
    tr = float(num["trans_rel"])
    most = {}
    share = 0.0
    for dl in ((-1, -1), (0, 0), (1, 1), (-1, 1), (1, -1)):
        got, seen = _decide(kind, los, n1, n2, cst, d, A, widen, (dl[0] * tr, dl[1] * tr))
        bad = np.nonzero((got != -2) & (got != ref))[0]
        assert len(bad) == 0, (name, dl, A[bad[:3]], B[bad[:3]], got[bad[:3]], ref[bad[:3]])
        share = max(share, float(np.mean(got == -2)))
        # how much of its tolerance the error takes, near an edge (of pairs that the
        # other axis does not drop)
        for axis, (x, tol) in seen.items():
            if axis == "mu":
                want = ex["mun"]
            else:
                e = e1 if axis == "s" else e2
                want = (np.sqrt(ex["v1" if axis == "s" else "v2"]) - e[0]) / (e[-1] - e[0]) * (len(e) - 1)
            near = np.isfinite(want) & np.isfinite(x) & (np.abs(want - np.rint(want)) <= tol) & (tol < 0.5) & (tol > 0)
            if kind == "spi":
                near &= (ex["v1"] <= e1[-1] ** 2 * 1.001) & (ex["v2"] <= e2[-1] ** 2 * 1.001)
            if near.any():
                most[axis] = max(most.get(axis, 0.0), float(np.max(np.abs(x[near] - want[near]) / tol[near])))
    print(f"[computed] {name}{' tree' if tree else ''}: {len(A)} pairs, rechecked {share:.3f}, largest share of a "
          f"tolerance: " + ", ".join(f"{k} {v:.3f}" for k, v in most.items()))
    assert all(v < 1.0 for v in most.values()), most


@pytest.mark.parametrize("i", range(len(_cases())), ids=[g[0] for g in _cases()])
def test_grid_decisions_match_the_oracle(i):
    _check(_cases()[i], False, 2000 + i)


@pytest.mark.parametrize("i", range(len(_cases())), ids=[g[0] for g in _cases()])
def test_tree_decisions_match_the_oracle(i):
    _check(_cases()[i], True, 3000 + i)


def test_tables_where_an_axis_is_not_uniform():
    lin = synth.linear_edges(0, 100, 20)
    for kind, e1, e2, uniform in (("s", lin, None, 1), ("s", synth.log_edges(0.1, 50.0, 50), None, 0),
                                  ("s", lin + np.where(np.arange(21) == 7, 1e-5, 0.0), None, 0),
                                  ("spi", lin, lin ** 1.01, 0), ("spi", lin ** 1.01, lin, 0), ("spi", lin, lin, 1),
                                  ("s", synth.linear_edges(0, 1, 16000), None, 1),
                                  ("s", 400.0 + synth.linear_edges(0, 0.01, 100), None, 0)):
        p = fcfc.Plan(kind, e1, e2, box=1000.0, n_hint=10000)
        c = p.computed()
        p.close()
        assert c["uniform"] == uniform, (kind, c)
        if not uniform:
            assert not any(v for k, v in c.items())
