"""Segment merging at the sizes where its pair search and its fit change: ends
that fill no, one and many waves, more pairs than a queue holds, few and many
components (16 and 8 lanes each), hits per segment around the lanes' steps.
Cut-up helices with displaced pieces, so that pairs fall on both sides of every
cut, and curvatures on both sides of the straight-line limit."""
import numpy as np
import pytest

import oracle

from _helix_frames import B, NROW, row_x_fx
from test_gpu_merge import FIELDS, _gpu_merge

pytestmark = pytest.mark.gpu

CURV = np.array([0.0, 0.99999e-4, 1.00001e-4, -1e-4, 4e-4, -3e-3, 0.006, -0.012, 0.03])
LENGTHS = np.array([1, 2, 3, 7, 8, 9, 15, 16, 17, 24, 33])


def cut_helices(n, n_units, seed):
    """n segments of helices in random sectors, and their clusters."""
    rng = np.random.default_rng(seed)
    xr = row_x_fx(np.arange(NROW)) / 65536.0
    unit, row, y, z, par, hs = [], [], [], [], [], [0]
    while len(par) < n:
        u, C, tgl = rng.integers(n_units), rng.choice(CURV), rng.uniform(-2, 2)
        s0, y0, z0 = rng.uniform(-0.2, 0.2), rng.uniform(-14, 14), rng.uniform(20, 240)
        r = int(rng.integers(0, 30))
        xa = xr[r]
        while len(par) < n:
            m = int(rng.choice(LENGTHS))
            rr = np.arange(r, min(r + m, NROW))
            s = s0 + C * (xr[rr] - xa)
            rr, s = rr[np.abs(s) < 0.95], s[np.abs(s) < 0.95]
            if not len(rr):
                break
            dx, f0, f = xr[rr] - xa, np.arcsin(s0), np.arcsin(s)
            if C:
                yy, arc = y0 + (np.cos(f0) - np.cos(f)) / C, (f - f0) / C
            else:
                yy, arc = y0 + dx * np.tan(f0), dx / np.cos(f0)
            yy, zz = yy + rng.normal(0, 0.25), z0 + tgl * arc + rng.normal(0, 0.7)
            unit.append(np.full(len(rr), u))
            row.append(rr)
            y.append(np.rint(yy * 65536))
            z.append(np.rint(np.clip(zz, 0, 255) * 65536))
            par.append((yy[0], 0.0, s[0] + rng.normal(0, 0.03), tgl + rng.normal(0, 0.02),
                        -C * (1 + rng.normal(0, 0.1)) / B))
            hs.append(hs[-1] + len(rr))
            r = int(rr[-1]) + int(rng.integers(1, 12))
            if r >= NROW:
                break
    unit, row, y, z = (np.concatenate(a).astype(np.int64) for a in (unit, row, y, z))
    ur = unit * NROW + row
    order = np.argsort(ur, kind="stable")
    hits = np.empty(len(ur), np.uint32)
    hits[order] = np.arange(len(ur))
    hs = np.array(hs, np.uint32)
    nc = len(ur)
    crow = np.searchsorted(ur[order], np.arange(n_units * NROW + 1))
    cl = dict(crow_start=crow.astype(np.uint32),
              y_fx=y[order].astype(np.int32), z_fx=z[order].astype(np.int32),
              qtot=np.ones(nc, np.uint16), qmax=np.ones(nc, np.uint16),
              flags=np.zeros(nc, np.uint8))
    tr = dict(par=np.array(par, np.float32), row=row[hs[:-1]].astype(np.uint8),
              z_anchor=z[hs[:-1]].astype(np.int32), hit_start=hs, hits=hits)
    return cl, tr


@pytest.mark.parametrize("n,n_units", [(1, 1), (2, 1), (31, 1), (32, 1), (33, 1), (700, 1),
                                       (4000, 36), (33000, 36)])
def test_labels(n, n_units):
    # (labels and counts: the circle through three almost collinear hits of a
    # piece has no bound against the oracle; the fits are the next test's)
    cl, tr = cut_helices(n, n_units, n)
    o = oracle.merge_tracks(cl, tr, n_units)
    g = _gpu_merge(cl, tr, n_units, 1000)
    if n >= 700:  # the pieces do join
        assert len(np.unique(o["label"])) < 0.8 * n
    assert np.array_equal(g["label"].astype(np.int64), o["label"])
    assert g["n_merged"] == len(np.unique(o["label"]))
    for k in ("n_segments", "n_hits"):
        assert np.array_equal(g[k], o[k]), k


def test_fit_widths():
    # 2000 segments alone (16 lanes per component, the width of the frames that
    # other tests hold against the oracle) and followed by a frame of 33000 (8
    # lanes): the same sums in the same order, so the same bits
    a, ta = cut_helices(2000, 36, 5)
    b, tb = cut_helices(33000, 36, 6)
    nc, nh = len(a["y_fx"]), len(ta["hits"])
    cl = {k: np.concatenate([a[k], b[k]]) for k in a if k != "crow_start"}
    cl["crow_start"] = np.concatenate([a["crow_start"][:-1], b["crow_start"] + np.uint32(nc)])
    tr = {k: np.concatenate([ta[k], tb[k]]) for k in ("par", "row", "z_anchor")}
    tr["hit_start"] = np.concatenate([ta["hit_start"][:-1], tb["hit_start"] + np.uint32(nh)])
    tr["hits"] = np.concatenate([ta["hits"], tb["hits"] + np.uint32(nc)])
    alone, both = _gpu_merge(a, ta, 36, 1000), _gpu_merge(cl, tr, 72, 1000)
    for k in ("label", "near_tie") + FIELDS:
        assert np.array_equal(alone[k], both[k][:2000]), k


@pytest.mark.parametrize("dy,dz", [(30, 0), (30, 3), (0.5, 0), (0.5, 5), (0.25, 1), (0.6, 1),
                                   (4, 1)])
def test_ties_are_flagged(dy, dz):
    # two straight segments of one hit in one row, exactly at the cut on the gap,
    # the distance off the line or the drift, whether or not another cut is missed
    cl = dict(crow_start=np.where(np.arange(NROW + 1) > 40, 2, 0).astype(np.uint32),
              y_fx=(np.array([0, dy]) * 65536 - 65536).astype(np.int32),
              z_fx=(np.array([100, 100 + dz]) * 65536).astype(np.int32),
              qtot=np.ones(2, np.uint16), qmax=np.ones(2, np.uint16), flags=np.zeros(2, np.uint8))
    tr = dict(par=np.zeros((2, 5), np.float32), row=np.full(2, 40, np.uint8),
              z_anchor=cl["z_fx"], hit_start=np.arange(3, dtype=np.uint32),
              hits=np.arange(2, dtype=np.uint32))
    o, g = oracle.merge_tracks(cl, tr, 1), _gpu_merge(cl, tr, 1, 1000)
    assert o["near_tie"].all() and g["near_tie"].astype(bool).all()
