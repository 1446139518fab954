"""A malformed frame over many workgroups ends as an error, and the context then
serves the next frame as a new one does: workgroups that start while others latch
the error leave as a whole or run as a whole."""
import numpy as np
import pytest

import oracle
from paper_2208_07412_amd import tpc

pytestmark = pytest.mark.gpu

NPADS, _, _ = oracle.geometry()
T = 1000


def unit(seed, overfull):
    """(row, time, pad, adc) of one sector: noise in every row, and in a few rows
    every cell of 40 bins three times over (more samples than a window has cells)."""
    rng = np.random.default_rng(seed)
    out = []
    for r in range(152):
        k = np.unique(rng.integers(0, T * int(NPADS[r]), 600))
        t, p = k // int(NPADS[r]), k % int(NPADS[r])
        if overfull and r in (130, 151):
            tt, pp = np.divmod(np.repeat(np.arange(40 * int(NPADS[r])), 3), int(NPADS[r]))
            keep = t >= 40
            t, p = np.concatenate([tt, t[keep]]), np.concatenate([pp, p[keep]])
        out.append((t, p, rng.integers(1, 200, len(t))))
    return out


def frame(bad, n_units=36):
    units = [unit(5, False), unit(5, True)]
    rows = [v for u in range(n_units) for v in units[int(u % bad == 1) if bad else 0]]
    t, p, a = (np.concatenate([v[i] for v in rows]).astype(np.uint16) for i in range(3))
    rs = np.concatenate([[0], np.cumsum([len(v[0]) for v in rows])]).astype(np.uint32)
    return tpc.to_device_zs(p, t, a, rs, n_units, T), len(t)


def test_overfull_windows_among_many():
    good, ng = frame(0)
    bad = [frame(b) for b in (2, 5, 35)]
    cap = max([ng] + [n for _, n in bad])

    def clusters(reco):
        cl = reco.alloc_clusters(36, T, ng)
        reco.cluster(good, cl)
        reco.sync()
        return tpc.clusters_to_host(cl, 36)

    fresh = tpc.Reco(36, T, cap, 64, max_samples=cap)
    want = clusters(fresh)
    fresh.close()
    reco = tpc.Reco(36, T, cap, 64, max_samples=cap)
    for zs, _ in bad * 3:
        reco.cluster(zs, reco.alloc_clusters(36, T, cap))
        assert reco.sync(raise_on_error=False)["status"] == -3
        got = clusters(reco)
        for k in want:
            assert np.array_equal(got[k], want[k]), k
    reco.close()
