"""The shared-window peak pass where its parts meet: clusters, moments and
labels bit-exact against the oracle at window and row edges, at peak lists of
one entry and of several batches, at windows below and above the samples that a
wave prefetches, and in both prefetch depths (chosen by the mean occupancy)."""
import numpy as np
import pytest

import oracle
import tpcsynth

from _parity import compare_clusters, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

NPADS, _, _ = oracle.geometry()


def event(rows, T):
    """rows: {row: [(time, pad, adc)]} of one unit."""
    s = sorted((r, t, p, a) for r, v in rows.items() for t, p, a in v)
    col = lambda i: np.array([x[i] for x in s], np.uint16)
    start = np.zeros(153, np.uint32)
    for r, *_ in s:
        start[r + 1] += 1
    cfg = tpcsynth.config_small(0, n_time_bins=T)
    return tpcsynth.Event(cfg, col(2), col(1), col(3), np.cumsum(start).astype(np.uint32), 1, T,
                          {}, {}, None)


def edges(T):
    """Lone peaks, plateaus and saturated blobs on every window edge and pad edge."""
    out = {}
    for r in (0, 1, 75, 151):
        n = int(NPADS[r])
        v = []
        for t in range(0, T, 8):
            for p in (0, n // 2, n - 1):
                v.append((t + (p % 3 == 0), p, 1023 if t % 64 == 32 else 20 + t % 7))
        out[r] = [(t, p, a) for t, p, a in set((min(t, T - 1), p, a) for t, p, a in v)]
        seen = {}
        for t, p, a in out[r]:
            seen[(t, p)] = a
        for t in range(30, min(T, 66)):  # a ridge across two window edges, ties along it
            for p in (n // 3, n // 3 + 1):
                seen[(t, p)] = 50 + (t % 5 == 0)
        out[r] = [(t, p, a) for (t, p), a in seen.items()]
    return out


def lattice(T, step):
    """A peak every `step` bins and pads: more peaks than one list holds."""
    return {r: [(t, p, 9 + (t * 7 + p) % 5) for t in range(0, T, step)
                for p in range(0, int(NPADS[r]), step)] for r in (3, 100)}


def noise(T, share, rows, seed):
    rng = np.random.default_rng(seed)
    out = {}
    for r in rows:
        t, p = np.nonzero(rng.random((T, int(NPADS[r]))) < share)
        out[r] = [(int(a), int(b), int(c)) for a, b, c in zip(t, p, rng.integers(1, 60, len(t)))]
    return out


CASES = {
    "edges": (lambda: edges(131), 131),
    "lattice2": (lambda: lattice(97, 2), 97),
    "lattice3": (lambda: lattice(64, 3), 64),
    "one_sample": (lambda: {151: [(0, 137, 1023)]}, 1),
    "short_frame": (lambda: noise(7, 0.5, (0, 151), 1), 7),
    "few_rows_dense": (lambda: noise(200, 0.6, (10, 150), 2), 200),   # more steps than prefetched
    "all_rows_dense": (lambda: noise(70, 0.12, range(152), 3), 70),   # the deeper prefetch
    "full": (lambda: noise(72, 1.0, (151,), 4), 72),
}


@pytest.mark.parametrize("w,k", [(32, 8), (24, 8), (32, 4), (32, 16)])
@pytest.mark.parametrize("name", sorted(CASES))
def test_shared_windows(name, w, k):
    make, T = CASES[name]
    ev = event(make(), T)
    g = run_gpu(ev, labels=True, max_tracklets=1024,
                tuning=dict(cl_window=w, cl_chunk=k, cl_mode=2))
    o = run_oracle(ev, labels=True)
    compare_clusters(g["clusters"], o["clusters"], labels=True)


@pytest.mark.parametrize("bins", [53 * 512, 53 * 512 + 1])
def test_windows_per_workgroup_by_frame_size(bins):
    # 8056 and 8208 workgroups of 16 windows: 8 windows each below the line, 16 above
    ev = event(noise(bins, 0.002, (0, 75, 151), 3), bins)
    g, o = run_gpu(ev, labels=True, max_tracklets=4096), run_oracle(ev, labels=True)
    compare_clusters(g["clusters"], o["clusters"], labels=True)
