"""Codec paths against the oracle, word for word: records of few and many hits
(one and several 64-hit rounds), of no hits, with gaps between rows, with codes
that one kept word holds, that two hold and that are coded anew; runs of records
shorter and longer than the LDS they are put together in; rows whose clusters on
no track fill a list exactly, overfill it, or are none; decoding in two steps and
(outputs larger than the context's clusters) in one."""
import numpy as np
import pytest
import torch

import oracle
from paper_2208_07412_amd import tpc

from test_gpu_compress import _same_decoded

pytestmark = pytest.mark.gpu
NROW = 152


def frame(seed, n_units, tracks, loose, spread):
    """tracks: (unit, rows of its hits); loose: {(unit, row): clusters on no
    track}; spread: scale of positions about zero.  One cluster per hit."""
    rng = np.random.default_rng(seed)
    per = [[[] for _ in range(NROW)] for _ in range(n_units)]
    for j, (u, rows) in enumerate(tracks):
        for r in rows:
            per[u][r].append(j)
    for (u, r), n in loose.items():
        per[u][r] += [-1] * n
    crow, ct, where = [0], [], {}
    for u in range(n_units):
        for r in range(NROW):
            order = rng.permutation(len(per[u][r]))
            for k in order:
                j = per[u][r][k]
                if j >= 0:
                    where[(j, r)] = len(ct)
                ct.append(j)
            crow.append(len(ct))
    n = len(ct)
    clusters = dict(crow_start=np.array(crow, np.uint32), n_units=n_units,
                    y_fx=rng.normal(0, spread, n).clip(-2**30, 2**30).astype(np.int32),
                    z_fx=np.abs(rng.normal(0, spread, n)).clip(0, 2**30).astype(np.int32),
                    qtot=(65536 * rng.random(n) ** 4).astype(np.uint16),
                    qmax=(65536 * rng.random(n) ** 6).astype(np.uint16),
                    flags=rng.integers(0, 4, n).astype(np.uint8),
                    ptime=np.zeros(n, np.uint16), ppad=np.zeros(n, np.uint16))
    hits = [where[(j, r)] for j, (u, rows) in enumerate(tracks) for r in rows]
    hs = np.concatenate([[0], np.cumsum([len(rows) for _, rows in tracks])]).astype(np.uint32)
    m = len(tracks)
    par = np.stack([rng.normal(0, 5, m), rng.normal(0, 5, m), rng.uniform(-0.9, 0.9, m),
                    rng.uniform(-1, 1, m), rng.normal(0, 3, m)], 1).astype(np.float32)
    first = [rows[0] if rows else 7 for _, rows in tracks]
    row = [max(0, f - int(rng.integers(0, 3))) for f in first]
    tr = dict(tracklet=np.arange(m, dtype=np.uint32), par=par, row=np.array(row, np.uint8),
              z_anchor=rng.integers(0, 2**24, m).astype(np.int32), hit_start=hs,
              hits=np.array(hits, np.uint32), cluster_track=np.array(ct, np.int32))
    return clusters, tr


def some_rows(rng, n, gap):
    r, out = int(rng.integers(0, 4)), []
    while len(out) < n and r < NROW:
        out.append(r)
        r += 1 + (int(rng.integers(0, gap)) if rng.random() < 0.3 else 0)
    return out


def make(name):
    rng = np.random.default_rng(len(name))
    if name == "lengths":
        lens = [1, 2, 63, 64, 65, 100, 127, 128, 129, 152, 0, 0, 5, 36, 0] * 3
        t = [(int(rng.integers(0, 2)), list(range(NROW))[:n]) for n in lens]
        return frame(1, 2, t, {(0, 5): 3, (1, 151): 64, (1, 150): 65}, 2e4)
    if name == "gaps":
        t = [(u % 3, some_rows(rng, 40, 30)) for u in range(50)]
        return frame(2, 3, t, {(2, 0): 1}, 2e4)
    if name == "wide_codes":  # residuals of many bits: two words, and coded anew
        t = [(0, some_rows(rng, 30, 3)) for _ in range(40)] + [(0, list(range(NROW)))] * 0
        return frame(3, 1, t, {}, 4e8)
    if name == "mixed_codes":
        c, t = frame(4, 1, [(0, some_rows(rng, 50, 3)) for _ in range(60)], {(0, 9): 200}, 2e4)
        far = np.random.default_rng(5).random(len(c["y_fx"]))
        c["y_fx"] = np.where(far < 0.02, c["y_fx"] * 1000, c["y_fx"]).astype(np.int32)
        c["z_fx"] = np.where(far > 0.99, c["z_fx"] * 3000, c["z_fx"]).astype(np.int32)
        return c, t
    if name == "long_runs":
        return frame(6, 1, [(0, list(range(NROW))) for _ in range(30)], {}, 3e6)
    if name == "row_lists":
        return frame(7, 1, [(0, [3, 4, 5])], {(0, 10): 4096, (0, 11): 4097, (0, 12): 255,
                                              (0, 13): 256, (0, 14): 257, (0, 151): 9000}, 1e6)
    return frame(8, 1, [], {}, 1.0)


@pytest.mark.parametrize("name", ["lengths", "gaps", "wide_codes", "mixed_codes", "long_runs",
                                  "row_lists", "nothing"])
def test_paths(name):
    clusters, tracks = make(name)
    n, n_units = len(clusters["y_fx"]), clusters["n_units"]
    o = oracle.compress(clusters, tracks, n_units,
                        capacity_words=4096 + n_units * 200 + (n + 60 * len(tracks["row"])) * 10)
    assert o["status"] == 0
    reco = tpc.Reco(n_units, 500, max(n, 1), max(len(tracks["row"]), 1))
    small = tpc.Reco(n_units, 500, 1, max(len(tracks["row"]), 1), max_samples=1)
    try:
        cl = reco.clusters_from_host(clusters, n_units, 500)
        tr = reco.tracks_from_host(tracks, max(n, 1))
        comp = reco.alloc_compressed(o["n_words"] + 3)
        for _ in range(2):
            reco.compress(cl, tr, comp)
            reco.sync()
        got = tpc.compressed_to_host(comp)
        assert got["n_words"] == o["n_words"]
        bad = np.nonzero(got["words"] != o["words"])[0]
        assert len(bad) == 0, f"{len(bad)} words differ, first {bad[:5]}"
        assert np.array_equal(got["hist"], o["hist"])
        ref = oracle.decompress(o["words"])
        for r in (reco, small):  # in two steps, and in one
            dec = r.alloc_decoded(max(n, 1))
            r.decompress(comp["stream"], dec, got["n_words"])
            r.sync()
            _same_decoded(tpc.decoded_to_host(dec), ref)
    finally:
        reco.close()
        small.close()


@pytest.mark.parametrize("name", ["lengths", "gaps"])
def test_malformed_records(name):
    """A bit flipped in a record's codes or fixed fields, a chunk or a row: both
    decoders report it exactly where the oracle rejects the stream."""
    clusters, tracks = make(name)
    n, n_units = len(clusters["y_fx"]), clusters["n_units"]
    w = oracle.compress(clusters, tracks, n_units)["words"]
    m = len(tracks["row"])
    dir_words = 8 + m + 1 + n_units * NROW + 1
    rng = np.random.default_rng(11)
    reco = tpc.Reco(n_units, 500, n, m)
    small = tpc.Reco(n_units, 500, 1, m, max_samples=1)
    try:
        rejected = 0
        for _ in range(40):
            a = w.copy()
            a[int(rng.integers(dir_words, len(w)))] ^= np.uint32(1 << int(rng.integers(0, 32)))
            ref = oracle.decompress(a)
            for r in (reco, small):
                dec = r.alloc_decoded(n)
                r.decompress(torch.from_numpy(a.view(np.int32)).cuda(), dec)
                st = r.sync(raise_on_error=False)["status"]
                assert (st != 0) == (ref["status"] != 0)
                if st == 0:
                    _same_decoded(tpc.decoded_to_host(dec), ref)
            rejected += ref["status"] != 0
        assert rejected > 0
    finally:
        reco.close()
        small.close()
