"""Conflict resolution on its own: from the exported hit tables, every cluster
goes to the tracklet with most hits (the lower index on a tie) and a track keeps
the hits it won, recomputed here and compared exactly.  Numbers of tracklets
around the groups of four that a wave takes, up to a full collision."""
import numpy as np
import pytest
import torch

import tpcsynth
from paper_2208_07412_amd import pipeline, tpc

from _parity import run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tracks,sectors", [(1, 1), (2, 1), (3, 1), (5, 1), (9, 1), (60, 1),
                                            (400, 1), (3000, 36)])
def test_claims_from_hit_tables(tracks, sectors):
    cfg = tpcsynth.config_small(tracks) if sectors == 1 else tpcsynth.config_c2()
    ev = tpcsynth.generate(cfg, 77)
    mc, mt = ev.n_samples // 4 + 64, ev.n_samples // 16 + 64
    reco = tpc.Reco(ev.n_units, ev.n_time_bins, mc, mt, max_samples=ev.n_samples)
    try:
        zs = tpc.to_device_zs(ev.pad, ev.time, ev.adc, ev.row_start, ev.n_units, ev.n_time_bins)
        cl, links = reco.alloc_clusters(ev.n_units, ev.n_time_bins, mc), reco.alloc_links(mc)
        tl, tr = reco.alloc_tracklets(mt), reco.alloc_tracks(mt, mc, mc, mt)
        reco.process(zs, cl, links, tl, tr)
        c = reco.sync()
        out = tpc.tracks_to_host(tr, c["n_clusters"], c["n_tracklets"])
        min_hits = reco.params.min_track_hits
    finally:
        reco.close()
    H = out["follow_hits"].astype(np.int64)
    nh = (H >= 0).sum(1)
    bids = nh >= min_hits
    key = (nh << 24) | (0xFFFFFF - np.arange(len(H)))
    owner = np.zeros(c["n_clusters"], np.int64)
    for t in np.nonzero(bids)[0]:
        np.maximum.at(owner, H[t][H[t] >= 0], key[t])
    won = (H >= 0) & bids[:, None] & (owner[np.maximum(H, 0)] == key[:, None])
    n = won.sum(1)
    hs, tlt = out["hit_start"].astype(np.int64), out["tracklet"]
    assert np.array_equal(np.diff(hs), n[tlt]) and (n[tlt] >= min_hits).all()
    for j, t in enumerate(tlt):
        assert np.array_equal(out["hits"][hs[j]:hs[j + 1]], H[t][won[t]])
    ct = np.full(c["n_clusters"], -1)
    ct[out["hits"]] = np.repeat(np.arange(len(tlt)), np.diff(hs))
    assert np.array_equal(out["cluster_track"], ct)
    # what kept enough hits and is no track failed its refit
    assert (n >= min_hits).sum() - len(tlt) <= c["n_refit_fail"] + c["n_fallback_fail"]


def test_claims_with_streams_at_work():
    # four parts on streams of their own, again and again: every pass has the
    # hits of one call over the whole frame
    ev = tpcsynth.generate(tpcsynth.config_chunk(404, 3, n_coll=6), 4043)
    full = run_gpu(ev, moments=False, follow=False)["tracks"]["hits"].astype(np.int64)
    zs = tpc.to_device_zs(ev.pad, ev.time, ev.adc, ev.row_start, ev.n_units, ev.n_time_bins)
    p = pipeline.Pipeline(zs, 4, stagger="none")
    want = None
    for i in range(200):
        p.enqueue()
        torch.cuda.synchronize()
        got = [sl.tr["hits"][:int(sl.tr["n_hits"].item())].clone() for sl in p.slices]
        if want is None:
            off = np.cumsum([0] + [int(sl.cl["n_clusters"].item()) for sl in p.slices])
            n = np.cumsum([0] + [len(g) for g in got])
            assert n[-1] == len(full)
            want = [torch.from_numpy((full[n[k]:n[k + 1]] - off[k]).astype(np.int32)).cuda()
                    for k in range(4)]
        assert all(torch.equal(g, w) for g, w in zip(got, want)), i
    p.close()
