"""The following's ways of dealing tracklets to lanes give one result.

A sort group's tracklets are spread over its waves with 4, 2 or 1 lanes each,
or taken from a queue, by their number.  Copies of one event batched together
reach each of them; every copy's tracks have to equal those of the event alone
followed one tracklet per lane in one launch (which the oracle tests hold).
"""
import numpy as np
import pytest

import tpcsynth
from paper_2208_07412_amd import tpc

pytestmark = pytest.mark.gpu

FIELDS = ("par", "cov", "chi2", "ndf", "row", "flags", "z_anchor")


def reconstruct(ev, tuning=None):
    mc, mt = ev.n_samples // 8 + 4096, ev.n_samples // 64 + 1024
    reco = tpc.Reco(ev.n_units, ev.n_time_bins, mc, mt, max_samples=max(ev.n_samples, 1))
    if tuning:
        reco.set_tuning(**tuning)
    zs = tpc.to_device_zs(ev.pad, ev.time, ev.adc, ev.row_start, ev.n_units, ev.n_time_bins)
    cl, links = reco.alloc_clusters(ev.n_units, ev.n_time_bins, mc), reco.alloc_links(mc)
    tl, tr = reco.alloc_tracklets(mt), reco.alloc_tracks(mt, mc, mc)
    reco.process(zs, cl, links, tl, tr)
    c = reco.sync()
    out = tpc.tracks_to_host(tr, c["n_clusters"], 0)
    reco.close()
    return c, out


# copies of a central collision (19,600 tracklets): 4 and 2 lanes per
# tracklet, one lane each, lanes refilled from the queue
@pytest.mark.parametrize("tracks,copies", [(1, 1), (40, 1), (3600, 1), (3600, 4), (3600, 8),
                                           (3600, 14)])
def test_spread_equals_one_lane_each(tracks, copies):
    sector = tracks < 100
    cfg = tpcsynth.config_small(tracks) if sector else tpcsynth.config_c2()
    ev = tpcsynth.generate(cfg, 29)
    c1, ref = reconstruct(ev, dict(follow_mode=1))
    c, got = reconstruct(tpcsynth.stack([ev] * copies) if copies > 1 else ev)
    assert c["n_tracklets"] == copies * c1["n_tracklets"]
    assert c["n_tracks"] == copies * c1["n_tracks"] and c["n_hits"] == copies * c1["n_hits"]
    for k in FIELDS:
        assert np.array_equal(got[k], np.concatenate([ref[k]] * copies)), k
    hits = got["hits"].reshape(copies, -1) - (np.arange(copies) * c1["n_clusters"])[:, None]
    assert np.array_equal(hits, np.broadcast_to(ref["hits"], hits.shape))
