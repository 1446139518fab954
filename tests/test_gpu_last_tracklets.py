"""The last tracklet ids a context can have (2^24 of them), in the group of four
that a wave resolves, some bidding and the last one not: the same tracks as the
bidding tracklets alone give."""
import numpy as np
import pytest
import torch

import tpcsynth
from paper_2208_07412_amd import tpc

pytestmark = pytest.mark.gpu

CAP = 1 << 24


# tracklet ids in use from the end, 0 the last; the count of tracklets
@pytest.mark.parametrize("last,count", [((3, 2, 1), CAP), ((3,), CAP), ((1, 0), CAP),
                                        ((3, 2, 1), CAP - 1)])
def test_last_group(last, count):
    ev = tpcsynth.generate(tpcsynth.config_small(60), 31)
    mc = ev.n_samples
    reco = tpc.Reco(ev.n_units, ev.n_time_bins, mc, CAP, max_samples=mc)
    try:
        zs = tpc.to_device_zs(ev.pad, ev.time, ev.adc, ev.row_start, ev.n_units, ev.n_time_bins)
        cl, links = reco.alloc_clusters(ev.n_units, ev.n_time_bins, mc), reco.alloc_links(mc)
        tl, tr = reco.alloc_tracklets(CAP), reco.alloc_tracks(4096, mc, mc)
        reco.process(zs, cl, links, tl, tr)
        c = reco.sync()
        n, n_cl = c["n_tracklets"], c["n_clusters"]
        assert c["n_tracks"] > 20

        def fit(ids, total):
            """The first len(ids) tracklets as tracklets `ids` of `total`, the others broken."""
            start = torch.full((CAP,), -1, dtype=torch.int32, device="cuda")
            length = torch.full((CAP,), 5, dtype=torch.int16, device="cuda")
            at = torch.tensor(ids, device="cuda")
            start[at], length[at] = tl["start"][:len(ids)], tl["len"][:len(ids)]
            t = reco.alloc_tracklets(CAP)
            t["start"].copy_(start)
            t["len"].copy_(length)
            t["n_tracklets"].fill_(total)
            torch.cuda.synchronize()
            reco.fit_tracks(cl, links, t, tr)
            reco.sync()
            return tpc.tracks_to_host(tr, n_cl)

        k = len(last)
        ids = list(range(n - k)) + [count - 1 - i for i in last]
        got, want = fit(ids, count), fit(list(range(n)), n)
        assert np.array_equal(got.pop("tracklet"), np.array(ids, np.uint32)[want.pop("tracklet")])
        for f in want:
            assert np.array_equal(got[f], want[f]), f
    finally:
        reco.close()
