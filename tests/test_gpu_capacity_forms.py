"""The forms that scans and sorts take by capacity (one workgroup, sums added up
by their users, sums scanned by a launch of their own; sorts that add up their
counts or scan them) give one result: the same sector reconstructed and merged
with buffers on both sides of every line."""
import numpy as np
import pytest

import tpcsynth
from paper_2208_07412_amd import tpc

pytestmark = pytest.mark.gpu

ONE, SELF, DIRECT = 16384, 2048 * 2048, 512 * 1024  # elements; clusters; tracklets


def reconstruct(ev, mc, mt):
    reco = tpc.Reco(ev.n_units, ev.n_time_bins, mc, mt, max_samples=ev.n_samples)
    try:
        zs = tpc.to_device_zs(ev.pad, ev.time, ev.adc, ev.row_start, ev.n_units, ev.n_time_bins)
        cl, links = reco.alloc_clusters(ev.n_units, ev.n_time_bins, mc), reco.alloc_links(mc)
        tl, tr = reco.alloc_tracklets(mt), reco.alloc_tracks(mt, mc, mc)
        mg = reco.alloc_merged(mt)
        reco.process(zs, cl, links, tl, tr)
        reco.merge_tracks(cl, tr, mg)
        c = reco.sync()
        return (c, tpc.clusters_to_host(cl, ev.n_units), tpc.links_to_host(links, c["n_clusters"]),
                tpc.tracklets_to_host(tl), tpc.tracks_to_host(tr, c["n_clusters"]),
                tpc.merged_to_host(mg, c["n_tracks"]))
    finally:
        reco.close()


@pytest.fixture(scope="module")
def event():
    ev = tpcsynth.generate(tpcsynth.config_small(60), 31)
    return ev, reconstruct(ev, 15000, 4000)


@pytest.mark.parametrize("mc,mt", [(ONE, ONE), (ONE + 1, ONE + 1), (2 * ONE, 2 * ONE + 1),
                                   (SELF, 20000), (SELF + 1, 20000), (2 * SELF, 20000),
                                   (20000, DIRECT), (20000, DIRECT + 1)])
def test_same_results(event, mc, mt):
    ev, ref = event
    got = reconstruct(ev, mc, mt)
    assert ref[0]["n_tracks"] > 20
    assert got[0] == ref[0]
    for a, b in zip(got[1:], ref[1:]):
        for k in b:
            assert np.array_equal(a[k], b[k]), k


def test_stages_equal_the_whole(event):
    # called stage by stage the fit walks the tracklets itself
    ev, ref = event
    mc, mt = 15000, 4000
    reco = tpc.Reco(ev.n_units, ev.n_time_bins, mc, mt, max_samples=ev.n_samples)
    try:
        zs = tpc.to_device_zs(ev.pad, ev.time, ev.adc, ev.row_start, ev.n_units, ev.n_time_bins)
        cl, links = reco.alloc_clusters(ev.n_units, ev.n_time_bins, mc), reco.alloc_links(mc)
        tl, tr = reco.alloc_tracklets(mt), reco.alloc_tracks(mt, mc, mc)
        reco.cluster(zs, cl)
        reco.find_neighbours(cl, links)
        reco.build_tracklets(cl, links, tl)
        reco.fit_tracks(cl, links, tl, tr)
        c = reco.sync()
        got = tpc.tracklets_to_host(tl), tpc.tracks_to_host(tr, c["n_clusters"])
    finally:
        reco.close()
    for a, b in zip(got, ref[3:5]):
        for k in b:
            assert np.array_equal(a[k], b[k]), k
