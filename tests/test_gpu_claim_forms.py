"""Conflict resolution of tracklets whose chains share clusters, as a caller of the
fit may give them (starts inside other chains, tracklets twice): every cluster goes
to the tracklet with most hits, the lower index on a tie, and the claims by chains
that the whole call makes give the same tracks as the claims of each hit."""
import numpy as np
import pytest
import torch

import tpcsynth
from paper_2208_07412_amd import tpc

pytestmark = pytest.mark.gpu


def resolve(H, n_clusters, min_hits):
    """Owner of every cluster and the hits that each tracklet of the table H keeps."""
    nh = (H >= 0).sum(1)
    bids = nh >= min_hits
    key = (nh << 24) | (0xFFFFFF - np.arange(len(H)))
    owner = np.zeros(n_clusters, np.int64)
    for t in np.nonzero(bids)[0]:
        np.maximum.at(owner, H[t][H[t] >= 0], key[t])
    return (H >= 0) & bids[:, None] & (owner[np.maximum(H, 0)] == key[:, None])


@pytest.mark.parametrize("form", ["chains", "twice", "inside", "reversed"])
@pytest.mark.parametrize("tracks,sectors", [(60, 1), (3000, 36)])
def test_overlapping_tracklets(tracks, sectors, form):
    ev = tpcsynth.generate(tpcsynth.config_small(tracks) if sectors == 1 else tpcsynth.config_c2(), 78)
    mc, mt = ev.n_samples // 4 + 64, ev.n_samples // 4 + 64
    reco = tpc.Reco(ev.n_units, ev.n_time_bins, mc, mt, max_samples=ev.n_samples)
    try:
        zs = tpc.to_device_zs(ev.pad, ev.time, ev.adc, ev.row_start, ev.n_units, ev.n_time_bins)
        cl, links = reco.alloc_clusters(ev.n_units, ev.n_time_bins, mc), reco.alloc_links(mc)
        tl, tr = reco.alloc_tracklets(mt), reco.alloc_tracks(mt, mc, mc, mt)
        reco.process(zs, cl, links, tl, tr)
        c = reco.sync()
        n_cl = c["n_clusters"]
        whole = tpc.tracks_to_host(tr, n_cl, c["n_tracklets"])
        h = tpc.tracklets_to_host(tl)
        upc = links["upc"].cpu().numpy()
        start, length = h["tl_start"].astype(np.int64), h["tl_len"].astype(np.int64)
        if form == "twice":
            start, length = np.repeat(start, 2), np.repeat(length, 2)
        elif form == "inside":  # every chain again, from its second cluster on
            long = length > 5
            start = np.concatenate([start, upc[start[long]]])
            length = np.concatenate([length, length[long] - 1])
        elif form == "reversed":
            start, length = start[::-1].copy(), length[::-1].copy()
        n = len(start)
        tl["start"][:n] = torch.from_numpy(start.astype(np.int32)).cuda()
        tl["len"][:n] = torch.from_numpy(length.astype(np.int16)).cuda()
        tl["n_tracklets"].fill_(n)
        torch.cuda.synchronize()
        reco.fit_tracks(cl, links, tl, tr)
        c = reco.sync()
        out = tpc.tracks_to_host(tr, n_cl, n)
        min_hits = reco.params.min_track_hits
    finally:
        reco.close()
    if form == "chains":
        for k in whole:
            assert np.array_equal(out[k], whole[k]), k
    won = resolve(out["follow_hits"].astype(np.int64), n_cl, min_hits)
    kept, hs, tlt = won.sum(1), out["hit_start"].astype(np.int64), out["tracklet"]
    assert np.array_equal(np.diff(hs), kept[tlt]) and (kept[tlt] >= min_hits).all()
    for j, t in enumerate(tlt):
        assert np.array_equal(out["hits"][hs[j]:hs[j + 1]], out["follow_hits"][t][won[t]])
    assert (kept >= min_hits).sum() - len(tlt) <= c["n_refit_fail"] + c["n_fallback_fail"]


@pytest.mark.parametrize("name", ["sector", "central", "noise"])
def test_chains_share_no_cluster(name):
    # what the claims by chains rest on: each word is stored by one tracklet
    ev = tpcsynth.generate(tpcsynth.config_c2() if name == "central" else
                           tpcsynth.config_small(100), 79)
    # (wide windows on noise: most links are wrong, and chains still share nothing)
    over = dict(win_y=1 << 20, win_z=1 << 20, s_max=1 << 42) if name == "noise" else {}
    mc, mt = ev.n_samples // 2 + 64, ev.n_samples // 4 + 64
    reco = tpc.Reco(ev.n_units, ev.n_time_bins, mc, mt, max_samples=ev.n_samples,
                    param_overrides=over)
    try:
        zs = tpc.to_device_zs(ev.pad, ev.time, ev.adc, ev.row_start, ev.n_units, ev.n_time_bins)
        cl, links = reco.alloc_clusters(ev.n_units, ev.n_time_bins, mc), reco.alloc_links(mc)
        tl, tr = reco.alloc_tracklets(mt), reco.alloc_tracks(mt, mc, mc, mt)
        reco.process(zs, cl, links, tl, tr)
        c = reco.sync()
        h, hits = tpc.tracklets_to_host(tl), tpc.tracks_to_host(tr, 1, c["n_tracklets"])["follow_hits"]
        upc = links["upc"].cpu().numpy()
    finally:
        reco.close()
    at, left = h["tl_start"].astype(np.int64), h["tl_len"].astype(np.int64)
    row = np.searchsorted(cl["crow_start"].cpu().numpy(), at, side="right") - 1
    seen = np.zeros(c["n_clusters"], np.int64)
    t = np.arange(len(at))
    assert len(at) > 20
    while len(at):
        np.add.at(seen, at, 1)
        found = hits[t, row % 152]  # a hit in a row of the chain is the chain's cluster
        assert ((found < 0) | (found == at)).all()
        on = left > 1
        at, left, row, t = upc[at[on]].astype(np.int64), left[on] - 1, row[on] + 1, t[on]
    assert seen.max() == 1
