"""GPU sector merger (C8) and chain refit (C9) against the oracle.

Bars: the oracle's links between tracks that both sides found (same start
position) are reproduced for >= 99.5% of links, and >= 99.5% of the GPU's links
are oracle links; every chain with the same clusters on both sides and a
successful refit on both has refit parameters within 1e-4 relative (floors as
for tracks) and covariance diagonals within 1e-3 relative; chains are valid
(every track in exactly one chain, cluster lists = the segments' lists in
chain order).  A refit fails when the state reaches |sin phi| >= s_max (a
looper near its turning point); whether that happens on a chain within
rounding of the limit can differ between the two sides, so at most 0.5% of
the compared chains may succeed on one side only.
"""
import numpy as np
import pytest

from oracle import oracle
from paper_2502_09138_amd import synth
from paper_2502_09138_amd.config import default_config

import parity

pytestmark = pytest.mark.gpu
R = synth.N_ROWS


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _compare(ev, phys, label):
    from paper_2502_09138_amd.tracker import Tracker
    cfg = default_config()
    tr = Tracker(cfg, max_clusters=ev.n_clusters, max_sectors=ev.n_sectors)
    tracks, mg = tr.track_and_merge(ev.y, ev.z, ev.row_offsets, ev.sector_z_lo, ev.sector_z_hi, phys, host=True)
    tr.close()
    run = oracle.Run.from_event(cfg.as_dict(), ev).run_all()
    res = run.result()
    mo = oracle.merge(run, phys)
    # chains are a partition of the tracks; cluster lists are the segments' lists in chain order
    n = tracks.n_tracks
    assert len(mg["next"]) == n and len(mg["heads"]) == len(mg["nseg"])
    assert np.array_equal(np.sort(np.unique(mg["head_of"])), np.sort(mg["heads"]))
    for c, h in enumerate(mg["heads"]):
        ids, t = [], int(h)
        while t >= 0:
            ids.append(tracks.cluster_ids[tracks.first[t]:tracks.first[t + 1]])
            t = int(mg["next"][t])
        assert np.array_equal(np.concatenate(ids), mg["clusters"][mg["first"][c]:mg["first"][c + 1]])
    # links: GPU track index <-> oracle track index by start position
    st_o = res["starts"][res["trk_tracklet"]].astype(np.int64)
    o_of = {int(s): k for k, s in enumerate(st_o)}
    g2o = np.array([o_of.get(int(s), -1) for s in tracks.start], np.int64)
    o_links = {(a, int(b)) for a, b in enumerate(mo["next"]) if b >= 0}
    g_links = {(int(g2o[a]), int(g2o[b])) for a, b in enumerate(mg["next"]) if b >= 0}
    both = {(a, b) for a, b in o_links if a in set(g2o.tolist()) and b in set(g2o.tolist())}
    found = len(both & g_links)
    print(label, "tracks", n, "oracle links", len(o_links), "GPU links", len(g_links), "common", found, flush=True)
    assert found >= 0.995 * len(both) and found >= 0.995 * len(g_links)
    # refit parity on chains with the same clusters
    oc = {}
    for c, h in enumerate(mo["heads"]):
        oc[int(st_o[h])] = c
    n_same = bad_p = bad_c = 0
    one_sided = []
    for c, h in enumerate(mg["heads"]):
        if mg["nseg"][c] < 2:
            continue
        k = oc.get(int(tracks.start[h]))
        if k is None or mo["nseg"][k] != mg["nseg"][c]:
            continue
        if not np.array_equal(np.sort(mg["clusters"][mg["first"][c]:mg["first"][c + 1]]),
                              np.sort(mo["clusters"][mo["first"][k]:mo["first"][k + 1]])):
            continue
        n_same += 1
        if (mg["ndf"][c] < 0) != (mo["ndf"][k] < 0):
            one_sided.append((int(h), int(mg["ndf"][c]), int(mo["ndf"][k])))
            continue
        if mg["ndf"][c] < 0:
            continue
        assert mg["ndf"][c] == mo["ndf"][k]
        po = mo["param"][k]
        dp = np.abs(mg["param"][c].astype(np.float64) - po)
        bad_p += int(np.any(dp > parity.PARAM_RTOL * np.maximum(np.abs(po), parity.FLOORS)))
        do = np.diag(parity.unpack_cov(mo["cov"][k]))
        dg = np.diag(parity.unpack_cov(mg["cov"][c].astype(np.float64)))
        bad_c += int(np.any(np.abs(dg - do) > parity.COV_RTOL * np.abs(do)))
    print(label, "merged chains compared", n_same, "beyond 1e-4", bad_p, "cov beyond 1e-3", bad_c,
          "refit failed on one side only", one_sided, flush=True)
    assert n_same > 0 and bad_p == 0 and bad_c == 0
    assert len(one_sided) <= 0.005 * n_same
    return mg


def test_merge_boundary_crossers(torch_cuda):
    ev = synth.boundary_crossers(seed=7)
    print("case: boundary_crossers seed=7 N=", ev.n_clusters, flush=True)
    mg = _compare(ev, [0, 1, 2], "boundary_crossers")
    assert (mg["nseg"] > 1).sum() >= 30


def test_merge_central_event(torch_cuda):
    ev = synth.central_event(seed=2)
    print("case: central_event seed=2 N=", ev.n_clusters, flush=True)
    _compare(ev, np.arange(36), "central_event")


def test_merge_time_frame_sectors(torch_cuda):
    ev = synth.time_frame(seed=3).sector_slice(range(6))
    print("case: time_frame seed=3 sectors 0-5 N=", ev.n_clusters, flush=True)
    _compare(ev, np.arange(6), "time_frame sectors 0-5")


def test_merge_without_neighbours_changes_nothing(torch_cuda):
    from paper_2502_09138_amd.tracker import Tracker
    ev = synth.uneven_chunks(chunks=range(6))
    tr = Tracker(default_config(), max_clusters=ev.n_clusters, max_sectors=ev.n_sectors)
    tracks, mg = tr.track_and_merge(ev.y, ev.z, ev.row_offsets, ev.sector_z_lo, ev.sector_z_hi, None, host=True)
    assert np.all(mg["next"] == -1) and len(mg["heads"]) == tracks.n_tracks
    assert np.array_equal(mg["param"], tracks.param) and np.array_equal(mg["clusters"], tracks.cluster_ids)
    tr.close()


@pytest.mark.parametrize("n_tracks, windows", [(1, {}), (30, {}), (700, {}),
                                               (60, dict(merge_dtanl=10.0, merge_dqpt=100.0, merge_dz=1e4)),
                                               (300, dict(merge_dtanl=1e-4, merge_dz=0.3))])
def test_merge_candidates_over_sizes_and_windows(torch_cuda, n_tracks, windows):
    """The candidate lists (tan(lambda) bins, reachable z) against the oracle's walk over every pair: sectors of a
    few tracks, more than one wave of slots, windows wider than the bins and narrower than one.  A link may
    differ where a track or a score differs within rounding, so at most 0.5% (the file's bar), and at most one
    where there are fewer than 200 links."""
    from paper_2502_09138_amd.tracker import Tracker
    ev = synth.boundary_crossers(seed=11, n_tracks=n_tracks)
    print("case: boundary_crossers n_tracks", n_tracks, windows, "N=", ev.n_clusters, flush=True)
    cfg = default_config(**windows)
    tr = Tracker(cfg, max_clusters=max(64, ev.n_clusters), max_sectors=ev.n_sectors)
    tracks, mg = tr.track_and_merge(ev.y, ev.z, ev.row_offsets, ev.sector_z_lo, ev.sector_z_hi, [0, 1, 2], host=True)
    tr.close()
    run = oracle.Run.from_event(cfg.as_dict(), ev).run_all()
    res, mo = run.result(), oracle.merge(run, [0, 1, 2])
    st_o = res["starts"][res["trk_tracklet"]].astype(np.int64)
    start = tracks.start.astype(np.int64)
    o_links = {(int(st_o[a]), int(st_o[b])) for a, b in enumerate(mo["next"]) if b >= 0}
    g_links = {(int(start[a]), int(start[b])) for a, b in enumerate(mg["next"]) if b >= 0}
    print("links", len(o_links), len(g_links), "common", len(o_links & g_links), flush=True)
    assert len(o_links ^ g_links) <= max(1, 0.005 * len(o_links))


def _links_over_all_pairs(sector, x_ref, param, cov, phys, cfg):
    """C8 in double over every pair of the given tracks, without a candidate list: next[] (-1: none)."""
    n, p = len(sector), param.astype(np.float64)
    x, phys = x_ref.astype(np.float64), np.asarray(phys)
    cyy, czz = cov[:, 0].astype(np.float64), cov[:, 2].astype(np.float64)
    r_in = np.sqrt(x * x + p[:, 0] * p[:, 0])
    bk, smax = -0.00299792458 * cfg.bz, cfg.s_max
    succ, succ_score = np.full(n, -1), np.full(n, np.inf)
    pred, pred_score = np.full(n, -1), np.full(n, np.inf)
    for a in range(n):
        ph = int(phys[sector[a]])
        for step in (-1, 1) if ph >= 0 else ():
            where = np.flatnonzero(phys == ph // 18 * 18 + (ph % 18 + step) % 18)
            if not len(where):
                continue
            b = np.flatnonzero((sector == where[0]) & (r_in > r_in[a]))
            d = step * np.deg2rad(20.0)
            y, z, s, t, k = p[a]
            cs = np.sqrt((1 - s) * (1 + s))
            s1, c1 = s * np.cos(d) - cs * np.sin(d), cs * np.cos(d) + s * np.sin(d)
            if not (c1 > 0 and abs(s1) < smax):
                continue
            dx = x[b] - (x[a] * np.cos(d) + y * np.sin(d))
            s2 = s1 + bk * k * dx
            b, dx, s2 = (v[np.abs(s2) < smax] for v in (b, dx, s2))
            dy = dx * (s1 + s2) / (np.sqrt((1 - s1) * (1 + s1)) + np.sqrt((1 - s2) * (1 + s2)))
            L = np.sqrt(dx * dx + dy * dy)
            u = 0.5 * bk * k * L
            b, dx, s2, dy, L, u = (v[np.abs(u) < 1] for v in (b, dx, s2, dy, L, u))
            S = np.sign(dx) * L * np.where(u == 0, 1.0, np.arcsin(u) / np.where(u == 0, 1.0, u))
            dy = -x[a] * np.sin(d) + y * np.cos(d) + dy - p[b, 0]
            dz = z + t * S - p[b, 1]
            ok = ((np.abs(dy) <= cfg.merge_dy) & (np.abs(dz) <= cfg.merge_dz) & (np.abs(s2 - p[b, 2]) <= cfg.merge_dsinphi) &
                  (np.abs(t - p[b, 3]) <= cfg.merge_dtanl) & (np.abs(k - p[b, 4]) <= cfg.merge_dqpt))
            score = dy * dy / (cyy[b] + cfg.sigma_y ** 2) + dz * dz / (czz[b] + cfg.sigma_z ** 2)
            for j, sc in zip(b[ok], score[ok]):   # ascending j; a ascends, too
                if sc < succ_score[a] or (sc == succ_score[a] and j < succ[a]):
                    succ[a], succ_score[a] = j, sc
                if sc < pred_score[j]:
                    pred[j], pred_score[j] = a, sc
    return np.array([s if s >= 0 and pred[s] == a else -1 for a, s in enumerate(succ)], np.int64)


@pytest.mark.parametrize("n_tracks, windows, at_least",
                         [(1, {}, 1), (3, {}, 2), (30, {}, 10), (60, dict(merge_dtanl=10.0, merge_dqpt=100.0, merge_dz=1e4), 20),
                          (200, dict(merge_dtanl=1 / 64, merge_dqpt=0.1), 40), (300, dict(merge_dtanl=1e-3, merge_dz=0.3), 10),
                          (700, {}, 200), (1500, dict(merge_dtanl=0.3, merge_dz=20.0, merge_dsinphi=0.2, merge_dy=6.0), 300)])
def test_merge_links_are_those_of_all_pairs(torch_cuda, n_tracks, windows, at_least):
    """The links exactly, against a walk over every pair of the GPU's own tracks in double: no candidate may be lost by the
    tan(lambda) bins or the reach in z.  Chains, their cluster lists and single segments' results with them."""
    from paper_2502_09138_amd.tracker import Tracker
    ev = synth.boundary_crossers(seed=11, n_tracks=n_tracks)
    print("case: merge over all pairs", n_tracks, windows, "N=", ev.n_clusters, flush=True)
    cfg = default_config(**windows)
    tr = Tracker(cfg, max_clusters=max(64, ev.n_clusters), max_sectors=ev.n_sectors)
    tracks, mg = tr.track_and_merge(ev.y, ev.z, ev.row_offsets, ev.sector_z_lo, ev.sector_z_hi, [0, 1, 2], host=True)
    tr.close()
    ref = _links_over_all_pairs(tracks.sector, tracks.x_ref, tracks.param, tracks.cov, [0, 1, 2], cfg)
    print("tracks", tracks.n_tracks, "links", int((ref >= 0).sum()), flush=True)
    assert (ref >= 0).sum() >= at_least
    assert np.array_equal(mg["next"], ref)
    heads = np.setdiff1d(np.arange(tracks.n_tracks), ref)
    assert np.array_equal(mg["heads"], heads) and len(mg["first"]) == len(heads) + 1
    for c, h in enumerate(heads):
        chain = [int(h)]
        while ref[chain[-1]] >= 0:
            chain.append(int(ref[chain[-1]]))
        ids = np.concatenate([tracks.cluster_ids[tracks.first[t]:tracks.first[t + 1]] for t in chain])
        assert np.array_equal(mg["clusters"][mg["first"][c]:mg["first"][c + 1]], ids)
        assert mg["nseg"][c] == len(chain) and np.all(mg["head_of"][chain] == h)
        assert mg["ndf"][c] in ((2 * len(ids) - 5,) if len(chain) == 1 else (2 * len(ids) - 5, -1))
        if len(chain) == 1 or mg["ndf"][c] == -1:
            assert np.array_equal(mg["param"][c], tracks.param[h]) and np.array_equal(mg["cov"][c], tracks.cov[h])
            assert mg["chi2"][c] == tracks.chi2[h]


def test_merge_of_a_frame_without_tracks(torch_cuda):
    """Nothing to link: empty arrays, also after a frame with chains on the same tracker."""
    from paper_2502_09138_amd.tracker import Tracker
    ev = synth.boundary_crossers(seed=11, n_tracks=30)
    few = synth.boundary_crossers(seed=12, n_tracks=1)
    print("case: merge without tracks N=", ev.n_clusters, flush=True)
    tr = Tracker(default_config(), max_clusters=ev.n_clusters, max_sectors=3)
    for e, some in ((ev, True), (few.sector_slice(range(3)), True), (ev, True)):
        _, mg = tr.track_and_merge(e.y, e.z, e.row_offsets, e.sector_z_lo, e.sector_z_hi, [0, 1, 2], host=True)
        assert (len(mg["heads"]) > 0) == some
        # a few clusters of one row: no tracks
        n = 5
        off = np.zeros(3 * R + 1, np.uint32)
        off[40:] = n
        tracks, mg = tr.track_and_merge(e.y[:n], e.z[:n], off, e.sector_z_lo, e.sector_z_hi, [0, 1, 2], host=True)
        assert tracks.n_tracks == 0 and mg["first"].tolist() == [0]
        assert all(len(v) == 0 for k, v in mg.items() if k != "first")
    tr.close()
