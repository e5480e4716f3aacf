"""The starting order of the lane-per-tracklet waves changes no result: bucket-ordered refits (ordered waves)
against tracklet-ordered ones (plain order) and the row-synchronous kernel, bit for bit, from a frame of less than
one wave to several waves per XCD with sectors that end inside a wave."""
import numpy as np
import pytest

from paper_2502_09138_amd import synth
from paper_2502_09138_amd.config import default_config

pytestmark = pytest.mark.gpu
FIELDS = ("sector", "start", "first", "cluster_ids", "x_ref", "param", "cov", "chi2", "ndf")


@pytest.mark.parametrize("kind, size", [("sector", 3), ("sector", 10), ("sector", 90), ("chunks", 7), ("frame", 1)])
def test_wave_order_changes_nothing(kind, size):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_09138_amd.tracker import Tracker
    ev = {"sector": lambda: synth.single_sector(seed=size, n_tracks=size),
          "chunks": lambda: synth.uneven_chunks(chunks=range(size), n_max=20000),
          "frame": lambda: synth.time_frame(seed=61, n_orbits=size)}[kind]()
    print("case: wave order", kind, size, "N=", ev.n_clusters, flush=True)
    tr = Tracker(default_config(), max_clusters=ev.n_clusters, max_sectors=ev.n_sectors)
    got = []
    for knobs in (dict(schedule=1, refit_order=0), dict(schedule=1, refit_order=1), dict(schedule=2, refit_order=0)):
        tr.set_knobs(**knobs)
        got.append(tr.track_event(ev, host=True))
    tr.close()
    assert got[0].n_tracks > 0
    for other in got[1:]:
        assert other.n_tracklets == got[0].n_tracklets
        for k in FIELDS:
            np.testing.assert_array_equal(getattr(got[0], k), getattr(other, k), err_msg=k)


@pytest.mark.parametrize("kind, size", [("event", (1, 2)), ("event", (1, 45)), ("event", (2, 100)), ("event", (36, 12)),
                                        ("event", (36, 80)), ("chunks", 90), ("pp", 4)])
def test_resident_sectors_change_nothing(kind, size):
    """Frames whose sectors are swept resident in LDS (from two tracks, 16 lanes a tracklet, to sectors of about 13k
    hits, two lanes and no room for the links; chunks of very uneven sizes) against the lane-per-tracklet pipeline, bit
    for bit, row -> hit columns included."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_09138_amd import tracker as T
    if kind == "event":
        ev = synth.single_sector(seed=3, n_tracks=size[1]) if size[0] == 1 else \
            synth.central_event(seed=4, n_primaries=size[1] * 36, sectors=range(size[0]))
    else:
        ev = synth.uneven_chunks(chunks=range(size), n_max=6000) if kind == "chunks" else \
            synth.pp_time_frame(seed=54, n_orbits=size)
    print("case: resident sectors", kind, size, "N=", ev.n_clusters, "largest sector",
          int(np.diff(ev.row_offsets[::synth.N_ROWS].astype(np.int64)).max()), flush=True)
    tr = T.Tracker(default_config(), max_clusters=ev.n_clusters, max_sectors=ev.n_sectors)
    got = []
    for schedule in (2, 1):
        tr.set_knobs(schedule=schedule)
        out = tr.track_event(ev, host=True)
        info = tr.debug(T.TPC_DBG_TK_INFO, np.int32).reshape(4, -1)[:, :out.n_tracklets]
        col = tr.debug(T.TPC_DBG_TK_ROWHIT, np.int32).reshape(synth.N_ROWS, -1)[:, :out.n_tracklets]
        row = np.arange(synth.N_ROWS)[:, None]
        held = (info[0] > 0) & (row >= info[1]) & (row <= info[2])
        got.append((out, info[0], np.where(info[0] > 0, info, 0), np.where(held, col, -2)))
    tr.close()
    assert got[0][0].n_tracklets == got[1][0].n_tracklets > 0
    for k in FIELDS:
        np.testing.assert_array_equal(getattr(got[0][0], k), getattr(got[1][0], k), err_msg=k)
    for a, b in zip(got[0][1:], got[1][1:]):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("overrides", [dict(), dict(gate_nsigma=40.0, win_cap=4.0), dict(gate_nsigma=40.0, win_cap=15.0),
                                       dict(gate_nsigma=12.0, grid_hits_per_bin=1), dict(win_cap=0.02)])
def test_wave_search_changes_nothing(overrides):
    """Searches shared by the lanes of a wave (the lane-per-tracklet pipeline) against searches by the lanes of one
    tracklet (row-synchronous): windows of no candidate, of one item, of several rounds of items, of two runs of bins and
    of more.  The order of equal deviations is the same, so every result is, bit for bit."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_09138_amd.tracker import Tracker
    ev = synth.single_sector(seed=21, n_tracks=500)
    print("case: wave search", overrides, "N=", ev.n_clusters, flush=True)
    tr = Tracker(default_config(**overrides), max_clusters=ev.n_clusters, max_sectors=1)
    got = []
    for schedule in (2, 1):
        tr.set_knobs(schedule=schedule)
        got.append(tr.track_event(ev, host=True))
    tr.close()
    assert got[0].n_tracklets == got[1].n_tracklets > 0
    for k in FIELDS:
        np.testing.assert_array_equal(getattr(got[0], k), getattr(got[1], k), err_msg=k)


@pytest.mark.parametrize("sectors, primaries, n_min, n_max, staged",
                         [(1, 220, 20000, 1 << 17, True), (1, 700, 20000, 1 << 17, False), (5, 240, 1 << 17, 1 << 18, True),
                          (2, 700, 1 << 17, 1 << 18, False), (10, 240, 1 << 18, 1 << 20, True),
                          (3, 900, 1 << 18, 1 << 20, False), (36, 330, 3 << 19, 3 << 20, False),
                          (8, 1600, 3 << 19, 3 << 20, False)])
def test_row_by_row_lanes_change_nothing(sectors, primaries, n_min, n_max, staged):
    """Row-by-row sweeps with 8, 4, 2 lanes and one lane a tracklet, rows staged or too large for it, and the
    schedule left to the device (few enough tracklets, and too many), against the lane-per-tracklet pipeline, bit for bit."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_09138_amd.tracker import Tracker
    ev = synth.central_event(seed=8, n_primaries=primaries * 36, sectors=range(sectors))
    widest = int(np.diff(ev.row_offsets.astype(np.int64)).max())
    print("case: row by row", sectors, primaries, "N=", ev.n_clusters, "widest row", widest, flush=True)
    assert n_min < ev.n_clusters <= n_max and (widest <= 320) == staged
    tr = Tracker(default_config(), max_clusters=ev.n_clusters, max_sectors=ev.n_sectors)
    got = []
    for schedule in (0, 1):
        tr.set_knobs(schedule=schedule)
        got.append(tr.track_event(ev, host=True))
    tr.close()
    assert got[0].n_tracklets == got[1].n_tracklets > 0
    for k in FIELDS:
        np.testing.assert_array_equal(getattr(got[0], k), getattr(got[1], k), err_msg=k)


@pytest.mark.parametrize("kind, size, lanes", [("one", 30, 16), ("one", 100, 16), ("pp", 1, 8), ("pp", 2, 4), ("pp", 4, 2),
                                               ("short", 600, 2)])
def test_resident_columns_read_by_other_lanes(kind, size, lanes):
    """The row -> hit column of a resident tracklet is written by one of its lanes and read by all of them, through every
    number of lanes, and taken over by the next tracklet of the same lanes (short: one sector of 360 chains of three
    hits, more than its two workgroups hold at once): the columns and results of the lane-per-tracklet pipeline, bit for
    bit."""
    import types

    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_09138_amd import tracker as T
    cfg = default_config()
    if kind == "pp":
        ev = synth.pp_time_frame(seed=54, n_orbits=size)
    elif kind == "one":
        ev = synth.single_sector(seed=3, n_tracks=size)
    else:
        cfg = default_config(min_tracklet_hits=3, min_track_hits=3)
        R, S, at = synth.N_ROWS, size, size - 1
        y = np.array([[y + 5.0 * (r // 5 % 2) - 2.5 for y in (-8.0, 0.0, 8.0) for z in range(4)] for r in range(R)])
        z = np.array([[20.0 + 20.0 * z + 0.01 * r for y in range(3) for z in range(4)] for r in range(R)])
        off = np.zeros(S * R + 1, np.uint32)
        off[at * R:(at + 1) * R + 1] = np.arange(0, y.size + 1, 12)
        ev = types.SimpleNamespace(y=y.astype(np.float32).ravel(), z=z.astype(np.float32).ravel(), row_offsets=off,
                                   n_clusters=y.size, n_sectors=S, sector_z_lo=np.zeros(S, np.float32),
                                   sector_z_hi=np.full(S, 250.0, np.float32))
    print("case: resident columns", kind, size, "N=", ev.n_clusters, flush=True)
    tr = T.Tracker(cfg, max_clusters=ev.n_clusters, max_sectors=ev.n_sectors, max_tracklets=ev.n_clusters)
    got = []
    for schedule in (2, 1):
        tr.set_knobs(schedule=schedule)
        out = tr.track_event(ev, host=True)
        info = tr.debug(T.TPC_DBG_TK_INFO, np.int32).reshape(4, -1)[:, :out.n_tracklets]
        col = tr.debug(T.TPC_DBG_TK_ROWHIT, np.int32).reshape(synth.N_ROWS, -1)[:, :out.n_tracklets]
        row = np.arange(synth.N_ROWS)[:, None]
        held = (info[0] > 0) & (row >= info[1]) & (row <= info[2])
        got.append((out, np.where(info[0] > 0, info, 0), np.where(held, col, -2)))
    tr.close()
    n, parts = got[0][0].n_tracklets, (768 + ev.n_sectors - 1) // ev.n_sectors
    if kind == "short":
        assert n > 128 * parts
    else:
        assert next(v for v in (16, 8, 4, 2) if v == 2 or n * v <= 49152) == lanes
    assert got[1][0].n_tracklets == n and got[0][0].n_tracks > 0
    for k in FIELDS:
        np.testing.assert_array_equal(getattr(got[0][0], k), getattr(got[1][0], k), err_msg=k)
    for a, b in zip(got[0][1:], got[1][1:]):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("sectors, per_row", [(4, 330), (6, 340), (30, 340)])
def test_sparse_frames_are_not_swept_row_by_row(sectors, per_row):
    """Hits without particles in rows too large to stage: a few short tracklets, far apart.  The automatic schedule gives the
    results of both others, bit for bit, and its tracklet pass takes at most 1.6 times that of the faster one (it took 2.5
    to 3 times while such frames were swept row by row)."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_09138_amd.tracker import Tracker
    R, N = synth.N_ROWS, sectors * synth.N_ROWS * per_row
    rng = np.random.default_rng(sectors)
    half_y = synth.row_geometry()[1]
    y = torch.from_numpy((rng.uniform(-1, 1, (sectors, R, per_row)) * half_y[None, :, None]).astype(np.float32).ravel()).cuda()
    z = torch.from_numpy(rng.uniform(0, 250, N).astype(np.float32)).cuda()
    frame = (y, z, np.arange(0, N + 1, per_row, dtype=np.uint32), np.zeros(sectors, np.float32),
             np.full(sectors, 250.0, np.float32))
    print("case: sparse frame", sectors, per_row, "N=", N, flush=True)
    tr = Tracker(default_config(min_tracklet_hits=4, min_track_hits=4), max_clusters=N, max_sectors=sectors)
    got, us = [], []
    for schedule in (0, 1, 2):
        tr.set_knobs(schedule=schedule)
        tr.set_timing(passes=("tracklets",))
        t = []
        for _ in range(9):
            rid = tr.submit(*frame)
            tr.get_device(rid)
            t.append(1e3 * tr.pass_times()["tracklets"])
            tr.release(rid)
        us.append(float(np.median(t)))
        got.append(tr.track(*frame))
    tr.close()
    print("tracklets", got[0].n_tracklets, "tracks", got[0].n_tracks, "us: automatic %.0f, pipeline %.0f, rows %.0f" % tuple(us),
          flush=True)
    assert got[0].n_tracks > 0
    for other in got[1:]:
        assert other.n_tracklets == got[0].n_tracklets
        for k in FIELDS:
            np.testing.assert_array_equal(getattr(got[0], k), getattr(other, k), err_msg=k)
    assert us[0] <= 1.6 * min(us[1:])


def _k5_us(tr, ev, schedule):
    """Median time of the tracklet pass under a schedule, us."""
    import torch
    y, z = torch.from_numpy(ev.y).cuda(), torch.from_numpy(ev.z).cuda()
    tr.set_knobs(schedule=schedule)
    tr.set_timing(passes=("tracklets",))
    t = []
    for _ in range(11):
        rid = tr.submit(y, z, ev.row_offsets, ev.sector_z_lo, ev.sector_z_hi)
        tr.get_device(rid)
        t.append(1e3 * tr.pass_times()["tracklets"])
        tr.release(rid)
    return float(np.median(t))


@pytest.mark.parametrize("size, sectors, others", [(100, 100, 0), (100, 400, 0), (30, 700, 0), (100, 200, 4)])
def test_a_full_sector_among_small_ones_is_swept_at_once(size, sectors, others):
    """One full sector, the others empty or of a few tracks: its tracklets run side by side, so the tracklet pass takes at
    most 1.25 times the pipeline's (1.4 to 1.9 times when the lanes of a tracklet were chosen by the whole frame's
    tracklets, and a full sector's were swept in several rounds)."""
    import types

    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_09138_amd.tracker import Tracker
    full, few = synth.single_sector(seed=3, n_tracks=size), synth.single_sector(seed=3, n_tracks=max(1, others))
    counts, y, z = np.zeros((sectors, synth.N_ROWS), np.int64), [], []
    for s in range(sectors):
        e = full if s == sectors // 2 else few if others else None
        if e is not None:
            counts[s] = np.diff(e.row_offsets.astype(np.int64))
            y.append(e.y)
            z.append(e.z)
    ev = types.SimpleNamespace(y=np.concatenate(y), z=np.concatenate(z), n_sectors=sectors,
                               row_offsets=np.concatenate([[0], np.cumsum(counts)]).astype(np.uint32),
                               sector_z_lo=np.full(sectors, full.sector_z_lo[0], np.float32),
                               sector_z_hi=np.full(sectors, full.sector_z_hi[0], np.float32))
    ev.n_clusters = len(ev.y)
    print("case: full sector", size, sectors, others, "N=", ev.n_clusters, flush=True)
    tr = Tracker(default_config(), max_clusters=ev.n_clusters, max_sectors=sectors)
    got = []
    for schedule in (0, 1):
        tr.set_knobs(schedule=schedule)
        got.append(tr.track_event(ev, host=True))
    us = [_k5_us(tr, ev, s) for s in (0, 1)]
    tr.close()
    print("tracklets", got[0].n_tracklets, "us: automatic %.0f, pipeline %.0f" % tuple(us), flush=True)
    for k in FIELDS:
        np.testing.assert_array_equal(getattr(got[0], k), getattr(got[1], k), err_msg=k)
    assert us[0] <= 1.25 * us[1]


def test_wide_windows_are_not_searched_twice():
    """The pipeline with windows of more than two runs of bins in many lanes: its tracklet pass takes at most 2.2 times that
    of the row-by-row schedule, what it took lane by lane (2.35 while a wave searched such windows alone and then the
    others together)."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_09138_amd.tracker import Tracker
    ev = synth.central_event(seed=2)
    print("case: wide windows, time N=", ev.n_clusters, flush=True)
    tr = Tracker(default_config(gate_nsigma=40.0, win_cap=15.0), max_clusters=ev.n_clusters, max_sectors=ev.n_sectors)
    us = [_k5_us(tr, ev, s) for s in (1, 2)]
    tr.close()
    print("us: pipeline %.0f, row by row %.0f, ratio %.2f" % (us[0], us[1], us[0] / us[1]), flush=True)
    assert us[0] <= 2.2 * us[1]
