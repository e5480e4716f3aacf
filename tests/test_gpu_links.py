"""C2 links over the sizes where the neighbour finder takes another path, bit-exact against the oracle: candidate lists
that overflow (in rows that always fit the stage, and in larger ones that go to the large stage), runs larger than
either stage, rows of a few hits and rows of a whole number of tiles.  Coordinates on a coarse lattice add many ties."""
import types

import numpy as np
import pytest

from oracle import oracle
from paper_2502_09138_amd import synth
from paper_2502_09138_amd.config import default_config

import parity

pytestmark = pytest.mark.gpu
R = synth.N_ROWS


def _event(n, y_cm, z_cm, lattice, seed):
    """n hits in each of the rows 60..64, in a patch of y_cm by z_cm."""
    rng = np.random.default_rng(seed)
    rows = range(60, 65)
    y = rng.uniform(-0.5 * y_cm, 0.5 * y_cm, 5 * n)
    z = rng.uniform(120.0, 120.0 + z_cm, 5 * n)
    if lattice:
        y, z = np.rint(y / lattice) * lattice, np.rint(z / lattice) * lattice
    counts = np.zeros(R, np.int64)
    counts[list(rows)] = n
    return types.SimpleNamespace(y=y.astype(np.float32), z=z.astype(np.float32), n_clusters=5 * n, n_sectors=1,
                                 row_offsets=np.concatenate([[0], np.cumsum(counts)]).astype(np.uint32),
                                 sector_z_lo=np.zeros(1, np.float32), sector_z_hi=np.full(1, 250.0, np.float32))


@pytest.mark.parametrize("slots", [4, 8])
@pytest.mark.parametrize("n, y_cm, z_cm, lattice", [(1, 1, 1, 0), (64, 20, 100, 0), (40, 6, 6, 0.25), (65, 3, 3, 0.5),
                                                    (256, 20, 60, 0), (257, 20, 60, 0.5), (300, 9, 12, 0), (700, 25, 40, 0),
                                                    (1300, 20, 12, 0)])
def test_links_match_the_oracle(n, y_cm, z_cm, lattice, slots):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_09138_amd.tracker import Tracker
    ev = _event(n, y_cm, z_cm, lattice, seed=n + slots)
    print("case: links", n, y_cm, z_cm, lattice, slots, flush=True)
    cfg = default_config()
    # lattices make chains fork at every hit: room for a tracklet per hit
    tr = Tracker(cfg, max_clusters=ev.n_clusters, max_sectors=1, max_tracklets=ev.n_clusters)
    tr.set_knobs(link_slots=slots)
    g = parity.gpu_run(tr, ev, tracklets=False)
    tr.close()
    run = oracle.Run.from_event(cfg.as_dict(), ev).run_all()
    o = run.result()
    o["_row_offsets"] = ev.row_offsets
    if n > 1:
        assert (o["up0"] >= 0).any()
    parity.compare_c1_c4(g, o, R)


@pytest.mark.parametrize("slots", [4, 8])
@pytest.mark.parametrize("n, y_cm, z_cm, lattice, overrides",
                         [(256, 6, 6, 0, {}), (250, 5, 5, 0.25, {}), (256, 60, 200, 0, dict(grid_hits_per_bin=1)),
                          (255, 30, 30, 0, dict(grid_hits_per_bin=1)), (33, 1, 1, 0, {}), (700, 7, 7, 0, {}), (1500, 12, 12, 0, {}),
                          (900, 60, 200, 0, dict(grid_hits_per_bin=1)), (200, 30, 60, 0, dict(win_b_y=6.0, win_b_z=9.0)),
                          (1000, 30, 60, 0.5, dict(win_b_y=3.0, win_b_z=4.0))])
def test_crowded_windows_match_the_oracle(n, y_cm, z_cm, lattice, overrides, slots):
    """Windows of more hits than any list holds (so each list is filled several times), in runs that fit the small stage, the
    large one and neither; rows of few hits with more bins than the small stage."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_09138_amd.tracker import Tracker
    ev = _event(n, y_cm, z_cm, lattice, seed=n + slots)
    print("case: crowded windows", n, y_cm, z_cm, lattice, overrides, slots, flush=True)
    cfg = default_config(**overrides)
    tr = Tracker(cfg, max_clusters=ev.n_clusters, max_sectors=1, max_tracklets=ev.n_clusters)
    tr.set_knobs(link_slots=slots)
    g = parity.gpu_run(tr, ev, tracklets=False)
    tr.close()
    o = oracle.Run.from_event(cfg.as_dict(), ev).run_all().result()
    o["_row_offsets"] = ev.row_offsets
    assert (o["up0"] >= 0).any()
    parity.compare_c1_c4(g, o, R)


@pytest.mark.parametrize("n, sectors, most", [(256, 4, 50.0), (600, 2, 150.0)])
def test_crowded_windows_are_not_searched_pair_by_pair_in_memory(n, sectors, most):
    """K2 on rows whose hits lie in one patch (windows of a dozen to 60 hits: lists that overflow, runs larger than the large
    stage) against the same number of hits spread over the sector.  Walking the upper window in global memory for every
    lower hit made it 418 times as long in rows of 256 hits, and 1222 times in rows of 600; a list at a time 17 and 58."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_09138_amd.tracker import Tracker
    N = sectors * R * n
    rng = np.random.default_rng(n)
    off = np.arange(0, N + 1, n, dtype=np.uint32)
    lo, hi = np.zeros(sectors, np.float32), np.full(sectors, 250.0, np.float32)
    us = []
    for y_cm, z_cm in ((20.0, 25.0), (60.0, 230.0)):
        print("case: crowded windows, time", n, sectors, y_cm, z_cm, flush=True)
        y = torch.from_numpy(rng.uniform(-0.5 * y_cm, 0.5 * y_cm, N).astype(np.float32)).cuda()
        z = torch.from_numpy(rng.uniform(10.0, 10.0 + z_cm, N).astype(np.float32)).cuda()
        tr = Tracker(default_config(), max_clusters=N, max_sectors=sectors, max_tracklets=N)
        tr.set_timing(passes=("neighbours",))
        t = []
        for _ in range(9):
            rid = tr.submit(y, z, off, lo, hi)
            tr.get_device(rid)
            t.append(1e3 * tr.pass_times()["neighbours"])
            tr.release(rid)
        tr.close()
        us.append(float(np.median(t)))
    print("K2 us: crowded %.0f, spread %.0f, ratio %.1f" % (us[0], us[1], us[0] / us[1]), flush=True)
    assert us[0] <= most * us[1]
