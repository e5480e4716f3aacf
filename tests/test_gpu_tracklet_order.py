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
