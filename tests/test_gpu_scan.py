"""Prefix sums by one workgroup and by three launches: frames of equal sectors on both sides of the two limits (rows of a
frame, tracklet capacity) and of a workgroup's tile.  Every sector has to repeat what it gives alone."""
import numpy as np
import pytest

from paper_2502_09138_amd import synth
from paper_2502_09138_amd.config import default_config

pytestmark = pytest.mark.gpu
R = synth.N_ROWS


@pytest.mark.parametrize("sectors, max_tracklets", [(1, 4000), (26, 65536), (27, 65537), (107, 65536), (108, 65536),
                                                    (108, 65537)])
def test_equal_sectors_repeat(sectors, max_tracklets):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_09138_amd.tracker import Tracker
    ev = synth.single_sector(seed=9, n_tracks=20)
    n, S = ev.n_clusters, sectors
    one = Tracker(default_config(), max_clusters=n, max_sectors=1).track_event(ev, host=True)
    assert one.n_tracks > 5
    offs = np.concatenate([[0]] + [ev.row_offsets[1:].astype(np.int64) + k * n for k in range(S)]).astype(np.uint32)
    print("case: scans", S, "rows", S * R, "tracklets", S * one.n_tracklets, "capacity", max_tracklets, flush=True)
    tr = Tracker(default_config(), max_clusters=S * n, max_sectors=S, max_tracklets=max_tracklets)
    for host in (True, False, True):
        y, z = np.tile(ev.y, S), np.tile(ev.z, S)
        if not host:
            y, z = torch.from_numpy(y).to("cuda:0"), torch.from_numpy(z).to("cuda:0")
        got = tr.track(y, z, offs, np.tile(ev.sector_z_lo, S), np.tile(ev.sector_z_hi, S), host=host)
        assert (got.n_tracks, got.n_tracklets, got.error_flags) == (S * one.n_tracks, S * one.n_tracklets, 0)
        nc = len(one.cluster_ids)
        want = {"sector": np.repeat(np.arange(S), one.n_tracks),
                "start": np.concatenate([one.start.astype(np.int64) + k * n for k in range(S)]),
                "first": np.concatenate([[0]] + [one.first[1:].astype(np.int64) + k * nc for k in range(S)]),
                "cluster_ids": np.concatenate([one.cluster_ids.astype(np.int64) + k * n for k in range(S)])}
        for f in ("x_ref", "param", "cov", "chi2", "ndf"):
            v = getattr(one, f)
            want[f] = np.tile(v, (S,) + (1,) * (v.ndim - 1))
        for f, v in want.items():
            np.testing.assert_array_equal(getattr(got, f), v, err_msg=f)
    tr.close()
