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
