"""Performance cases: track finding, sector merging and the track-model codec, over the range of their sizes.

Every case goes through the Python binding (``paper_2502_09138_amd.tracker.Tracker``) as a user's
program does.  The clusters are made on the GPU from a seed with the detector model of
``paper_2502_09138_amd.synth`` (the same geometry, helices, resolution, efficiency and noise): events,
continuous-readout time frames and independent chunks, from one small chunk to the 512-chunk request.

Fields of a case:

``call``      "device"  submit, wait, device views of the outputs, release (tracks stay in HBM)
              "host"    the same through the pinned host copy of every output array, as the server
                        reads it, and from there into the program's own arrays
              "numpy"   numpy clusters in, numpy tracks out (``Tracker.track(..., host=True)``)
              "merge"   sector merger and chain refit on a tracked frame
              "encode"  track-model encoding of a tracked frame
              "decode"  track-model decoding of a stream
``kind``      "event" (physical z), "frame" (continuous readout, drift coordinate), "chunks"
              (independent sector-sized chunks, log-uniform occupancy)
``sectors``   sectors of an event or frame, chunks of a "chunks" request
``tracks``    generated particles (events and frames); chunks follow from their occupancies
``orbits``    length of a time frame in LHC orbits
``rate_khz``  its collision rate
``lo``, ``hi``  occupancy range of the chunks, clusters

How many tracks a frame has is known only once it is tracked, so the outputs are kept in arrays of a
fixed capacity, zero beyond the tracks: the workspace's own output arrays for "device", arrays of the
program elsewhere.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2502_09138_amd import synth
from paper_2502_09138_amd.config import default_config
from paper_2502_09138_amd.tracker import Tracker

R = synth.N_ROWS
DEV = "cuda"
PER_TRACK = 140.0          # clusters per generated particle (all sectors), noise included
TRACKS_OUT = 1.77          # tracks found per generated particle
Q_Y, Q_Z = 0.01, 0.015     # codec quanta: a tenth of the cluster resolution

# the tuned setting of the 32-orbit frame's shape class, as the benchmark runs it
TUNED = {"schedule": 1, "select_tile_rows": 4, "refit_order": 0, "link_slots": 4, "link_group": -1,
         "select_threads": 1024}


def _event(name, call, sectors, tracks):
    return {"name": name, "call": call, "kind": "event", "sectors": sectors, "tracks": tracks}


def _frame(name, call, orbits, rate_khz, tracks, **more):
    return {"name": name, "call": call, "kind": "frame", "sectors": 36, "tracks": tracks, "orbits": orbits,
            "rate_khz": rate_khz, **more}


def _chunks(name, call, chunks, lo, hi):
    return {"name": name, "call": call, "kind": "chunks", "sectors": chunks, "lo": lo, "hi": hi}


def listed():
    return [
        # one small chunk from host arrays, as a script or a test tracks it: latency and launches only
        _event("chunk_5k_numpy", "numpy", 1, 37),
        # one ordinary sector (the plain per-sector path issues 36 of these per frame)
        _event("sector_27k", "host", 1, 200),
        # the smallest and the largest pp frames that the serving trace asks for, tracks to the host
        _frame("pp_1_orbit", "host", 1, 650.0, 694),
        _frame("pp_4_orbits", "host", 4, 650.0, 2775),
        # one central heavy-ion event, tracks left on the device (as the next step on the GPU reads them)
        _event("central_event", "device", 36, 8800),
        # a medium heavy-ion frame of the serving trace
        _frame("heavy_ion_8_orbits", "device", 8, 50.0, 17750),
        # the benchmark's frame with its tuned knobs, tracks left on the device
        _frame("time_frame", "device", 32, 50.0, 71000, **TUNED),
        # 512 chunks of uneven occupancy in one request: the largest call
        _chunks("uneven_chunks", "device", 512, 1000, 200000),
        # one dense chunk alone: rows too large to be staged, too few tracklets to fill the card
        _event("dense_sector", "device", 1, 1600),
        # merger and refit, codec: the steps after tracking, on heavy-ion frames
        _frame("merge_8_orbits", "merge", 8, 50.0, 17750),
        _frame("encode_time_frame", "encode", 32, 50.0, 71000),
        {"name": "decode_time_frame", "call": "decode", "tracks": 126001},
    ]


def draw(rng):
    """One more case: the calls above over the whole range of sizes, odd ones among them."""
    def log(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    call = rng.choice(["numpy", "host", "host", "device", "device", "device", "merge", "encode", "decode"])
    if call == "decode":
        return {"call": call, "tracks": log(40, 126000)}
    if call == "numpy":
        case = _event("", call, rng.randint(1, 3), log(20, 600))
    elif (kind := rng.choice(["event", "frame", "frame", "chunks"])) == "event":
        sectors = rng.choice([1, 2, 3, 7, 18, 36])
        case = _event("", call, sectors, log(20 * sectors, 1600 * sectors))
    elif kind == "frame":
        orbits = rng.randint(1, 32)
        if rng.random() < 0.4:
            case = _frame("", call, orbits, 650.0, int(690 * orbits * rng.uniform(0.8, 1.2)))
        else:
            case = _frame("", call, orbits, 50.0, int(2200 * orbits * rng.uniform(0.5, 1.0)))
    else:
        case = _chunks("", call, log(3, 400), 1000, rng.choice([20000, 60000, 200000]))
    del case["name"]
    return case


def _clusters_of(case):
    if case["kind"] == "chunks":
        lo, hi = case["lo"], case["hi"]
        return case["sectors"] * (hi - lo) / math.log(hi / lo)
    return case["tracks"] * PER_TRACK


def _caps(case):
    """Capacities of a frame's clusters and tracks."""
    n = int(1.25 * _clusters_of(case)) + 4000
    return n, n // 40


def work(case):
    """Bytes of one pass: clusters in, tracks out.  Operations: per track cluster one Kalman step (state
    and covariance transport and update) outward and one inward, per cluster one neighbour search."""
    if case["call"] == "decode":
        nc = case["tracks"] * 74.0
        return {"bytes": case["tracks"] * 32.0 + nc * (5 + 9) + 0.067 * nc * 18, "flops": nc * 12.0}
    n = _clusters_of(case)
    nt, nc = n / PER_TRACK * TRACKS_OUT, 0.937 * n
    if case["call"] == "encode":
        return {"bytes": nc * (4 + 8 + 1 + 4 + 8) + (n - nc) * 17 + nt * (28 + 32), "flops": nc * 14.0}
    if case["call"] == "merge":
        return {"bytes": nt * 2 * 104.0 + nc * 8, "flops": 0.3 * nc * 400.0}
    return {"bytes": n * 8.0 + nt * 104.0 + nc * 4.0, "flops": nc * 800.0 + n * 60.0}


# ---------------------------------------------------------------------------
# Clusters
# ---------------------------------------------------------------------------
class _Rng:
    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(int(seed))

    def uniform(self, n, a=0.0, b=1.0):
        return a + (b - a) * torch.rand(n, generator=self.g, device=DEV, dtype=torch.float64)

    def normal(self, n, sigma):
        return sigma * torch.randn(n, generator=self.g, device=DEV, dtype=torch.float64)


def _geometry():
    x, half = synth.row_geometry()
    return torch.from_numpy(x).to(DEV), torch.from_numpy(half).to(DEV)


def _cross(p, kap, alpha, x):
    """First outward crossing of the row planes x within the first half-turn: (ok, y, z), [pairs, rows]."""
    ca, sa = torch.cos(alpha)[:, None], torch.sin(alpha)[:, None]
    vx, vy = p["vx"][:, None], p["vy"][:, None]
    kap = kap[:, None]
    x0, y0 = vx * ca + vy * sa, -vx * sa + vy * ca
    psi0 = p["phi"][:, None] - alpha[:, None]
    v = torch.sin(psi0) + kap * (x[None, :] - x0)
    psi = torch.asin(v.clamp(-1.0, 1.0))
    d = torch.where(kap > 0, torch.remainder(psi - psi0, 2 * math.pi), -torch.remainder(psi0 - psi, 2 * math.pi))
    s = d / kap
    y = y0 + 2.0 * torch.sin(0.5 * (psi + psi0)) * (torch.sin(0.5 * d) / kap)
    z = p["tanl"][:, None] * s
    return (v.abs() < 1.0) & (d.abs() <= math.pi) & (s >= 0.0) & (z.abs() < synth.TPC_HALF_LENGTH), y, z


def _kappa(p):
    return -synth.C_LIGHT_B * synth.BZ_TESLA * p["q"] / p["pt"]


def _particles(g, n, eta_lo, eta_hi):
    """Primaries of pT = 0.1 + Exp(0.5) GeV; every eleventh comes from a displaced vertex (r < 50 cm)."""
    eta = g.uniform(n, eta_lo, eta_hi)
    r = torch.where(torch.arange(n, device=DEV) % 11 == 10, 50.0 * torch.sqrt(g.uniform(n)), g.uniform(n) * 0.0)
    a = g.uniform(n, 0.0, 2 * math.pi)
    return dict(pt=0.1 - 0.5 * torch.log1p(-g.uniform(n)), tanl=torch.sinh(eta), phi=g.uniform(n, 0.0, 2 * math.pi),
                q=torch.where(g.uniform(n) < 0.5, -1.0, 1.0).double(), vx=r * torch.cos(a), vy=r * torch.sin(a))


def _pairs(p, sectors):
    """(particle, sector) pairs of the sectors that a particle's arc enters, sector = 0..17 A side, 18..35 C."""
    kap = _kappa(p)[:, None]
    s = torch.minimum(math.pi / kap.abs(), torch.full_like(kap, 530.0)) * torch.linspace(0, 1, 64, device=DEV)[None, :]
    ang = p["phi"][:, None] + kap * s
    x = p["vx"][:, None] + (torch.sin(ang) - torch.sin(p["phi"])[:, None]) / kap
    y = p["vy"][:, None] - (torch.cos(ang) - torch.cos(p["phi"])[:, None]) / kap
    r = torch.hypot(x, y)
    sec = torch.floor(torch.remainder(torch.atan2(y, x), 2 * math.pi) / (math.pi / 9)).long() % 18
    mask = torch.zeros(len(kap), 19, dtype=torch.bool, device=DEV)
    mask.scatter_(1, torch.where((r > 75.0) & (r < 252.0), sec, 18), True)
    i, sec = torch.nonzero(mask[:, :18], as_tuple=True)
    sec = sec + 18 * (p["tanl"][i] < 0).long()
    keep = sec < sectors
    return i[keep], sec[keep]


def _clusters(case, seed):
    """A frame as a user holds it: y, z on the device, row offsets and sector z ranges on the host."""
    g = _Rng(seed)
    rows, half = _geometry()
    S, kind = case["sectors"], case["kind"]
    shift = None
    if kind == "chunks" or S == 1:
        # sector-0 frame: particles aimed into the sector at r = 160 cm
        if kind == "chunks":
            u = (torch.randperm(S, generator=g.g, device=DEV).double() + g.uniform(S)) / S
            want = case["lo"] * torch.exp(u * math.log(case["hi"] / case["lo"]))
            per = (want / 115.0).round().clamp(min=3).long()
        else:
            per = torch.full((1,), case["tracks"], device=DEV).long()
        sec = torch.repeat_interleave(torch.arange(S, device=DEV), per)
        p = _particles(g, len(sec), 0.0, 0.9)
        theta = g.uniform(len(sec), 0.0, math.pi / 9)
        p["phi"] = theta - torch.asin((_kappa(p) * 80.0).clamp(-1, 1))
        p["vx"], p["vy"] = p["vx"] * 0.0, p["vy"] * 0.0
        part = torch.arange(len(sec), device=DEV)
        alpha = torch.full((len(sec),), math.pi / 18, device=DEV, dtype=torch.float64)
        z_lo, z_hi = np.zeros(S, np.float32), np.full(S, synth.TPC_HALF_LENGTH, np.float32)
    else:
        p = _particles(g, case["tracks"] * 36 // S if kind == "event" else case["tracks"], -0.9, 0.9)
        part, sec = _pairs(p, S)
        alpha = (sec % 18).double() * (math.pi / 9) + math.pi / 18
        side = np.arange(S) < 18
        z_lo = np.where(side, 0.0, -synth.TPC_HALF_LENGTH).astype(np.float32)
        z_hi = np.where(side, synth.TPC_HALF_LENGTH, 0.0).astype(np.float32)
        if kind == "frame":
            t_frame = case["orbits"] * synth.ORBIT_US
            nc = max(2, int(round(case["rate_khz"] * 1e-3 * t_frame)))
            if case["rate_khz"] < 200.0:   # heavy-ion multiplicities vary exponentially, pp ones are alike
                share = torch.cumsum(-torch.log1p(-g.uniform(nc)), 0)
            else:
                share = torch.cumsum(torch.ones(nc, device=DEV, dtype=torch.float64), 0)
            coll = torch.searchsorted(share, g.uniform(len(p["pt"])) * share[-1]).clamp(max=nc - 1)
            shift = synth.DRIFT_VELOCITY * g.uniform(nc, 0.0, t_frame)[coll]
            z_lo = np.zeros(S, np.float32)
            z_hi = np.full(S, synth.DRIFT_VELOCITY * t_frame + synth.TPC_HALF_LENGTH, np.float32)
    kap = _kappa(p)
    cols = []
    for a in range(0, len(part), 1 << 18):   # blocks of pairs bound the [pairs, rows] temporaries
        i, s, al = part[a:a + (1 << 18)], sec[a:a + (1 << 18)], alpha[a:a + (1 << 18)]
        ok, y, z = _cross({k: v[i] for k, v in p.items()}, kap[i], al, rows)
        ok &= y.abs() <= half[None, :] + 2.0
        k, r = torch.nonzero(ok, as_tuple=True)
        y, z = y[k, r], z[k, r]
        if shift is not None:
            z = (synth.TPC_HALF_LENGTH - z.abs()) + shift[i[k]]
        y, z = y + g.normal(len(k), synth.SIGMA_Y), z + g.normal(len(k), synth.SIGMA_Z)
        keep = (g.uniform(len(k)) < 0.95) & (y.abs() <= half[r])
        cols.append((s[k][keep] * R + r[keep], y[keep], z[keep]))
    key, y, z = (torch.cat([c[j] for c in cols]) for j in range(3))
    n = int(0.05 * len(key))                 # noise: 5%, as many per sector as its signal asks for
    nsec = torch.div(key[torch.randint(len(key), (n,), generator=g.g, device=DEV)], R, rounding_mode="floor")
    nrow = torch.randint(R, (n,), generator=g.g, device=DEV)
    lo, hi = torch.from_numpy(z_lo).to(DEV).double(), torch.from_numpy(z_hi).to(DEV).double()
    key = torch.cat([key, nsec * R + nrow])
    y = torch.cat([y, (2.0 * g.uniform(n) - 1.0) * half[nrow]])
    z = torch.cat([z, lo[nsec] + g.uniform(n) * (hi - lo)[nsec]])
    mix = torch.randperm(len(key), generator=g.g, device=DEV)     # random order inside each row
    order = mix[torch.sort(key[mix], stable=True).indices]
    offs = torch.zeros(S * R + 1, dtype=torch.int64, device=DEV)
    offs[1:] = torch.cumsum(torch.bincount(key, minlength=S * R), 0)
    return y[order].float(), z[order].float(), offs.cpu().numpy().astype(np.uint32), z_lo, z_hi


def _stream(tracks, seed):
    """A compressed stream with a few escaped clusters."""
    g = _Rng(seed)
    rows, _ = _geometry()
    # 12 to 138 clusters per track and one row in twenty missing; the multiset of lengths is the size's own
    length = (12 + torch.arange(tracks, device=DEV) * 97 % 127)[torch.randperm(tracks, generator=g.g, device=DEV)]
    gaps = torch.div(length, 20, rounding_mode="floor")
    r0 = (g.uniform(tracks) * (R + 1 - length - gaps)).long()
    grid = torch.arange(R, device=DEV)[None, :]
    inside = (grid >= r0[:, None]) & (grid < (r0 + length + gaps)[:, None])
    order = torch.where(inside, torch.rand(tracks, R, generator=g.g, device=DEV), 2.0).argsort(1)
    rank = torch.empty_like(order).scatter_(1, order, grid.expand(tracks, R))
    held = inside & (rank >= gaps[:, None])
    t, row = torch.nonzero(held, as_tuple=True)
    nc = len(t)
    coef = torch.stack([g.uniform(tracks, -30, 30), g.normal(tracks, 0.25), g.normal(tracks, 8e-4),
                        g.uniform(tracks, 0, 7500), g.normal(tracks, 0.5), g.normal(tracks, 2e-4)], 1).float()
    first = torch.zeros(tracks + 1, dtype=torch.int32, device=DEV)
    first[1:] = torch.cumsum(held.sum(1), 0)
    code = torch.stack([g.normal(nc, 10.0), g.normal(nc, 10.0)], 1).round().to(torch.int16)
    raw = torch.zeros(nc, 2, device=DEV)
    esc = torch.randperm(nc, generator=g.g, device=DEV)[:max(1, nc // 100000)]
    code[esc, 0], code[esc, 1] = -32768, 0
    raw[esc] = torch.stack([g.uniform(len(esc), -30, 30), g.uniform(len(esc), 0, 7500)], 1).float()
    nu = int(0.067 * nc)
    stream = dict(coef=coef, x_ref=rows[r0].float(), first=first, row=row.to(torch.uint8), code=code, raw=raw,
                  un_row=(g.uniform(nu) * R).to(torch.uint8),
                  un_yz=torch.stack([g.uniform(nu, -30, 30), g.uniform(nu, 0, 7500)], 1).float())
    return stream, dict(n_tracks=tracks, n_track_clusters=nc, n_unassigned=nu, n_escaped=int((code[:, 0] == -32768).sum()))


# ---------------------------------------------------------------------------
# Calls
# ---------------------------------------------------------------------------
def prepare(case, seed):
    call = case["call"]
    if call == "decode":
        stream, counts = _stream(case["tracks"], seed)
        return dict(call=call, tracker=Tracker(default_config(), max_clusters=1024, max_sectors=1), stream=stream,
                    counts=counts)
    y, z, offs, z_lo, z_hi = _clusters(case, seed)
    S = case["sectors"]
    cap, cap_t = _caps(case)
    tr = Tracker(default_config(), max_clusters=cap, max_sectors=S)
    st = dict(call=call, tracker=tr, caps=(cap, cap_t))
    if call == "numpy":
        y, z = y.cpu().numpy(), z.cpu().numpy()
    if call == "device":
        # the tracker on memory of this program, so that its outputs can be read as tensors
        need = tr.workspace_bytes_for(cap, S)
        st["buf"] = buf = torch.zeros(need + 256, dtype=torch.uint8, device=DEV)
        tr.bind_workspace((buf.data_ptr() + 255) // 256 * 256, need, cap, S)
    tr.set_knobs(**{k: case[k] for k in TUNED if k in case})
    st["frame"] = (y, z, offs, z_lo, z_hi)
    if call in ("merge", "encode"):
        st["rid"] = tr.submit(*st["frame"])
        tr.get_counts(st["rid"])
        st["phys"] = np.arange(S, dtype=np.int32) if case["kind"] != "chunks" else None
    tracks, clusters = dict(param=5, cov=15), {}
    if call == "merge":
        tracks.update(next=0, head_of=0, heads=0, nseg=0, chi2=0, ndf=0)
        clusters = {"clusters": np.uint32}
    elif call in ("host", "numpy"):
        tracks.update(sector=0, start=0, x_ref=0, chi2=0, ndf=0)
        clusters = {"cluster_ids": np.uint32}
    if clusters:
        ints = {"next": np.int32, "nseg": np.int32, "ndf": np.int32, "head_of": np.uint32, "heads": np.uint32,
                "sector": np.uint32, "start": np.uint32}
        st["out"] = {k: np.zeros((cap_t, w) if w else cap_t, ints.get(k, np.float32)) for k, w in tracks.items()}
        st["out"].update({k: np.zeros(cap, t) for k, t in clusters.items()}, first=np.zeros(cap_t + 1, np.uint32))
    elif call == "encode":
        f32 = dict(dtype=torch.float32, device=DEV)
        st["out"] = dict(coef=torch.zeros(cap_t, 6, **f32), x_ref=torch.zeros(cap_t, **f32),
                         first=torch.zeros(cap_t + 1, dtype=torch.int32, device=DEV),
                         row=torch.zeros(cap, dtype=torch.uint8, device=DEV),
                         code=torch.zeros(cap, 2, dtype=torch.int16, device=DEV), raw=torch.zeros(cap, 2, **f32),
                         un_row=torch.zeros(cap, dtype=torch.uint8, device=DEV), un_yz=torch.zeros(cap, 2, **f32))
    torch.cuda.synchronize()
    return st


def _view(buf, address, n, dtype):
    off = address - buf.data_ptr()
    return buf[off:off + 4 * n].view(dtype)


def _keep(out, got):
    """The arrays of one pass, into the program's own (which are as long as they ever get)."""
    for k, to in out.items():
        to[:len(got[k])] = got[k]
    return out


def run(state):
    tr, call = state["tracker"], state["call"]
    if call == "device":
        rid = tr.submit(*state["frame"])
        got = tr.get_device(rid)
        tr.release(rid)
        buf, (cap, cap_t) = state["buf"], state["caps"]
        return dict(n_tracks=got["n_tracks"], n_track_clusters=got["n_track_clusters"], n_tracklets=got["n_tracklets"],
                    first=_view(buf, got["track_first"], cap_t + 1, torch.int32),
                    cluster_ids=_view(buf, got["cluster_ids"], cap, torch.int32),
                    param=_view(buf, got["param"], 5 * cap_t, torch.float32).view(cap_t, 5),
                    cov=_view(buf, got["cov"], 15 * cap_t, torch.float32).view(cap_t, 15))
    if call == "host":
        return tr.track_to_host(*state["frame"], lambda t: _keep(state["out"], vars(t)))
    if call == "numpy":
        return _keep(state["out"], vars(tr.track(*state["frame"], host=True)))
    if call == "merge":
        return _keep(state["out"], tr.merge(state["rid"], state["phys"]))
    if call == "encode":
        stream, counts = tr.encode(state["rid"], Q_Y, Q_Z)
        return dict(_keep(state["out"], stream), **counts)
    y, z, row = tr.decode(state["stream"], state["counts"], Q_Y, Q_Z)
    return dict(y=y, z=z, row=row)


# ---------------------------------------------------------------------------
# The same in 64 bits, from the definitions in include/tpc_tracker.h: the decisions of C1 and C2 are
# float32 by definition (one rounding per operation); everything of C5 is float64.
# ---------------------------------------------------------------------------
EXACT_CLUSTERS = 450_000


def exact(case, seed):
    if case["call"] == "decode":
        return _exact_decode(*_stream(case["tracks"], seed))
    # no value for merged chains, nor for larger frames: among millions of searches some candidate lies within
    # float32 rounding of its window's edge, and one track more or less moves all that follow it
    if case["call"] == "merge" or _clusters_of(case) > EXACT_CLUSTERS:
        return None
    trk = _exact_tracks(*_clusters(case, seed))
    cap_t = _caps(case)[1]

    def full(v):
        out = torch.zeros(cap_t, *v.shape[1:], dtype=torch.float64, device=DEV)
        out[:len(v)] = v
        return out

    trk = {k: full(v) for k, v in trk.items()}
    if case["call"] == "encode":
        p, x_ref = trk["param"], trk["x_ref"]
        kap = -synth.C_LIGHT_B * synth.BZ_TESLA * p[:, 4]
        ic = 1.0 / torch.sqrt(1.0 - p[:, 2] ** 2)
        coef = torch.stack([p[:, 0], p[:, 2] * ic, 0.5 * kap * ic ** 3, p[:, 1], p[:, 3] * ic,
                            0.5 * p[:, 3] * p[:, 2] * kap * ic ** 3], 1)
        return dict(coef=coef, x_ref=x_ref)
    if case["call"] == "device":
        return dict(param=trk["param"], cov=trk["cov"])
    return trk


def _exact_decode(s, counts):
    rows, _ = _geometry()
    length = (s["first"][1:] - s["first"][:-1]).long()
    t = torch.repeat_interleave(torch.arange(len(length), device=DEV), length)
    u = rows[s["row"].long()] - s["x_ref"].double()[t]
    c = s["coef"].double()[t]
    code = s["code"].double()
    esc = s["code"][:, 0] == -32768
    out = {}
    for k, (name, q) in enumerate((("y", Q_Y), ("z", Q_Z))):
        v = c[:, 3 * k] + u * (c[:, 3 * k + 1] + u * c[:, 3 * k + 2]) + code[:, k] * float(np.float32(q))
        v = torch.where(esc, s["raw"][:, k].double(), v)
        out[name] = torch.cat([v, s["un_yz"][:, k].double()])
    return out


def _exact_tracks(y, z, offs, z_lo, z_hi):
    cfg = default_config()
    S = (len(offs) - 1) // R
    N = len(y)
    ro = torch.from_numpy(offs.astype(np.int64)).to(DEV)
    n_row = ro[1:] - ro[:-1]
    X, Yh = _geometry()
    srow = torch.repeat_interleave(torch.arange(S * R, device=DEV), n_row)      # (sector, row) slot of each hit
    # C1: grid order
    ly = torch.ceil(20.0 * Yh).long().repeat(S)
    lz = torch.ceil(10.0 * (torch.from_numpy(z_hi.astype(np.float64) - z_lo).to(DEV))).long().repeat_interleave(R)
    B = torch.div(n_row, cfg.grid_hits_per_bin, rounding_mode="floor").clamp(min=1)
    q = torch.div(B * ly, lz, rounding_mode="floor")
    s = torch.floor(torch.sqrt(q.double())).long()
    s = torch.where(s * s > q, s - 1, s)
    s = torch.where((s + 1) * (s + 1) <= q, s + 1, s)
    ny = torch.minimum(s.clamp(min=1), B)
    nz = torch.div(B, ny, rounding_mode="floor").clamp(min=1)

    def bins(v, lo, inv, n):
        u = (v - lo) * (n.float() * inv)
        u = torch.where(u >= 0, u, torch.zeros_like(u))
        return torch.minimum(u, (n - 1).float()).long()

    ylo, iwy = (-Yh).float().repeat(S), (1.0 / (2.0 * Yh)).float().repeat(S)
    zl = torch.from_numpy(z_lo).to(DEV).repeat_interleave(R)
    iwz = (1.0 / torch.from_numpy(z_hi.astype(np.float64) - z_lo).to(DEV)).float().repeat_interleave(R)
    b = bins(z, zl[srow], iwz[srow], nz[srow]) * ny[srow] + bins(y, ylo[srow], iwy[srow], ny[srow])
    order = torch.sort(srow * (1 << 20) + b, stable=True).indices
    hy, hz = y[order], z[order]                                                  # float32, sorted positions
    # hits of a row padded to the widest row: [S, R, M]
    M = int(n_row.max())
    slot = torch.arange(M, device=DEV)[None, :]
    pos = torch.where(slot < n_row[:, None], ro[:-1, None] + slot, -1).view(S, R, M)
    py = torch.where(pos >= 0, hy[pos.clamp(min=0)], torch.full((), 1e9, device=DEV))
    pz = torch.where(pos >= 0, hz[pos.clamp(min=0)], torch.full((), 1e9, device=DEV))
    # C2: links (float32 as written), C3
    up0 = torch.full((N,), -1, dtype=torch.int64, device=DEV)
    dn0 = up0.clone()
    rho = float(np.float32((cfg.sigma_y / cfg.sigma_z) ** 2))

    def near(a, c, wy, wz):
        """Up to K hits of row c in the window of each hit of row a: slots [S, M, K] (M where none)."""
        m = ((py[:, a, :, None] - py[:, c, None, :]).abs() <= wy) & ((pz[:, a, :, None] - pz[:, c, None, :]).abs() <= wz)
        m &= (pos[:, a, :, None] >= 0) & (pos[:, c, None, :] >= 0)
        K = max(1, int(m.sum(-1).max()))
        idx = torch.where(m, slot[None], M)
        return torch.topk(idx, min(K, M), dim=-1, largest=False).values

    big = torch.iinfo(torch.int64).max
    for r in range(1, R - 1):
        du, dd = float(X[r + 1] - X[r]), float(X[r] - X[r - 1])
        tt = dd / (dd + du)
        f32 = lambda v: float(np.float32(v))   # noqa: E731
        ku = near(r, r + 1, f32(cfg.win_a_y * du + cfg.win_b_y), f32(cfg.win_a_z * du + cfg.win_b_z))
        kd = near(r, r - 1, f32(cfg.win_a_y * dd + cfg.win_b_y), f32(cfg.win_a_z * dd + cfg.win_b_z))
        dmax = f32((cfg.link_nsigma ** 2 * cfg.sigma_y ** 2) * ((1 + tt * tt) + (1 - tt) * (1 - tt)))
        t32 = torch.tensor(tt, dtype=torch.float32, device=DEV)

        def take(v, c, k):
            return torch.gather(torch.nn.functional.pad(v[:, c], (0, 1)), 1, k.view(S, -1)).view(k.shape)

        yu, zu, yd, zd = take(py, r + 1, ku), take(pz, r + 1, ku), take(py, r - 1, kd), take(pz, r - 1, kd)
        yu, zu, yd, zd = yu[..., None, :], zu[..., None, :], yd[..., :, None], zd[..., :, None]
        ey = py[:, r, :, None, None] - (yd + t32 * (yu - yd))
        ez = pz[:, r, :, None, None] - (zd + t32 * (zu - zd))
        dev = ey * ey + torch.tensor(rho, dtype=torch.float32, device=DEV) * (ez * ez)
        ok = (dev <= dmax) & (ku[..., None, :] < M) & (kd[..., :, None] < M)
        dev = torch.where(ok, dev, torch.full((), math.inf, device=DEV))
        best = dev.amin((-1, -2), keepdim=True)
        # ties: the smaller position up, then down
        rank = torch.where(ok & (dev == best), ku[..., None, :] * (M + 1) + kd[..., :, None], big).amin((-1, -2))
        has = (rank < big) & (pos[:, r] >= 0)
        h = pos[:, r][has]
        base = torch.arange(S, device=DEV)[:, None].expand(S, M)[has]
        up0[h] = pos[base, r + 1, torch.div(rank[has], M + 1, rounding_mode="floor")]
        dn0[h] = pos[base, r - 1, rank[has] % (M + 1)]
    ids = torch.arange(N, device=DEV)
    up1 = torch.where((up0 >= 0) & (dn0[up0.clamp(min=0)] == ids), up0, -1)
    dn1 = torch.where((dn0 >= 0) & (up0[dn0.clamp(min=0)] == ids), dn0, -1)
    start = torch.nonzero((dn1 < 0) & (up1 >= 0) & (up1[up1.clamp(min=0)] >= 0)).view(-1)
    # C5 in float64, one row of all tracklets at a time
    T = len(start)
    sec = torch.div(srow[start], R, rounding_mode="floor")
    r0 = srow[start] % R
    held = torch.full((T, R), -1, dtype=torch.int64, device=DEV)
    cur, n = start.clone(), torch.zeros(T, dtype=torch.int64, device=DEV)
    tid = torch.arange(T, device=DEV)
    while bool((cur >= 0).any()):
        on = cur >= 0
        held[tid[on], (r0 + n)[on]] = cur[on]
        n = n + on.long()
        cur = torch.where(on, up1[cur.clamp(min=0)], -1)
    rl = r0 + n - 1
    rm = r0 + torch.div(n - 1, 2, rounding_mode="floor")
    Hy, Hz = hy.double(), hz.double()
    bk = -synth.C_LIGHT_B * cfg.bz
    vy, vz = cfg.sigma_y ** 2, cfg.sigma_z ** 2

    def asin_over(u):
        return torch.where(u.abs() < 1e-4, 1.0 + u * u / 6.0, torch.asin(u) / torch.where(u.abs() < 1e-4, 1.0, u))

    def dasin_over(u):
        v = torch.where(u.abs() < 1e-2, 0.5, u)
        far = (v / torch.sqrt(1 - v * v) - torch.asin(v)) / (v * v)
        return torch.where(u.abs() < 1e-2, u * (1 / 3 + u * u * (3 / 10 + u * u * (15 / 56 + u * u * 35 / 144))), far)

    x0, xm, xl = X[r0], X[rm], X[rl]
    h0, hm, hl = start, held[tid, rm], held[tid, rl]
    ax, ay, bx, by, cx, cy = xm - x0, Hy[hm] - Hy[h0], xl - xm, Hy[hl] - Hy[hm], xl - x0, Hy[hl] - Hy[h0]
    lc = torch.hypot(cx, cy)
    kap = 2 * (ax * by - ay * bx) / (torch.hypot(ax, ay) * torch.hypot(bx, by) * lc)
    u = 0.5 * kap * lc
    ok = u.abs() < 1
    u = torch.where(ok, u, 0.0)
    phi0 = torch.atan2(cy, cx) - torch.asin(u)
    p = torch.stack([Hy[h0], Hz[h0], torch.sin(phi0), (Hz[hl] - Hz[h0]) / (lc * asin_over(u)),
                     (kap / bk).clamp(-cfg.seed_qpt_max, cfg.seed_qpt_max)], 1)
    ok &= (torch.cos(phi0) > 0) & (p[:, 2].abs() < cfg.s_max)
    c0 = torch.diag(torch.tensor([vy, vz, cfg.c0_sinphi, cfg.c0_tanl, cfg.c0_qpt], dtype=torch.float64, device=DEV))
    Cv = c0.expand(T, 5, 5).clone()
    eye = torch.eye(5, dtype=torch.float64, device=DEV)

    def move(p, Cv, dx):
        s1, tl = p[:, 2], p[:, 3]
        k = bk * p[:, 4]
        s2 = s1 + k * dx
        good = (s1.abs() < cfg.s_max) & (s2.abs() < cfg.s_max)
        s1, s2 = torch.where(good, s1, 0.0), torch.where(good, s2, 0.0)
        c1, c2 = torch.sqrt(1 - s1 * s1), torch.sqrt(1 - s2 * s2)
        dy = dx * (s1 + s2) / (c1 + c2)
        L = torch.sqrt(dx * dx + dy * dy)
        u = 0.5 * k * L
        good &= u.abs() < 1
        u = torch.where(good, u, 0.0)
        sg = torch.sign(dx)
        ds = sg * L * asin_over(u)
        # derivatives of dy in s1 (s2 moves with it) and in kappa
        D = (1 + c1 * c2 + s1 * s2) / (c1 + c2) ** 2
        a = dx * D * (1 / c1 + 1 / c2)
        bq = dx * dx * (D / c2) * bk
        dl = dy / L
        sl, sk = sg / torch.sqrt(1 - u * u), sg * 0.5 * L * L * dasin_over(u)
        F = eye.expand(len(p), 5, 5).clone()
        F[:, 0, 2], F[:, 0, 4] = a, bq
        F[:, 1, 2], F[:, 1, 3], F[:, 1, 4] = tl * sl * dl * a, ds, tl * (sl * dl * bq + sk * bk)
        F[:, 2, 4] = bk * dx
        p2 = p.clone()
        p2[:, 0] += dy
        p2[:, 1] += tl * ds
        p2[:, 2] = s2
        return good, p2, F @ Cv @ F.transpose(1, 2).contiguous()

    def measure(p, Cv, h):
        r = torch.stack([Hy[h], Hz[h]], 1) - p[:, :2]
        a, b, c = Cv[:, 0, 0] + vy, Cv[:, 0, 1], Cv[:, 1, 1] + vz
        inv = (torch.stack([c, -b, -b, a], 1) / (a * c - b * b)[:, None]).view(-1, 2, 2)
        K = Cv[:, :, :2].contiguous() @ inv
        J = eye.expand(len(p), 5, 5).clone()
        J[:, :, :2] -= K
        V = torch.diag(torch.tensor([vy, vz], dtype=torch.float64, device=DEV)).expand(len(p), 2, 2).contiguous()
        Cn = J @ Cv @ J.transpose(1, 2).contiguous() + K @ V @ K.transpose(1, 2).contiguous()
        return p + (K @ r[:, :, None])[:, :, 0], Cn, (r[:, None, :] @ inv @ r[:, :, None]).view(-1)

    def search(p, Cv, s, r):
        sy, sz = Cv[:, 0, 0] + vy, Cv[:, 1, 1] + vz
        wy = (cfg.gate_nsigma * torch.sqrt(sy)).clamp(max=cfg.win_cap)
        wz = (cfg.gate_nsigma * torch.sqrt(sz)).clamp(max=cfg.win_cap)
        dy, dz = py[s, r].double() - p[:, :1], pz[s, r].double() - p[:, 1:2]
        d = dy * dy / sy[:, None] + dz * dz / sz[:, None]
        d = torch.where((dy.abs() <= wy[:, None]) & (dz.abs() <= wz[:, None]), d, math.inf)
        best, j = d.min(1)
        return torch.where(best < math.inf, pos[s, r, j], -1)

    def keep(sel, old, new):
        return torch.where(sel.view(-1, *([1] * (old.dim() - 1))), new, old)

    xp, rout, pout = X[r0].clone(), rl.clone(), p.clone()
    miss = torch.zeros(T, dtype=torch.int64, device=DEV)
    up = ok.clone()
    for r in range(1, R):
        i = torch.nonzero(up & (r0 < r)).view(-1)
        if not len(i):
            continue
        good, p2, C2 = move(p[i], Cv[i], X[r] - xp[i])
        chain = rl[i] >= r
        ok[i] &= good | ~chain
        go = good & (chain | (p2[:, 0].abs() <= float(Yh[r]) + cfg.edge_margin))
        up[i] = go
        i, p2, C2, chain = i[go], p2[go], C2[go], chain[go]
        xp[i] = X[r]
        h = torch.where(chain, held[i, r], -1)
        h = torch.where(chain, h, search(p2, C2, sec[i], r))
        held[i, r] = h
        hit = h >= 0
        pn, Cn, _ = measure(p2, C2, h.clamp(min=0))
        p[i], Cv[i] = keep(hit, p2, pn), keep(hit, C2, Cn)
        far = hit & (rl[i] <= r)
        pout[i[far]], rout[i[far]], miss[i[far]] = p[i[far]], r, 0
        miss[i[~hit]] += 1
        up[i] = miss[i] <= cfg.max_miss
    p = pout.clone()
    ho = held[tid, rout]
    p[:, 0], p[:, 1] = Hy[ho], Hz[ho]
    Cv = c0.expand(T, 5, 5).clone()
    xp, rin, nh = X[rout].clone(), rout.clone(), torch.ones_like(rout)
    chi2 = torch.zeros(T, dtype=torch.float64, device=DEV)
    pin, Cin = p.clone(), Cv.clone()
    miss[:] = 0
    down = ok.clone()
    for r in range(R - 2, -1, -1):
        held[:, r] = torch.where((r0 > r) | (rout < r), -1, held[:, r])
        i = torch.nonzero(down & (rout > r)).view(-1)
        if not len(i):
            continue
        good, p2, C2 = move(p[i], Cv[i], X[r] - xp[i])
        below = r0[i] > r
        go = good & ~(below & (p2[:, 0].abs() > float(Yh[r]) + cfg.edge_margin))
        down[i] = go
        i, p2, C2, below = i[go], p2[go], C2[go], below[go]
        xp[i] = X[r]
        h = held[i, r]
        h = torch.where(h >= 0, h, search(p2, C2, sec[i], r))
        held[i, r] = h
        hit = h >= 0
        pn, Cn, x2 = measure(p2, C2, h.clamp(min=0))
        p[i], Cv[i] = keep(hit, p2, pn), keep(hit, C2, Cn)
        j = i[hit]
        pin[j], Cin[j], rin[j] = p[j], Cv[j], r
        nh[j] += 1
        chi2[j] += x2[hit]
        miss[i[hit & below]] = 0
        miss[i[~hit & below]] += 1
        down[i] = miss[i] <= cfg.max_miss
    # C6: each hit goes to the tracklet with the most hits, ties to the smaller start
    grid = torch.arange(R, device=DEV)[None, :]
    valid = ok & (nh >= cfg.min_tracklet_hits)
    mine = (held >= 0) & (grid >= rin[:, None]) & (grid <= rout[:, None]) & valid[:, None]
    rank = nh * T + (T - 1 - tid)
    t, r = torch.nonzero(mine, as_tuple=True)
    W = torch.full((N,), -1, dtype=torch.int64, device=DEV)
    W.scatter_reduce_(0, held[t, r], rank[t], "amax")
    owned = torch.zeros(T, dtype=torch.int64, device=DEV)
    owned.index_add_(0, t, (W[held[t, r]] == rank[t]).long())
    take = valid & (owned >= cfg.min_track_hits) & (owned.double() >= cfg.min_owned_frac * nh.double())
    i, j = (torch.tril_indices(5, 5, device=DEV))
    return dict(x_ref=X[rin[take]], param=pin[take], cov=Cin[take][:, i, j], chi2=chi2[take])
