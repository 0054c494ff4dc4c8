"""Performance cases of the TPC tracker: the calls a user's program makes, over
the range of events it sees, with seeded inputs made on the GPU.

A case names what is called (`kind`), the shape of the events and how clusters
and tracks travel:

  kind       "track"   clusters -> tracks
             "merge"   the cross-sector merger on an event tracked before
             "chain"   tracking, then merging
             "calib"   drift correction, accumulation and fit on a tracked event
             "serve"   a burst of requests through the continuous-batching server
  shape      "sector"  one sector, tracks from the origin (one link's data)
             "pp"      36 sectors, soft spectrum, 5% noise
             "pbpb"    36 sectors, primaries, secondaries and loopers, 10% noise
  primaries  particles of the (largest) event; for "sector" its tracks
  events     events of the call; a "pbpb" batch of several has multiplicities
             spread over their logarithm between 50 and `primaries`
  api        "event" (one launch per step), "graph" (replay of the slot's
             graph), "sector" (the per-sector call), "flight" (every event on a
             tracker and stream of its own)
  source     where the clusters are: "device" or "host" (pinned)
  read       where the tracks go: "device" (views of the tracker's arrays, the
             counts read back) or "host" (pinned); the arrays have room for more
             than such an event gives, zero beyond the counts
  x0_cm      radiation length of the scattering model, 0 without it
  tl_block, row_batch   launch shape, as the autotuner may set it
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1712_09416_amd import TRACK_DTYPE, Tracker
from paper_1712_09416_amd._lib import check
from paper_1712_09416_amd.serve import Request, Server
from paper_1712_09416_amd.tracker import calib_fit

N_SECTORS, N_ROWS = 36, 159
Z_MAX, BZ, R_EXIT, C_LIGHT = 250.0, 0.5, 250.0, 0.00299792458
TAN_HALF = float(np.float32(math.tan(math.radians(10.0))))
SIGMA = {"sector": (0.1, 0.0, 0.15, 0.0), "pp": (0.1, 0.0, 0.15, 0.0), "pbpb": (0.1, 0.1, 0.1, 0.1)}
NOISE = {"sector": 0.05, "pp": 0.05, "pbpb": 0.10}
EFFICIENCY = {"sector": 1.0, "pp": 0.98, "pbpb": 0.98}
# clusters of an event per primary, noise included, as these shapes give them on
# average; every event of a case is brought to exactly this number by its noise
CLUSTERS_PER_PRIMARY = {"sector": 95.0, "pp": 179.0, "pbpb": 233.0}
DRIFT_EPS = 0.004
SERVE_MIX = (0.70, 0.25, 0.05)        # pp / peripheral / central


def _case(name, kind, shape, primaries, events=1, api="event", source="device", read="device",
          x0_cm=0.0, tl_block=64, row_batch=8):
    c = dict(kind=kind, shape=shape, primaries=int(primaries), events=int(events), api=api,
             source=source, read=read, x0_cm=float(x0_cm), tl_block=int(tl_block),
             row_batch=int(row_batch))
    return dict(c, name=name) if name else c


def listed():
    return [
        # one detector link's part of an event, tracked on its own
        _case("sector_200", "track", "sector", 200, api="sector", read="host"),
        # the smallest ordinary call: one pp event, where launches and latency count
        _case("pp_60", "track", "pp", 60, read="host"),
        # a serving slot of small events, tracked together and read back
        _case("pp_batch_32", "track", "pp", 60, events=32, read="host"),
        # a peripheral event, as most heavy-ion events are
        _case("peripheral_2000", "track", "pbpb", 2000),
        # the same with the scattering model on, from host memory, segments joined
        _case("peripheral_chain_ms", "chain", "pbpb", 2000, source="host", read="host", x0_cm=31000.0),
        # a central event resident on the GPU: the largest single event
        _case("central_15000", "track", "pbpb", 15000),
        # the same end to end, pinned host memory to pinned host memory
        _case("central_host", "track", "pbpb", 15000, source="host", read="host"),
        # central events pipelined, each on its own tracker and stream
        _case("central_flight_3", "track", "pbpb", 15000, events=3, api="flight"),
        # 64 events of uneven size in one slot, replayed from its graph: the largest call
        _case("batch_64", "track", "pbpb", 15000, events=64, api="graph"),
        # the merger alone on a central event (global reconstruction step)
        _case("merge_15000", "merge", "pbpb", 15000, read="host"),
        # the drift-velocity side task on a central event
        _case("calib_15000", "calib", "pbpb", 15000),
        # a burst of requests of the serving mix through the server
        _case("serve_24", "serve", "pbpb", 15000, events=24, source="host", read="host"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["track"] * 6 + ["merge", "chain", "calib", "serve"])
    x0 = rng.choice([0.0, 0.0, 31000.0])
    shape = dict(tl_block=rng.choice([64, 64, 128, 256]), row_batch=rng.choice([4, 8, 8, 16]))
    if kind == "serve":
        return _case(None, kind, "pbpb", _log_int(rng, 1000, 15000), events=rng.randint(6, 24),
                     source="host", read="host", **shape)
    if kind != "track":
        sh = "pbpb" if kind == "calib" else rng.choice(["pp", "pbpb"])
        n = _log_int(rng, 20, 400) if sh == "pp" else _log_int(rng, 300 if kind == "calib" else 50, 15000)
        src = rng.choice(["device", "host"]) if kind == "chain" else "device"
        read = "device" if kind == "calib" else "host"
        return _case(None, kind, sh, n, source=src, read=read, x0_cm=x0, **shape)
    sh = rng.choice(["sector", "pp", "pbpb", "pbpb"])
    src, read = rng.choice(["device", "device", "host"]), rng.choice(["device", "host"])
    if sh == "sector":
        return _case(None, kind, sh, _log_int(rng, 8, 2000), api=rng.choice(["sector", "event"]),
                     source=src, read=read, x0_cm=x0, **shape)
    events = rng.choice([1, _log_int(rng, 2, 48)])
    api = rng.choice(["event", "graph"])
    if events <= 4 and events > 1 and rng.random() < 0.5:
        api = "flight"
    n = _log_int(rng, 15, 400) if sh == "pp" else _log_int(rng, 60, 15000)
    return _case(None, kind, sh, n, events=events, api=api, source=src, read=read, x0_cm=x0, **shape)


# ---------------------------------------------------------------------------
# events: exact helices in 0.5 T; every crossing of a pad-row plane inside a
# sector's acceptance is a cluster, smeared, thinned, with uniform noise and
# in random order
# ---------------------------------------------------------------------------
def _row_x():
    r = np.arange(N_ROWS, dtype=np.float64)
    x = np.where(r < 63, 85.225 + 0.75 * r, np.where(r < 127, 135.1 + (r - 63), 199.35 + 1.5 * (r - 127)))
    return x.astype(np.float32)


def _geometry(shape):
    s = SIGMA[shape]
    return dict(n_sectors=N_SECTORS, n_rows=N_ROWS, row_x=_row_x(), bz_tesla=np.float32(BZ),
                tan_half_angle=np.float32(TAN_HALF), z_max=np.float32(Z_MAX),
                sigma_y0=np.float32(s[0]), sigma_y1=np.float32(s[1]), sigma_z0=np.float32(s[2]),
                sigma_z1=np.float32(s[3]))


def _multiplicities(case):
    n, k = case["primaries"], case["events"]
    if case["shape"] != "pbpb" or k == 1 or case["api"] == "flight":
        return [n] * k
    lo = min(50, n)
    # spread over the logarithm, large and small ones mixed
    return [int(round(lo * (n / lo) ** (((i * 37) % k + 0.5) / k))) for i in range(k)]


def _n_clusters(shape, primaries):
    return max(1, round(CLUSTERS_PER_PRIMARY[shape] * primaries))


def _max_tracks(n):
    """Track records that the result arrays have room for: events of n
    clusters give about n / 78."""
    return n // 32 + 64


class _Rand:
    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed))

    def uniform(self, n, lo=0.0, hi=1.0):
        return lo + (hi - lo) * torch.rand(n, generator=self.g, device="cuda", dtype=torch.float64)

    def normal(self, n):
        return torch.randn(n, generator=self.g, device="cuda", dtype=torch.float64)


def _pt_tail(u, slope=0.5, lo=0.1, pj=2.0, hi=20.0):
    """exp(-pT/slope) from lo to pj, then a pT^-4 tail to hi, by inversion."""
    e0, e1 = math.exp(-lo / slope), math.exp(-pj / slope)
    w0, w1 = slope * (e0 - e1), e1 * pj / 3.0 * (1.0 - (hi / pj) ** -3.0)
    f = u * (w0 + w1)
    soft = -slope * torch.log((e0 - f / slope).clamp_min(e1 * 0.5))
    v = ((f - w0) / w1).clamp(0.0, 1.0)
    tail = pj * (1.0 + v * ((hi / pj) ** -3.0 - 1.0)) ** (-1.0 / 3.0)
    return torch.where(f < w0, soft, tail)


def _particles(R, shape, n):
    """Columns vx, vy, vz, pT, phi, eta, charge of one event's particles."""
    zero = torch.zeros(n, device="cuda", dtype=torch.float64)
    sign = torch.where(R.uniform(n) < 0.5, -1.0, 1.0).to(torch.float64)
    if shape == "sector":
        pt = torch.exp(R.uniform(n, math.log(0.2), math.log(5.0)))
        return torch.stack([zero, zero, zero, pt, R.uniform(n, 0.0, math.radians(20.0)),
                            R.uniform(n, 0.0, 0.9), sign])
    if shape == "pp":
        pt = 0.1 - 0.5 * torch.log1p(-R.uniform(n))
        return torch.stack([zero, zero, zero, pt, R.uniform(n, 0.0, 2 * math.pi), R.uniform(n, -0.9, 0.9), sign])
    prim = torch.stack([zero, zero, zero, _pt_tail(R.uniform(n)), R.uniform(n, 0.0, 2 * math.pi),
                        R.uniform(n, -0.9, 0.9), sign])
    ns, nl = round(0.2 * n), round(0.05 * n)
    r, a, ev = R.uniform(ns, 0.0, 60.0), R.uniform(ns, 0.0, 2 * math.pi), R.uniform(ns, -0.9, 0.9)
    sec = torch.stack([r * torch.cos(a), r * torch.sin(a), r * torch.sinh(ev), _pt_tail(R.uniform(ns)),
                       a + R.uniform(ns, -0.5, 0.5), R.uniform(ns, -0.9, 0.9),
                       torch.where(R.uniform(ns) < 0.5, -1.0, 1.0).to(torch.float64)])
    z = torch.zeros(nl, device="cuda", dtype=torch.float64)
    loop = torch.stack([z, z, z, R.uniform(nl, 0.05, 0.15), R.uniform(nl, 0.0, 2 * math.pi),
                        R.uniform(nl, -0.9, 0.9), torch.where(R.uniform(nl) < 0.5, -1.0, 1.0).to(torch.float64)])
    return torch.cat([prim, sec, loop], 1)


def _crossings(p, ev):
    """(event, sector, row, y, z) of every pad-row crossing of the particles."""
    vx, vy, vz, pt, phi0, eta, q = p
    rad = pt / (C_LIGHT * BZ)
    h = -q
    hr = h * rad
    xc, yc = vx - hr * torch.sin(phi0), vy + hr * torch.cos(phi0)
    T = torch.sinh(eta)
    rho, psi = torch.hypot(xc, yc), torch.atan2(yc, xc)
    w = (R_EXIT ** 2 - rho ** 2 - rad ** 2) / (2.0 * hr * rho)
    aw = torch.asin(w.clamp(-1.0, 1.0))
    l_max = 4.0 * math.pi * rad                       # at most two turns
    for sol in (psi + aw, psi + math.pi - aw):
        l_exit = rad * torch.remainder(h * (sol - phi0), 2 * math.pi)
        l_max = torch.where(w.abs() <= 1.0, torch.minimum(l_max, l_exit), l_max)
    l_z = torch.where(T != 0, (torch.sign(T) * Z_MAX - vz) / T, torch.full_like(T, math.inf))
    l_max = torch.minimum(l_max, l_z)
    # azimuths reached inside the chamber (samples of the path and their neighbours)
    t = torch.linspace(0.0, 1.0, 96, device="cuda", dtype=torch.float64)[None, :] * l_max[:, None]
    ph = phi0[:, None] + h[:, None] * t / rad[:, None]
    X, Y = xc[:, None] + hr[:, None] * torch.sin(ph), yc[:, None] - hr[:, None] * torch.cos(ph)
    sec = torch.floor(torch.remainder(torch.atan2(Y, X), 2 * math.pi) / math.radians(20.0)).long() % 18
    inside = (torch.hypot(X, Y) >= 70.0).to(torch.float32)
    near = torch.zeros((len(pt), 18), device="cuda")
    near.scatter_reduce_(1, sec, inside, "amax")
    near = torch.maximum(torch.maximum(near, near.roll(1, 1)), near.roll(-1, 1))
    ip, ia = torch.nonzero(near > 0, as_tuple=True)
    al = torch.deg2rad((ia.to(torch.float64) + 0.5) * 20.0)
    ca, sa = torch.cos(al), torch.sin(al)
    nc, yl = xc[ip] * ca + yc[ip] * sa, -xc[ip] * sa + yc[ip] * ca
    xr = torch.from_numpy(_row_x()).to("cuda", torch.float64)
    v = (xr[None, :] - nc[:, None]) / hr[ip][:, None]
    reach = v.abs() <= 1.0
    asv = torch.asin(v.clamp(-1.0, 1.0))
    out = []
    for dphi in (asv, math.pi - asv):
        y = yl[:, None] - hr[ip][:, None] * torch.cos(dphi)
        in_y = reach & (y.abs() <= xr[None, :] * TAN_HALF)
        th = torch.remainder(h[ip][:, None] * (al[:, None] + dphi - phi0[ip][:, None]), 2 * math.pi)
        for turn in (0.0, 2 * math.pi):
            l = rad[ip][:, None] * (th + turn)
            z = vz[ip][:, None] + T[ip][:, None] * l
            k, r = torch.nonzero(in_y & (l > 0) & (l <= l_max[ip][:, None]) & (z.abs() <= Z_MAX), as_tuple=True)
            zk = z[k, r]
            out.append((ev[ip[k]], ia[k] + torch.where(zk >= 0, 0, 18), r, y[k, r], zk))
    return [torch.cat(c) for c in zip(*out)]


def _clusters(shape, mult, seed):
    """Event offsets (numpy) and the clusters sector, row, y, z (device) of
    len(mult) concatenated events."""
    R = _Rand(seed)
    tab = [_particles(R, shape, n) for n in mult]
    ev = torch.cat([torch.full((t.shape[1],), e, device="cuda") for e, t in enumerate(tab)])
    tab = torch.cat(tab, 1)
    parts = [_crossings(tab[:, a:a + 16384], ev[a:a + 16384]) for a in range(0, tab.shape[1], 16384)]
    ev, sec, row, y, z = [torch.cat(c) for c in zip(*parts)]
    if shape == "sector":
        keep = sec == 0
    else:
        keep = R.uniform(len(y)) < EFFICIENCY[shape]
    ev, sec, row, y, z = (c[keep] for c in (ev, sec, row, y, z))
    s = SIGMA[shape]
    y = y + R.normal(len(y)) * (s[0] + s[1] * z.abs() / Z_MAX)
    zm = z + R.normal(len(y)) * (s[2] + s[3] * z.abs() / Z_MAX)
    # the number of clusters is the case's: surplus crossings are dropped at
    # random, the noise fills the rest
    want = torch.tensor([_n_clusters(shape, m) for m in mult], device="cuda")
    most = (want.to(torch.float64) * (1.0 - 0.5 * NOISE[shape])).long()
    order = torch.argsort(R.uniform(len(y)))
    order = order[torch.argsort(ev[order], stable=True)]
    ev, sec, row, y, zm = (c[order] for c in (ev, sec, row, y, zm))
    per = torch.bincount(ev, minlength=len(mult))
    first = torch.cumsum(per, 0) - per
    keep = torch.arange(len(ev), device="cuda") - first[ev] < most[ev]
    ev, sec, row, y, zm = (c[keep] for c in (ev, sec, row, y, zm))
    nn = want - torch.minimum(per, most)
    nev = torch.repeat_interleave(torch.arange(len(mult), device="cuda"), nn)
    k = len(nev)
    nsec = torch.zeros(k, device="cuda", dtype=torch.long) if shape == "sector" else \
        torch.randint(0, N_SECTORS, (k,), generator=R.g, device="cuda")
    nrow = torch.randint(0, N_ROWS, (k,), generator=R.g, device="cuda")
    xr = torch.from_numpy(_row_x()).to("cuda", torch.float64)
    ny = R.uniform(k, -1.0, 1.0) * xr[nrow] * TAN_HALF
    nz = R.uniform(k, 0.0, Z_MAX) * torch.where(nsec < 18, 1.0, -1.0)
    ev, sec, row = torch.cat([ev, nev]), torch.cat([sec, nsec]), torch.cat([row, nrow])
    y, zm = torch.cat([y, ny]), torch.cat([zm, nz])
    order = torch.argsort(R.uniform(len(y)))
    order = order[torch.argsort(ev[order], stable=True)]
    offs = np.concatenate([[0], np.cumsum(want.cpu().numpy())]).astype(np.int64)
    return offs, [sec[order].to(torch.uint8), row[order].to(torch.uint8), y[order].to(torch.float32),
                  zm[order].to(torch.float32)]


def _pinned(t):
    h = torch.empty(t.shape, dtype=t.dtype, pin_memory=True)
    h.copy_(t)
    return h


# ---------------------------------------------------------------------------
class _Slot:
    """One tracker with its staged clusters and, for host reads, its result buffers."""

    def __init__(self, case, offs, cl):
        self.api, self.read = case["api"], case["read"]
        n, ne = int(offs[-1]), len(offs) - 1
        self.trk = Tracker(_geometry(case["shape"]), max_events=ne, max_clusters=max(n, 1),
                           x0_cm=case["x0_cm"], tl_block=case["tl_block"], row_batch=case["row_batch"])
        self.offs, self.ne = offs, ne
        if case["source"] == "host":
            self.held = [_pinned(c) for c in cl]
            self.cl = [h.numpy() for h in self.held]
        else:
            self.cl = cl
        # result arrays, as long as the case's events can need
        self.mt, self.n = _max_tracks(n), n
        if self.read == "host":
            self.held_t = torch.zeros(self.mt * TRACK_DTYPE.itemsize, dtype=torch.uint8, pin_memory=True)
            self.held_h = torch.zeros(n, dtype=torch.int32, pin_memory=True)
            self.tracks, self.hits = self.held_t.numpy().view(TRACK_DTYPE), self.held_h.numpy()
            self.nseg = np.zeros(self.mt, np.int32)
            self.totals = np.zeros(2, np.int64)
        else:
            self.trk.workspace.zero_()
        torch.cuda.synchronize()
        if self.api == "graph" and case["source"] == "device":
            self.load()

    def load(self):
        if self.ne == 1:
            self.trk.load(0, *self.cl)
        else:
            self.trk.load_batch(0, self.offs, *self.cl)

    def track(self):
        if self.api != "graph" or isinstance(self.cl[0], np.ndarray):
            self.load()
        if self.api == "graph":
            self.trk.track_events([0])
        elif self.api == "sector":
            self.trk.track_sector(0, 0)
        else:
            self.trk.track_event(0)

    def results(self):
        if self.read == "host":
            got = self.trk.get_slot_tracks(0, self.tracks, self.hits)
            counts = np.array([[len(t), len(h)] for t, h in got], np.int64)
            return dict(_records(self.tracks), hits=self.hits, counts=counts)
        t = self.trk
        tk, hits, tof, hof, tot = (p - t.workspace.data_ptr() for p in t.device_results(0))
        with torch.cuda.stream(t.stream):
            nt, nh = t.workspace[tot:tot + 8].view(torch.int32).tolist()
        if nt > self.mt:
            raise RuntimeError("more tracks than the result array holds")
        rec = t.workspace[tk:tk + self.mt * TRACK_DTYPE.itemsize]
        return dict(tracks=rec.view(torch.int32).view(self.mt, -1)[:, :10],
                    fit=rec.view(torch.float64).view(self.mt, -1)[:, 5:],
                    hits=t.workspace[hits:hits + 4 * self.n].view(torch.int32),
                    counts=np.array([nt, nh], np.int64),
                    track_off=t.workspace[tof:tof + 4 * self.ne + 4].view(torch.int32),
                    hit_off=t.workspace[hof:hof + 4 * self.ne + 4].view(torch.int32))

    def merged(self):
        """The merger's output into the pinned arrays (the C entry: the
        caller's own buffers)."""
        t, n = self.trk, self.totals
        check(t.L.tpc_get_merged(t.ctx, 0, 0, self.tracks.ctypes.data, self.mt, self.hits.ctypes.data,
                                 self.n, self.nseg.ctypes.data, n[0:].ctypes.data, n[1:].ctypes.data),
              t.ctx)
        return dict(_records(self.tracks), hits=self.hits, counts=n, segments=self.nseg)


def _records(tracks):
    """The whole and the fitted values of track records."""
    return dict(tracks=tracks.view(np.int32).reshape(len(tracks), -1)[:, :10],
                fit=tracks.view(np.float64).reshape(len(tracks), -1)[:, 5:])


def _serve_groups(case):
    k, n = case["events"], case["primaries"]
    npp, nce = round(SERVE_MIX[0] * k), max(1, round(SERVE_MIX[2] * k))
    return [("pp", [60] * npp), ("pbpb", [min(2000, n)] * (k - npp - nce)), ("pbpb", [n] * nce)]


def prepare(case, seed):
    kind = case["kind"]
    if kind == "serve":
        reqs, cap = [], 0
        for gi, (shape, mult) in enumerate(_serve_groups(case)):
            if not mult:
                continue
            offs, cl = _clusters(shape, mult, seed * 4 + gi)
            host = [c.cpu() for c in cl]
            for e in range(len(mult)):
                part = [h[offs[e]:offs[e + 1]] for h in host]
                # large events arrive in pinned memory, small ones as numpy arrays
                part = [_pinned(c) for c in part] if len(part[0]) >= 100_000 else [c.numpy().copy() for c in part]
                cap = max(cap, len(part[0]))
                reqs.append(part)
        # an even mix over the burst
        order = sorted(range(len(reqs)), key=lambda i: (i * 0.6180339887498949) % 1.0)
        reqs = [Request(0.0, *reqs[i]) for i in order]
        srv = Server(_geometry("pbpb"), cap_clusters=cap + (1 << 19), tl_block=case["tl_block"],
                     row_batch=case["row_batch"])
        n = sum(r.n for r in reqs)
        return dict(case=case, srv=srv, reqs=reqs, tracks=np.zeros(_max_tracks(n), TRACK_DTYPE),
                    hits=np.zeros(n, np.int32))
    mult = _multiplicities(case)
    if case["api"] == "flight":
        slots = []
        for e, m in enumerate(mult):
            slots.append(_Slot(case, *_clusters(case["shape"], [m], seed * 64 + e)))
        return dict(case=case, slots=slots)
    offs, cl = _clusters(case["shape"], mult, seed)
    slot = _Slot(case, offs, cl)
    state = dict(case=case, slots=[slot])
    if kind in ("merge", "calib"):
        slot.track()
        slot.trk.synchronize()
    if kind == "calib":
        state.update(raw=cl[3].clone(), z=cl[3].clone(), sector=cl[0],
                     hist=torch.zeros((2, 4000), dtype=torch.int32, device="cuda"),
                     out=torch.zeros(4, dtype=torch.float64, device="cuda"))
    return state


def run(state):
    kind = state["case"]["kind"]
    if kind == "serve":
        stats = state["srv"].run(state["reqs"], collect=True)
        # every request's tracks, in the order of the requests
        nt = nh = 0
        counts = np.zeros((len(stats.results), 2), np.int64)
        for i, (t, h) in enumerate(stats.results):
            counts[i] = len(t), len(h)
            state["tracks"][nt:nt + len(t)] = t
            state["hits"][nh:nh + len(h)] = h
            nt, nh = nt + len(t), nh + len(h)
        return dict(_records(state["tracks"]), hits=state["hits"], counts=counts)
    slots = state["slots"]
    trk = slots[0].trk
    if kind == "calib":
        with torch.cuda.stream(trk.stream):
            state["z"].copy_(state["raw"])
            state["hist"].zero_()
            trk.calib_correct_z(state["sector"], state["z"], DRIFT_EPS)
            trk.calib_accumulate(0, state["hist"])
            calib_fit(state["hist"], state["out"], Z_MAX, DRIFT_EPS, stream=trk.stream)
        return dict(z=state["z"], hist=state["hist"], fit=state["out"])
    if kind in ("merge", "chain"):
        if kind == "chain":
            slots[0].track()
        trk.merge(0)
        return slots[0].merged()
    for s in slots:
        s.track()
    out = [s.results() for s in slots]
    return out[0] if len(out) == 1 else out


def work(case):
    """Clusters in (10 bytes each), track records and hit IDs out; the least
    filter steps: each track hit filtered out- and inward and refitted three
    times, about 220 operations a step."""
    if case["kind"] == "serve":
        n = sum(_n_clusters(shape, m) for shape, mult in _serve_groups(case) for m in mult)
    else:
        n = sum(_n_clusters(case["shape"], m) for m in _multiplicities(case))
    hits = 0.85 * n
    tracks = n / 78.0
    if case["kind"] == "calib":
        # z in and out, the side of each cluster; one transport to the axis a track
        return dict(bytes=9.0 * n + 72.0 * tracks + 32000.0, flops=4.0 * n + 50 * 40.0 * tracks)
    out = 4.0 * hits + 216.0 * tracks
    if case["kind"] == "merge":
        # tracks and their clusters in, merged tracks out; one outward pass, three inward
        return dict(bytes=2.0 * out + 9.0 * hits, flops=4 * 220.0 * hits)
    steps = 5 if case["kind"] != "chain" else 9
    return dict(bytes=10.0 * n + out, flops=steps * 220.0 * hits)


def exact(case, seed):
    """The corrected z of the calibration in 64 bits; tracks have no value
    without the tracker's own decisions."""
    if case["kind"] != "calib":
        return None
    _, cl = _clusters(case["shape"], _multiplicities(case), seed)
    side = torch.where(cl[0] < 18, 1.0, -1.0).to(torch.float64)
    z = (cl[3].to(torch.float64) + side * DRIFT_EPS * Z_MAX) / (1.0 + DRIFT_EPS)
    return dict(z=z, hist=None, fit=None)
