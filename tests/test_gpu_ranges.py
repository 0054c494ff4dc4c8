"""Sizes at which the kernels change their split of the work, against the
oracle.  Tolerance: none; links, tracks and fits are the oracle's bits (the
same operations in the same precision and order, so no split may change them).
"""
import types

import numpy as np
import pytest

import tpcgen
from test_gpu_parity import ORACLE_THREADS, compare_links, compare_tracks, dev, gpu_run, merge_case  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GEO = tpcgen.geometry.geometry_dict(tpcgen.geometry.SIGMA_PBPB)


def event(name, sector, row, y, z):
    return types.SimpleNamespace(name=name, n=len(y), sector=np.asarray(sector, np.uint8),
                                 row=np.asarray(row, np.uint8), y=np.asarray(y, np.float32),
                                 z=np.asarray(z, np.float32), geometry=lambda: GEO)


def oracle_run(oracle_lib, ev):
    return oracle_lib.run(ev.sector, ev.row, ev.y, ev.z, GEO, precision=32, nthreads=ORACLE_THREADS)


def chains(n, rows=12):
    """n origin-pointing chains of `rows` hits each, far apart, on the pad rows
    in groups of `rows` with an empty row between: n start hits."""
    per = 156 // (rows + 1)                       # groups of a sector
    cells = 36 * per
    ny = 8 if n > 4 * 10 * cells else 4
    k = np.arange(n)
    cell, slot = k % cells, k // cells
    sector, group = cell % 36, cell // 36
    ty = ((slot % ny) + 0.5) / ny * 0.3 - 0.15    # y / x
    tz = ((slot // ny) + 0.5) / 20 * 0.9          # |z| / x
    side = np.where(sector < 18, 1.0, -1.0)
    x = tpcgen.geometry.row_x().astype(np.float64)
    r = (group * (rows + 1))[:, None] + np.arange(rows)
    rng = np.random.default_rng(n)
    y = ty[:, None] * x[r] + rng.normal(size=r.shape) * 0.03
    z = (tz * side)[:, None] * x[r] + rng.normal(size=r.shape) * 0.03
    order = rng.permutation(r.size)
    return event(f"{n} chains", np.repeat(sector, rows)[order], r.ravel()[order], y.ravel()[order],
                 z.ravel()[order])


# a wave a tracklet; two; groups of 32 and of 16 lanes, of 8 and a lane each;
# the selection's two ways
@pytest.mark.parametrize("n", [1, 2047, 2049, 4096, 4097, 16384, 16385, 65536, 65537])
def test_tracklet_counts(dev, oracle_lib, n):  # noqa: F811
    ev = chains(n)
    tracks, hits, lk = gpu_run(ev, dev)
    assert np.count_nonzero((lk["upc"] >= 0) & (lk["dnc"] < 0)) == n
    ref = oracle_run(oracle_lib, ev)
    compare_links(lk, ref)
    compare_tracks(tracks, hits, ref)


# the merger's outer fits and positions: a tile of tracks and one either side
@pytest.mark.parametrize("n", [1, 1023, 1024, 1025])
def test_merged_track_counts(dev, oracle_lib, n):  # noqa: F811
    from paper_1712_09416_amd import Tracker
    ev = chains(n)
    trk = Tracker(GEO, max_clusters=max(ev.n, 4096))
    trk.load(0, *[torch.from_numpy(a).to(dev) for a in (ev.sector, ev.row, ev.y, ev.z)])
    trk.track_event(0)
    assert len(trk.get_tracks(0)[0]) > 0
    trk.merge(0)
    merge_case(trk, 0, 0, ev, oracle_lib, geometry=GEO)
    trk.close()


# rows at the row sort's and the group search's limits, spread over the sector
# or so dense that a hit has more neighbours than a list holds
@pytest.mark.parametrize("dense", [False, True])
def test_row_sizes(dev, oracle_lib, dense):  # noqa: F811
    counts = [1, 15, 16, 17, 128, 129, 255, 256, 257, 0, 300, 1023, 1024, 1025, 900, 4096, 4095, 4096]
    rng = np.random.default_rng(5)
    row = np.concatenate([np.full(c, 20 + i) for i, c in enumerate(counts)])
    x = tpcgen.geometry.row_x().astype(np.float64)[row]
    n = len(row)
    if dense:
        y, z = rng.uniform(-0.05, 0.05, n) * x, rng.uniform(0.5, 0.7, n) * x
    else:
        y, z = rng.uniform(-0.17, 0.17, n) * x, rng.uniform(0.0, 2.0, n) * x
    order = rng.permutation(n)
    ev = event("rows", np.full(n, 7), row[order], y[order], z[order])
    tracks, hits, lk = gpu_run(ev, dev)
    ref = oracle_run(oracle_lib, ev)
    compare_links(lk, ref)
    compare_tracks(tracks, hits, ref)


# events that end at, before and after a tile of the output order, empty ones,
# and as many as go by argument and one more
@pytest.mark.parametrize("n_events", [7, 128, 129])
def test_event_sizes(dev, oracle_lib, n_events):  # noqa: F811
    from paper_1712_09416_amd import Tracker
    sizes = [1024, 0, 1023, 1025, 1, 2048, 3000]
    sizes += [13 * (e % 3) for e in range(n_events - len(sizes))]
    evs = []
    for e, n in enumerate(sizes):
        c = chains(-(-n // 12) or 1)
        evs.append(event(f"event {e}", c.sector[:n], c.row[:n], c.y[:n], c.z[:n]))
    offs = np.concatenate([[0], np.cumsum(sizes)])
    cat = [np.concatenate([getattr(ev, k) for ev in evs]) for k in ("sector", "row", "y", "z")]
    trk = Tracker(GEO, max_events=n_events, max_clusters=int(offs[-1]))
    trk.load_batch(0, offs, *[torch.from_numpy(a).to(dev) for a in cat])
    trk.track_event(0)
    got = trk.get_slot_tracks(0)
    trk.close()
    for ev, (tracks, hits) in zip(evs, got):
        compare_tracks(tracks, hits, oracle_run(oracle_lib, ev))


# so many clusters that the kernels for few tracklets are left out, but few
# tracklets: every second row full, which no chain can follow
def test_many_clusters_few_tracklets(dev, oracle_lib):  # noqa: F811
    c = chains(100)
    per = -(-(32 * 16384 * 5 + 1) // (36 * 78))
    assert per <= 4096 - 200
    rng = np.random.default_rng(6)
    sector = np.repeat(np.arange(36), 78 * per)
    row = np.tile(np.repeat(2 * np.arange(78) + 1, per), 36)
    x = tpcgen.geometry.row_x().astype(np.float64)[row]
    y = rng.uniform(-0.17, 0.17, len(row)) * x
    z = rng.uniform(0.0, 240.0, len(row)) * np.where(sector < 18, 1.0, -1.0)
    ev = event("alternate rows", np.concatenate([c.sector, sector]), np.concatenate([c.row, row]),
               np.concatenate([c.y, y]), np.concatenate([c.z, z]))
    tracks, hits, lk = gpu_run(ev, dev)
    assert np.count_nonzero((lk["upc"] >= 0) & (lk["dnc"] < 0)) <= 16384
    ref = oracle_run(oracle_lib, ev)
    compare_links(lk, ref)
    compare_tracks(tracks, hits, ref)


# candidates of a hit in the rows above and below, around what its list holds
# (47): both rows listed; the down row paired as it is read; neither listed
@pytest.mark.parametrize("nu,nd", [(46, 1), (24, 23), (24, 24), (47, 1), (48, 1), (1, 46), (1, 47), (60, 60)])
def test_neighbour_list_limits(dev, oracle_lib, nu, nd):  # noqa: F811
    rng = np.random.default_rng(100 * nu + nd)
    x = tpcgen.geometry.row_x().astype(np.float64)
    cols = []
    for sector in (2, 30):
        for r in (1, 40, 63, 100, 150, 157):      # the middle row of three
            side = 1.0 if sector < 18 else -1.0
            for row, n in ((r - 1, nd), (r, 3), (r + 1, nu)):
                # inside the window of every middle hit: 3 cm around the line
                # from the origin
                cols.append((np.full(n, sector), np.full(n, row), 0.05 * x[row] + rng.uniform(-1.2, 1.2, n),
                             side * (0.6 * x[row] + rng.uniform(-1.2, 1.2, n))))
    sector, row, y, z = [np.concatenate(c) for c in zip(*cols)]
    order = rng.permutation(len(row))
    ev = event(f"{nu} up, {nd} down", sector[order], row[order], y[order], z[order])
    _, _, lk = gpu_run(ev, dev)
    ref = oracle_run(oracle_lib, ev)
    compare_links(lk, ref)
    assert np.count_nonzero(lk["up"] >= 0) >= 12


# groups of 64, 32, 16 and 8 lanes and a lane each, at the counts where the
# next one takes over: three events of short chains (rows short on average,
# 2048 waves), one of longer ones (rows of 17 hits or more, 1408 waves)
@pytest.mark.parametrize("events,rows,n", [(3, 12, 2048), (3, 12, 2049), (3, 12, 4096), (3, 12, 4097),
                                           (3, 12, 8192), (3, 12, 8193), (3, 12, 16384), (3, 12, 16385),
                                           (1, 100, 1408), (1, 100, 1409), (1, 40, 2816), (1, 40, 2817),
                                           (1, 20, 5632), (1, 20, 5633), (1, 12, 11264), (1, 12, 11265)])
def test_lane_group_counts(dev, oracle_lib, events, rows, n):  # noqa: F811
    from paper_1712_09416_amd import Tracker
    evs = [chains((n + e) // events, rows) for e in range(events)]
    offs = np.concatenate([[0], np.cumsum([ev.n for ev in evs])])
    assert (offs[-1] // (events * 36 * 159) <= 16) == (events == 3)
    cat = [np.concatenate([getattr(ev, k) for ev in evs]) for k in ("sector", "row", "y", "z")]
    trk = Tracker(GEO, max_events=events, max_clusters=int(offs[-1]))
    trk.set_profiling(True)
    trk.load_batch(0, offs, *[torch.from_numpy(a).to(dev) for a in cat])
    trk.track_event(0)
    got = trk.get_slot_tracks(0)
    assert trk.profile()[1]["tracklets"] == n
    trk.close()
    for ev, (tracks, hits) in zip(evs, got):
        compare_tracks(tracks, hits, oracle_run(oracle_lib, ev))
