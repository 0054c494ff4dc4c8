"""The filter's short square roots and reciprocals against the general
operations, and events whose covariances leave the range they hold in.
Tolerance: none, all are correctly rounded."""
import ctypes
import os

import numpy as np
import pytest

import tpcgen
from test_gpu_parity import compare_links, compare_tracks, dev, gpu_run  # noqa: F401
from test_gpu_ranges import event

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    from paper_1712_09416_amd import build
    if not os.path.exists(build.TEST_LIB):
        build.build_tests()
    return ctypes.CDLL(build.TEST_LIB)


def ptr(t):
    return ctypes.c_void_p(t.data_ptr())


def test_floats_in_the_whole_middle_range(dev, lib):  # noqa: F811
    """Every float in [2^-100, 2^100]."""
    lo, hi = (int(np.float32(x).view(np.uint32)) for x in (2.0 ** -100, 2.0 ** 100))
    bad = torch.zeros(5, dtype=torch.int64, device=dev)
    example = torch.zeros(5, dtype=torch.int32, device=dev)
    assert lib.roots_floats(ctypes.c_uint32(lo), ctypes.c_uint32(hi - lo + 1), ptr(bad), ptr(example),
                            None) == 0
    torch.cuda.synchronize()
    seen = dict(zip(("root", "reciprocal", "root in double", "reciprocal in double", "determinant"),
                    zip(bad.tolist(), [hex(e & 0xFFFFFFFF) for e in example.tolist()])))
    assert all(n == 0 for n, _ in seen.values()), seen


def test_determinants_outside_the_middle_range(dev, lib):  # noqa: F811
    """Zero, denormal, smallest and largest numbers, infinities and NaN take
    the general division."""
    e = np.concatenate([np.arange(0, 0x0D800000, 4099), np.arange(0x71800000, 0x7F800001, 4099),
                        [0, 1, 0x007FFFFF, 0x00800000, 0x0D7FFFFF, 0x0D800000, 0x71800000, 0x71800001,
                         0x7F7FFFFF, 0x7F800000, 0x7FC00000]]).astype(np.uint32)
    x = np.concatenate([e, e | np.uint32(0x80000000)]).view(np.float32)
    out = torch.empty(len(x), dtype=torch.float32, device=dev)
    assert lib.roots_dets(ptr(torch.from_numpy(x).to(dev)), ptr(out), ctypes.c_int64(len(x)), None) == 0
    with np.errstate(all="ignore"):
        want = np.float32(1.0) / x
    assert np.array_equal(out.cpu().numpy(), want, equal_nan=True)


def test_doubles(dev, lib):  # noqa: F811
    """Random mantissas and those next to the powers of two, the last ones
    before the next power among them, over the exponents the fits meet."""
    rng = np.random.default_rng(3)
    mant = np.concatenate([rng.integers(0, 1 << 52, 1 << 13), np.arange(64), (1 << 52) - 1 - np.arange(64),
                           (1 << 51) + np.arange(-32, 32)]).astype(np.uint64)
    exp = np.arange(1023 - 300, 1023 + 301).astype(np.uint64)
    x = ((exp[:, None] << np.uint64(52)) | mant[None, :]).ravel().view(np.float64)
    d = torch.from_numpy(x).to(dev)
    root, rcp = torch.empty_like(d), torch.empty_like(d)
    assert lib.roots_doubles(ptr(d), ptr(root), ptr(rcp), ctypes.c_int64(len(x)), None) == 0
    assert np.array_equal(root.cpu().numpy(), np.sqrt(x))
    assert np.array_equal(rcp.cpu().numpy(), 1.0 / x)


# Cluster errors so small that determinants (2^-26 cm), and variances too
# (2^-52), leave the middle range: straight tracks on rows and slopes that
# floats hold exactly, with rows left out so that windows are searched; prior
# variances of the same size (with wide ones the updates would be refused).
@pytest.mark.parametrize("sigma", [2.0 ** -26, 2.0 ** -30, 2.0 ** -52])
@pytest.mark.parametrize("copies", [1, 40])
def test_tiny_cluster_errors(dev, oracle_lib, sigma, copies):  # noqa: F811
    geo = dict(tpcgen.geometry.geometry_dict())
    geo.update(row_x=(64.0 + np.arange(159)).astype(np.float32), sigma_y0=np.float32(sigma),
               sigma_z0=np.float32(sigma), sigma_y1=np.float32(0), sigma_z1=np.float32(0))
    cols = []
    for c in range(copies):
        for sector in (0, 5, 20):
            side = 1.0 if sector < 18 else -1.0
            rows = np.array([r for r in range(159) if r % 23 != 11 + c % 7])
            x = 64.0 + rows
            a, b = ((c % 8) - 4) / 32.0 * (c > 0), side * (c // 8) / 8.0
            cols.append((np.full(len(rows), sector), rows, a * x, b * x))
    sector, row, y, z = [np.concatenate(c) for c in zip(*cols)]
    keep = np.abs(z) < 249.0
    order = np.random.default_rng(1).permutation(np.flatnonzero(keep))
    ev = event("tiny errors", sector[order], row[order], y[order], z[order])
    cuts = dict(c_s0=4.0 * sigma ** 2, c_t0=4.0 * sigma ** 2, c_q0=16.0 * sigma ** 2)
    tracks, hits, lk = gpu_run(ev, dev, geometry=geo, **cuts)
    ref = oracle_lib.run(ev.sector, ev.row, ev.y, ev.z, geo, precision=32, nthreads=4,
                         params=oracle_lib.make_params(**cuts))
    assert np.count_nonzero(ref.upc >= 0) > 100
    if sigma > 2.0 ** -52:
        assert len(ref.tracks) >= 3
    compare_links(lk, ref)
    compare_tracks(tracks, hits, ref)
