"""What making a context and reading its first results may not disturb: a
stream capture in progress, in the same thread or in another one."""
import ctypes
import os
import subprocess
import sys
import threading

import numpy as np
import pytest

import tpcgen
from paper_1712_09416_amd import _lib

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

COUNTER = r"""
int calls;
int hipHostMalloc(void **p, unsigned long n, unsigned f) { ++calls; return 2; }
int hipMalloc(void **p, unsigned long n) { ++calls; return 2; }
int hipHostFree(void *p) { ++calls; return 0; }
int hipGetLastError(void) { ++calls; return 0; }
"""
MAKE = r"""
import ctypes, sys
stub = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)          # before the HIP runtime
from paper_1712_09416_amd import _lib
from paper_1712_09416_amd.tracker import default_params, make_geometry
import tpcgen
L = _lib.load()
p = default_params(max_clusters=1 << 10)
need = L.tpc_workspace_bytes(ctypes.byref(p))
ctx, g = ctypes.c_void_p(), make_geometry(tpcgen.geometry.geometry_dict())
before = ctypes.c_int.in_dll(stub, "calls").value
assert L.tpc_init_geometry(ctypes.byref(ctx), ctypes.byref(g), ctypes.byref(p), 0x100000, need, None) == 0
print("calls", ctypes.c_int.in_dll(stub, "calls").value - before)
"""


def test_making_a_context_allocates_nothing(tmp_path):
    """tpc_init_geometry allocates no memory through HIP: the runtime's
    allocation calls, replaced by counting ones, stay at zero."""
    src, lib = tmp_path / "stub.c", tmp_path / "stub.so"
    src.write_text(COUNTER)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(lib), str(src)], check=True)
    r = subprocess.run([sys.executable, "-c", MAKE, str(lib)], cwd=ROOT, capture_output=True, text=True,
                       timeout=300, env=dict(os.environ, PYTHONPATH=ROOT))
    assert r.returncode == 0, r.stderr
    assert r.stdout.split()[-2:] == ["calls", "0"], r.stdout


def _beside_capture(work, mode, other):
    """`work` run while a stream is captured, by the capturing thread or by
    another one; its result, after the captured graph was replayed."""
    torch = pytest.importorskip("torch")
    x = torch.zeros(8, device="cuda:0")
    g = torch.cuda.CUDAGraph()
    got = []
    with torch.cuda.graph(g, stream=torch.cuda.Stream(), capture_error_mode=mode):
        x.add_(1)
        if other:
            t = threading.Thread(target=lambda: got.append(work()))
            t.start()
            t.join(20)
        else:
            got.append(work())
        x.add_(1)
    for k in range(1, 4):
        g.replay()
        torch.cuda.synchronize()
        assert x.tolist() == [2.0 * k] * 8
    return got[0]


@pytest.mark.gpu
@pytest.mark.parametrize("mode", ["global", "thread_local"])
@pytest.mark.parametrize("other", [False, True])
def test_context_made_beside_a_capture(mode, other):
    torch = pytest.importorskip("torch")
    from paper_1712_09416_amd.tracker import default_params, make_geometry
    L = _lib.load()
    p = default_params(max_clusters=1 << 10)
    need = L.tpc_workspace_bytes(ctypes.byref(p))
    ws, st = torch.empty(need, dtype=torch.uint8, device="cuda:0"), torch.cuda.Stream()
    geo, ctx = make_geometry(tpcgen.geometry.geometry_dict()), ctypes.c_void_p()
    rc = _beside_capture(lambda: L.tpc_init_geometry(ctypes.byref(ctx), ctypes.byref(geo), ctypes.byref(p),
                                                     ws.data_ptr(), need, st.cuda_stream), mode, other)
    assert rc == _lib.TPC_OK
    assert L.tpc_destroy(ctx) == _lib.TPC_OK


@pytest.mark.gpu
def test_first_results_read_beside_another_threads_capture():
    torch = pytest.importorskip("torch")
    from paper_1712_09416_amd import Tracker
    ev = tpcgen.tiny_event(7, n_tracks=4)
    ins = [torch.from_numpy(a).to("cuda:0") for a in (ev.sector, ev.row, ev.y, ev.z)]
    trk, again = (Tracker(ev.geometry(), max_clusters=1 << 12) for _ in range(2))
    for t in (trk, again):
        t.load(0, *ins)
        t.track_event(0)
        t.synchronize()

    def read_and_close():
        out = trk.get_tracks(0)
        trk.close()
        return out

    tracks, hits = _beside_capture(read_and_close, "thread_local", True)
    want_tracks, want_hits = again.get_tracks(0)
    again.close()
    assert len(tracks) >= 1 and np.array_equal(hits, want_hits)
    assert tracks.tobytes() == want_tracks.tobytes()


@pytest.mark.gpu
def test_destroying_a_context_waits_for_its_own_stream_only():
    """Trackers read and closed while another stream works: that work is still
    running afterwards; results read into blocks left by closed contexts are
    the same, by several threads at once too."""
    torch = pytest.importorskip("torch")
    from paper_1712_09416_amd import Tracker
    ev = tpcgen.tiny_event(7, n_tracks=4)
    ins = [torch.from_numpy(a).to("cuda:0") for a in (ev.sector, ev.row, ev.y, ev.z)]

    def one():
        trk = Tracker(ev.geometry(), max_clusters=1 << 12)
        trk.load(0, *ins)
        trk.track_event(0)
        tracks, hits = trk.get_tracks(0)
        trk.close()
        return tracks.tobytes() + hits.tobytes()

    want = one()
    other, done = torch.cuda.Stream(), torch.cuda.Event()
    torch.cuda.synchronize()
    with torch.cuda.stream(other):
        torch.cuda._sleep(400_000_000)              # some 170 ms
        done.record()
    assert one() == want
    assert not done.query()
    torch.cuda.synchronize()
    got = []
    threads = [threading.Thread(target=lambda: got.extend(one() for _ in range(8))) for _ in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    assert got == [want] * 32
