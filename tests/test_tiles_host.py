"""The library's own choice of tiles, as far as the host decides it (no GPU: the
pointers are never used).  Each check runs in a process of its own without
devices; KM_FAULT_INJECT=launch makes a call that reaches its launch return
KM_E_HIP."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SETUP = f"""
import ctypes, sys
sys.path.insert(0, {ROOT!r})
from paper_1204_1225_amd import _lib
lib = _lib.load()
p = ctypes.c_void_p(0x1000)
def args(n=4, n_t=10, nx=2, ny=1, nz=3, bins=1, prec=0):
    t = _lib.KmTraces(n_traces=n, n_samples=n_t, dtype=0, trace_stride=n_t, t_first=0.0, dt=0.004, data=p, scale=None,
                      src=p, rec=p, bin=p)
    g = _lib.KmGrid(nx=nx, ny=ny, nz=nz, n_bins=bins, x=p, y=p)
    return t, g, _lib.KmTraveltime(t0sq=p, s2=p, r2=p, time_precision=prec), _lib.KmWeight(kind=1)
def migrate(tile=-1, **kw):
    t, g, tt, w = args(**kw)
    return lib.kirchhoff_migrate(ctypes.byref(t), ctypes.byref(g), ctypes.byref(tt), ctypes.byref(w), p, 0, tile, None)
def demigrate(tile=-1, **kw):
    t, g, tt, w = args(**kw)
    return lib.kirchhoff_demigrate(p, ctypes.byref(g), ctypes.byref(tt), ctypes.byref(w), ctypes.byref(t), 0, tile, None)
def static_batch(tile=-1, **kw):
    t, g, tt, w = args(**kw)
    pr = (_lib.KmProblem * 1)(_lib.KmProblem(traces=t, grid=g, tt=tt, weight=w, image=p))
    return lib.km_batch_migrate_static(pr, 1, tile, None)
def said(text): return text in lib.km_last_error().decode()
"""


def run(body, **env):
    e = dict(os.environ, HIP_VISIBLE_DEVICES="", KM_FAULT_INJECT="launch", **{k: str(v) for k, v in env.items()})
    e.setdefault("KM_TUNE_CACHE", "")
    r = subprocess.run([sys.executable, "-c", SETUP + body], env=e, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


def test_tuned_tile_gives_way_where_its_items_do_not_fit():
    # 1 048 576 work items with tile 8, 131 072 with the default; room for about 460 000.  The
    # static batch goes on to ask for its device (there is none).
    run("""
big = dict(n_t=500, nx=4096, ny=256, nz=1000)
assert lib.km_tune_record(0, 0, 0, 0, 1000, 500, 8, 1.0) == _lib.KM_OK
assert static_batch(8, **big) == _lib.KM_E_UNSUPPORTED and said("work items")  # asked for: refused
assert static_batch(-1, **big) == _lib.KM_E_HIP, lib.km_last_error()
""")
