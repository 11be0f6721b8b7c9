"""The library's own choice of tiles, as far as the host decides it (no GPU: the
pointers are never used).  Each check runs in a process of its own without
devices; KM_FAULT_INJECT=launch makes a call that reaches its launch return
KM_E_HIP."""
import json
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
def tables(nz, n, grid=None):
    # (migrate, demigrate) through one-way time tables of 2 rows, on a node grid or invariant
    t, g, tt, w = args(n=n, nz=nz, n_t=500)
    if grid:
        tab = _lib.KmLtable(n_gx=1, n_gy=1, gx0=0.0, gy0=0.0, gdx=1.0, gdy=1.0, n_h=2, dh=10.0, t=p, r2=p)
        names = lib.kirchhoff_migrate_ltable, lib.kirchhoff_demigrate_ltable
    else:
        tab = _lib.KmTtable(n_h=2, dh=10.0, t=p, r2=p)
        names = lib.kirchhoff_migrate_table, lib.kirchhoff_demigrate_table
    G, T, X = ctypes.byref(g), ctypes.byref(tab), ctypes.byref(t)
    return names[0](X, G, T, p, 0, -1, None), names[1](p, G, T, X, 0, -1, None)
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


DEEP = "deep = dict(n_t=500, nz=5000000)\n"  # tile 8 holds 64 depths: more chunks than a launch has


def entry(tile, size=None, op=0, ntb=1, nzb=39063):
    e = dict(arch="unknown", op=op, dtype=0, kind=0, precision=0, nz_bucket=nzb, nt_bucket=ntb, tile=tile, ms=1.0)
    return e if size is None else dict(e, size_bucket=size)


def cache(tmp_path, version, *entries):
    path = tmp_path / "tune.json"
    path.write_text(json.dumps({"format": "km_tune_cache", "version": version, "entries": list(entries)}))
    return path


def test_tuned_tile_is_for_its_size(tmp_path):
    # a tile tuned on 2 columns x 1 bin (size bucket 1) is taken there and not on 16 columns
    path = cache(tmp_path, 2, entry(8, 1))
    run(DEEP + """
assert migrate(nx=2, **deep) == _lib.KM_E_UNSUPPORTED and said("depth chunks")
assert migrate(nx=16, **deep) == _lib.KM_E_HIP and said("injected")
assert migrate(nx=2, bins=8, **deep) == _lib.KM_E_HIP and said("injected")
assert lib.km_tune_lookup(0, 0, 0, 0, 5000000, 500) == 8
""", KM_TUNE_CACHE=path)
    # the adjoint's size is its traces: a tile of no shape that holds 65535 x 64 depths at 4 traces only
    path = cache(tmp_path, 2, entry(3, 2, op=1))
    run(DEEP + """
assert demigrate(n=4, **deep) == _lib.KM_E_UNSUPPORTED and said("depth chunks")
assert lib.km_tune_record(1, 0, 0, 0, 5000000, 500, 0, 1.0) == _lib.KM_OK  # every size, in its place
assert demigrate(n=4, **deep) == _lib.KM_E_HIP and demigrate(n=400, **deep) == _lib.KM_E_HIP
""", KM_TUNE_CACHE=path)
    assert [(e["tile"], e["size_bucket"]) for e in json.loads(path.read_text())["entries"]] == [(0, -1)]


def test_tuned_tile_without_a_size_is_for_its_class(tmp_path):
    # a file of version 1, and beside it a tile of one size
    path = cache(tmp_path, 1, entry(8))
    run(DEEP + """
for nx in (2, 16, 300): assert migrate(nx=nx, **deep) == _lib.KM_E_UNSUPPORTED and said("depth chunks")
""", KM_TUNE_CACHE=path)
    path = cache(tmp_path, 2, entry(8, -1), entry(2, 4))
    run(DEEP + """
assert migrate(nx=2, **deep) == _lib.KM_E_UNSUPPORTED and said("depth chunks")
assert migrate(nx=16, **deep) == _lib.KM_E_HIP and said("injected")
assert lib.km_tune_lookup(0, 0, 0, 0, 5000000, 500) == 2  # recorded last
""", KM_TUNE_CACHE=path)


def test_deep_tables_keep_their_chunks():
    # 65535 chunks of 128 depths (migrate: 256 with lateral tables) whatever the number of traces
    run("""
for n in (4, 1500, 5000, 20000, 30000):
    assert tables(8300000, n) == (_lib.KM_E_HIP, _lib.KM_E_HIP), n
    assert tables(8300000, n, grid=True) == (_lib.KM_E_HIP, _lib.KM_E_HIP), n
    assert tables(9000000, n) == (_lib.KM_E_UNSUPPORTED, _lib.KM_E_UNSUPPORTED), n
    assert tables(16700000, n, grid=True) == (_lib.KM_E_HIP, _lib.KM_E_UNSUPPORTED), n
    assert tables(16800000, n, grid=True) == (_lib.KM_E_UNSUPPORTED, _lib.KM_E_UNSUPPORTED), n
""")
