"""The library on the stand-in device of tests/native/host_device.cpp, in a
process of its own (run by tests/test_host_launch.py as
`host_launch.py <stand-in> <check>`): set-up, tuning and launches run on host
memory, no kernel runs and no result is computed."""
import ctypes
import importlib
import os
import sys

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
DEV = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)     # before the library: its runtime calls go here
_lib = importlib.import_module("paper_2412_17543_amd._lib")
LIB = _lib.load()


def best(**grids):
    for part, grid in grids.items():
        DEV.host_device_best_grid(part.encode(), ctypes.c_long(grid))


def grid(part):
    DEV.host_device_last_grid.restype = ctypes.c_long
    return DEV.host_device_last_grid(part.encode())


def partition(nx, cells):
    c = (np.arange(nx) * cells) // nx
    return (c[None, None, :] + cells * (c[None, :, None] + cells * c[:, None, None])).ravel().astype(np.int32)


def setup(nx, cells, **opts):
    e2s, coef = partition(nx, cells), np.ones(nx ** 3)
    o = _lib.Opts()
    LIB.bddc_default_opts(ctypes.byref(o))
    for k, v in opts.items():
        if k == "product_cfg":
            o.product_cfg[:] = v
        else:
            setattr(o, k, v)
    mesh = _lib.Mesh(nx, nx, nx, 1.0 / nx, None, None)
    part = _lib.Partition(cells ** 3, e2s.ctypes.data, 0, None)
    ctx = ctypes.c_void_p()
    _lib.check(LIB.bddc_setup(ctypes.byref(mesh), ctypes.byref(part), coef.ctypes.data, ctypes.byref(o), None,
                              ctypes.byref(ctx)))
    return ctx


def tuning(ctx):
    a = (ctypes.c_double * 14)()
    _lib.check(LIB.bddc_tuning(ctx, a))
    return [int(v) for v in a[:5]], [int(v) for v in a[7:12]]


def sizes(ctx):
    a = (ctypes.c_int64 * 16)()
    _lib.check(LIB.bddc_info(ctx, a))
    return int(a[0]), int(a[1])


def apply(ctx):
    """One A p and one M^{-1} r: the grids of their products."""
    n = sizes(ctx)[1]
    x, y = np.zeros(n), np.zeros(n)
    DEV.host_device_forget()
    _lib.check(LIB.bddc_apply_schur(ctx, x.ctypes.data, y.ctypes.data))
    _lib.check(LIB.bddc_apply_precond(ctx, x.ctypes.data, y.ctypes.data))
    return grid("OpSchur"), grid("OpNeumann")


def check_pinned(schur, neumann):
    """Whatever the tuner picks can be read back and pinned, at set-up and later."""
    best(OpSchur=schur, OpNeumann=neumann)
    a = setup(16, 2)
    s, n = tuning(a)
    print("tuned", s, n, flush=True)
    assert apply(a) == (s[0], n[0])
    cfg = s[1:] + n[1:]
    b = setup(16, 2, product_cfg=cfg)
    assert tuning(b) == (s, n) and apply(b) == (s[0], n[0])
    _lib.check(LIB.bddc_set_launch(b, 2, (ctypes.c_int32 * 8)(*([-1] * 8))))
    assert tuning(b) != (s, n)
    _lib.check(LIB.bddc_set_launch(b, 2, (ctypes.c_int32 * 8)(*cfg)))
    assert tuning(b) == (s, n) and apply(b) == (s[0], n[0])
    LIB.bddc_destroy(a)
    LIB.bddc_destroy(b)


def check_interior(schur, interior):
    """Small interfaces: the interior product gets the split that is best for
    it, whatever is best for the Schur product and its sums."""
    got = []
    for best_schur in (schur, interior):
        best(OpSchur=best_schur, OpInterior=interior)
        c = setup(16, 2)
        n_nodes, n_gamma = sizes(c)
        F, b = np.zeros(n_nodes), np.zeros(n_gamma)
        DEV.host_device_forget()
        _lib.check(LIB.bddc_condense(c, F.ctypes.data, b.ctypes.data))
        got.append(grid("OpInterior"))
        LIB.bddc_destroy(c)
    print("interior blocks", got, flush=True)
    assert got[0] == got[1] and abs(got[0] - interior) <= interior // 8


def check_refused(*cfg):
    """A refused launch configuration changes nothing, whichever product it is
    refused for (the products' buffers are sized together)."""
    good, ref = [4, 1, 8, 4], [1, 4, 4, 4]
    for bad in (list(cfg) + good, good + list(cfg)):
        c = setup(16, 2, autotune=0, product_cfg=ref * 2)
        was = tuning(c), apply(c)
        assert LIB.bddc_set_launch(c, 2, (ctypes.c_int32 * 8)(*bad)) == -1
        assert (tuning(c), apply(c)) == was, bad
        LIB.bddc_destroy(c)


def check_failed(*cfg):
    """A launch configuration that finds no memory, at whichever allocation,
    leaves the one before in place; the same call later takes it."""
    for fn in ("host_device_live", "host_device_bad"):
        getattr(DEV, fn).restype = ctypes.c_long
    cfg8 = (ctypes.c_int32 * 8)(*(cfg + cfg))
    want = setup(16, 2, autotune=0, product_cfg=cfg + cfg)
    ref = tuning(want), apply(want)
    failures = 0
    while True:
        c = setup(16, 2, autotune=0, product_cfg=[1, 4, 4, 4] * 2)
        was = tuning(c), apply(c)
        DEV.host_device_fail_in(ctypes.c_long(failures))
        rc = LIB.bddc_set_launch(c, 2, cfg8)
        DEV.host_device_fail_in(ctypes.c_long(-1))
        if rc == 0:
            break
        failures += 1
        assert rc == -2, rc
        now = tuning(c), apply(c)
        _lib.check(LIB.bddc_set_launch(c, 2, (ctypes.c_int32 * 8)(*([1, 4, 4, 4] * 2))))
        assert (tuning(c), apply(c)) == was
        _lib.check(LIB.bddc_set_launch(c, 2, cfg8))
        assert (tuning(c), apply(c)) == ref
        assert now == was, (now, was)
        LIB.bddc_destroy(c)
    print("allocations", failures, flush=True)
    assert failures >= 1 and DEV.host_device_bad() == 0
    LIB.bddc_destroy(c)
    LIB.bddc_destroy(want)
    assert DEV.host_device_live() == 0


CHECKS = {"pinned": check_pinned, "interior": check_interior, "refused": check_refused, "failed": check_failed}

if __name__ == "__main__":
    CHECKS[sys.argv[2]](*[int(v) for v in sys.argv[3:]])
    print("ok", flush=True)
