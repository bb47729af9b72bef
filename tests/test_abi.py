"""The C-ABI library loads and exports every entry point include/lsrtm.h
declares; host-side argument validation (no GPU needed)."""
import ctypes
import os
import re

import pytest

from paper_2508_10405_amd import lsrtm

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include", "lsrtm.h")


def _declared():
    src = open(HEADER).read()
    return sorted(set(re.findall(r"^\s*(?:lsrtm_status|void|const char\s*\*)\s*(lsrtm_\w+)\s*\(", src, re.M)))


def test_header_declares_the_api():
    names = _declared()
    for n in ("lsrtm_create", "lsrtm_set_model", "lsrtm_set_acquisition", "lsrtm_forward", "lsrtm_born",
              "lsrtm_adjoint", "lsrtm_cgnr", "lsrtm_dot", "lsrtm_destroy", "lsrtm_strerror"):
        assert n in names


def test_library_exports_every_declared_symbol():
    L = lsrtm.lib()
    for name in _declared():
        assert hasattr(L, name), name
        assert name in lsrtm.SIGNATURES, name


def test_create_validates_grid_on_host():
    L = lsrtm.lib()

    def create(**kw):
        g = lsrtm.Grid()
        g.ndim = kw.get("ndim", 2)
        n = kw.get("n", (10, 12, 1))
        for a in range(3):
            g.n[a] = n[a]
            g.h[a] = kw.get("h", 10.0)
        g.npml, g.pml_R, g.pml_f0 = kw.get("npml", 4), kw.get("R", 1e-4), 10.0
        g.nt, g.dt = kw.get("nt", 10), kw.get("dt", 1e-3)
        g.ckpt_every, g.ckpt_dtype = kw.get("ck", 0), kw.get("ckd", 0)
        h = ctypes.c_void_p()
        st = L.lsrtm_create(ctypes.byref(g), None, ctypes.byref(h))
        if st == 0:
            L.lsrtm_destroy(h)
        return st

    assert create() == lsrtm.OK
    assert create(ndim=3, n=(5, 6, 7)) == lsrtm.OK
    assert create(ndim=4) == lsrtm.EINVAL
    assert create(n=(0, 12, 1)) == lsrtm.EINVAL
    assert create(n=(10, 12, 3)) == lsrtm.EINVAL      # 2D needs ny = 1
    assert create(h=-1.0) == lsrtm.EINVAL
    assert create(nt=0) == lsrtm.EINVAL
    assert create(dt=0.0) == lsrtm.EINVAL
    assert create(npml=-1) == lsrtm.EINVAL
    assert create(R=1.5) == lsrtm.EINVAL
    assert create(ckd=3) == lsrtm.EINVAL
    assert L.lsrtm_create(None, None, None) == lsrtm.EINVAL


def test_strerror_and_tiles():
    L = lsrtm.lib()
    assert L.lsrtm_strerror(lsrtm.EUNSTABLE).decode().startswith("CFL")
    assert lsrtm.tile_shape(2, 4) == (64, 8)
    assert lsrtm.tile_shape(2, 1) == (32, 16)
    with pytest.raises(lsrtm.LsrtmError):
        lsrtm.tile_shape(2, 99)


def test_calls_before_setup_report_state():
    L = lsrtm.lib()
    g = lsrtm.Grid()
    g.ndim = 2
    g.n[0], g.n[1], g.n[2] = 10, 12, 1
    g.h[0] = g.h[1] = g.h[2] = 10.0
    g.npml, g.pml_R, g.pml_f0, g.nt, g.dt = 4, 1e-4, 10.0, 10, 1e-3
    h = ctypes.c_void_p()
    assert L.lsrtm_create(ctypes.byref(g), None, ctypes.byref(h)) == 0
    assert L.lsrtm_born(h, ctypes.c_void_p(16), ctypes.c_void_p(16)) == lsrtm.ESTATE
    assert L.lsrtm_set_acquisition(h, 1, None, None, None, None, None) == lsrtm.ESTATE
    step = (ctypes.c_double * 5)()
    assert L.lsrtm_cgnr_step(h, step) == lsrtm.ESTATE          # no CGNR run begun
    assert L.lsrtm_cgnr_step(h, None) == lsrtm.EINVAL
    assert L.lsrtm_set_option(h, 99, 0) == lsrtm.EINVAL
    assert L.lsrtm_set_option(h, lsrtm.OPT_TILE, 42) == lsrtm.EINVAL
    assert L.lsrtm_set_option(h, lsrtm.OPT_REPLAY_CACHE_MB, -1) == lsrtm.EINVAL
    assert L.lsrtm_set_option(h, lsrtm.OPT_REPLAY_CACHE_MB, 512) == lsrtm.OK   # planned with the acquisition
    assert L.lsrtm_set_option(h, lsrtm.OPT_GRAPH_CACHE, -1) == lsrtm.EINVAL
    assert L.lsrtm_set_option(h, lsrtm.OPT_GRAPH_CACHE, 4) == lsrtm.OK
    # counts that would wrap in an int and sizes whose byte count would
    # overflow are argument errors, not silently different plans
    assert L.lsrtm_set_option(h, lsrtm.OPT_SHOTS_PER_LAUNCH, 2 ** 31) == lsrtm.EINVAL
    assert L.lsrtm_set_option(h, lsrtm.OPT_GRAPH_CACHE, 2 ** 32) == lsrtm.EINVAL
    assert L.lsrtm_set_option(h, lsrtm.OPT_MEM_BUDGET_MB, 2 ** 44) == lsrtm.EINVAL
    assert L.lsrtm_set_option(h, lsrtm.OPT_REPLAY_CACHE_MB, 2 ** 44) == lsrtm.EINVAL
    assert L.lsrtm_set_option(h, lsrtm.OPT_MEM_BUDGET_MB, 2 ** 30) == lsrtm.OK
    assert L.lsrtm_set_option(h, lsrtm.OPT_MEM_BUDGET_MB, 0) == lsrtm.OK
    assert L.lsrtm_set_option(h, lsrtm.OPT_SHOTS_PER_LAUNCH, 0) == lsrtm.OK
    # the streaming calibration refuses unsupported mixes and grids that do
    # not match n before it touches the device
    ms = ctypes.c_double()
    buf = ctypes.c_void_p(16)
    assert L.lsrtm_stream_mix(h, buf, 1024, 3, 3, None, ctypes.byref(ms)) == lsrtm.EINVAL
    assert L.lsrtm_stream_mix(h, None, 1024, 10, 6, None, ctypes.byref(ms)) == lsrtm.EINVAL
    assert L.lsrtm_stream_mix(h, buf, 0, 10, 6, None, ctypes.byref(ms)) == lsrtm.EINVAL
    grid = (ctypes.c_int * 4)(40, 8, 4, 32)      # n would be 32 * 8 * 4; nz > ldz
    assert L.lsrtm_stream_mix(h, buf, 1024, 10, 6, grid, ctypes.byref(ms)) == lsrtm.EINVAL
    grid = (ctypes.c_int * 4)(30, 8, 4, 32)
    assert L.lsrtm_stream_mix(h, buf, 1000, 10, 6, grid, ctypes.byref(ms)) == lsrtm.EINVAL
    out = (ctypes.c_longlong * 15)(*([-7] * 15))
    assert L.lsrtm_sizes(h, out, 15) == lsrtm.OK
    # no segment held and no graph before a plan; 14 entries written
    assert out[12] == 0 and out[13] == 0 and out[14] == -7
    L.lsrtm_destroy(h)


def test_every_entry_point_refuses_a_null_context():
    """A NULL context is an invalid argument for every entry point that takes
    one (checked before anything else, also where another argument is bad
    too, such as a negative iteration count); destroy ignores it and
    last_error returns an empty string.  Every other pointer passed here is a
    dummy that must not be touched."""
    L = lsrtm.lib()
    P = ctypes.c_void_p(16)
    dbl = ctypes.c_double()
    dbls = (ctypes.c_double * 16)()
    lls = (ctypes.c_longlong * 16)()
    grid = (ctypes.c_int * 4)(32, 8, 4, 32)
    calls = {
        "set_option": lambda: L.lsrtm_set_option(None, lsrtm.OPT_TILE, 0),
        "set_model": lambda: L.lsrtm_set_model(None, P, P),
        "set_acquisition": lambda: L.lsrtm_set_acquisition(None, 1, P, P, P, P, P),
        "autotune": lambda: L.lsrtm_autotune(None, 4, 0, dbls),
        "sizes": lambda: L.lsrtm_sizes(None, lls, 15),
        "stats": lambda: L.lsrtm_stats(None, dbls, 16),
        "forward": lambda: L.lsrtm_forward(None, P),
        "born": lambda: L.lsrtm_born(None, P, P),
        "adjoint": lambda: L.lsrtm_adjoint(None, P, P, 0),
        "dot": lambda: L.lsrtm_dot(None, P, P, 4, ctypes.byref(dbl)),
        "axpy": lambda: L.lsrtm_axpy(None, 1.0, P, P, 4),
        "stream_mix": lambda: L.lsrtm_stream_mix(None, P, 1024, 10, 6, grid, ctypes.byref(dbl)),
        "cgnr_begin": lambda: L.lsrtm_cgnr_begin(None, P, P),
        "cgnr_iterate": lambda: L.lsrtm_cgnr_iterate(None, P, dbls),
        "cgnr": lambda: L.lsrtm_cgnr(None, P, 1, P, dbls),
        "cgnr negative niter": lambda: L.lsrtm_cgnr(None, P, -1, P, dbls),
        "cgnr_step": lambda: L.lsrtm_cgnr_step(None, dbls),
        "cgnr_state": lambda: L.lsrtm_cgnr_state(None, 1, P, P, P, dbls),
        "pseudo_hessian": lambda: L.lsrtm_pseudo_hessian(None, P, P, 1e-3),
        "set_preconditioner": lambda: L.lsrtm_set_preconditioner(None, P),
        "psf_images": lambda: L.lsrtm_psf_images(None, 4, P),
        "psf_apply": lambda: L.lsrtm_psf_apply(None, P, 4, 0, 0, P, P),
        "psf_cgnr": lambda: L.lsrtm_psf_cgnr(None, P, 4, 0, P, 1, P, dbls),
        "mute": lambda: L.lsrtm_mute(None, P, 1500.0, 0.0, 0),
        "mute_noalloc": lambda: L.lsrtm_mute_noalloc(None, P, 1500.0, 0.0, 0),
        "wiener": lambda: L.lsrtm_wiener(None, P, P, P, 1, 16, 1e-3, P),
    }
    got = {name: call() for name, call in calls.items()}
    assert got == {name: lsrtm.EINVAL for name in calls}
    L.lsrtm_destroy(None)
    assert L.lsrtm_last_error(None) == b""


def test_calls_before_the_model_report_state():
    """On a fresh context (no model, no acquisition) every call that needs
    them returns ESTATE before it touches its (dummy) device pointers, and
    leaves a description in last_error."""
    L = lsrtm.lib()
    g = lsrtm.Grid()
    g.ndim = 2
    g.n[0], g.n[1], g.n[2] = 10, 12, 1
    g.h[0] = g.h[1] = g.h[2] = 10.0
    g.npml, g.pml_R, g.pml_f0, g.nt, g.dt = 4, 1e-4, 10.0, 10, 1e-3
    h = ctypes.c_void_p()
    assert L.lsrtm_create(ctypes.byref(g), None, ctypes.byref(h)) == 0
    P = ctypes.c_void_p(16)
    dbls = (ctypes.c_double * 16)()
    calls = {
        "autotune": lambda: L.lsrtm_autotune(h, 4, 0, dbls),
        "forward": lambda: L.lsrtm_forward(h, P),
        "born": lambda: L.lsrtm_born(h, P, P),
        "adjoint": lambda: L.lsrtm_adjoint(h, P, P, 0),
        "cgnr_begin": lambda: L.lsrtm_cgnr_begin(h, P, P),
        "cgnr_iterate": lambda: L.lsrtm_cgnr_iterate(h, P, dbls),
        "cgnr": lambda: L.lsrtm_cgnr(h, P, 2, P, dbls),
        "cgnr_state": lambda: L.lsrtm_cgnr_state(h, 1, P, P, P, dbls),
        "pseudo_hessian": lambda: L.lsrtm_pseudo_hessian(h, P, P, 1e-3),
        "psf_images": lambda: L.lsrtm_psf_images(h, 4, P),
        "psf_cgnr": lambda: L.lsrtm_psf_cgnr(h, P, 4, 0, P, 1, P, dbls),
        "mute": lambda: L.lsrtm_mute(h, P, 1500.0, 0.0, 0),
        "mute_noalloc": lambda: L.lsrtm_mute_noalloc(h, P, 1500.0, 0.0, 0),
    }
    try:
        for name, call in calls.items():
            assert call() == lsrtm.ESTATE, name
            assert L.lsrtm_last_error(h), name
        # a negative iteration count is refused as an argument error first
        assert L.lsrtm_cgnr(h, P, -1, P, dbls) == lsrtm.EINVAL
    finally:
        L.lsrtm_destroy(h)


def test_binding_constants_match_the_header():
    """Every option key, status code, snapshot storage code and the kernel
    class count the binding passes are the header's values."""
    src = open(HEADER).read()
    opts = dict((k, int(v)) for k, v in re.findall(r"LSRTM_OPT_(\w+)\s*=\s*(\d+)", src))
    assert opts, "no options found"
    for name, val in opts.items():
        assert getattr(lsrtm, f"OPT_{name}") == val, name
    status = dict((k, int(v)) for k, v in re.findall(r"LSRTM_(OK|E[A-Z]+)\s*=\s*(-?\d+)", src))
    for name, val in status.items():
        assert getattr(lsrtm, name) == val, name
    ck = dict((k.lower(), int(v)) for k, v in re.findall(r"LSRTM_CKPT_(\w+)\s*=\s*(\d+)", src))
    assert ck == lsrtm.CKPT
    nk = int(re.search(r"LSRTM_NKERNEL\s*=\s*(\d+)", src).group(1))
    assert nk == lsrtm.NKERNEL == len(lsrtm.KERNEL_NAMES)


def test_resident_state_of_a_fresh_context():
    """lsrtm_resident: nothing planned, nothing run, nothing given up; three
    entries written; NULL arguments refused."""
    L = lsrtm.lib()
    g = lsrtm.Grid()
    g.ndim = 2
    g.n[0], g.n[1], g.n[2] = 10, 12, 1
    g.h[0] = g.h[1] = g.h[2] = 10.0
    g.npml, g.pml_R, g.pml_f0, g.nt, g.dt = 4, 1e-4, 10.0, 10, 1e-3
    h = ctypes.c_void_p()
    assert L.lsrtm_create(ctypes.byref(g), None, ctypes.byref(h)) == 0
    out = (ctypes.c_longlong * 4)(*([-7] * 4))
    assert L.lsrtm_resident(h, out, 4) == lsrtm.OK
    assert list(out) == [0, 0, 0, -7]
    assert L.lsrtm_resident(h, None, 3) == lsrtm.EINVAL
    assert L.lsrtm_resident(None, out, 3) == lsrtm.EINVAL
    for v in (0, 1, 2, 7, -1):
        assert L.lsrtm_set_option(h, lsrtm.OPT_RESIDENT, v) == lsrtm.OK
    L.lsrtm_destroy(h)
