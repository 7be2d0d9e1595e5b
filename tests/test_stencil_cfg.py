"""Host-side checks of the stencil launch configurations (no launch): what bri_stencil_time and bri_set_stencil_cfg
accept."""

import ctypes

import paper_1701_00726_amd as bri


def _time(L, prec, nrhs, cfg):
    g = bri._geom(L)
    us = ctypes.c_double()
    P = ctypes.c_void_p
    return bri.load().bri_stencil_time(ctypes.byref(g), P(1 << 24), prec, P(1 << 28), P(1 << 29), nrhs, ctypes.byref(cfg),
                                       1, ctypes.byref(us), None)


def test_wave_counts_beyond_four_are_refused():
    """nsplit is 1, 2 or 4 for one right-hand side per thread: twelve waves a tile are a default of the library
    that callers cannot ask for."""
    L = (8, 8, 8, 8)
    for nsplit in (0, 3, 8, 12):
        cfg = bri.StencilCfg(8, 8, 1, 1, 2, nsplit, 0, 1, 0)
        assert _time(L, bri.F64, 1, cfg) == bri.EINVAL, nsplit
        g = bri._geom(L)
        assert bri.load().bri_set_stencil_cfg(ctypes.byref(g), bri.F64, 1, ctypes.byref(cfg)) == bri.EINVAL, nsplit
