"""Host-side checks of the stencil launch configurations (no launch): what bri_stencil_time and bri_set_stencil_cfg
accept, and that what is reported stands for what launches."""

import ctypes

import pytest

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


@pytest.mark.parametrize("L", [(20, 12, 28, 24), (24, 24, 24, 48), (8, 8, 8, 8), (48, 8, 4, 4), (32, 32, 32, 64)])
def test_reported_configuration_is_the_one_that_launches(L):
    """The configuration reported without an entry stands for the launch that runs: of variant VARIANT_LIBRARY where
    the fields cannot express it (line tiles, blocks of 16 or 48 sites, twelve waves), and installing it, under
    either variant, leaves the defaults in place."""
    for prec in (bri.F64, bri.F32, bri.F32_BF16W):
        for nrhs in (1, 4, 12):
            d = bri.get_stencil_cfg(L, prec, nrhs).as_dict()
            if L == (32, 32, 32, 64):
                assert d["variant"] != bri.VARIANT_LIBRARY, (prec, nrhs)
            elif nrhs == 1 or L in ((20, 12, 28, 24), (24, 24, 24, 48)):
                assert d["variant"] == bri.VARIANT_LIBRARY, (prec, nrhs)
            try:
                bri.set_stencil_cfg(L, prec, nrhs, bri.StencilCfg(*[d[f] for f, _ in bri.StencilCfg._fields_]))
                assert bri.get_stencil_cfg(L, prec, nrhs).as_dict() == d, (prec, nrhs)
                # an entry of the cut tiles is reported as itself, and the library's variant removes it
                bri.set_stencil_cfg(L, prec, nrhs, bri.StencilCfg(0, 0, 0, 0, 0, 4, 0, 1, 0))
                assert bri.get_stencil_cfg(L, prec, nrhs).variant == 0
                bri.set_stencil_cfg(L, prec, nrhs, bri.StencilCfg(variant=bri.VARIANT_LIBRARY))
                assert bri.get_stencil_cfg(L, prec, nrhs).as_dict() == d, (prec, nrhs)
            finally:
                bri.set_stencil_cfg(L, prec, nrhs, None)
