"""Installing the stencil configuration that is reported leaves the launches as they are, bit for bit, where the
default is one that the fields cannot express, and so does the winner of a tuning run (the sums of the kernels run
in different orders, so another launch would show)."""

import numpy as np
import pytest

import paper_1701_00726_amd as bri
import synth
from tests._gpu import need_gpu, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,L,nrhs", [(bri.F32, (20, 12, 8, 16), 3), (bri.F64, (8, 4, 4, 8), 1),
                                         (bri.F64, (24, 6, 7, 12), 4)])
def test_set_of_get_keeps_the_launch(prec, L, nrhs):
    need_gpu()
    W = bri.build_links(L, bri.links_to_device(synth.random_links(L, 0.6, 6200)), prec)
    x = bri.spinor_to_device(synth.gaussian_source(L, 6201, nrhs=nrhs), prec)
    print(f"[cfg] {L} prec {prec}", flush=True)
    want = bri.apply(L, W, prec, -0.9, x)
    try:
        d = bri.get_stencil_cfg(L, prec, nrhs)
        assert d.variant == bri.VARIANT_LIBRARY
        bri.set_stencil_cfg(L, prec, nrhs, d)
        assert torch.equal(bri.apply(L, W, prec, -0.9, x), want)
        assert bri.stencil_time(L, W, prec, x, cfg=d, reps=1) > 0
        best, us = bri.autotune(L, W, prec, x, reps=2)
        tuned = bri.apply(L, W, prec, -0.9, x)
        bri.set_stencil_cfg(L, prec, nrhs, best)
        assert us > 0 and torch.equal(bri.apply(L, W, prec, -0.9, x), tuned)
        assert np.isfinite(float(torch.linalg.vector_norm(tuned)))
    finally:
        bri.set_stencil_cfg(L, prec, nrhs, None)
