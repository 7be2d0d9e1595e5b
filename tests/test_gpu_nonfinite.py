"""A non-finite entry of the input reaches the same output entries whichever kernel a launch uses: the sites within
one hop per direction, and of their spins those that the spin matrix of the displacement couples (a zero weight
adds nothing, where 0 * inf would be NaN).  The defaults against the tiles of 64 sites.

Tolerance of the finite entries: 81 terms of 3 complex products in two orders, 243 roundings of the largest
entry: 3e-14 in FP64 and 1.5e-5 in FP32, held to 1e-13 and 5e-5."""

import pytest

import paper_1701_00726_amd as bri
import synth
from tests._gpu import need_gpu, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,L,nrhs", [
    (bri.F64, (4, 4, 4, 8), 1),  # blocks of 16 sites
    (bri.F32, (8, 8, 8, 8), 2),
    (bri.F32_BF16W, (5, 4, 4, 8), 1),
    (bri.F64, (24, 6, 7, 12), 4),  # four right-hand sides on 48 sites
    (bri.F32, (24, 4, 14, 16), 4),
    (bri.F32, (20, 12, 8, 16), 3),  # line tiles
])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_nonfinite_entries_spread_alike(prec, L, nrhs, bad):
    need_gpu()
    W = bri.build_links(L, bri.links_to_device(synth.random_links(L, 0.6, 6400 + L[0])), prec)
    x = bri.spinor_to_device(synth.gaussian_source(L, 6401, nrhs=nrhs), prec)
    site = L[0] * L[1] * L[2] + L[0] * L[1] + L[0] + 2  # (2, 1, 1, 1)
    x[nrhs - 1, 1, 2, site] = bad
    print(f"[nonfinite] {L} prec {prec} {bad}", flush=True)
    for fn in (bri.apply, bri.apply_dag):
        got = torch.view_as_real(fn(L, W, prec, -0.9, x))
        try:
            bri.set_stencil_cfg(L, prec, nrhs, bri.StencilCfg(0, 0, 0, 0, 0, 4, 0, 1, 0))
            want = torch.view_as_real(fn(L, W, prec, -0.9, x))
        finally:
            bri.set_stencil_cfg(L, prec, nrhs, None)
        ok = torch.isfinite(want)
        assert not bool(ok.all())
        assert torch.equal(torch.isfinite(got), ok)
        d = (got - want)[ok].abs().max() / want[ok].abs().max()
        assert float(d) < (5e-5 if prec else 1e-13)
