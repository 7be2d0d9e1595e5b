"""The four-right-hand-side stencil (48 sites a block, 12-, 24- and 48-site lines): the Brillouin operator and
its adjoint against the oracle (App. C.1 stencil), with full and incomplete groups, odd extents, the clover
term and antiperiodic time, and the solver epilogues (Sec. 3.3).

Tolerances: the operator is a sum of 81 terms of 3 products with weights summing to about 4, so a relative L2
error of a few units of roundoff: 1e-14 in FP64 (45 eps), 2e-6 in FP32 (17 eps); the overlap apply
carries its CG tolerance 1e-12 and is held to 1e-10."""

import numpy as np
import pytest

import oracle
import paper_1701_00726_amd as bri
import synth
from tests._gpu import need_gpu, rel_l2, round_links

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [(12, 8, 8, 16), (24, 6, 9, 12), (48, 3, 5, 20), (12, 4, 1, 260)])
@pytest.mark.parametrize("prec,tol", [(bri.F64, 1e-14), (bri.F32, 2e-6), (bri.F32_BF16W, 2e-6)])
def test_rows_match_oracle(L, prec, tol):
    need_gpu()
    U = synth.random_links(L, 0.6, 5700 + L[0])
    W = bri.build_links(L, bri.links_to_device(U), prec)
    Wr = round_links(oracle.links(L, U), prec)
    print(f"[rows] {L} prec {prec}", flush=True)
    for nrhs in (3, 4, 7) if prec == bri.F64 else (4, 8):
        psi = synth.gaussian_source(L, 5710 + nrhs, nrhs=nrhs).astype(np.complex64 if prec else np.complex128)
        x = bri.spinor_to_device(psi.astype(np.complex128), prec)
        got, gotd = (bri.spinor_to_host(f(L, W, prec, -0.9, x)) for f in (bri.apply, bri.apply_dag))
        ref = oracle.dirac(L, Wr, -0.9, psi.astype(np.complex128))
        refd = oracle.dirac_adj(L, Wr, -0.9, psi.astype(np.complex128))
        for r in range(nrhs):
            assert rel_l2(got[r], ref[r]) < tol, (nrhs, r)
            assert rel_l2(gotd[r], refd[r]) < tol, (nrhs, r)


@pytest.mark.parametrize("csw,tbc", [(0.0, 0), (1.0, 1)])
def test_rows_in_the_solver(csw, tbc):
    """The norm and residual epilogues of a batch, one column empty, against single right-hand sides."""
    need_gpu()
    L = (12, 8, 4, 8)
    U = bri.links_to_device(synth.smeared_links(L, 0.5, 5720, 0.6, 1))
    W = bri.build_links(L, U, bri.F64, tbc=tbc, csw=csw)
    b = synth.gaussian_source(L, 5721, nrhs=7)
    b[2] = 0.0
    print(f"[rows] overlap {csw} {tbc}", flush=True)
    got = bri.spinor_to_host(bri.OverlapOp(L, W, kl_n=6, tol=1e-12, nrhs=7, tbc=tbc).apply(bri.spinor_to_device(b))[0])
    one = bri.OverlapOp(L, W, kl_n=6, tol=1e-12, nrhs=1, tbc=tbc)
    assert np.count_nonzero(got[2]) == 0
    for r in (0, 1, 3, 4, 5, 6):
        ref = bri.spinor_to_host(one.apply(bri.spinor_to_device(b[r:r + 1]))[0])[0]
        assert rel_l2(got[r], ref) < 1e-10, r


def test_rows_low_precision_phase():
    need_gpu()
    L = (12, 8, 8, 16)
    U = bri.links_to_device(synth.smeared_links(L, 0.5, 5730, 0.6, 1))
    W, Wlo = bri.build_links(L, U, bri.F64), bri.build_links(L, U, bri.F32)
    b = synth.gaussian_source(L, 5731, nrhs=4)
    op = bri.OverlapOp(L, W, kl_n=6, tol=1e-12, nrhs=4, Wlo=Wlo, inner=bri.F32)
    got = bri.spinor_to_host(op.apply(bri.spinor_to_device(b))[0])
    one = bri.OverlapOp(L, W, kl_n=6, tol=1e-12, nrhs=1)
    for r in range(4):
        ref = bri.spinor_to_host(one.apply(bri.spinor_to_device(b[r:r + 1]))[0])[0]
        assert rel_l2(got[r], ref) < 1e-10, r
