"""The four-right-hand-side stencil at the fill of its rounds of blocks where it takes over (12-, 24- and 48-site
lines, one block of 48 sites and four right-hand sides per CU): the Brillouin operator and its adjoint against
the oracle (App. C.1 stencil), just inside and just outside the line.

Tolerances: the operator is a sum of 81 terms of 3 products with weights summing to about 4, so a relative L2
error of a few units of roundoff: 1e-14 in FP64 (45 eps), 2e-6 in FP32 (17 eps)."""

import numpy as np
import pytest

import oracle
import paper_1701_00726_amd as bri
import synth
from tests._gpu import need_gpu, rel_l2, round_links

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,L,nrhs", [
    (bri.F64, (24, 6, 7, 12), 4),  # 252 of 256 blocks; the last CUs idle
    (bri.F64, (48, 3, 7, 12), 7),  # two rounds, the second group of three
    (bri.F64, (12, 4, 12, 16), 4),  # 192 of 256: left to the line tiles
    (bri.F64, (24, 4, 4, 8), 8),  # 128 of 256: left to the line tiles
    (bri.F32, (24, 4, 14, 16), 4),  # 448 of 512
    (bri.F32_BF16W, (48, 2, 14, 16), 8),  # 896 of 1024
    (bri.F32, (12, 8, 12, 12), 4),  # 288 of 512: left to the line tiles
    (bri.F32_BF16W, (12, 8, 8, 20), 12),  # 960 of 1024 in three groups
])
def test_rows_at_the_fill_of_their_rounds(prec, L, nrhs):
    need_gpu()
    U = synth.random_links(L, 0.6, 6100 + L[0])
    W = bri.build_links(L, bri.links_to_device(U), prec)
    Wr = round_links(oracle.links(L, U), prec)
    psi = synth.gaussian_source(L, 6110 + nrhs, nrhs=nrhs).astype(np.complex64 if prec else np.complex128)
    x = bri.spinor_to_device(psi.astype(np.complex128), prec)
    print(f"[rows] rounds {L} prec {prec} nrhs {nrhs}", flush=True)
    got, gotd = (bri.spinor_to_host(f(L, W, prec, -0.9, x)) for f in (bri.apply, bri.apply_dag))
    ref = oracle.dirac(L, Wr, -0.9, psi.astype(np.complex128))
    refd = oracle.dirac_adj(L, Wr, -0.9, psi.astype(np.complex128))
    tol = 2e-6 if prec else 1e-14
    for r in range(nrhs):
        assert rel_l2(got[r], ref[r]) < tol, r
        assert rel_l2(gotd[r], refd[r]) < tol, r
