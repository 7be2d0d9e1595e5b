"""The fused vector launches of ov_solve: combinations that also leave the compacted copy the kernel
level's stencil reads, take its result in or form dot products, with finished and empty columns.

A batch with an empty column in the middle (so the kernel level works on a compacted copy from the first
step on, also in FP64) reaches, column by column, the solutions of single-source solves, with their
number of outer iterations.  Tolerance: both sides stop at 1e-11 relative residual; with condition
numbers of a few at m = 0.3 the solutions agree to 1e-9 relative (L2).  A column's recurrence is the same
in both up to rounding, so the batch takes the iterations of its slowest column, give or take one.
"""

import numpy as np
import pytest

import paper_1701_00726_amd as bri
import synth
from tests._gpu import need_gpu, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [(4, 4, 4, 6), (8, 8, 8, 8), (12, 12, 8, 12)])  # blocks: 18, 192, all 512 and a second round
@pytest.mark.parametrize("kprec", [bri.F64, bri.F32])
def test_batch_with_an_empty_column_matches_single_solves(L, kprec):
    need_gpu()
    U = bri.links_to_device(synth.smeared_links(L, 0.5, 5600, 0.6, 1))
    W = bri.build_links(L, U, bri.F64)
    op = bri.OverlapOp(L, W, kl_n=4, tol=1e-13, max_iter=3000, Wlo=bri.build_links(L, U, bri.F32))
    levels = [bri.Level(1, tol=0.1, max_iter=30, ms_tol=1e-8), bri.Level(0, tol=0.1, max_iter=30, inner=kprec)]
    b = synth.gaussian_source(L, 5601, nrhs=3)
    b[1] = 0.0
    b[2] *= 1e-5
    print(f"[solve] {L} {kprec}", flush=True)
    x, st = op.solve(bri.spinor_to_device(b), 0.3, complete=True, tol=1e-11, prec=levels)
    got = bri.spinor_to_host(x)
    assert st.status == bri.OK and st.rel_resid < 1e-10
    assert np.count_nonzero(got[1]) == 0
    its = []
    for c in (0, 2):
        xs, ss = op.solve(bri.spinor_to_device(b[c:c + 1]), 0.3, complete=True, tol=1e-11, prec=levels)
        assert rel_l2(got[c], bri.spinor_to_host(xs)[0]) < 1e-9, c
        its.append(ss.iters)
    assert abs(st.iters - max(its)) <= 1, (st.iters, its)
