"""Launches on tiles of whole x-lines that do not fill a wave's 64 lanes, or a tile row that does not
divide L_y, the twelve-wave launch and the small-lattice kernel: the Brillouin and Wilson operators, their
adjoints and the solver epilogues against the oracle (App. C.1 stencil, eq. (def_wils), Sec. 3.3).

Tolerances: the operator is a sum of 81 terms of 3 products with weights summing to about 4, so a
relative L2 error of a few units of roundoff: 1e-14 in FP64 (45 eps), 2e-6 in FP32 (17 eps); the
overlap apply carries its CG tolerance 1e-12 and is held to 1e-10."""

import numpy as np
import pytest

import oracle
import paper_1701_00726_amd as bri
import synth
from tests._gpu import need_gpu, rel_l2, round_links

pytestmark = pytest.mark.gpu

LATTICES = [
    (20, 7, 8, 16),  # 3 lines a tile (60 lanes), the last tile row holds one
    (33, 4, 8, 16),  # 1 line a tile, 33 lanes
    (24, 12, 6, 12),  # 2 lines a tile (48 lanes), columns of several tile rows and planes
    (9, 8, 8, 8),  # 7 lines, then 1; twelve waves a tile in FP64
    (64, 3, 4, 4),  # the small-lattice kernel, eight and four waves, and full 64-site lines
    (5, 4, 4, 8),  # the small-lattice kernel up to all 9 right-hand sides
    (4, 4, 4, 1),  # extents of one site: a slab's both neighbours coincide
]


@pytest.fixture(scope="module")
def fields():
    out = {}
    for L in LATTICES:
        U = synth.random_links(L, 0.6, 5100 + L[0])
        out[L] = (bri.links_to_device(U), oracle.links(L, U))
    return out


@pytest.mark.parametrize("L", LATTICES)
@pytest.mark.parametrize("prec,tol", [(bri.F64, 1e-14), (bri.F32, 2e-6), (bri.F32_BF16W, 2e-6)])
def test_line_tiles_match_oracle(fields, L, prec, tol):
    need_gpu()
    Ud, Wo = fields[L]
    W = bri.build_links(L, Ud, prec)
    Wr = round_links(Wo, prec)
    print(f"[lines] {L} prec {prec}", flush=True)
    for nrhs in (1, 2, 3, 5, 9):
        psi = synth.gaussian_source(L, 5200 + nrhs, nrhs=nrhs).astype(np.complex64 if prec else np.complex128)
        x = bri.spinor_to_device(psi.astype(np.complex128), prec)
        got, gotd = (bri.spinor_to_host(f(L, W, prec, -0.9, x)) for f in (bri.apply, bri.apply_dag))
        ref = oracle.dirac(L, Wr, -0.9, psi.astype(np.complex128))
        refd = oracle.dirac_adj(L, Wr, -0.9, psi.astype(np.complex128))
        for r in range(nrhs):
            assert rel_l2(got[r], ref[r]) < tol, (nrhs, r)
            assert rel_l2(gotd[r], refd[r]) < tol, (nrhs, r)


@pytest.mark.parametrize("L", LATTICES)
def test_line_tiles_wilson(fields, L):
    need_gpu()
    Ud, _ = fields[L]
    K = oracle.WilsonKernel(np.transpose(Ud.cpu().numpy(), (0, 3, 1, 2)))
    W = bri.build_links(L, Ud, bri.F64)
    print(f"[lines] wilson {L}", flush=True)
    for nrhs in (1, 4):
        psi = synth.gaussian_source(L, 5300 + nrhs, nrhs=nrhs)
        x = bri.spinor_to_device(psi)
        got = bri.spinor_to_host(bri.wilson_apply(L, W, bri.F64, -0.8, x))
        gotd = bri.spinor_to_host(bri.wilson_apply_dag(L, W, bri.F64, -0.8, x))
        for r in range(nrhs):
            assert rel_l2(got[r], oracle.dirac(L, K, -0.8, psi[r])) < 1e-14, r
            assert rel_l2(gotd[r], oracle.dirac_adj(L, K, -0.8, psi[r])) < 1e-14, r


@pytest.mark.parametrize("L,nrhs", [((20, 7, 4, 8), 1), ((20, 7, 4, 8), 4), ((9, 8, 8, 8), 1), ((33, 4, 4, 8), 3),
                                    ((5, 4, 4, 8), 1), ((5, 4, 4, 8), 5)])
def test_line_tiles_in_the_solver(L, nrhs):
    """The norm and residual epilogues: one pair of partial sums per tile, idle lanes adding nothing."""
    need_gpu()
    U = synth.smeared_links(L, 0.5, 5400, 0.6, 1)
    W = bri.build_links(L, bri.links_to_device(U), bri.F64)
    Wo = oracle.links(L, U)
    b = synth.gaussian_source(L, 5401, nrhs=nrhs)
    print(f"[lines] overlap {L} {nrhs}", flush=True)
    out, _ = bri.OverlapOp(L, W, kl_n=6, tol=1e-12, nrhs=nrhs).apply(bri.spinor_to_device(b))
    got = bri.spinor_to_host(out)
    for r in range(nrhs):
        ref, _, _ = oracle.ov_apply(L, Wo, 1.0, 6, b[r], tol=1e-13)
        assert rel_l2(got[r], ref) < 1e-10, r


@pytest.mark.parametrize("L", [(32, 8, 8, 64), (16, 16, 16, 34), (12, 12, 12, 12)])
def test_alpha_formed_by_the_stencil(L):
    """Up to 2048 partial sums the residual stencil of a single column forms alpha itself; four columns on the
    kernels with several columns per thread take it from a launch of its own.  Both stop at the same bound."""
    need_gpu()
    U = synth.smeared_links(L, 0.5, 5500, 0.6, 1)
    W = bri.build_links(L, bri.links_to_device(U), bri.F64)
    b = bri.spinor_to_device(synth.gaussian_source(L, 5501, nrhs=4))
    print(f"[lines] alpha {L}", flush=True)
    four, _ = bri.OverlapOp(L, W, kl_n=4, tol=1e-12, nrhs=4).apply(b)
    one, _ = bri.OverlapOp(L, W, kl_n=4, tol=1e-12, nrhs=1).apply(b[2:3].contiguous())
    assert rel_l2(bri.spinor_to_host(one)[0], bri.spinor_to_host(four)[2]) < 1e-10


@pytest.mark.parametrize("prec,L,nrhs", [(bri.F64, (16, 16, 16, 14), 1), (bri.F64, (16, 16, 16, 14), 2),
                                         (bri.F32, (24, 14, 16, 18), 4), (bri.F32, (30, 12, 16, 17), 1)])
def test_adjoint_backwards(prec, L, nrhs):
    """Links between 256 and 512 MiB: the adjoint walks tiles and slabs backwards; <x, D y> = <D^dag x, y>
    for vectors of unit variance holds to the operator's tolerance times |x| |D y|."""
    need_gpu()
    V = int(np.prod(L))
    assert (256 << 20) < V * 360 * (16 if prec == bri.F64 else 8) <= (512 << 20)
    W = bri.build_links(L, bri.links_to_device(synth.random_links(L, 0.6, 5900)), prec)
    x, y = (bri.spinor_to_device(synth.gaussian_source(L, 5901 + k, nrhs=nrhs), prec) for k in (0, 1))
    print(f"[lines] adjoint {L} prec {prec}", flush=True)
    Dy, Dx = (bri.spinor_to_host(f(L, W, prec, -0.9, v)).astype(complex)
              for f, v in ((bri.apply, y), (bri.apply_dag, x)))
    hx, hy = bri.spinor_to_host(x).astype(complex), bri.spinor_to_host(y).astype(complex)
    for r in range(nrhs):
        bound = np.linalg.norm(hx[r]) * np.linalg.norm(Dy[r])
        assert abs(np.vdot(hx[r], Dy[r]) - np.vdot(Dx[r], hy[r])) < (1e-14 if prec == bri.F64 else 2e-6) * bound
