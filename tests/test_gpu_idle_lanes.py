"""Tiles whose lanes are not all at work, in the forms that the plain FP64 operator does not reach: the Wilson
operator in low precision, its norm and residual epilogues and in-kernel alpha inside the overlap (eqs. (def_wils),
(def_over)), the clover term with antiperiodic time, and the four-right-hand-side kernel in a mixed-precision batch
against a stored FP64 oracle output.

Tolerances: 2e-6 in FP32 against links rounded alike (17 eps for 9 terms of 3 products); 1e-14 in FP64 and, against
unrounded links, 1e-6 and 1e-2 (their own roundings, 6e-8 and 4e-3) with the clover term; 1e-10 for the overlap,
whose CG stops at 1e-12 and whose result bound at 1e-11."""

import numpy as np
import pytest

import oracle
import paper_1701_00726_amd as bri
import synth
from tests._gpu import need_gpu, rel_l2, round_links, torch
from tests.test_gpu_overlap_golden import _check, _field, _load, _source

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [bri.F32, bri.F32_BF16W])
@pytest.mark.parametrize("L", [(20, 7, 8, 16), (33, 4, 8, 16), (9, 8, 8, 8)])
def test_wilson_low_precision(L, prec):
    need_gpu()
    U = synth.random_links(L, 0.6, 6500 + L[0])
    W = bri.build_links(L, bri.links_to_device(U), prec)
    K = oracle.WilsonKernel(round_links(U, prec))
    print(f"[idle] wilson {L} prec {prec}", flush=True)
    for nrhs in (1, 4):
        psi = synth.gaussian_source(L, 6510 + nrhs, nrhs=nrhs).astype(np.complex64).astype(np.complex128)
        x = bri.spinor_to_device(psi, prec)
        got = bri.spinor_to_host(bri.wilson_apply(L, W, prec, -0.8, x))
        gotd = bri.spinor_to_host(bri.wilson_apply_dag(L, W, prec, -0.8, x))
        for r in range(nrhs):
            assert rel_l2(got[r], oracle.dirac(L, K, -0.8, psi[r])) < 2e-6, (nrhs, r)
            assert rel_l2(gotd[r], oracle.dirac_adj(L, K, -0.8, psi[r])) < 2e-6, (nrhs, r)


@pytest.mark.parametrize("inner", [bri.F64, bri.F32])
@pytest.mark.parametrize("L,nrhs", [((20, 7, 4, 8), 1), ((33, 4, 4, 8), 3)])
def test_wilson_overlap(L, nrhs, inner):
    need_gpu()
    U = synth.smeared_links(L, 0.5, 6520, 0.6, 1)
    Ud = bri.links_to_device(U)
    W = bri.build_links(L, Ud, bri.F64)
    Wlo = None if inner == bri.F64 else bri.build_links(L, Ud, inner)
    b = synth.gaussian_source(L, 6521, nrhs=nrhs)
    print(f"[idle] wilson overlap {L} {nrhs} inner {inner}", flush=True)
    op = bri.OverlapOp(L, W, kl_n=4, tol=1e-12, max_iter=5000, Wlo=Wlo, inner=inner, nrhs=nrhs,
                       kernel=bri.KERNEL_WILSON)
    got = bri.spinor_to_host(op.apply(bri.spinor_to_device(b))[0])
    K = oracle.WilsonKernel(U)
    for r in range(nrhs):
        assert rel_l2(got[r], oracle.ov_apply(L, K, 1.0, 4, b[r], tol=1e-13)[0]) < 1e-10, r


@pytest.mark.parametrize("prec,L,nrhs,tol", [
    (bri.F64, (20, 7, 8, 16), 1, 1e-14), (bri.F64, (20, 7, 8, 16), 3, 1e-14), (bri.F32, (20, 7, 8, 16), 3, 1e-6),
    (bri.F64, (9, 8, 8, 8), 1, 1e-14),  # twelve waves a tile
    (bri.F32, (24, 4, 14, 16), 4, 1e-6), (bri.F32_BF16W, (24, 4, 14, 16), 4, 1e-2)])  # 48 sites a block
def test_clover_antiperiodic(prec, L, nrhs, tol):
    need_gpu()
    U = synth.random_links(L, 0.6, 6530 + L[0])
    W = bri.build_links(L, bri.links_to_device(U), prec, tbc=1, csw=1.0)
    K = oracle.BrillouinKernel(oracle.links(L, U, tbc=1), oracle.clover_field(L, U, 1.0))
    psi = synth.gaussian_source(L, 6531, nrhs=nrhs)
    print(f"[idle] clover {L} prec {prec} nrhs {nrhs}", flush=True)
    x = bri.spinor_to_device(psi, prec)
    assert rel_l2(bri.spinor_to_host(bri.apply(L, W, prec, -0.9, x)), oracle.dirac(L, K, -0.9, psi)) < tol
    assert rel_l2(bri.spinor_to_host(bri.apply_dag(L, W, prec, -0.9, x)), oracle.dirac_adj(L, K, -0.9, psi)) < tol


def test_mixed_batch_24_48():
    """Twelve sources, the stored point and Gaussian ones among them, at the benchmark's precision and stopping."""
    need_gpu()
    gp, gg = _load("24x24x24x48_point0"), _load("24x24x24x48_gauss")
    L, (U, W) = _field(gp)
    Wlo = bri.build_links(L, U, bri.F32)
    b = synth.point_sources_12(L)
    b[5] = _source(L, gg)[0]
    assert np.array_equal(b[int(gp["source_arg"])], _source(L, gp)[0])
    print("[24^3x48] mixed batch of 12", flush=True)
    op = bri.OverlapOp(L, W, kl_n=16, rho=1.0, tol=1e-11, relax=bri.RELAX_BOUND, max_iter=5000, Wlo=Wlo,
                       inner=bri.F32, nrhs=12)
    out, st = op.apply(bri.spinor_to_device(b))
    _check(out[int(gp["source_arg"])], gp, f"24^3x48 point, mixed batch ({st.iters} iterations)")
    _check(out[5], gg, f"24^3x48 gauss, mixed batch ({st.iters} iterations, {st.refine} in low precision)")
    del op, out, Wlo
    torch.cuda.empty_cache()


@pytest.mark.parametrize("prec,L,tol", [(bri.F64, (16, 16, 16, 14), 1e-13), (bri.F64, (20, 12, 14, 16), 1e-13),
                                        (bri.F32, (30, 12, 16, 17), 1e-5)])
def test_adjoint_in_reverse_order(prec, L, tol):
    """Links between 256 and 512 MiB, where the adjoint takes the tiles in reverse order, at sampled sites: the
    corners of the lattice, of the first and the last tile, and random ones."""
    need_gpu()
    V = int(np.prod(L))
    assert (256 << 20) < V * 360 * (16 if prec == bri.F64 else 8) <= (512 << 20)
    U = synth.random_links(L, 0.6, 6540)
    W = bri.build_links(L, bri.links_to_device(U), prec, tbc=1)
    psi = synth.gaussian_source(L, 6541)
    sites = [0, 1, L[0] - 1, 63, 64, V - 1, V - 64, V - 65]
    sites += [int(v) for v in np.random.default_rng(6542).integers(0, V, 56)]
    print(f"[idle] adjoint {L} prec {prec}", flush=True)
    got = bri.spinor_to_host(bri.apply_dag(L, W, prec, -0.9, bri.spinor_to_device(psi, prec)))[0]
    ref = oracle.dirac_adj_at(L, U, 1, -0.9, psi[0], sites)
    assert np.abs(got[sites] - ref).max() <= tol * np.abs(ref).max()
