"""ov_solve in several host threads, each with its own operator and stream: the partial sums of a solve go to memory
of its thread, so concurrent solves, and a later solve of another batch size in the same thread, give the bits
of solves run alone (every reduction has a fixed order)."""

import threading

import pytest

import paper_1701_00726_amd as bri
import synth
from tests._gpu import need_gpu, torch

pytestmark = pytest.mark.gpu


def test_concurrent_solves_match_solves_alone():
    need_gpu()
    L = (4, 4, 4, 8)
    U = bri.links_to_device(synth.smeared_links(L, 0.5, 6300, 0.6, 1))
    W, Wlo = bri.build_links(L, U, bri.F64), bri.build_links(L, U, bri.F32)
    levels = [bri.Level(1, tol=0.1, max_iter=30, ms_tol=1e-8), bri.Level(0, tol=0.1, max_iter=30, inner=bri.F32)]
    b = bri.spinor_to_device(synth.gaussian_source(L, 6301, nrhs=5))

    def solves(stream=None):
        op = bri.OverlapOp(L, W, kl_n=4, tol=1e-13, max_iter=3000, Wlo=Wlo)
        return [op.solve(b[:n].contiguous(), 0.3, tol=1e-11, prec=levels, stream=stream)[0] for n in (2, 5, 1)]

    want = solves()
    torch.cuda.synchronize()
    got, errors = {}, []

    def work(k):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                got[k] = solves(s)
            s.synchronize()
        except Exception as e:  # a failure in a thread fails the test below
            errors.append((k, e))

    print("[solve] two threads", flush=True)
    ts = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errors, errors
    for k in range(2):
        for x, y in zip(got[k], want):
            assert torch.equal(x, y), k
