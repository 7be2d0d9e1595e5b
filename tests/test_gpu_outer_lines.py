"""The outer products of the link gradient, three x-displacements a wave (Sec. 9 force): lattices whose lines
are shorter or longer than a block's 64 sites, of one or two sites, or end inside a block, with one, two
(both staging buffers) and five pairs, against the oracle's path-by-path product rule.

Tolerance: the force is a sum of O(10^4) FP64 terms per link, 1e-12 of max |F|."""

import numpy as np
import pytest

import oracle
import paper_1701_00726_amd as bri
import synth
from tests._gpu import need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [(5, 3, 2, 7), (1, 4, 3, 6), (2, 3, 4, 5), (70, 2, 1, 3), (16, 4, 2, 2)])
@pytest.mark.parametrize("npairs", [1, 2, 5])
def test_link_force_line_lengths(L, npairs):
    need_gpu()
    V = int(np.prod(L))
    rng = np.random.default_rng(50 + npairs)
    U = synth.random_links(L, 0.6, 5800 + L[0])
    psi = [rng.standard_normal((2, V, 4, 3)) + 1j * rng.standard_normal((2, V, 4, 3)) for _ in range(npairs)]
    pairs = [(1.0 - 0.7 * k, p[0], p[1]) for k, p in enumerate(psi)]
    ref = oracle.link_force(L, U, 1, pairs)
    Ud = bri.links_to_device(U)
    W = bri.build_links(L, Ud, bri.F64, tbc=1)
    print(f"[outer] {L} {npairs}", flush=True)
    dev = [(w, bri.spinor_to_device(u[None])[0], bri.spinor_to_device(v[None])[0]) for w, u, v in pairs]
    F, _ = bri.link_grad(L, Ud, W, dev, tbc=1)
    got = np.ascontiguousarray(np.transpose(F.cpu().numpy(), (0, 2, 1)))
    assert np.abs(got - ref).max() <= 1e-12 * np.abs(ref).max()
