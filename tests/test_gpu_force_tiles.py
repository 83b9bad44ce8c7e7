"""The force kernel's 4D tiles at their edges: lattices smaller than a tile,
extents that no tile divides, each choice of the two long tile directions,
and the slice pairing at odd, even and single Ls, against the oracle."""
import numpy as np
import pytest

import dwf_inputs as din
import oracle
from helpers import to_dev

pytestmark = pytest.mark.gpu

# sums of 4 Ls products per element in FP64: a few hundred units of 1.1e-16
TOL = 1e-12


@pytest.mark.parametrize("L,Ls,aperiodic", [
    ((2, 2, 2, 2), 1, True), ((4, 4, 2, 2), 2, True), ((2, 2, 4, 4), 3, False), ((6, 2, 10, 4), 5, True),
    ((2, 6, 4, 6), 8, False), ((10, 6, 6, 2), 7, True), ((4, 6, 6, 8), 4, True),
])
def test_force_tiles(L, Ls, aperiodic):
    from paper_1611_00298_amd import Context
    m1, m2 = 0.05, 0.9
    print(f"force tiles: L={L} Ls={Ls}", flush=True)
    U = din.random_gauge(L, 0.4, 701)
    chiL, chiR = din.gaussian_5d(L, Ls, 702), din.gaussian_5d(L, Ls, 703)
    lat = oracle.Lattice(L, Ls, M5=1.8, alpha=2.0, antiperiodic_t=aperiodic)
    Fr, Gr = oracle.force(lat, U, m1, m2, chiL, chiR)
    with Context(L, Ls, to_dev(U), M5=1.8, alpha=2.0, antiperiodic_t=aperiodic) as ctx:
        F, G, _ = ctx.eofa_force(m1, m2, chiL=to_dev(chiL), chiR=to_dev(chiR), want_grad=True)
        F0, G0, _ = ctx.eofa_force(m1, m2, chiL=to_dev(chiL), chiR=to_dev(chiR))
        assert G0 is None
        F, G, F0 = F.cpu().numpy(), G.cpu().numpy(), F0.cpu().numpy()
    assert np.array_equal(F, F0)
    assert np.abs(F - Fr).max() <= TOL * np.abs(Fr).max()
    assert np.abs(G - Gr).max() <= TOL * np.abs(Gr).max()
