"""The force on lattices with few tiles, where several workgroups share a tile's
slice pairs: ranges of uneven length, both sides of the lines in Ls and in the
number of tiles, ragged tiles, against the oracle; and the time it is for."""
import numpy as np
import pytest

import dwf_inputs as din
import oracle
from helpers import to_dev

pytestmark = pytest.mark.gpu

# sums of 4 Ls products per element in FP64: a few hundred units of 1.1e-16
TOL = 1e-12


@pytest.mark.parametrize("L,Ls", [((2, 2, 2, 2), 8), ((4, 4, 4, 4), 7), ((4, 6, 2, 10), 8), ((6, 4, 4, 2), 9), ((2, 4, 4, 2), 23),
                                  ((4, 2, 4, 4), 63), ((2, 2, 4, 4), 64), ((8, 8, 8, 16), 8), ((8, 8, 8, 18), 8)])
def test_force_split(L, Ls):
    from paper_1611_00298_amd import Context
    m1, m2 = 0.05, 0.9
    print(f"force split: L={L} Ls={Ls}", flush=True)
    U = din.random_gauge(L, 0.4, 771)
    chiL, chiR = din.gaussian_5d(L, Ls, 772), din.gaussian_5d(L, Ls, 773)
    Fr, Gr = oracle.force(oracle.Lattice(L, Ls, M5=1.8, alpha=2.0), U, m1, m2, chiL, chiR)
    with Context(L, Ls, to_dev(U), M5=1.8, alpha=2.0) as ctx:
        for _ in range(2):   # the second call on the first one's workspace
            F, G, _ = ctx.eofa_force(m1, m2, chiL=to_dev(chiL), chiR=to_dev(chiR), want_grad=True)
            assert np.abs(F.cpu().numpy() - Fr).max() <= TOL * np.abs(Fr).max()
            assert np.abs(G.cpu().numpy() - Gr).max() <= TOL * np.abs(Gr).max()


def test_many_slices_on_an_idle_gpu():
    """Eight times the slices on 4^4 take less than four times the GPU time:
    one workgroup per tile that walks them all in a row takes eight times."""
    from paper_1611_00298_amd import Context
    L, t = (4, 4, 4, 4), {}
    U = to_dev(din.random_gauge(L, 0.4, 774))
    for Ls in (8, 64):
        chi = to_dev(din.gaussian_5d(L, Ls, 775))
        with Context(L, Ls, U, M5=1.8, alpha=2.0) as ctx:
            for _ in range(20):
                ctx.timing_enable()
                ctx.eofa_force(0.05, 0.9, chiL=chi, chiR=chi)
                t[Ls] = min(t.get(Ls, 1e9), ctx.timing_query("force")["ms"])
    print(f"force on 4^4: {t}", flush=True)
    assert t[64] < 4 * t[8]
