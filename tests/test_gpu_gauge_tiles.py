"""The gauge force's plane tiles at their edges: extents below a tile, uneven
splits, a tile and one more, both actions, written and accumulated, against
the oracle."""
import numpy as np
import pytest

import dwf_inputs as din
import oracle
from helpers import to_dev

pytestmark = pytest.mark.gpu

# sums of a few hundred FP64 products of unitary matrices per element, against the largest force
TOL = 1e-12


@pytest.mark.parametrize("c1", [oracle.IWASAKI_C1, 0.0])
@pytest.mark.parametrize("L", [(2, 2, 2, 2), (4, 2, 8, 6), (8, 10, 2, 4), (10, 4, 18, 2), (2, 4, 4, 14), (6, 12, 4, 2)])
def test_gauge_force_tiles(L, c1):
    from paper_1611_00298_amd import Context
    beta = 2.13
    print(f"gauge tiles: L={L} c1={c1}", flush=True)
    U = din.random_gauge(L, 0.5, 731)
    F0 = din.gaussian_momenta(L, 732)
    ref = oracle.gauge_force(U, beta, c1)
    Ud = to_dev(U)
    with Context(L, 4, Ud) as ctx:
        out = to_dev(np.full(U.shape, np.nan + 0j))
        ctx.gauge_force(Ud, beta, c1, out=out)
        acc = to_dev(F0)
        ctx.gauge_force(Ud, beta, c1, out=acc, accumulate=True)
        out, acc = out.cpu().numpy(), acc.cpu().numpy()
    assert np.abs(out - ref).max() <= TOL * np.abs(ref).max()
    assert np.abs(acc - (ref + F0)).max() <= TOL * np.abs(ref).max()
