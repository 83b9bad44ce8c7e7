"""EOFA_TILE reorders the hops on small lattices too: the sums over workgroups,
and with them the last bits of a solution, follow the order that it asks for (in FP64: 32-bit scalars round the
difference away)."""
import pytest

import dwf_inputs as din
from helpers import rel, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("inner", ["fp64", "fp64_fused"])
@pytest.mark.parametrize("L,Ls", [((4, 8, 8, 16), 8), ((8, 4, 4, 8), 24)])
def test_order_is_followed(L, Ls, inner, monkeypatch):
    import torch
    from paper_1611_00298_amd import Context
    U, phi = to_dev(din.random_gauge(L, 0.4, 791)), to_dev(din.gaussian_4d(L, 792))
    chi = []
    for tile in ("none", "none", "p2,2,2,2,2,1,t"):
        monkeypatch.setenv("EOFA_TILE", tile)
        with Context(L, Ls, U, M5=1.8, alpha=2.0) as ctx:
            chi.append(ctx.eofa_solve(phi, 0.1, 0.8, tol=1e-11, inner=inner)[0])
    assert torch.equal(chi[0], chi[1]) and not torch.equal(chi[0], chi[2])
    # residuals of 1e-11 times the inverse's norm (smallest singular value above 0.01 here)
    assert rel(chi[2].cpu().numpy(), chi[0].cpu().numpy()) <= 1e-9
