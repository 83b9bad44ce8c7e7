"""The solver over the hop's forms and the places its sums ride in: per-site and
block-sharing throughput hops with all sums inside other launches (small
lattices, EOFA_BLOCKS=0 and 2, and 8^3x34), the FP64 throughput form among
one-wavefront workgroups (8^3x18), and grids of more than 2048 workgroups, where
|z|^2 has a launch of its own; every inner precision, against the oracle's
operator."""
import pytest

import dwf_inputs as din
import oracle
from helpers import rel, to_dev

pytestmark = pytest.mark.gpu

M1, M2 = 0.2, 1.0


def _sources(lat, phi):
    om_m, om_p, _ = oracle.omega_k(lat, M1, M2)
    vL, vR = lat.zeros5(), lat.zeros5()
    vL[..., 2:, :] = om_m[:, None, None, None, None, None, None] * phi[None, ..., 2:, :]
    vR[..., :2, :] = om_p[:, None, None, None, None, None, None] * phi[None, ..., :2, :]
    return vL, vR


SMALL = [((4, 2, 6, 4), 10), ((4, 6, 4, 2), 8), ((8, 4, 4, 8), 24)]
LARGE = [((8, 8, 8, 34), 16), ((8, 8, 8, 18), 16), ((16, 16, 16, 32), 8), ((16, 16, 16, 16), 24)]


@pytest.mark.parametrize("inner", ["fp64", "fp64_fused", "fp32", "fp16", "bf16"])
@pytest.mark.parametrize("L,Ls,blocks", [c + (b,) for c in SMALL for b in ("0", "2")] + [c + ("1",) for c in LARGE])
def test_solve_forms(L, Ls, blocks, inner, monkeypatch):
    from paper_1611_00298_amd import Context
    monkeypatch.setenv("EOFA_BLOCKS", blocks)
    print(f"solve forms: L={L} Ls={Ls} blocks={blocks} {inner}", flush=True)
    U, phi = din.random_gauge(L, 0.3, 821), din.gaussian_4d(L, 822)
    lat = oracle.Lattice(L, Ls, M5=1.8, alpha=2.0)
    with Context(L, Ls, to_dev(U), M5=1.8, alpha=2.0) as ctx:
        chiL, chiR, _, _, st = ctx.eofa_solve(to_dev(phi), M1, M2, tol=1e-10, inner=inner, want_mphi=False)
    arith = "fp64" if inner == "fp64_fused" else inner
    assert st["converged"] and st["inner_used"] == [arith, arith], st
    vL, vR = _sources(lat, phi)
    assert rel(oracle.H_op(lat, U, M1, M1, chiL.cpu().numpy()), vL) <= 1e-10
    assert rel(oracle.H_op(lat, U, M1, M2, chiR.cpu().numpy()), vR) <= 1e-10


@pytest.mark.parametrize("blocks", ["0", "1", "2"])
@pytest.mark.parametrize("L,Ls", SMALL)
def test_fp64_iterates(L, Ls, blocks, monkeypatch):
    """Six iterations of the plain FP64 solver are the oracle's, in every form."""
    from paper_1611_00298_amd import Context
    monkeypatch.setenv("EOFA_BLOCKS", blocks)
    U, phi = din.random_gauge(L, 0.3, 823), din.gaussian_4d(L, 824)
    lat = oracle.Lattice(L, Ls, M5=1.8, alpha=2.0)
    with Context(L, Ls, to_dev(U), M5=1.8, alpha=2.0) as ctx:
        chi = ctx.eofa_solve(to_dev(phi), M1, M2, tol=1e-30, maxiter=6, want_mphi=False, allow_noconv=True)[:2]
    for v, mm, x in zip(_sources(lat, phi), (M1, M2), chi):
        y, _, _ = oracle.solve_ddwf_eo(lat, U, M1, mm, oracle.g5r5(lat, v), fixed=6)
        assert rel(x.cpu().numpy(), oracle.apply_chiral(lat, "dtilde", M1, mm, y)) <= 1e-12
