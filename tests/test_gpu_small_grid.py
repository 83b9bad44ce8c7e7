"""The hop's latency form and one-wavefront workgroups on grids that leave the
GPU idle, against the oracle: every Ls class (one work-item per site, partial
wavefronts, links in several batches, matrix cores, the largest Ls), with the
throughput forms (per site, and block sharing where it applies) on the same
lattice; and the two sides of the grid-size line."""
import pytest

import dwf_inputs as din
import oracle
from helpers import PREC_TOL, region_rel, rel, to_dev

pytestmark = pytest.mark.gpu


def _check(L, Ls, precs):
    from paper_1611_00298_amd import Context
    mp, mm = 0.07, 0.8
    U, psi = din.random_gauge(L, 0.4, 741), din.gaussian_5d(L, Ls, 742)
    lat = oracle.Lattice(L, Ls, M5=1.8, alpha=2.0)
    with Context(L, Ls, to_dev(U), M5=1.8, alpha=2.0) as ctx:
        x = to_dev(psi)
        for dag in (False, True):
            full = oracle.ddwf(lat, U, mp, mm, psi, dagger=dag)
            schur = oracle.schur(lat, U, mp, mm, psi, dagger=dag)
            for prec in precs:
                print(f"small grid: L={L} Ls={Ls} dagger={dag} {prec}", flush=True)
                out = ctx.dwf_apply(x, mp, mm, dagger=dag, prec=prec).cpu().numpy()
                assert region_rel(out, full) <= PREC_TOL[prec]
                out = ctx.dwf_apply(x, mp, mm, dagger=dag, eo=True, prec=prec).cpu().numpy()
                assert rel(out, schur) <= PREC_TOL[prec]


@pytest.mark.parametrize("form", ["1", "0", "2"])
@pytest.mark.parametrize("Ls", [1, 3, 7, 8, 10, 12, 24, 33, 64])
def test_hop_forms(Ls, form, monkeypatch):
    monkeypatch.setenv("EOFA_BLOCKS", form)
    _check((4, 2, 6, 4), Ls, ("fp64", "fp32", "fp16", "bf16"))


@pytest.mark.parametrize("L,Ls", [((8, 8, 8, 32), 16), ((8, 8, 8, 34), 16), ((8, 8, 4, 16), 24), ((8, 8, 4, 18), 24)])
def test_grid_size_line(L, Ls):
    """2048 wavefronts of full lanes and 1024 of 48, and just above each."""
    _check(L, Ls, ("fp64", "fp16"))


@pytest.mark.parametrize("inner", ["fp64", "fp64_fused", "fp32", "fp16", "bf16"])
@pytest.mark.parametrize("Ls", [8, 10])
def test_solve_on_small_grid(inner, Ls):
    """The CG whose reductions run inside the hops and the direction update:
    the solutions' true residuals and the action, against the plain solver's."""
    from paper_1611_00298_amd import Context
    L = (4, 2, 6, 4)
    U, phi = din.random_gauge(L, 0.4, 751), din.gaussian_4d(L, 752)
    with Context(L, Ls, to_dev(U), M5=1.8, alpha=2.0) as ctx:
        ref = ctx.eofa_solve(to_dev(phi), 0.05, 1.0, tol=1e-12)
        got = ctx.eofa_solve(to_dev(phi), 0.05, 1.0, tol=1e-11, inner=inner)
    assert got[4]["converged"] and max(got[4]["true_resid"]) <= 1e-11
    # residual 1e-11 times the inverse's norm (smallest singular value above 0.01 here)
    assert rel(got[0].cpu().numpy(), ref[0].cpu().numpy()) <= 1e-9
    assert rel(got[1].cpu().numpy(), ref[1].cpu().numpy()) <= 1e-9
    assert abs(got[3] - ref[3]) <= 1e-9 * abs(ref[3])
