"""Where the FP64 hop takes its latency form: the operator on both sides of each
line against the oracle, and solves beyond the lines, which may not be slower
than with the throughput form forced."""
import time

import pytest

import dwf_inputs as din
import oracle
from helpers import PREC_TOL, region_rel, rel, to_dev

pytestmark = pytest.mark.gpu


# wavefronts: 1024 and 1152 of 16 slices; 768 and 816 of 4; 1536 and 1792 of 32; one and two slices
@pytest.mark.parametrize("L,Ls", [((8, 8, 8, 16), 16), ((8, 8, 8, 18), 16), ((8, 8, 12, 32), 4), ((8, 8, 12, 34), 4),
                                  ((8, 8, 8, 12), 32), ((8, 8, 8, 14), 32), ((4, 6, 8, 4), 1), ((4, 6, 8, 4), 2)])
def test_operator_at_the_lines(L, Ls):
    from paper_1611_00298_amd import Context
    mp, mm = 0.07, 0.8
    U, psi = din.random_gauge(L, 0.4, 781), din.gaussian_5d(L, Ls, 782)
    lat = oracle.Lattice(L, Ls, M5=1.8, alpha=2.0)
    with Context(L, Ls, to_dev(U), M5=1.8, alpha=2.0) as ctx:
        x = to_dev(psi)
        for dag in (False, True):
            full, schur = oracle.ddwf(lat, U, mp, mm, psi, dagger=dag), oracle.schur(lat, U, mp, mm, psi, dagger=dag)
            for prec in ("fp64", "fp32", "fp16"):
                print(f"hop lines: L={L} Ls={Ls} dagger={dag} {prec}", flush=True)
                out = ctx.dwf_apply(x, mp, mm, dagger=dag, prec=prec).cpu().numpy()
                assert region_rel(out, full) <= PREC_TOL[prec]
                out = ctx.dwf_apply(x, mp, mm, dagger=dag, eo=True, prec=prec).cpu().numpy()
                assert rel(out, schur) <= PREC_TOL[prec]


@pytest.mark.parametrize("L,Ls", [((12, 12, 12, 24), 4), ((12, 12, 12, 12), 8), ((12, 12, 12, 12), 1)])
def test_no_slower_than_the_throughput_form(L, Ls, monkeypatch):
    """30 iterations of the plain FP64 solver: the default against EOFA_BLOCKS=0
    (per-site throughput form), the two timed in turn."""
    import torch
    from paper_1611_00298_amd import Context
    U, phi = to_dev(din.random_gauge(L, 0.4, 783)), to_dev(din.gaussian_4d(L, 784))
    default = Context(L, Ls, U, M5=1.8, alpha=2.0)
    monkeypatch.setenv("EOFA_BLOCKS", "0")
    forced = Context(L, Ls, U, M5=1.8, alpha=2.0)
    t = [1e9, 1e9]
    for _ in range(8):
        for i, ctx in enumerate((default, forced)):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            ctx.eofa_solve(phi, 0.05, 1.0, tol=1e-30, maxiter=30, want_mphi=False, allow_noconv=True)
            t[i] = min(t[i], time.perf_counter() - t0)
    print(f"hop lines: L={L} Ls={Ls} default {t[0] * 1e3:.2f} ms, throughput form {t[1] * 1e3:.2f} ms", flush=True)
    assert t[0] <= 1.07 * t[1]
    default.close()
    forced.close()
