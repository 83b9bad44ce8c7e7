"""The plain FP64 solver's launches on a grid of more than 2048 workgroups: a
converged system leaves no iteration's second half unused."""
import pytest

import dwf_inputs as din
from helpers import to_dev

pytestmark = pytest.mark.gpu


def test_no_work_after_convergence():
    from paper_1611_00298_amd import Context
    L, Ls = (16, 16, 16, 32), 8
    U, phi = to_dev(din.random_gauge(L, 0.4, 801)), to_dev(din.gaussian_4d(L, 802))
    with Context(L, Ls, U, M5=1.8, alpha=2.0) as ctx:
        def hops(**kw):
            ctx.timing_enable()
            out = ctx.eofa_solve(phi, 0.2, 0.8, **kw)
            return ctx.timing_query("hop")["count"], out[0], out[1], out[4]
        # per system: z = Mhat^dag r, then four hops an iteration, two in the last
        other = hops(tol=1e-30, maxiter=1, allow_noconv=True)[0] - 2 * 4
        n, cl, cr, st = hops(tol=1e-6)
        assert st["converged"] and n == other + 4 * sum(st["iters"])
        # a warm start that needs few iterations
        n, _, _, st = hops(tol=2e-7, x0=(cl, cr))
        print(f"warm start: iterations {st['iters']}, hops {n}", flush=True)
        guess = 2 * 2   # the residual of each system's guess
        assert st["converged"] and n == other + guess + 4 * sum(st["iters"])
