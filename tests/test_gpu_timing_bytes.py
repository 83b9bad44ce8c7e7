"""The algorithmic bytes that the timing entry point reports for the FP64 hops of
a mixed-precision solve: a reliable update reads five FP64 fields and writes one
and, in the inner precision, the residual."""
import pytest

import dwf_inputs as din
from helpers import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("inner,width", [("fp16", 52), ("bf16", 48), ("fp32", 96)])
def test_residual_hop_bytes(inner, width):
    from paper_1611_00298_amd import Context
    L, Ls = (4, 4, 4, 4), 8
    Vh = 4 ** 4 // 2
    with Context(L, Ls, to_dev(din.random_gauge(L, 0.4, 811)), M5=1.8, alpha=2.0) as ctx:
        phi, got = to_dev(din.gaussian_4d(L, 812)), []
        for tol in (1e-6, 1e-11):
            ctx.timing_enable()
            st = ctx.eofa_solve(phi, 0.1, 0.8, tol=tol, inner=inner)[4]
            q = ctx.timing_query("hop64")
            got.append((sum(st["reliable_updates"]), q["count"], q["bytes"]))
    (n0, c0, b0), (n1, c1, b1) = got
    assert n1 > n0 and c1 - c0 == 2 * (n1 - n0)
    links = 72 * 16 * Vh
    assert b1 - b0 == (n1 - n0) * (Vh * Ls * (5 * 192 + width) + 2 * links)
