"""Natural <-> device layout passes and the FP64 operator whose last hop reads
and writes the natural layout, at the edges of their workgroups: Ls that
leaves ragged rows, the largest Ls, lattices with inactive rows, block and
per-site hops, against the oracle; in reduced precision against the stated
bounds.  The even sites of a Schur complement's input may hold anything."""
import numpy as np
import pytest

import dwf_inputs as din
import oracle
from helpers import PREC_TOL, region_rel, rel, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,Ls", [((2, 2, 2, 2), 1), ((2, 2, 2, 2), 64), ((4, 6, 2, 10), 5), ((6, 2, 4, 6), 13),
                                  ((4, 4, 4, 4), 24), ((2, 4, 6, 2), 32), ((10, 4, 2, 4), 18)])
def test_apply_layouts(L, Ls):
    import torch
    from paper_1611_00298_amd import Context
    mp, mm = 0.07, 0.6
    U, psi = din.random_gauge(L, 0.4, 711), din.gaussian_5d(L, Ls, 712)
    lat = oracle.Lattice(L, Ls, M5=1.8, alpha=2.0)
    with Context(L, Ls, to_dev(U), M5=1.8, alpha=2.0) as ctx:
        x = to_dev(psi)
        t, z, y, w = np.indices(psi.shape[1:5])
        odd = (t + z + y + w) % 2 == 1
        xo = x.clone()
        xo[:, to_dev(~odd)] = float("nan")
        for dag in (False, True):
            full, schur = oracle.ddwf(lat, U, mp, mm, psi, dagger=dag), oracle.schur(lat, U, mp, mm, psi, dagger=dag)
            for prec in ("fp64", "fp32", "fp16", "bf16"):
                print(f"layouts: L={L} Ls={Ls} dagger={dag} {prec}", flush=True)
                out = torch.full_like(x, float("nan"))
                ctx.dwf_apply(x, mp, mm, dagger=dag, prec=prec, out=out)
                assert region_rel(out.cpu().numpy(), full) <= PREC_TOL[prec]
                out.fill_(float("nan"))
                ctx.dwf_apply(xo if prec == "fp64" else x, mp, mm, dagger=dag, eo=True, prec=prec, out=out)
                o = out.cpu().numpy()
                assert rel(o, schur) <= PREC_TOL[prec]
                assert not o[:, ~odd].any()


def test_solution_layout_round_trip():
    """A converged solution handed back as the guess: the two layout passes
    return it, and the solve needs no iterations."""
    from paper_1611_00298_amd import Context
    L, Ls = (4, 6, 2, 4), 5
    U, phi = din.random_gauge(L, 0.4, 721), din.gaussian_4d(L, 722)
    with Context(L, Ls, to_dev(U), M5=1.8, alpha=2.0) as ctx:
        cl, cr, _, S, st = ctx.eofa_solve(to_dev(phi), 0.1, 0.8, tol=1e-12)
        assert min(st["iters"]) > 0
        cl2, cr2, _, S2, st2 = ctx.eofa_solve(to_dev(phi), 0.1, 0.8, tol=1e-11, x0=(cl, cr))
        assert st2["iters"] == [0, 0]
        assert rel(cl2.cpu().numpy(), cl.cpu().numpy()) <= 1e-13 and rel(cr2.cpu().numpy(), cr.cpu().numpy()) <= 1e-13


@pytest.mark.parametrize("L,Ls", [((4, 4, 4, 4), 8), ((8, 8, 16, 16), 12)])
def test_overlapping_operands(L, Ls):
    """A result whose memory overlaps an operand's gives what separate memory
    does, bit for bit: D_DWF and the Schur operator one slice further in the
    same buffer, in both directions, and the force and its gradient inside
    chi_L and chi_R."""
    import torch
    from paper_1611_00298_amd import Context
    from paper_1611_00298_amd._lib import check
    U = to_dev(din.random_gauge(L, 0.4, 723))
    x, y = to_dev(din.gaussian_5d(L, Ls, 724)), to_dev(din.gaussian_5d(L, Ls, 725))
    with Context(L, Ls, U, M5=1.8, alpha=2.0) as ctx:
        for dag in (False, True):
            for eo in (False, True):
                ref = ctx.dwf_apply(x, 0.1, 0.8, dagger=dag, eo=eo)
                for i, o in ((0, 1), (1, 0)):
                    print(f"overlap: L={L} Ls={Ls} dagger={dag} eo={eo} {i}->{o}", flush=True)
                    buf = torch.zeros((Ls + 1,) + tuple(x.shape[1:]), dtype=x.dtype, device=x.device)
                    buf[i:i + Ls] = x
                    assert torch.equal(ctx.dwf_apply(buf[i:i + Ls], 0.1, 0.8, dagger=dag, eo=eo, out=buf[o:o + Ls]), ref)
        Fr, Gr, _ = ctx.eofa_force(0.1, 0.8, chiL=x, chiR=y, want_grad=True)
        xa, ya, n = x.clone(), y.clone(), U.numel()
        F, G = xa.view(-1)[:n], ya.view(-1)[-n:]
        check(ctx.lib.eofa_force(ctx.handle, 0.1, 0.8, None, xa.data_ptr(), ya.data_ptr(), F.data_ptr(), G.data_ptr(),
                                 None, None))
        assert torch.equal(F, Fr.reshape(-1)) and torch.equal(G, Gr.reshape(-1))
