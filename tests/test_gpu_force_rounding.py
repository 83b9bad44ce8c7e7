"""Rounding error of the force's sum over the fifth dimension, against 80-bit
arithmetic: no larger than that of a plain FP64 sum which forms each slice's
term first and then adds the slices of one system one by one."""
import numpy as np
import pytest

import dwf_inputs as din
from helpers import to_dev

pytestmark = pytest.mark.gpu


def _lower(mu, v):
    """(A_mu v)_j, A_k = -i sigma_k and A_t = 1, on two spins (last axis but one)."""
    a, b = v[..., 0, :], v[..., 1, :]
    return np.stack([(-1j * b, -1j * a), (-b, a), (-1j * a, 1j * b), (a, b)][mu], axis=-2)


def _sums(chiL, chiR, dtype):
    """B_mu(x) = sum_s sum_j h_j(x, s) g_j(x + mu, Ls-1-s)^dag of chi_L minus that of chi_R."""
    out = []
    for mu in range(4):
        per_system = []
        for chi in (chiL.astype(dtype), chiR.astype(dtype)):
            up, lo = chi[..., :2, :], _lower(mu, chi[..., 2:, :])
            h, g = up + lo, np.roll((up - lo)[::-1], -1, axis=4 - mu)
            b = 0
            for s in range(len(chi)):
                b = b + sum(h[s][..., j, :, None] * g[s][..., j, None, :].conj() for j in range(2))
            per_system.append(b)
        out.append(per_system[0] - per_system[1])
    return np.stack(out)


@pytest.mark.parametrize("L,Ls", [((4, 4, 4, 4), 16), ((4, 4, 4, 4), 64), ((8, 8, 8, 16), 24), ((8, 8, 8, 8), 7)])
def test_gradient_rounding(L, Ls):
    from paper_1611_00298_amd import Context
    chiL, chiR = din.gaussian_5d(L, Ls, 761), din.gaussian_5d(L, Ls, 762)
    with Context(L, Ls, to_dev(din.random_gauge(L, 0.4, 763)), M5=1.8, alpha=2.0, antiperiodic_t=False) as ctx:
        _, G, _ = ctx.eofa_force(0.05, 0.9, chiL=to_dev(chiL), chiR=to_dev(chiR), want_grad=True)
    B = _sums(chiL, chiR, np.clongdouble)

    def error(a):   # G = -k B: the factor is fitted, its own rounding is not the sum's
        f = np.sum(a * B.conj()) / np.sum(np.abs(B) ** 2)
        return float(np.sqrt(np.mean(np.abs(a - f * B) ** 2) / np.mean(np.abs(f * B) ** 2)))

    got, plain = error(G.cpu().numpy().astype(np.clongdouble)), error(_sums(chiL, chiR, np.complex128).astype(np.clongdouble))
    print(f"force rounding: L={L} Ls={Ls} {got:.3e}, plain sum {plain:.3e}", flush=True)
    # 72 V values or more: their mean square is known to 2 % or better; G adds one rounding of its own, at most 2.2e-16 / sqrt(12)
    assert got <= 1.05 * np.hypot(plain, 2.2e-16 / np.sqrt(12))
