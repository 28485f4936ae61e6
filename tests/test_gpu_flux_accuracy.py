"""Double precision: how far one explicit step's flux update is from the same update
in 80-bit arithmetic.  Cells come in runs of three equal ones, so every slope is
zero and a face between two runs is a Riemann problem of the two states; the
reference is the scheme's formulas in numpy's longdouble.  LEVEL is the rms error,
in units of 2^-53 E, of the kernels with an IEEE division and square root in every
place; refined hardware estimates, an ulp or less off each, may add 4 % (taking
s = sqrt(4 - 3 f^2) as the rounded product of 4 - 3 f^2 with 1 / s added 9 % to
the error of Fx)."""
import numpy as np
import pytest

from paper_2606_26268_amd import inputs as I
from tests.gpu_common import say

pytestmark = pytest.mark.gpu

RUNS = 1 << 15
LEVEL = dict(E=0.3883, Fx=0.1821, Fy=0.1227, Fz=0.1227)


def _reference(E, F, x):
    """Phi at the faces between runs (and within them) and the updated states."""
    def side(E, F):
        f2 = (F * F).sum(axis=0) / E ** 2
        s = np.sqrt(4 - 3 * f2)
        phi = F[0] / E
        m = 2 * phi / (2 + s)
        zeta = np.sqrt((s - 1) * (2 * s / 3 - phi * m))
        flux = np.stack([F[0], 3 * m / 2 * F[0] + (s - 1) / 3 * E, 3 * m / 2 * F[1], 3 * m / 2 * F[2]])
        return (phi - zeta) / s, (phi + zeta) / s, flux
    U = np.concatenate([E[None], F])
    L, R = U[:, :-1], U[:, 1:]
    lL, hL, pL = side(L[0], L[1:])
    lR, hR, pR = side(R[0], R[1:])
    SL, SR = np.minimum(np.minimum(lL, lR), 0), np.maximum(np.maximum(hL, hR), 0)
    phi = (SR * pL - SL * pR + SL * SR * (R - L)) / (SR - SL)
    return U[:, 1:-1] - x * (phi[:, 1:] - phi[:, :-1])


def test_flux_update_against_80_bit_arithmetic():
    from paper_2606_26268_amd import m1
    rng = np.random.default_rng(5)
    n = 3 * RUNS
    E = np.repeat(np.exp(0.5 * rng.standard_normal(RUNS)), 3)
    d = rng.standard_normal((3, RUNS))
    F = np.repeat(0.9 * rng.random(RUNS) * d / np.sqrt((d * d).sum(axis=0)), 3, axis=1) * E
    one = np.ones((1, 1, n))
    p = I.Problem("riemann", I.CARTESIAN, 1, (n, 1, 1), [np.arange(n + 1.0), np.array([0.0, 1.0]), np.array([0.0, 1.0])],
                  [[I.OUTFLOW] * 2] + [[I.PERIODIC] * 2] * 2, c_hat=1.0, c=1.0,
                  opacity=dict(kind=I.OPAC_CONSTANT, kP=0.0, kR=0.0, sigma=0.0),
                  fields=dict(E=E.reshape(1, 1, n), Fx=F[0].reshape(1, 1, n), Fy=F[1].reshape(1, 1, n), Fz=F[2].reshape(1, 1, n),
                              rho=one, mx=0 * one, my=0 * one, mz=0 * one, Eg=one))
    s = m1.Solver(p, "p64")
    m1.m1_step_explicit(s.ctx, 0.25)
    got = s.transported()
    assert s.diagnostics()["counters"][:2] == [0, 0]
    s.close()
    want = _reference(E.astype(np.longdouble), F.astype(np.longdouble), np.longdouble(0.25))
    rms = {}
    for k, w in zip(("E", "Fx", "Fy", "Fz"), want):
        e = (got[k].ravel()[1:-1].astype(np.longdouble) - w) / E[1:-1]
        rms[k] = float(np.sqrt((e * e).mean())) / 2.0 ** -53
    say("  rms error in units of 2^-53 E: " + " ".join(f"{k} {v:.4f}" for k, v in rms.items()))
    for k, v in rms.items():
        assert v < 1.04 * LEVEL[k], k
