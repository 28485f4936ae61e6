"""A uniform isotropic radiation field at rest on a grid of thin rings or shells stays
at rest: the pressures of a cell's two unequal faces and the geometric source
cancel up to roundings of terms of the source's size.  With u the unit roundoff and
x = dt c_hat times the source's factor ((b - a) / ring, (b^2 - a^2) / (2 shell),
and cot(theta) times that in the polar direction), one step leaves at most some five
roundings of products and sums of x E / 3, twice as large in the spherical radial
direction: 5 u x E.  Two area factors rounded by themselves leave u dt c_hat E / (3
dR) instead, R / dR times that."""
import numpy as np
import pytest

from paper_2606_26268_amd import inputs as I
from tests.gpu_common import say

pytestmark = pytest.mark.gpu


def _step(geom, ndim, n, faces, bc, precision):
    from paper_2606_26268_amd import m1
    shape = (n[2], n[1], n[0])
    one, zero = np.ones(shape), np.zeros(shape)
    p = I.Problem("static", geom, ndim, n, faces, bc, c_hat=3.0, c=3.0,
                  opacity=dict(kind=I.OPAC_CONSTANT, kP=0.0, kR=0.0, sigma=0.0),
                  fields=dict(E=1.3 * one, Fx=zero, Fy=zero, Fz=zero, rho=one, mx=zero, my=zero, mz=zero, Eg=one))
    s = m1.Solver(p, precision)
    dt = s.max_dt(0.4)
    m1.m1_step_explicit(s.ctx, dt)
    got = s.transported()
    s.close()
    return got, 3.0 * dt


U = [("f32", 2.0 ** -24), ("p64", 2.0 ** -53)]


@pytest.mark.parametrize("precision,u", U)
@pytest.mark.parametrize("n,ndim", [((3000, 1, 1), 1), ((2000, 6, 1), 2), ((500, 16, 1), 2), ((700, 10, 7), 3)])
def test_static_isotropic_rings(precision, u, n, ndim):
    faces = [np.linspace(1.0, 2.0, n[0] + 1), np.linspace(0.0, 2 * np.pi, n[1] + 1), np.linspace(-1.0, 1.0, n[2] + 1)]
    got, dtc = _step(I.CYLINDRICAL, ndim, n, faces, [[I.OUTFLOW] * 2, [I.PERIODIC] * 2, [I.OUTFLOW] * 2], precision)
    a, b = faces[0][:-1], faces[0][1:]
    x = dtc * (b - a) / (0.5 * (b * b - a * a))
    worst = (np.abs(got["Fx"]) / (u * x * 1.3)).max()
    say(f"  {precision} {n}: largest radial flux {worst:.2f} u x E")
    assert worst <= 5
    assert (got["Fy"] == 0).all() and (got["Fz"] == 0).all()


@pytest.mark.parametrize("precision,u", U)
@pytest.mark.parametrize("n,ndim", [((2000, 6, 1), 2), ((20, 700, 1), 2), ((500, 16, 1), 2), ((300, 40, 7), 3)])
def test_static_isotropic_shells(precision, u, n, ndim):
    faces = [np.linspace(1.0, 2.0, n[0] + 1), np.linspace(0.4, 1.4, n[1] + 1), np.linspace(0.0, 2 * np.pi, n[2] + 1)]
    got, dtc = _step(I.SPHERICAL, ndim, n, faces, [[I.OUTFLOW] * 2, [I.OUTFLOW] * 2, [I.PERIODIC] * 2], precision)
    a, b = faces[0][:-1], faces[0][1:]
    x = dtc * (b * b - a * a) / (2 * (b ** 3 - a ** 3) / 3)
    t0, t1 = faces[1][:-1], faces[1][1:]
    cot = ((np.sin(t1) - np.sin(t0)) / (np.cos(t0) - np.cos(t1)))[:, None]
    worst = [(np.abs(got[k]) / (u * f * 1.3)).max() for k, f in (("Fx", x), ("Fy", cot * x))]
    say(f"  {precision} {n}: largest radial flux {worst[0]:.2f} u x E, polar {worst[1]:.2f} u x cot E")
    assert max(worst) <= 5
    assert (got["Fz"] == 0).all()
