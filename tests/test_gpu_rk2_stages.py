"""The second-order step where one kernel takes a stage's transport and
implicit step together (constant, power-law and tabulated opacities), against
the oracle: every dimension and geometry, grids that end inside a tile, a wave
or a z chunk, periodic wrap shorter than the stencil, irradiation and
absorption, the 1D/2D variants, and its place in a run beside the split
steps (the power law's optical depths change hands between the stages)."""
import numpy as np
import pytest

from paper_2606_26268_amd import inputs as I
from tests.gpu_common import TOL_P64, assert_close, assert_close_f32, fp32_response, say

pytestmark = pytest.mark.gpu

POWER = dict(kind=1, k0=0.7, rho0=1.1, alpha=0.8, T0=0.9, beta=-2.5, sigma=0.3)
CONST = dict(kind=0, kP=1.0, kR=2.0, sigma=0.5)


def _faces(geom, n, ndim):
    if geom == I.CARTESIAN:
        return [I.uniform_faces(n[d], 0.0, 1.0) if d < ndim else np.array([0.0, 1.0]) for d in range(3)]
    if geom == I.CYLINDRICAL:
        return [I.uniform_faces(n[0], 0.5, 2.0), I.uniform_faces(n[1], 0.0, 2 * np.pi), I.uniform_faces(n[2], -1.0, 1.0)]
    return [np.geomspace(1.0, 10.0, n[0] + 1), I.uniform_faces(n[1], 0.0, np.pi), I.uniform_faces(n[2], 0.0, 2 * np.pi)]


def _bc(geom):
    P, O = [I.PERIODIC] * 2, [I.OUTFLOW] * 2
    return {I.CARTESIAN: [P, O, P], I.CYLINDRICAL: [O, P, O], I.SPHERICAL: [O, O, P]}[geom]


def _problem(geom, n, ndim, opacity, seed, special=False):
    p = I.make_random_state(geom, n, ndim, seed, _faces(geom, n, ndim), _bc(geom), fmax=0.9, c_hat=3.0,
                            opacity=opacity, vmax=0.3)
    if special:
        p.irr = np.exp(np.random.default_rng(seed).standard_normal(p.shape)) * 0.5
        p.absorb_only = 1
    return p


def _check(orc, p, precision, steps, label, split=False):
    """`steps` second-order steps; with split, an Euler step before and after."""
    from paper_2606_26268_amd import m1
    say(f"case {label} {precision}")
    o = orc.Oracle(p)
    dt = o.max_dt(0.4)
    s = m1.Solver(p, precision, second_order=True)
    if split:
        s.step(dt)
    s.step(dt, steps, rk2=True)
    if split:
        s.step(dt)
    got, cnt = s.state(), s.diagnostics()["counters"]
    s.close()
    ref = p.fields
    if split:
        ref, _ = o.run(ref, dt, 1)
    ref, rcnt = o.run(ref, dt, steps, rk2=True)
    if split:
        ref, _ = o.run(ref, dt, 1)
    if precision == "p64":
        assert_close(got, ref, TOL_P64, label=label)
        if not split:
            assert cnt[:3] == list(rcnt[:3])
    else:
        assert_close_f32(got, ref, fp32_response(orc, p, steps, dt=dt, rk2=True), label=label)


@pytest.mark.parametrize("geom,n,ndim", [
    (I.CARTESIAN, (257, 1, 1), 1), (I.SPHERICAL, (50, 1, 1), 1), (I.CARTESIAN, (37, 23, 1), 2),
    (I.CYLINDRICAL, (29, 17, 1), 2), (I.CARTESIAN, (33, 17, 18), 3), (I.CARTESIAN, (5, 9, 1), 3),
    (I.CYLINDRICAL, (21, 13, 11), 3), (I.SPHERICAL, (64, 16, 3), 3)])
@pytest.mark.parametrize("opacity", ["constant", "powerlaw", "table"])
@pytest.mark.parametrize("precision", ["p64", "f32"])
def test_fused_stages_match_oracle(orc, geom, n, ndim, opacity, precision):
    op = {"constant": CONST, "powerlaw": POWER, "table": I.make_table()}[opacity]
    p = _problem(geom, n, ndim, op, seed=300 + 7 * geom + ndim)
    _check(orc, p, precision, 4, f"stages geom={geom} n={n} ndim={ndim} {opacity}")


@pytest.mark.parametrize("n,ndim", [((45, 11, 1), 2), ((34, 9, 7), 3)])
@pytest.mark.parametrize("opacity", ["constant", "powerlaw"])
def test_fused_stages_irradiated_absorbing(orc, n, ndim, opacity):
    p = _problem(I.CARTESIAN, n, ndim, CONST if opacity == "constant" else POWER, seed=17, special=True)
    _check(orc, p, "p64", 4, f"stages irradiated absorbing n={n} {opacity}")


def test_split_stages_past_the_cell_limit(orc):
    """FP64, power law, 3D: just past the cell count up to which stages fuse."""
    p = _problem(I.CARTESIAN, (89, 80, 74), 3, POWER, seed=5)
    _check(orc, p, "p64", 1, "stages past the cell limit")


@pytest.mark.parametrize("variant", [dict(recon=1, riemann=1), dict(limiter=1)])
def test_fused_stages_2d_variants(orc, variant):
    p = _problem(I.CARTESIAN, (41, 19, 1), 2, POWER, seed=23)
    for k, v in variant.items():
        setattr(p, k, v)
    _check(orc, p, "p64", 4, f"stages 2D {variant}")


@pytest.mark.parametrize("n,ndim", [((300, 1, 1), 1), ((35, 18, 9), 3)])
def test_fused_stages_between_split_steps(orc, n, ndim):
    p = _problem(I.CARTESIAN, n, ndim, POWER, seed=29)
    _check(orc, p, "p64", 3, f"stages between split steps n={n}", split=True)
