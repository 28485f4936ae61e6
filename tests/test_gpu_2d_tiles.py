"""2D transport in tiles (32 x 8 cells a block) and, on grids too thin for
them, a thread per cell: both sides of the rule that chooses (half of the
tiles' threads), whole and ragged tiles, every scheme variant and kind of
side, split and fused stages, against the oracle."""
import numpy as np
import pytest

from paper_2606_26268_amd import inputs as I
from tests.gpu_common import TOL_P64, TOL_P64_F1, assert_close, assert_close_f32, fp32_response, run_gpu, say
from tests.test_gpu_rk2_stages import CONST, _check, _problem

pytestmark = pytest.mark.gpu

# (cells, share of the tiles' threads): whole, one short, ragged in both
# directions, just past and just under half, thin either way
SIZES = [(32, 8), (31, 8), (64, 7), (100, 33), (33, 16), (32, 4), (5, 70), (70, 2), (1, 40)]


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("geom", [I.CARTESIAN, I.CYLINDRICAL, I.SPHERICAL])
@pytest.mark.parametrize("precision", ["p64", "f32"])
def test_sizes(orc, geom, n, precision):
    say(f"case 2d tiles geom={geom} n={n} {precision}")
    p = _problem(geom, n + (1,), 2, CONST, seed=500 + 10 * geom + n[0])
    o = orc.Oracle(p)
    dt = o.max_dt(0.4)
    ref, cnt = o.run(p.fields, dt, 3)
    got, diag = run_gpu(p, precision, 3, dt=dt)
    if precision == "p64":
        assert_close(got, ref, TOL_P64, label="2d tiles p64")
        assert diag["counters"][:3] == list(cnt[:3])
    else:
        assert_close_f32(got, ref, fp32_response(orc, p, 3, dt=dt), label="2d tiles f32")


@pytest.mark.parametrize("limiter,recon,riemann", [(0, 1, 0), (0, 0, 1), (0, 2, 0), (1, 0, 0), (1, 1, 1)])
@pytest.mark.parametrize("sides", ["reflect", "mixed"])
@pytest.mark.parametrize("rk2", [False, True])
@pytest.mark.parametrize("precision", ["p64", "f32"])
def test_variants(orc, limiter, recon, riemann, sides, rk2, precision):
    p = _problem(I.CARTESIAN, (45, 19, 1), 2, CONST, seed=600 + 4 * limiter + recon)
    p.limiter, p.recon, p.riemann = limiter, recon, riemann
    if sides == "reflect":
        p.bc = [[I.REFLECT, I.REFLECT], [I.REFLECT, I.REFLECT], p.bc[2]]
    else:
        p.bc = [[I.REFLECT, I.OUTFLOW], [I.OUTFLOW, I.REFLECT], p.bc[2]]
    label = f"2d variant limiter={limiter} recon={recon} riemann={riemann} {sides} rk2={rk2}"
    say(f"case {label} {precision}")
    o = orc.Oracle(p)
    dt = o.max_dt(0.4)
    ref, _ = o.run(p.fields, dt, 3, rk2=rk2)
    from paper_2606_26268_amd import m1
    s = m1.Solver(p, precision, second_order=rk2)
    s.step(dt, 3, rk2=rk2)
    got = s.state()
    s.close()
    if precision == "p64":
        # the PLUTO and clip treatments put faces at f = 1 exactly
        assert_close(got, ref, TOL_P64 if recon == 0 else TOL_P64_F1, label=label)
    else:
        assert_close_f32(got, ref, fp32_response(orc, p, 3, dt=dt, rk2=rk2), label=label, f1=recon == 2)


@pytest.mark.parametrize("n", [(40, 21), (6, 50)])
@pytest.mark.parametrize("opacity", ["powerlaw", "table"])
@pytest.mark.parametrize("precision", ["p64", "f32"])
def test_fused_stages(orc, n, opacity, precision):
    op = dict(kind=1, k0=0.7, rho0=1.1, alpha=0.8, T0=0.9, beta=-2.5, sigma=0.3) if opacity == "powerlaw" else I.make_table()
    _check(orc, _problem(I.SPHERICAL, n + (1,), 2, op, seed=700 + n[0]), precision, 3, f"2d stages {opacity} n={n}")
