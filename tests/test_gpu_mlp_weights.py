"""Inference of the opacity network with second-layer weights of ordinary and
of very large size (the packed image scales them into half precision and the
hidden values by the inverse), against the oracle's exact network."""
import numpy as np
import pytest
import torch

from paper_2606_26268_amd import inputs as I
from tests.gpu_common import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", [1.0, 3e4, 3e6])
def test_inference_with_scaled_weights(orc, scale):
    """Ordinary weights: every point within the 2e-5 dex of the inference
    bound.  Scaled up by S the second layer saturates (h2 = -+1 exactly on
    both sides) wherever its pre-activation, spread over about S / 2, is past
    the -+25 where the FP32 activation is 1: all but 64 x 50 / (2.5 S / 2) of
    the points, 9 % at S = 3e4, have no other unit and keep the bound; the rest
    carry the rounding of pre-activations of that size and are finite."""
    from paper_2606_26268_amd import m1
    tab = I.make_table()
    p = I.make_uniform(I.CARTESIAN, (64, 1, 1), 1)
    p.opacity = tab
    rng = np.random.default_rng(3)
    th = I.mlp_init(7).astype(np.float64) + 0.05 * rng.normal(size=m1.M1_MLP_NPARAM)
    th[192:4288] *= scale                      # W2
    th = th.astype(np.float32)
    norm = np.array([f(tab[k].astype(np.float64)) for k in ("log10_kP", "log10_kR") for f in (np.mean, np.std)])
    s = m1.Solver(p, "p64")
    m1.m1_set_opacity_mlp(s.ctx, th, norm)
    n = 1027
    rho, T = 10 ** rng.uniform(-7.5, 5.5, n), 10 ** rng.uniform(-2.5, 2.5, n)
    dev = lambda a: torch.from_numpy(a).to("cuda")
    kP, kR = (torch.empty(n, dtype=torch.float64, device="cuda") for _ in range(2))
    m1.m1_opacity_eval(s.ctx, n, dev(rho), dev(T), kP, kR)
    s.sync()
    s.close()
    q = I.make_uniform(I.CARTESIAN, (2, 1, 1), 1)
    q.opacity = dict(tab, kind=I.OPAC_MLP)
    ref = orc.Oracle(q, dict(theta=th.astype(np.float64), norm=norm, bf16=False)).opacity(rho, T)
    share = 1.0 if scale == 1.0 else 1.0 - 64 * 50 / (2.5 * scale / 2) - 0.05
    for name, got, r in (("P", kP, ref[0]), ("R", kR, ref[1])):
        d = np.abs(np.log10(got.cpu().numpy()) - np.log10(r))
        say(f"  scale {scale:g} {name}: within 2e-5 dex {np.mean(d < 2e-5):.4f}, largest {d.max():.2e}")
        assert np.isfinite(d).all()
        assert np.mean(d < 2e-5) >= share
