"""Reference outputs of the opacity network in the double-precision form.

Both hidden layers run on the matrix cores with split operands and single
precision sums, so the network's last bits depend on how the operands are
split; in the double-precision form those bits reach the radiation flux.
network_step_p64.npz holds what the library gave with the 64 x 64 layer's
operands split into bfloat16 pairs (hi hi + hi lo + lo hi): the opacities at
seeded points, and the state after three Euler steps and one second-order
step of a small spherical grid.  Made on an MI355X by

    python tests/golden/make_network_reference.py tests/golden/network_step_p64.npz
"""
import os
import sys

import numpy as np

N_POINTS = 1031       # ragged against the 64 points of a wavefront


def make(device="cuda"):
    """The same calls on the library of the package on the path."""
    import torch

    from paper_2606_26268_amd import inputs as I
    from paper_2606_26268_amd import m1
    n = (13, 7, 10)
    faces = [np.geomspace(1.0, 10.0, n[0] + 1), I.uniform_faces(n[1], 0.0, np.pi), I.uniform_faces(n[2], 0.0, 2 * np.pi)]
    tab = I.make_table()
    p = I.make_random_state(I.SPHERICAL, n, 3, 41, faces, [[I.OUTFLOW] * 2, [I.OUTFLOW] * 2, [I.PERIODIC] * 2],
                            fmax=0.6, c_hat=3.0, opacity=dict(tab, kind=I.OPAC_MLP), vmax=0.2)
    rng = np.random.default_rng(7)
    theta = (I.mlp_init(7) + 0.05 * rng.standard_normal(m1.M1_MLP_NPARAM)).astype(np.float32)
    norm = np.array([f(tab[k].astype(np.float64)) for k in ("log10_kP", "log10_kR") for f in (np.mean, np.std)])
    s = m1.Solver(p, "p64", device=device, mlp=dict(theta=theta, norm=norm), second_order=True)
    rho = torch.from_numpy(10 ** rng.uniform(-7.5, 5.5, N_POINTS)).to(device)
    T = torch.from_numpy(10 ** rng.uniform(-2.5, 2.5, N_POINTS)).to(device)
    kP, kR = torch.empty_like(rho), torch.empty_like(rho)
    m1.m1_opacity_eval(s.ctx, N_POINTS, rho, T, kP, kR)
    dt = s.max_dt(0.4)
    s.step(dt, 3)
    s.step(dt, rk2=True)
    out = dict(s.state(), kP=kP.cpu().numpy(), kR=kR.cpu().numpy())
    s.close()
    return {k: v for k, v in out.items() if k != "rho"}


if __name__ == "__main__":
    sys.path.insert(0, os.environ.get("M1_ROOT", os.path.dirname(os.path.dirname(os.path.dirname(os.path.abspath(__file__))))))
    np.savez_compressed(sys.argv[1], **make())
