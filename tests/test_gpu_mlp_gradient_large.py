"""m1_mlp_gradient past the largest single launch: 2^29 samples are 2^23 blocks of
512 threads, 2^32 threads."""
import numpy as np
import pytest
import torch

from paper_2606_26268_amd import inputs as I
from tests.gpu_common import say

pytestmark = pytest.mark.gpu


def test_gradient_of_more_samples_than_one_launch_takes():
    """The same 2^16 samples over and over have the gradient of one of them.  The
    partial gradients are added in four runs of 2^21 single-precision sums:
    relative rounding of at most 2^21 x 2^-24 = 0.125 of the summed magnitudes
    (sums of one sign; 4e-4 was seen).  Blocks left out or read from elsewhere are
    half of them or more."""
    from paper_2606_26268_amd import m1
    n = 1 << 29
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < (170 << 30):
        pytest.skip("needs 170 GiB of free device memory")
    tab = I.make_table()
    p = I.make_uniform(I.CARTESIAN, (64, 1, 1), 1)
    p.opacity = tab
    s = m1.Solver(p, "p64")
    theta = (I.mlp_init(7) + 0.05 * np.random.default_rng(1).standard_normal(m1.M1_MLP_NPARAM)).astype(np.float32)
    norm = np.array([f(tab[k].astype(np.float64)) for k in ("log10_kP", "log10_kR") for f in (np.mean, np.std)])
    m1.m1_set_opacity_mlp(s.ctx, theta, norm)
    few = torch.from_numpy(I.mlp_samples(1 << 16, 3)).cuda()
    _, want = m1.m1_mlp_gradient(s.ctx, few, 1 << 16, theta)
    many = few.repeat(n >> 16, 1)
    torch.cuda.synchronize()
    loss, got = m1.m1_mlp_gradient(s.ctx, many, n, theta)
    s.close()
    err = np.linalg.norm(got.astype(np.float64) - want) / np.linalg.norm(want)
    say(f"  {n} samples: gradient rel-L2 {err:.1e}, loss {loss:.4g}")
    assert np.isfinite(loss) and loss > 0
    assert err < 0.125
