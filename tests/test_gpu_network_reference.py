"""The opacity network's arithmetic in the double-precision form stays that of
the stored reference (tests/golden/make_network_reference.py): the way the
64 x 64 layer's operands are split decides the last single-precision bits of
the opacities, and through the flux damping parts in 1e8 of the flux, far
beyond the rounding of the double-precision step itself."""
import os

import numpy as np
import pytest

from tests.golden import make_network_reference as ref
from tests.gpu_common import assert_close, say

pytestmark = pytest.mark.gpu

PATH = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "network_step_p64.npz")


def test_double_precision_network_steps_match_the_reference():
    """Opacities: the same FP32 operations in the same order, so the same
    numbers up to how the compiler fuses the last ones: one rounding of the
    exponent of 2^(log2 kappa), 2^-24 x 32 x ln 2 = 1.3e-6 for |log2 kappa| <
    32.  State: four steps of double-precision rounding (the parity bounds of
    that form, 1e-12 in L1 and 1e-10 in the maximum); another split of the
    operands moves the flux by 1e-8."""
    want, got = np.load(PATH), ref.make()
    for k in ("kP", "kR"):
        d = np.abs(got[k] / want[k] - 1.0)
        say(f"  {k}: largest relative difference {d.max():.2e}, differing {np.mean(d > 0):.3f}")
        assert np.abs(np.log2(want[k])).max() < 32
        assert d.max() < 1.3e-6
    assert_close(got, want, dict(l1=1e-12, linf=1e-10), fields=("E", "Fx", "Fy", "Fz", "mx", "my", "mz", "Eg"),
                 label="network, double precision")
