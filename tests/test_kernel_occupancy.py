"""What the header and the launch bounds rest on, from the compiler's resource
remarks of the built library: no kernel at all uses per-lane scratch or spills
vector registers (m1_step_noalloc promises that nothing sets scratch up), and the
tiled transport, the fused stages, the network and the training kernel keep the
waves per SIMD that their measurements were taken with."""
import json
import os
import re

import pytest

PATH = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_26268_amd", "_build",
                    "kernel_resources.json")


@pytest.fixture(scope="module")
def res():
    if not os.path.exists(PATH):
        pytest.skip("library not built in this tree")
    return json.load(open(PATH))


def test_no_scratch_and_no_vector_spill_anywhere(res):
    assert len(res) > 100
    assert not {k: v for k, v in res.items() if v["scratch"] or v["vgpr_spill"]}


# kernel and template arguments (R: d or f; geometry 0..2; then the flags) -> instances, waves per SIMD
@pytest.mark.parametrize("pattern,count,waves", [
    # <R, GEOM, GENERAL, TY, LIMO3>
    (r"k_transport3dIfLi\dELb[01]ELi(8|16)ELb[01]E", 12, 4),
    (r"k_transport3dIdLi\dELb0ELi8ELb0E", 3, 3),
    (r"k_transport3dIdLi\dELb1ELi8ELb[01]E", 6, 2),
    # <R, GEOM, GENERAL, LIMO3>
    (r"k_transport2dIfLi\dELb[01]ELb0E", 6, 6),
    (r"k_transport2dIfLi\dELb1ELb1E", 3, 4),
    (r"k_transport2dIdLi\dELb[01]ELb0E", 6, 3),
    (r"k_transport2dIdLi\dELb1ELb1E", 3, 2),
    # <R, GEOM, TY, CONST_OPAC>
    (r"k_stage3dIfLi\dELi(8|16)ELb[01]E", 12, 4),
    (r"k_stage3dIdLi\dELi8ELb1E", 3, 3),
    (r"k_stage3dIdLi\dELi8ELb0E", 3, 2),
    # <R, GEOM, GENERAL, LIMO3, CONST_OPAC>
    (r"k_stage2dIfLi\dELb[01]ELb0ELb[01]E", 12, 6),
    (r"k_stage2dIfLi\dELb1ELb1ELb[01]E", 6, 4),
    (r"k_stage2dIdLi\dELb[01]ELb0ELb[01]E", 12, 3),
    (r"k_stage2dIdLi\dELb1ELb1ELb[01]E", 6, 2),
    (r"k_implicit_mlpI[df]Lb[01]E", 4, 4),
    (r"k_mlp_fwd_bwdE", 1, 4),
])
def test_kernels_keep_their_waves(res, pattern, count, waves):
    ks = {k: v["waves_per_simd"] for k, v in res.items() if re.search(r"\d" + pattern, k)}
    assert len(ks) == count, sorted(ks)
    assert min(ks.values()) >= waves, ks
