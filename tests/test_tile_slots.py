"""The tiled transport's face stage writes x fluxes where x slopes lie in LDS, with
no workgroup barrier between the two: every slot is written by a lane of the
wavefront that holds all of its readers, after a wave barrier that follows those
reads (LimO3 reads the neighbour's slope from an array of its own).  The tasks
are those of transport_tile.h, with its sizes."""
import os
import re

import pytest

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_26268_amd", "csrc",
                      "transport_tile.h")


@pytest.fixture(scope="module")
def source():
    return re.sub(r"//[^\n]*", "", open(HEADER).read())


@pytest.mark.parametrize("TY", [8, 16])
def test_x_fluxes_stay_within_their_wavefront(source, TY):
    TX = int(re.search(r"TX = (\d+)", source).group(1))
    assert re.search(r"XS = TX \+ 2", source)
    XS = TX + 2
    reads, writes = {}, {}
    for tid in range(TX * TY):                                # pass 0: the face left of the thread's column
        xs = tid // TX * XS + tid % TX
        for slot in (xs, xs + 1):
            reads.setdefault(slot, set()).add((tid // 64, "pass 0", tid))
        writes.setdefault(xs, set()).add((tid // 64, "pass 0", tid))
    for t in range(TY):                                       # pass 2: the faces right of the last column
        for slot in (t * XS + TX, t * XS + TX + 1):
            reads.setdefault(slot, set()).add((t // 64, "pass 2", t))
        writes.setdefault(t * XS + TX + 1, set()).add((t // 64, "pass 2", t))
    for slot, by in writes.items():
        assert len(by) == 1, slot                             # one writer
        wave, when, lane = next(iter(by))
        for w, p, r in reads[slot]:
            assert w == wave and p == when, slot              # its readers: same wavefront, same pass
            assert r == lane or p == "pass 0", slot           # another lane only where the wave barrier stands


def test_a_wave_barrier_separates_the_reads_from_the_stores(source):
    face = source[source.index("slc[v] = LIMO3"):source.index("dst[v * fs + fo] = fl[v]")]
    assert re.search(r"if \(p == 0 && !LIMO3\)\s*\{\s*__builtin_amdgcn_fence\(__ATOMIC_ACQ_REL, \"wavefront\"\);\s*"
                     r"__builtin_amdgcn_wave_barrier\(\);", face)
    assert "static_assert(64 % TX == 0" in source
