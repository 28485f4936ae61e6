"""A bound opacity table is complete when m1_set_opacity_table returns: a context
that is given another, non-blocking stream right after it reads the new table's
records, however busy the stream was that the table was bound on."""
import numpy as np
import pytest
import torch

from paper_2606_26268_amd import inputs as I
from tests.gpu_common import say

pytestmark = pytest.mark.gpu


def _context(m1):
    faces = [I.uniform_faces(2, 0.0, 1.0), np.array([0.0, 1.0]), np.array([0.0, 1.0])]
    return m1.m1_create(1, (2, 1, 1), faces, [[I.PERIODIC] * 2] * 3, I.CARTESIAN, 1.0)


def _bind(m1, ctx, tab):
    m1.m1_set_opacity_table(ctx, tab["nr"], tab["nt"], tab["lr0"], tab["lr1"], tab["lt0"], tab["lt1"], tab["lr_off"],
                            tab["lt_off"], tab["log10_kP"], tab["log10_kR"], 0.0)


def _eval(m1, ctx, rho, T):
    kP, kR = torch.zeros_like(rho), torch.zeros_like(rho)
    torch.cuda.synchronize()
    m1.m1_opacity_eval(ctx, rho.numel(), rho, T, kP, kR)
    m1.m1_sync(ctx)
    return kP.cpu().numpy(), kR.cpu().numpy()


def test_table_bound_on_a_busy_stream_serves_the_next_stream():
    from paper_2606_26268_amd import m1
    tab = I.make_table()
    rng = np.random.default_rng(2)
    rho = torch.from_numpy(10 ** rng.uniform(-6, 4, 4099)).cuda()
    T = torch.from_numpy(10 ** rng.uniform(-2, 2, 4099)).cuda()
    ref = _context(m1)
    _bind(m1, ref, tab)
    want = _eval(m1, ref, rho, T)
    m1.m1_destroy(ref)
    busy, other = torch.cuda.Stream(), torch.cuda.Stream()     # both non-blocking
    ctx = _context(m1)
    m1.m1_set_stream(ctx, busy.cuda_stream)
    done = torch.cuda.Event()
    with torch.cuda.stream(busy):
        torch.cuda._sleep(20_000_000)                           # about 0.2 s at the counter's 100 MHz, else 10 ms
        done.record()
    _bind(m1, ctx, tab)
    say(f"  the busy stream's earlier work is done on return: {done.query()}")
    assert done.query()
    m1.m1_set_stream(ctx, other.cuda_stream)
    got = _eval(m1, ctx, rho, T)
    m1.m1_destroy(ctx)
    for a, b in zip(got, want):
        assert np.array_equal(a, b)
