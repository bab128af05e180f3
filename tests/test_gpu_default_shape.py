"""A default launch shape that gives way to (vec, 256) between runs: graphs captured
before, undrained records and the mask tables follow; populations are bitwise those of
plain steps, and every record is there."""
import numpy as np
import pytest
import torch

from paper_1901_08766_amd import inputs

pytestmark = pytest.mark.gpu

IO = ("inflow_eq", "outflow_zero_grad", "periodic", "periodic")


@pytest.mark.parametrize("storage", ["f16", "bf16"])
def test_narrowed_default_next_to_a_wide_one(lbvp, storage):
    p = inputs.random_state_problem(2305, 1153, seed=3, n_disks=4, bc=IO, tau_plus=0.8)
    q = inputs.random_state_problem(2048, 1200, seed=4, n_disks=3, bc=IO, tau_plus=0.8)
    stream = torch.cuda.Stream()
    a, b, plain = (lbvp.Solver(x, storage=storage, stream=stream) for x in (p, q, p))
    assert a.launch == (4, 128) and b.launch == (4, 256)
    a.step(4, graph=True)
    lbvp.lbvp_batch_step_static([a.ctx, b.ctx], 3, 0)
    assert a.launch == (4, 256)
    a.step(4, graph=True)
    plain.step(11)
    assert np.array_equal(a.populations(), plain.populations())
    (fa, ma, sa), (fb, mb, sb) = a.forces(), plain.forces()
    assert sa == sb == 1 and len(ma) == len(mb) == 11
    # the same FP64 partials grouped by other tiles: 2.7 M node values of order one
    assert np.max(np.abs(ma - mb)) <= 1e-12 * np.max(mb)
    assert np.max(np.abs(fa - fb)) <= 1e-9 * max(1.0, np.max(np.abs(fb)))
