"""Graphs are captured once per distinct run, not per call: the same call repeated
through LBVP_GRAPH captures as many graphs as it has record phases and lattice
parities, and every later call replays one of them, bitwise like plain launches."""
from math import gcd

import numpy as np
import pytest

from paper_1901_08766_amd import inputs

pytestmark = pytest.mark.gpu

IO = ("inflow_eq", "outflow_zero_grad", "periodic", "periodic")


# single steps (small domains, 2-byte storage, in place) and two steps a launch: odd
# and even calls, calls of an odd number of pairs, several record phases
@pytest.mark.parametrize("nx,ny,storage,launch,aa", [(96, 40, "f32", None, False), (96, 40, "f32", None, True),
                                                     (300, 64, "f16", (8, 64), False),
                                                     (1021, 760, "f64", (2, 128), False)])
@pytest.mark.parametrize("n,every", [(41, 1), (101, 1), (41, 3), (23, 3), (42, 5), (22, 8), (40, 0)])
def test_repeated_calls_replay(lbvp, nx, ny, storage, launch, aa, n, every):
    p = inputs.random_state_problem(nx, ny, seed=17, n_disks=2, bc=IO, tau_plus=0.7)
    flags = lbvp.LAYOUT_AA if aa else 0
    s, plain = (lbvp.Solver(p, storage=storage, force_every=every, flags=flags) for _ in range(2))
    for x in (s, plain):
        if launch:
            x.set_launch(*launch)
    phases = every // gcd(n, every) if every else 1
    warm = 2 * phases     # calls until phase and lattice parity come round
    for _ in range(warm):
        s.step(n, graph=True)
    seen = s.run_info[2]
    assert 1 <= seen <= 2 * phases
    for _ in range(warm):
        s.step(n, graph=True)
    assert s.run_info[2] == seen
    for _ in range(2 * warm):
        plain.step(n)
    if aa and (2 * warm * n) % 2:
        s.step(1)
        plain.step(1)
    assert np.array_equal(s.populations(), plain.populations())
    if every:
        (fa, ma, sa), (fb, mb, sb) = s.forces(), plain.forces()
        assert sa == sb and np.array_equal(fa, fb) and np.array_equal(ma, mb)
    s.close()
    plain.close()
