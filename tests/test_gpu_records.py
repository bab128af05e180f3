"""Force and mass records whose sums several blocks share: no body, fewer bodies
than shares, as many, more; runs of one to several steps (the last records of a
run are summed on their own); alone and in batches, whose domains get fewer
shares each. FP64 against the oracle, everything else bitwise."""
import numpy as np
import pytest

from paper_1901_08766_amd import inputs, inputs3

pytestmark = pytest.mark.gpu

SPLITS = ((12,), (1, 1, 2, 3, 5))


@pytest.mark.parametrize("n_bodies", [0, 1, 7, 8, 20])
@pytest.mark.parametrize("every", [1, 3])
def test_records_2d(lbvp, oracle, n_bodies, every):
    p = inputs.random_state_problem(150, 70, seed=100 + n_bodies, n_disks=n_bodies, tau_plus=0.8)
    o = oracle.RefSolver(p)
    want, mass = o.step(12, record=True)
    got = []
    for split in SPLITS:
        s = lbvp.Solver(p, storage="f64", force_every=every)
        for n in split:
            s.step(n)
        got.append(s.forces())
    stream = s.stream
    for n_dom in (2, 20, 70):      # four, two and one share per domain
        m = [lbvp.Solver(p, storage="f64", force_every=every, stream=stream) for _ in range(n_dom)]
        for x in m:
            x.set_launch(*s.launch)
        b = lbvp.Batch(m, *s.launch)
        for n in (5, 7):
            b.step(n)
        got += [m[0].forces(), m[-1].forces()]
        b.close()
    f, q, first = got[0]
    assert first == every and len(q) == 12 // every
    # summed in FP64 over under 10^4 nodes of O(1e-2) forces
    assert np.max(np.abs(f - want[every - 1::every]), initial=0.0) <= 1e-12 * max(1.0, np.max(np.abs(want), initial=0.0))
    assert np.max(np.abs(q - mass[every - 1::every])) <= 1e-13 * np.max(mass)
    for g, r, _ in got[1:]:
        assert np.array_equal(g, f) and np.array_equal(r, q)


@pytest.mark.parametrize("n_bodies", [0, 1, 9])
@pytest.mark.parametrize("every", [1, 2, 5])
def test_records_3d(lbvp3, ref3, n_bodies, every):
    p = inputs3.random_state_problem3(40, 22, 19, seed=7, n_spheres=n_bodies, tau_plus=0.8)
    o = ref3.RefSolver3(p)
    want, mass = o.step(12, record=True)
    got = []
    for split in SPLITS:
        s = lbvp3.Solver3(p, storage="f64", force_every=every)
        for n in split:
            s.step(n)
        got.append(s.forces())
    m = [lbvp3.Solver3(p, storage="f64", force_every=every, stream=s.stream) for _ in range(9)]
    b = lbvp3.Batch3(m, *s.launch)
    for n in (5, 7):
        b.step(n)
    got += [m[0].forces(), m[-1].forces()]
    b.close()
    f, q, first = got[0]
    assert first == every and len(q) == 12 // every
    assert np.max(np.abs(f - want[every - 1::every]), initial=0.0) <= 1e-12 * max(1.0, np.max(np.abs(want), initial=0.0))
    assert np.max(np.abs(q - mass[every - 1::every])) <= 1e-13 * np.max(mass)
    for g, r, _ in got[1:]:
        assert np.array_equal(g, f) and np.array_equal(r, q)
