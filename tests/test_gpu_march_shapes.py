"""Two steps per launch against single ones where lbvp_get_run_info says that pairs run:
strips of one column, ragged ends inside a vector, chunks of 2 to 6 rows with a shorter
last one, all x sides, record phases, graphs, state blobs and the oracle."""
import numpy as np
import pytest

from paper_1901_08766_amd import inputs

pytestmark = pytest.mark.gpu

IO = ("inflow_eq", "outflow_zero_grad", "periodic", "periodic")
OI = ("outflow_zero_grad", "inflow_eq", "periodic", "periodic")
OO = ("outflow_zero_grad", "outflow_zero_grad", "periodic", "periodic")
PP = ("periodic",) * 4


def _pair(lbvp, p, storage, every, launch, rows):
    s = [lbvp.Solver(p, storage=storage, force_every=every, mem_fill=0xFF) for _ in range(2)]
    for x in s:
        x.set_launch(*launch)
        assert x.run_info[:2] == (2, rows)
    return s


def _same(a, b):
    fa, fb = a.fields(), b.fields()
    for k in fa:
        assert np.array_equal(fa[k], fb[k]), k
    assert np.array_equal(a.populations(), b.populations())
    (ga, ma, sa), (gb, mb, sb) = a.forces(), b.forces()
    assert sa == sb and np.array_equal(ga, gb) and np.array_equal(ma, mb)


@pytest.mark.parametrize("nx,ny,storage,launch,rows,bc", [
    (513, 7201, "f32", (4, 128), 6, IO), (257, 14300, "f32", (4, 64), 6, PP), (1023, 2051, "f32", (4, 256), 3, OI),
    (1030, 2041, "f32", (4, 128), 4, OO), (2049, 1031, "f32", (4, 64), 4, PP),
    (257, 5361, "f64", (2, 128), 6, OI), (129, 10700, "f64", (2, 64), 6, IO), (515, 3309, "f64", (2, 256), 6, PP),
    (1024, 751, "f64", (2, 64), 2, IO), (1021, 755, "f64", (2, 256), 2, OO), (699, 2305, "f64", (2, 128), 5, PP)])
def test_pairs_are_bitwise_single_steps(lbvp, nx, ny, storage, launch, rows, bc):
    p = inputs.random_state_problem(nx, ny, seed=(nx, ny), n_disks=4, bc=bc,
                                    body_force=(0.0, 0.0) if bc == IO else (1e-5, -2e-5))
    a, b = _pair(lbvp, p, storage, 1, launch, rows)
    a.step(7, keep_fields=True)
    for i in range(7):
        b.step(1, keep_fields=i == 6)
    _same(a, b)
    a.close()
    b.close()


@pytest.mark.parametrize("every", [0, 1, 2, 3, 5])
@pytest.mark.parametrize("graph", [False, True])
def test_record_phases_and_graphs(lbvp, every, graph):
    p = inputs.random_state_problem(1021, 760, seed=5, n_disks=5, bc=IO)
    a, b = _pair(lbvp, p, "f64", every, (2, 128), 2)
    done = 0
    for n in (1, 6, 3, 6, 2, 6):
        a.step(n, graph=graph)
        for _ in range(n):
            b.step(1)
        done += n
        assert np.array_equal(a.populations(), b.populations()), done
    a.step(5, keep_fields=True, graph=graph)
    for i in range(5):
        b.step(1, keep_fields=i == 4)
    if every:
        _same(a, b)
    else:
        assert np.array_equal(a.populations(), b.populations())


def test_state_blobs_do_not_tell(lbvp):
    """A state saved after pairs is the one saved after single steps, byte for byte,
    and a run goes on from it."""
    p = inputs.random_state_problem(1024, 2101, seed=6, n_disks=3, bc=IO)   # rows without padding
    a, b = _pair(lbvp, p, "f32", 1, (4, 256), 3)
    a.step(6, keep_fields=True)
    for i in range(6):
        b.step(1, keep_fields=i == 5)
    _same(a, b)   # drains the records
    blob = a.save_state()
    assert np.array_equal(blob, b.save_state())
    b.load_state(blob)
    a.step(5, keep_fields=True)
    b.step(5, keep_fields=True)
    assert np.array_equal(a.populations(), b.populations())


@pytest.mark.parametrize("nx,ny,launch,rows", [(1024, 751, (2, 64), 2), (515, 3309, (2, 256), 6)])
def test_pairs_against_the_oracle(lbvp, oracle, nx, ny, launch, rows):
    p = inputs.random_state_problem(nx, ny, seed=9, n_disks=3, bc=IO)
    s, _ = _pair(lbvp, p, "f64", 1, launch, rows)
    o = oracle.RefSolver(p)
    s.step(11, keep_fields=True)
    want, mass = o.step(11, record=True)
    assert np.max(np.abs(s.populations() - o.populations())) <= 1e-12
    f, m, _ = s.forces()
    assert np.max(np.abs(f - want)) <= 1e-12 * max(1.0, np.max(np.abs(want)))
    assert np.max(np.abs(m - mass)) <= 1e-13 * np.max(mass)
