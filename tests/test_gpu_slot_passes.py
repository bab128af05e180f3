"""More bodies in one tile than the record sums take per pass over it (16 in a launch
of two steps, 8 in a D3Q19 step): forces on every body against the oracle, and bitwise
those of single steps."""
import numpy as np
import pytest

from paper_1901_08766_amd import inputs, inputs3

pytestmark = pytest.mark.gpu


def _bodies(n, width, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    b = np.zeros((n, width))
    b[:, 2 if width == 5 else 3] = rng.uniform(-0.02, 0.02, n)   # vx: the bodies' forces differ
    return b


# 16 bodies a tile fill one pass, 17 and 40 go on to a second and third
@pytest.mark.parametrize("n_bodies", [16, 17, 40])
@pytest.mark.parametrize("storage,launch,ny", [("f64", (2, 128), 760), ("f32", (4, 64), 2060)])
def test_pairs_of_steps(lbvp, oracle, n_bodies, storage, launch, ny):
    nx = 1021
    mask = np.zeros((ny, nx), dtype=np.uint8)
    cols = np.arange(nx)
    # rows of narrow strips, body after body, so that a tile of 256 nodes meets them all
    stripes = np.where(cols % 5 < 3, cols // 5 % n_bodies + 1, 0).astype(np.uint8)
    mask[3:40:2] = stripes
    mask[ny - 3] = stripes
    rng = np.random.Generator(np.random.PCG64(n_bodies))
    p = inputs.Problem(name="stripes", nx=nx, ny=ny, tau_plus=0.8, magic_lambda=0.25, eta=1e-3, mask=mask,
                       bodies=_bodies(n_bodies, 5, 1), ux_init=rng.uniform(-0.02, 0.02, (ny, nx)),
                       uy_init=rng.uniform(-0.02, 0.02, (ny, nx)))
    a, b = (lbvp.Solver(p, storage=storage, mem_fill=0xFF) for _ in range(2))
    for s in (a, b):
        s.set_launch(*launch)
        assert s.run_info[0] == 2
    a.step(6)
    for _ in range(6):
        b.step(1)
    (fa, ma, _), (fb, mb, _) = a.forces(), b.forces()
    assert np.array_equal(fa, fb) and np.array_equal(ma, mb)
    assert np.array_equal(a.populations(), b.populations())
    if storage == "f64":
        o = oracle.RefSolver(p)
        want, mass = o.step(6, record=True)
        assert np.abs(want).min(axis=(0, 2)).max() > 0.0
        # FP64 sums of under 10^4 node forces of O(1e-2)
        assert np.max(np.abs(fa - want)) <= 1e-12 * max(1.0, np.max(np.abs(want)))


@pytest.mark.parametrize("n_bodies", [8, 9, 30])
@pytest.mark.parametrize("launch", [(1, 128), (2, 64)])
def test_d3q19(lbvp3, ref3, n_bodies, launch):
    nx, ny, nz = 130, 12, 9
    mask = np.zeros((nz, ny, nx), dtype=np.uint8)
    cols = np.arange(nx)
    mask[2:6, 3:9] = np.where(cols % 4 < 3, cols // 4 % n_bodies + 1, 0)
    rng = np.random.Generator(np.random.PCG64(n_bodies))
    u = [rng.uniform(-0.02, 0.02, (nz, ny, nx)) for _ in range(3)]
    p = inputs3.Problem3(name="stripes", nx=nx, ny=ny, nz=nz, tau_plus=0.8, magic_lambda=0.25, eta=1e-3, mask=mask,
                         bodies=_bodies(n_bodies, 9, 2), ux_init=u[0], uy_init=u[1], uz_init=u[2])
    s = lbvp3.Solver3(p, storage="f64")
    s.set_launch(*launch)
    s.step(6)
    f, m, _ = s.forces()
    o = ref3.RefSolver3(p)
    want, mass = o.step(6, record=True)
    assert np.max(np.abs(f - want)) <= 1e-12 * max(1.0, np.max(np.abs(want)))
    assert np.max(np.abs(m - mass)) <= 1e-13 * np.max(mass)
