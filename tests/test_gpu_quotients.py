"""The FP64 step's quotients, 36 drho / 36 and 1 / (36 rho), are the correctly rounded
ones: a step from populations of one rounded sum gives bitwise the density and
velocity that IEEE division gives, at random densities, next to the powers of two and
just below them (mantissas of ones), and the same zeros, infinities and NaNs."""
from fractions import Fraction

import numpy as np
import pytest

from paper_1901_08766_amd import inputs, inputs3

pytestmark = pytest.mark.gpu


def _densities(n, rest):
    """n rest populations' deviations: densities 1 + rest h / 36 from 0.25 to 4 and
    runs of neighbouring doubles around 1, 2 and where 36 rho passes 32 and 64."""
    rng = np.random.Generator(np.random.PCG64(11))
    h = (np.exp(rng.uniform(np.log(0.25), np.log(4.0), size=n)) - 1.0) * 36.0 / rest
    k = np.arange(-200, 200)
    for i, rho in enumerate((1.0, 2.0, 32.0 / 36.0, 64.0 / 36.0)):
        h[400 * i:400 * (i + 1)] = (rho - 1.0) * 36.0 / rest + k * 2.0 ** -53
    return h


def _step_2d(lbvp, g):
    ny, nx = g.shape[1:]
    p = inputs.Problem(name="quotients", nx=nx, ny=ny, tau_plus=0.8, magic_lambda=0.25, eta=1e-4)
    s = lbvp.Solver(p, storage="f64")
    s.set_populations(g)
    s.step(1, keep_fields=True)
    f = s.fields()
    s.close()
    return f["rho"], f["ux"]


def _step_3d(lbvp3, g):
    nz, ny, nx = g.shape[1:]
    p = inputs3.Problem3(name="quotients", nx=nx, ny=ny, nz=nz, tau_plus=0.8, magic_lambda=0.25, eta=1e-4)
    s = lbvp3.Solver3(p, storage="f64")
    s.set_populations(g)
    s.step(1, keep_fields=True)
    f = s.fields()
    s.close()
    return f["rho"], f["ux"]


# weights, 36 w of the rest and axis populations, and the populations along +x and -x
W2 = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)
W3 = np.array([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12)
LATTICES = {"2d": (W2, 16.0, 4.0, 1, 3, (96, 512)), "3d": (W3, 12.0, 2.0, 1, 2, (12, 16, 256))}


def _populations(lattice, rest, east, west):
    """Full values with the given deviations of three populations, the others' zero,
    and the deviations as they are stored."""
    w, _, _, qe, qw, shape = LATTICES[lattice]
    h = np.zeros((len(w), *shape))
    h[0], h[qe], h[qw] = rest, east, west
    wq = w.reshape(-1, *[1] * len(shape))
    g = wq * (1.0 + h)
    return g, g / wq - 1.0


@pytest.mark.parametrize("lattice", ["2d", "3d"])
def test_correctly_rounded(lbvp, lbvp3, lattice):
    w, w_rest, w_axis, qe, qw, shape = LATTICES[lattice]
    rest = _densities(int(np.prod(shape)), w_rest).reshape(shape)
    g, h = _populations(lattice, rest, 0.0625, -0.03125)
    assert np.all(np.delete(h, [0, qe, qw], axis=0) == 0.0)
    a, b = float(h[qe].flat[0]), float(h[qw].flat[0])
    rho, ux = _step_2d(lbvp, g) if lattice == "2d" else _step_3d(lbvp3, g)
    # the weighted sum of the deviations, rounded once (one fused multiply-add)
    s36 = np.array([float(Fraction(x) * int(w_rest) + int(w_axis) * (Fraction(a) + Fraction(b))) for x in h[0].flat])
    want = 1.0 + s36.reshape(shape) / 36.0
    assert np.array_equal(rho, want)
    assert np.array_equal(ux, (w_axis * (a - b)) * (1.0 / (36.0 * want)))


@pytest.mark.parametrize("lattice", ["2d", "3d"])
def test_no_density_and_infinite_ones(lbvp, lbvp3, lattice):
    w, w_rest, w_axis, qe, qw, shape = LATTICES[lattice]
    step = (lambda g: _step_2d(lbvp, g)) if lattice == "2d" else (lambda g: _step_3d(lbvp3, g))
    g = np.zeros((len(w), *shape))
    g[qe], g[qw] = 0.25 * w[qe], -0.25 * w[qw]
    rho, ux = step(g)
    assert np.all(rho == 0.0) and np.all(ux == np.inf)
    g[qe], g[qw] = -g[qe], -g[qw]
    rho, ux = step(g)
    assert np.all(rho == 0.0) and np.all(ux == -np.inf)
    g[0] = np.inf
    rho, ux = step(g)
    assert np.all(rho == np.inf) and np.all(ux == 0.0)
    g[0] = -np.inf
    rho, ux = step(g)
    assert np.all(rho == -np.inf) and np.all(ux == 0.0)
    g[0] = np.nan
    rho, ux = step(g)
    assert np.all(np.isnan(rho)) and np.all(np.isnan(ux))
