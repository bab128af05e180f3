"""Reading field planes to the host: the values of the initial state, which the
library stores in the arithmetic type, come back exactly, over one and several
staging buffers, planes that share a buffer, odd row lengths and bands of rows."""
import numpy as np
import pytest

from paper_1901_08766_amd import inputs, inputs3

pytestmark = pytest.mark.gpu


def _field(shape, seed, lo, hi):
    return np.random.Generator(np.random.PCG64(seed)).uniform(lo, hi, size=shape)


# one value below, at and above a staging buffer of 2^19 floats or 2^18 doubles
# per plane, a plane of a few values, and several buffers
@pytest.mark.parametrize("nx,ny", [(3, 3), (65, 33), (512, 512), (1024, 512), (4099, 128), (1021, 1031)])
@pytest.mark.parametrize("storage", ["f32", "f64", "f16"])
def test_initial_fields_exact(lbvp, nx, ny, storage):
    rho, ux, uy = (_field((ny, nx), s, a, b) for s, a, b in ((1, 0.9, 1.1), (2, -0.1, 0.1), (3, -0.1, 0.1)))
    p = inputs.Problem(name="read", nx=nx, ny=ny, tau_plus=0.8, magic_lambda=0.25, eta=1e-4, rho_init=rho,
                       ux_init=ux, uy_init=uy)
    s = lbvp.Solver(p, storage=storage)
    r = np.float64 if storage == "f64" else np.float32
    f = s.fields()
    for name, want in (("rho", rho), ("ux", ux), ("uy", uy), ("fx", 0 * rho), ("fy", 0 * rho)):
        assert np.array_equal(f[name], want.astype(r).astype(np.float64)), name
    y0, n = ny // 3, max(1, ny // 2)
    band = s.fields(y0, n)
    for name in f:
        assert np.array_equal(band[name], f[name][y0:y0 + n]), name
    # some planes only, into the caller's arrays
    out = np.full((ny, nx), np.nan)
    assert lbvp.lib().lbvp_read_fields(s.ctx, None, None, out.ctypes.data, None, None) == lbvp.OK
    assert np.array_equal(out, f["uy"])
    s.close()


@pytest.mark.parametrize("shape", [(3, 3, 3), (97, 33, 5), (192, 64, 70)])
@pytest.mark.parametrize("storage", ["f32", "f64"])
def test_initial_fields_exact_3d(lbvp3, shape, storage):
    nx, ny, nz = shape
    a = [_field((nz, ny, nx), s, lo, hi) for s, lo, hi in ((1, 0.9, 1.1), (2, -0.1, 0.1), (3, -0.1, 0.1), (4, -0.1, 0.1))]
    p = inputs3.Problem3(name="read", nx=nx, ny=ny, nz=nz, tau_plus=0.8, magic_lambda=0.25, eta=1e-4, rho_init=a[0],
                         ux_init=a[1], uy_init=a[2], uz_init=a[3])
    s = lbvp3.Solver3(p, storage=storage)
    r = np.float64 if storage == "f64" else np.float32
    f = s.fields()
    want = a + [0 * a[0]] * 3
    for got, w in zip(f.values(), want):
        assert np.array_equal(got, w.astype(r).astype(np.float64))
    z0, n = nz // 3, max(1, nz // 2)
    for got, w in zip(s.fields(z0, n).values(), want):
        assert np.array_equal(got, w[z0:z0 + n].astype(r).astype(np.float64))
    s.close()
