"""The mask as the device holds it: after one step from a uniform stream, exactly the
solid nodes of a random mask carry a penalization force. One and several staging
buffers (2 MiB), rows that straddle them, odd row lengths."""
import numpy as np
import pytest

from paper_1901_08766_amd import inputs, inputs3

pytestmark = pytest.mark.gpu


def _mask(shape, seed):
    return np.random.Generator(np.random.PCG64(seed)).integers(0, 3, size=shape, dtype=np.uint8)


@pytest.mark.parametrize("nx,ny", [(3, 3), (65, 33), (64, 5), (2048, 1024), (2049, 1031), (1021, 4111)])
def test_mask_rows(lbvp, nx, ny):
    m = _mask((ny, nx), (nx, ny))
    p = inputs.Problem(name="mask", nx=nx, ny=ny, tau_plus=0.8, magic_lambda=0.25, eta=1e-4, mask=m,
                       bodies=np.zeros((2, 5)), ux_init=np.full((ny, nx), 0.05))
    s = lbvp.Solver(p, storage="f32", mem_fill=0xFF)
    s.step(1, keep_fields=True)
    assert np.array_equal(s.fields()["fx"] != 0.0, m > 0)
    f, _, _ = s.forces()
    fx = s.fields()["fx"]
    for b in (1, 2):   # by body: FP32 node forces, summed in FP64
        assert abs(f[0, b - 1, 0] + fx[m == b].sum()) <= 1e-12 * np.abs(fx).sum()
    s.close()


@pytest.mark.parametrize("shape", [(3, 3, 3), (97, 33, 5), (129, 129, 130)])
def test_mask_rows_3d(lbvp3, shape):
    nx, ny, nz = shape
    m = _mask((nz, ny, nx), shape)
    p = inputs3.Problem3(name="mask", nx=nx, ny=ny, nz=nz, tau_plus=0.8, magic_lambda=0.25, eta=1e-4, mask=m,
                         bodies=np.zeros((2, 9)), ux_init=np.full((nz, ny, nx), 0.05))
    s = lbvp3.Solver3(p, storage="f32")
    s.step(1, keep_fields=True)
    f = s.fields()
    assert np.array_equal(f["fx"] != 0.0, m > 0)
    s.close()
