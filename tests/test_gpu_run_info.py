"""Which kernel a context's steps take (lbvp_get_run_info): two steps a launch, with
the chunks the bitwise tests of pairs are written for, exactly where the rule puts
them (FP64 and FP32 vector launches of single-row tiles and more than 3072
wavefronts, a fixed mask and no cut), and one elsewhere."""
import numpy as np
import pytest

from paper_1901_08766_amd import inputs

pytestmark = pytest.mark.gpu

IO = ("inflow_eq", "outflow_zero_grad", "periodic", "periodic")


def _info(lbvp, nx, ny, storage, launch, flags=0, bc=IO, **kw):
    p = inputs.Problem(name="info", nx=nx, ny=ny, tau_plus=0.8, magic_lambda=0.25, eta=1e-4, bc=bc, **kw)
    s = lbvp.Solver(p, storage=storage, flags=flags)
    if launch:
        s.set_launch(*launch)
    info = s.run_info
    s.close()
    return info[:2]


# the grids and launch shapes that the tests of pairs compare with single steps;
# rows = ceil(wavefronts / 3072), at most 6
@pytest.mark.parametrize("nx,ny,storage,launch,rows", [
    (129, 3101, "f32", (4, 64), 2), (129, 3101, "f64", (2, 64), 3), (257, 3077, "f32", (4, 64), 3),
    (257, 3077, "f64", (2, 128), 5), (515, 1601, "f32", (4, 128), 3), (515, 1601, "f64", (2, 256), 5),
    (1023, 1551, "f32", (4, 256), 3), (1023, 1551, "f64", (2, 128), 5), (2049, 1031, "f32", (4, 64), 4),
    (2049, 1031, "f64", (2, 64), 6), (700, 1600, "f32", (4, 128), 3), (640, 1601, "f32", (4, 128), 3),
    (300, 1600, "f64", (2, 128), 3), (2048, 1153, "f32", (4, 128), 4), (8192, 4096, "f32", None, 6)])
def test_two_steps_a_launch(lbvp, nx, ny, storage, launch, rows):
    assert _info(lbvp, nx, ny, storage, launch) == (2, rows)


@pytest.mark.parametrize("nx,ny,storage,launch,kw", [
    (256, 3072, "f32", (4, 64), {}),                     # as many wavefronts as the chip holds
    (1024, 512, "f32", None, {}),                        # one node per thread
    (128, 8192, "f32", (4, 64), {}),                     # tiles of two rows
    (2049, 1031, "f16", (4, 64), {}), (2049, 1031, "bf16", (8, 64), {}),
    (2049, 1031, "f32", (4, 64), {"flags": 1}),          # the AA layout
    (2049, 1031, "f32", (1, 64), {"moving": True}),
    (2049, 1031, "f32", (4, 64), {"moving": True}),
    (2049, 1031, "f32", (4, 64), {"bc": ("neighbor", "outflow_zero_grad", "periodic", "periodic")})])
def test_one_step_a_launch(lbvp, nx, ny, storage, launch, kw):
    assert _info(lbvp, nx, ny, storage, launch, **kw) == (1, 0)


def test_one_row_past_the_line(lbvp):
    assert _info(lbvp, 256, 3073, "f32", (4, 64)) == (2, 2)


def test_partials_that_do_not_fit_four_times(lbvp):
    """Eight bodies in every tile: room for the partials of two records only."""
    nx, ny = 8192, 4096
    mask = np.broadcast_to((np.arange(nx) % 8 + 1).astype(np.uint8), (ny, nx))
    p = inputs.Problem(name="stripes", nx=nx, ny=ny, tau_plus=0.8, magic_lambda=0.25, eta=1e-4,
                       mask=np.ascontiguousarray(mask), bodies=np.zeros((8, 5)))
    s = lbvp.Solver(p, storage="f32")
    s.set_launch(4, 64)
    assert s.run_info[:2] == (1, 0)
    s.close()
