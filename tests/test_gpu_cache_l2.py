"""Vector launches over lattices about as large as the L2s, which store everything
non-temporal: a domain that repeats itself along y, beyond that window or within it,
stays, copy by copy, bitwise the smaller one; alone and in a batch."""
import dataclasses

import numpy as np
import pytest

from paper_1901_08766_amd import inputs

pytestmark = pytest.mark.gpu


# small and large within and past the window, below and within it
@pytest.mark.parametrize("nx,ny,storage,launch", [(767, 400, "f32", (4, 128)), (639, 240, "f32", (4, 64)),
                                                  (1439, 455, "f16", (4, 128)), (2177, 330, "bf16", (8, 64))])
@pytest.mark.parametrize("batched", [False, True])
def test_repeated_domain(lbvp, nx, ny, storage, launch, batched):
    p = inputs.random_state_problem(nx, ny, seed=(nx, ny), n_disks=4, rotating=False)
    rep = {k: np.concatenate([getattr(p, k)] * 2) for k in ("mask", "rho_init", "ux_init", "uy_init")}
    got = []
    for q in (p, dataclasses.replace(p, ny=2 * ny, **rep)):
        s = lbvp.Solver(q, storage=storage, mem_fill=0xFF)
        s.set_launch(*launch)
        run = lbvp.Batch([s], *launch) if batched else s
        run.step(5)
        run.step(1, keep_fields=True)
        got.append(s.fields())
    for k, small in got[0].items():
        for c in range(2):
            assert np.array_equal(got[1][k][c * ny:(c + 1) * ny], small), (k, c)
