"""Steps over lattices around the size of the last-level cache, where the rest of
the stores turn non-temporal: a domain that repeats itself along its last axis
stays, copy by copy, bitwise the smaller domain."""
import dataclasses

import numpy as np
import pytest

from paper_1901_08766_amd import inputs, inputs3

pytestmark = pytest.mark.gpu


def _repeat(p, **sizes):
    rep = {k: np.concatenate([getattr(p, k)] * 2) for k in ("mask", "rho_init", "ux_init", "uy_init", "uz_init")
           if hasattr(p, k)}
    return dataclasses.replace(p, **rep, **sizes)


def _same(small, large, copies=2):
    fs, fl = small.fields(), large.fields()
    for k in fs:
        n = fs[k].shape[0]
        for c in range(copies):
            assert np.array_equal(fl[k][c * n:(c + 1) * n], fs[k]), (k, c)


# half the lattices and all of them: within the cache and partly beyond it, partly
# beyond and far beyond it
@pytest.mark.parametrize("nx,ny,storage,launch", [(4095, 1152, "f16", (4, 256)), (4096, 2048, "bf16", (8, 128)),
                                                  (4096, 2048, "f16", (1, 128)), (2047, 1153, "f32", (4, 128)),
                                                  (1999, 1152, "f32", (1, 256)), (2048, 1024, "f64", (2, 128))])
def test_repeated_domain(lbvp, nx, ny, storage, launch):
    p = inputs.random_state_problem(nx, ny, seed=(nx, ny), n_disks=4, rotating=False)
    a = lbvp.Solver(p, storage=storage, mem_fill=0xFF)
    b = lbvp.Solver(_repeat(p, ny=2 * ny), storage=storage, mem_fill=0xFF)
    for s in (a, b):
        s.set_launch(*launch)
        s.step(5)                       # two steps a launch where they apply
        s.step(1, keep_fields=True)
    _same(a, b)


@pytest.mark.parametrize("nx,ny,nz,storage,launch", [(191, 104, 56, "f32", (1, 256)), (192, 104, 104, "f32", (4, 128)),
                                                     (190, 104, 104, "f16", (1, 64))])
def test_repeated_domain_3d(lbvp3, nx, ny, nz, storage, launch):
    p = inputs3.random_state_problem3(nx, ny, nz, seed=(nx, ny, nz), n_spheres=2, moving=False)
    a = lbvp3.Solver3(p, storage=storage)
    b = lbvp3.Solver3(_repeat(p, nz=2 * nz), storage=storage)
    for s in (a, b):
        s.set_launch(*launch)
        s.step(4, keep_fields=True)
    _same(a, b)
