"""Two steps per launch at full sizes, in the default launch: the 8192 x 4096 domain
that the benchmark times and one whose lattices hold more populations than 32-bit
offsets reach (32768 x 16384). Pairs against the same steps one per launch, bitwise:
every record of every step (each sums the whole domain), and the populations, of all
rows or of the first and last ones, those around chunk and offset limits and the rows
of the far-corner body."""
import numpy as np
import pytest
import torch

from paper_1901_08766_amd import inputs

pytestmark = pytest.mark.gpu


def _two(lbvp, prob, storage, steps):
    a, b = (lbvp.Solver(prob, storage=storage, force_every=1, force_capacity=64) for _ in range(2))
    assert a.run_info[:2] == (2, 6)
    print(f"case {prob.name} {storage} launch={a.launch} device bytes={a.footprint}", flush=True)
    a.step(steps)
    for _ in range(steps):
        b.step(1)
    (fa, ma, sa), (fb, mb, sb) = a.forces(), b.forces()
    assert sa == sb == 1 and len(ma) == steps and np.all(np.isfinite(ma)) and np.abs(fa).max() > 0.0
    assert np.array_equal(ma, mb) and np.array_equal(fa, fb)
    return a, b


def _done(a, b):
    a.close()
    b.close()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("storage", ["f32", "f64"])
def test_benchmark_domain(lbvp, storage):
    prob = inputs.large_domain()
    a, b = _two(lbvp, prob, storage, 6)
    for y0 in range(0, prob.ny, 512):
        assert np.array_equal(a.populations(y0, 512), b.populations(y0, 512)), y0
    a.step(3, keep_fields=True)    # a pair, then the step that keeps the fields
    for k in range(3):
        b.step(1, keep_fields=k == 2)
    for y0 in range(0, prob.ny, 1024):
        fa, fb = a.fields(y0, 1024), b.fields(y0, 1024)
        for k in fa:
            assert np.array_equal(fa[k], fb[k]), (k, y0)
    _done(a, b)


def test_maximum_size(lbvp):
    prob = inputs.huge_domain()
    nx, ny = prob.nx, prob.ny
    a, b = _two(lbvp, prob, "f32", 4)
    rows_of_body = np.nonzero((prob.mask == 2).any(axis=1))[0]    # body 2 lies in the far corner
    limits = [2 ** k // (9 * nx * s) for k, s in ((31, 1), (32, 1), (31, 4), (32, 4))]
    spans = [(0, 8), (ny - 8, 8), (int(rows_of_body.min()) - 2, len(rows_of_body) + 4)]
    spans += [(y - 4, 9) for y in limits if 4 <= y < ny - 8]
    assert len(spans) >= 6
    for y0, n in spans:
        n = min(n, ny - y0)
        assert np.array_equal(a.populations(y0, n), b.populations(y0, n)), (y0, n)
    _done(a, b)
