"""The HBM traffic that bench.py reports: bytes per step, from a counter summary of the
same kernel sources and of launches of as many steps; and the sources that decide it,
which stores bypass the caches among them, are in the hash."""
import importlib.util
import json
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture()
def bench(tmp_path, monkeypatch):
    spec = importlib.util.spec_from_file_location("bench_mod", os.path.join(ROOT, "bench.py"))
    m = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(m)
    for name, lat in m.LATTICES.items():
        path = tmp_path / f"{name}.json"
        path.write_text(json.dumps({"kernel_source_hash": m.kernel_source_hash(name), "per_storage": {
            "f32": {"nodes": 100, "hbm_bytes_per_launch": 2000, "steps_per_launch": 2},
            "f16": {"nodes": 100, "hbm_bytes_per_launch": 900}}}))
        monkeypatch.setitem(lat, "counters", str(path))
    return m


def test_bytes_per_step(bench):
    assert bench.measured_traffic("f32", 100, steps_per_launch=2) == 1000
    assert bench.measured_traffic("f32", 100, steps_per_launch=1) is None
    assert bench.measured_traffic("f16", 100) == 900
    assert bench.measured_traffic("f16", 100, steps_per_launch=2) is None
    assert bench.measured_traffic("f16", 99) is None


@pytest.mark.parametrize("lattice", ["d2q9", "d3q19"])
def test_sources_that_decide_the_traffic_are_hashed(bench, lattice):
    names = bench.LATTICES[lattice]["sources"]
    assert "lbvp_cache.h" in names     # plain or non-temporal stores
    csrc = os.path.join(ROOT, "paper_1901_08766_amd", "csrc")
    hashed = "".join(open(os.path.join(csrc, n)).read() for n in names)
    if lattice == "d2q9":
        assert "march_rows" in hashed  # the rows of a chunk, two of which are read twice
