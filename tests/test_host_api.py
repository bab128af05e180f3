"""The host side of the D2Q9 calls on the CPU, built against a stand-in for the HIP
runtime (fake_hip.h) with launches that do nothing: what contexts, batches and the
pool keep, accept and refuse."""
import host_build
import pytest


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    return host_build.build(str(tmp_path_factory.mktemp("host_api")), "host_api.cc",
                            ["lbvp_api.hip", "lbvp_pool.hip", "lbvp_readback.hip"])


@pytest.mark.parametrize("check", ["pool_staging", "static_capacity", "default_shape", "default_blocks", "tune_cuts"])
def test_host_side(program, check):
    host_build.run(program, check)
