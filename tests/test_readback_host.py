"""The host side of the staging buffers (csrc/lbvp_readback.hip) on the CPU, built
against a stand-in for the HIP runtime (fake_hip.h): what the calls do on several
devices and without pinned memory."""
import host_build
import pytest


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    return host_build.build(str(tmp_path_factory.mktemp("readback")), "readback_host.cc", ["lbvp_readback.hip"])


@pytest.mark.parametrize("check", ["devices", "pageable"])
def test_host_side(program, check):
    host_build.run(program, check)
