"""The host side of the staging buffers (csrc/lbvp_readback.hip) on the CPU, built
against a stand-in for the HIP runtime (readback_host.cc): what the calls do on
several devices and without pinned memory, and what they keep."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1901_08766_amd", "csrc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("readback")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    include = ["-I", CSRC, "-I", os.path.join(ROOT, "include")]
    objs = [str(d / "readback.o"), str(d / "host.o")]
    subprocess.run([hipcc, "--offload-arch=gfx950", "--cuda-host-only", "-fuse-cuid=none", "-O1", "-fPIC", "-std=c++17",
                    *include, "-c", "-o", objs[0], os.path.join(CSRC, "lbvp_readback.hip")], check=True)
    rocm = os.path.join(os.path.dirname(os.path.dirname(hipcc)), "include")
    subprocess.run(["g++", "-O1", "-fPIC", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-w", "-I", rocm, *include, "-c", "-o",
                    objs[1], os.path.join(ROOT, "tests", "readback_host.cc")], check=True)
    exe = str(d / "readback_host")
    subprocess.run(["g++", "-o", exe, *objs, "-lpthread"], check=True)
    return exe


@pytest.mark.parametrize("check", ["devices", "pageable"])
def test_host_side(program, check):
    r = subprocess.run([program, check], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
