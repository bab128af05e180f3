"""Builds the library's host code against the stand-in for the HIP runtime (fake_hip.h):
the named .hip sources compile for the host only and link with a test program."""
import concurrent.futures as cf
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1901_08766_amd", "csrc")
INCLUDE = ["-I", CSRC, "-I", os.path.join(ROOT, "include")]


def build(out_dir: str, program: str, sources) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    rocm = os.path.join(os.path.dirname(os.path.dirname(hipcc)), "include")
    objs = [os.path.join(out_dir, name + ".o") for name in (*sources, program)]
    cmds = [[hipcc, "--offload-arch=gfx950", "--cuda-host-only", "-fuse-cuid=none", "-O1", "-fPIC", "-std=c++17", *INCLUDE,
             "-c", "-o", o, os.path.join(CSRC, name)] for o, name in zip(objs, sources)]
    cmds.append(["g++", "-O1", "-fPIC", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-w", "-I", rocm, *INCLUDE, "-c", "-o",
                 objs[-1], os.path.join(ROOT, "tests", program)])
    with cf.ThreadPoolExecutor(max_workers=4) as ex:
        for r in ex.map(lambda c: subprocess.run(c, capture_output=True, text=True), cmds):
            assert r.returncode == 0, r.stderr
    exe = os.path.join(out_dir, os.path.splitext(program)[0])
    r = subprocess.run(["g++", "-Wl,--allow-multiple-definition", "-o", exe, *objs, "-lpthread"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


def run(exe: str, check: str):
    r = subprocess.run([exe, check], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
