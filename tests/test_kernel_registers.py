"""Registers and scratch of the step kernels in the built library: the wavefronts per
SIMD that their launch rules and measurements count on. Read from the metadata of the
gfx950 code objects that this build put into the library."""
import os
import re
import struct
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def kernels(lbvp, tmp_path_factory):
    """{mangled name: (vgprs, scratch bytes)} of every kernel."""
    d = tmp_path_factory.mktemp("objects")
    fat = str(d / "fat")
    subprocess.run([f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", lbvp.LIB_PATH, os.devnull], check=True)
    data = open(fat, "rb").read()
    out, at = {}, data.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + len(MAGIC))
        o = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, o)
            target = data[o + 24:o + 24 + idlen].decode()
            o += 24 + idlen
            if "gfx950" in target and size:
                path = str(d / "object")
                open(path, "wb").write(data[at + off:at + off + size])
                notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", path], capture_output=True, text=True,
                                       check=True).stdout
                for block in re.split(r"\n\s+- \.agpr_count", notes)[1:]:
                    name = re.search(r"\.name:\s+'?(\w+)", block).group(1)
                    out[name] = (int(re.search(r"\.vgpr_count:\s+(\d+)", block).group(1)),
                                 int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", block).group(1)))
        at = data.find(MAGIC, at + 1)
    return out


def _waves(vgprs):
    return min(8, 512 // ((vgprs + 7) // 8 * 8))


# at least this many wavefronts per SIMD: two steps a launch (MARCH_WAVES), the vector
# and single-node forms of the 2-D step, the 3-D forms of one node and of four 2-byte ones
# (without fields)
@pytest.mark.parametrize("pattern,waves", [
    (r"7k_marchI[df]Li\dELb[01]E", 3), (r"6k_stepIdLi2ELb1E", 4), (r"6k_stepIfLi4ELb1E", 4), (r"6k_stepIfLi1ELb1ELb0ELb0E", 8),
    (r"6k_stepIDF16[_b]Li4ELb1ELb0ELb0E", 7), (r"7k_step3IdLi1ELb1E", 4), (r"7k_step3IfLi1ELb1E", 5),
    (r"7k_step3IDF16[_b]Li4ELb[01]ELb0E", 3), (r"13k_step3_batchIDF16[_b]Li4ELb[01]ELb0E", 3), (r"7k_step3IDF16[_b]Li1ELb1E", 6)])
def test_wavefronts(kernels, pattern, waves):
    found = {k: v for k, v in kernels.items() if re.search(pattern, k)}
    assert found
    for name, (vgprs, scratch) in found.items():
        assert _waves(vgprs) >= waves, (name, vgprs)
        # the moving-mask forms spill a little; so does, two registers, the BF16 form for
        # lattices past 4 GiB
        assert scratch <= (68 if "6k_step" in name else 8), (name, scratch)
