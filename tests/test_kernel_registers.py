"""Vector registers of the kernels whose speed hangs on one more wave per SIMD
(CPU: read from the code object that the build put into libopf.so)."""
import os
import re
import struct
import subprocess

import pytest

from paper_2510_12897_amd import build

READELF = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")


def _code_objects(path):
    """The gfx950 ELF images of the library's offload bundles."""
    data = open(path, "rb").read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        p = at + len(magic)
        (n,) = struct.unpack_from("<Q", data, p)
        p += 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + idlen].decode()
            p += 24 + idlen
            if "gfx950" in name and size:
                yield data[at + off:at + off + size]
        at = data.find(magic, at + 1)


@pytest.fixture(scope="module")
def registers(tmp_path_factory):
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    if not os.path.exists(build.LIB):
        build.build()
    out = {}
    for k, elf in enumerate(_code_objects(build.LIB)):
        f = tmp_path_factory.mktemp("co") / f"{k}.elf"
        f.write_bytes(elf)
        txt = subprocess.run([READELF, "--notes", str(f)], check=True, capture_output=True, text=True).stdout
        for block in re.split(r"\n\s+- \.a", txt)[1:]:
            name, count = re.search(r"\.name:\s+(\S+)", block), re.search(r"\.vgpr_count:\s+(\d+)", block)
            if name and count:
                out[name[1]] = int(count[1])
    assert out
    return out


# 512 registers per SIMD lane in blocks of 8: 80 for six waves, 96 for five
@pytest.mark.parametrize("kernel,most", [("batch_bus_flatILi0ELb0ELb0E", 80), ("batch_bus_flatILi0ELb0ELb1E", 80),
                                         ("batch_bus_flatILi0ELb1ELb0E", 80), ("batch_bus_flatILi0ELb1ELb1E", 80),
                                         ("loss_fused_kernelILi256ELi2E", 96)])
def test_waves_per_simd(registers, kernel, most):
    counts = [v for k, v in registers.items() if kernel in k]
    assert len(counts) == 1 and counts[0] <= most, (kernel, counts)
