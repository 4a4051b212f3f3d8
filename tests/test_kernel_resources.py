"""Registers of the whole-tile GEMM kernels in the built library (CPU only): the metadata
that the compiler writes beside each kernel, read from the library's code objects.  Every
register of these kernels is taken (256 + 256 per lane), so a change that looks harmless
can push part of the main loop's state into memory."""
import re
import struct
import subprocess

import pytest

from paper_2607_28848_amd import build as pkg_build

READELF = pkg_build.ROCM + "/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(path):
    """The gfx950 ELF images of every bundle in the library."""
    data = open(path, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + idlen] and size:
                yield data[at + off:at + off + size]
            p += 24 + idlen
        at = data.find(MAGIC, at + 24)


@pytest.fixture(scope="module")
def spills(tmp_path_factory):
    out = {}
    for i, co in enumerate(_code_objects(pkg_build.LIB)):
        f = tmp_path_factory.mktemp("co") / ("%d.o" % i)
        f.write_bytes(co)
        notes = subprocess.run([READELF, "--notes", str(f)], capture_output=True, text=True, check=True).stdout
        for m in re.finditer(r"\.name:\s+(\S+)(.*?)\.vgpr_spill_count:\s+(\d+)", notes, re.S):
            if "kernel" in m.group(1):
                out[m.group(1)] = int(m.group(3))
    return out


@pytest.mark.parametrize("name", ["gemm16_kernelILb0ELb%dELb%dELb0EE" % (d, nn) for d in (0, 1) for nn in (0, 1)] +
                         ["gemm16_group_kernelILb%dELb%dELb0EE" % (d, nn) for d in (0, 1) for nn in (0, 1)])
def test_whole_tiles_keep_their_registers(spills, name):
    """Kernels of whole tiles spill at most a few registers (17 cost the grouped NN form
    4-7% of its time)."""
    found = [v for k, v in spills.items() if name in k]
    assert len(found) == 1, (name, sorted(spills))
    assert found[0] <= 4
