"""Registers of kernels whose occupancy decides, as the built library's own notes give them (no GPU)."""
import os
import re
import struct
import subprocess

import pytest

from paper_2307_05740_amd import _build


@pytest.fixture(scope="module")
def registers(tmp_path_factory):
    """Vector registers of every kernel of the library, by its mangled name."""
    with open(_build.ARROW_LIB, "rb") as f:
        lib = f.read()
    readelf = os.path.join(os.path.dirname(os.path.dirname(_build._hipcc())), "llvm", "bin", "llvm-readelf")
    found = {}
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", lib):
        at = m.end() + 8
        for _ in range(struct.unpack_from("<Q", lib, m.end())[0]):
            offset, size, name = struct.unpack_from("<QQQ", lib, at)
            target = lib[at + 24:at + 24 + name]
            at += 24 + name
            if b"gfx950" not in target or size == 0:
                continue
            path = tmp_path_factory.mktemp("code") / "gfx950.o"
            path.write_bytes(lib[m.start() + offset:m.start() + offset + size])
            notes = subprocess.run([readelf, "--notes", str(path)], stdout=subprocess.PIPE, text=True, check=True).stdout
            for kernel in re.split(r"\n  - ", notes):
                name_of, count = re.search(r"\.name: +(_Z\S+)", kernel), re.search(r"\.vgpr_count: +(\d+)", kernel)
                if name_of and count:
                    found[name_of.group(1)] = int(count.group(1))
    return found


# 512 registers of a SIMD's lane, given out eight at a time
@pytest.mark.parametrize("kernel,waves", [("chunks_kernelILi4ELi8ELb1E", 7), ("chunks_kernelILi4ELi16ELb1E", 7)])
def test_wavefronts_per_simd(registers, kernel, waves):
    """Products that are bound by rows of X on their way: A^5 of a 2m-vertex Chung-Lu graph, k = 32, 2464 us with seven wavefronts
    per SIMD and 2478 with six."""
    counts = [n for name, n in registers.items() if kernel in name]
    assert len(counts) == 1 and 512 // (-(-counts[0] // 8) * 8) >= waves, counts
