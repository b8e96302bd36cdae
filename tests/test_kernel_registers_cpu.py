"""Registers of the tile kernels as compiled: the forward kernels with general
products of up to three qubits keep their amplitudes in registers (no scratch). Read
from the metadata of the code objects in the built library."""
import os
import re
import struct
import subprocess

import pytest

from paper_2011_13524_amd import build as B

READELF = os.path.join(os.path.dirname(os.path.dirname(B.HIPCC)), "llvm", "bin", "llvm-readelf")


@pytest.fixture(scope="module")
def scratch(tmp_path_factory):
    """Kernel symbol -> bytes of scratch per lane."""
    data = open(B.OUT, "rb").read()
    d = tmp_path_factory.mktemp("objs")
    found = {}
    for m in re.finditer(rb"__CLANG_OFFLOAD_BUNDLE__", data):
        at = m.start()
        (count,) = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        if count > 16:
            continue
        for _ in range(count):
            off, size, tl = struct.unpack_from("<QQQ", data, p)
            triple = data[p + 24:p + 24 + tl]
            p += 24 + tl
            if b"gfx950" not in triple or size == 0:
                continue
            f = d / "o.elf"
            f.write_bytes(data[at + off:at + off + size])
            notes = subprocess.run([READELF, "--notes", str(f)], capture_output=True, text=True, timeout=120).stdout
            for kernel in notes.split("\n  - .agpr_count:")[1:]:
                name = re.search(r"\.name:\s+(\S+)", kernel).group(1)
                found[name] = int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", kernel).group(1))
    return found


def test_general_tile_kernels_have_no_scratch(scratch):
    names = [n for n in scratch if re.search(r"k_tile_regIfLi[34]ELi[023]E|k_tile_regIdLi[34]ELi[023]E|k_item_tileI[fd]Li[02]E", n)]
    assert len(names) >= 20
    assert {n: scratch[n] for n in names if scratch[n]} == {}
