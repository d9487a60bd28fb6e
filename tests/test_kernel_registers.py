"""What the built kernels keep outside their registers, from the metadata of the code objects in the library."""
import os
import re
import struct
import subprocess
import tempfile

import pytest

import paper_2406_15102_amd as hlq
from paper_2406_15102_amd.binding import LIB_PATH

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def _code_objects():
    blob = open(LIB_PATH, "rb").read()
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := blob.find(magic, at)) >= 0:
        n, = struct.unpack_from("<Q", blob, at + len(magic))
        p = at + len(magic) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", blob, p)
            if b"gfx950" in blob[p + 24:p + 24 + idlen] and size:
                yield blob[at + off:at + off + size]
            p += 24 + idlen
        at += len(magic)


def _spills():
    """kernel (mangled) -> vector registers spilled"""
    out = {}
    for obj in _code_objects():
        with tempfile.NamedTemporaryFile() as f:
            f.write(obj)
            f.flush()
            notes = subprocess.run([READELF, "--notes", f.name], stdout=subprocess.PIPE, text=True, check=True).stdout
        for name, spill in re.findall(r"\.name:\s+(_Z\w+)\n(?:(?!\.name:).)*?\.vgpr_spill_count:\s+(\d+)", notes, re.S):
            out[name] = int(spill)
    return out


@pytest.mark.skipif(not os.path.exists(READELF), reason="needs the compiler's readelf")
def test_front_of_small_weights_keeps_to_its_registers():
    # k_front_one<Tin, B, CODES, BASIS, CONV>: whatever the codes, no spills but those that the projection onto the sequency
    # basis has at B = 32 in fp32 (three wavefronts a SIMD are asked for)
    hlq.lib()
    spills = {k: v for k, v in _spills().items() if "k_front_one" in k}
    assert len(spills) == 72, len(spills)
    for name, n in spills.items():
        limit = 20 if re.search(r"k_front_oneIfLi32ELi\dELi1E", name) else 0
        assert n <= limit, (name, n)
