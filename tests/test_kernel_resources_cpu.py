"""What the compiler made of the kernels, read from the code objects of the library that was built here."""
import os
import re
import struct
import subprocess

import pytest

from paper_2601_12150_amd import build as nb_build

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def kernels(tmp_path):
    """{kernel name: spilled vector registers} of every gfx950 code object in libnsattn.so."""
    data = open(nb_build.LIB, "rb").read()
    found = {}
    for m in re.finditer(b"\x7fELF", data):
        at = m.start()
        if at == 0 or struct.unpack_from("<H", data, at + 18)[0] != 224:      # EM_AMDGPU
            continue
        shoff, = struct.unpack_from("<Q", data, at + 40)
        shentsize, shnum = struct.unpack_from("<HH", data, at + 58)
        path = tmp_path / ("%d.o" % at)
        path.write_bytes(data[at:at + shoff + shentsize * shnum])
        notes = subprocess.run([READELF, "--notes", str(path)], stdout=subprocess.PIPE, text=True, check=True).stdout
        for entry in notes.split("- .agpr_count:")[1:]:
            name = re.search(r"\.name:\s+(\S+)", entry).group(1)
            found[name] = int(re.search(r"\.vgpr_spill_count:\s+(\d+)", entry).group(1))
    return found


@pytest.mark.skipif(not (os.path.exists(nb_build.LIB) and os.path.exists(READELF)), reason="needs the built library and llvm-readelf")
def test_no_kernel_spills_vector_registers(tmp_path):
    """The attention kernels count their own memory requests: a reload of a spilled register in a key loop waits for
    every transfer in flight, tile by tile."""
    found = kernels(tmp_path)
    assert sum("attn_sweep_kernel" in n for n in found) == 6 and sum("attn_block16_kernel" in n for n in found) == 3
    assert {n: c for n, c in found.items() if c} == {}
