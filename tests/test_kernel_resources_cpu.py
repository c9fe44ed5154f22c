"""CPU check of the built library's kernels: their arrays live in registers.

An array that the compiler cannot keep in registers goes through scratch memory
(global memory, one access after the other), which no test of the results
shows.  The sizes are read from the kernel descriptors' metadata in the library."""
import os
import re
import subprocess

import pytest

from paper_1412_8266_amd import _abi

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def kernels(tmp_path):
    """{kernel name: scratch bytes per lane} of the library's device code."""
    data = open(_abi.LIB_PATH, "rb").read()
    out, at = {}, 0
    while (at := data.find(b"\x7fELF\x02\x01\x01\x40", at)) >= 0:  # ELF64 with the HSA ABI
        img = tmp_path / ("%d.elf" % at)
        img.write_bytes(data[at:])
        notes = subprocess.run([READELF, "--notes", str(img)], capture_output=True, text=True).stdout
        img.unlink()
        for m in re.finditer(r"\.name:\s+(\S+)(.*?)\.private_segment_fixed_size:\s+(\d+)", notes, re.S):
            out[m.group(1)] = int(m.group(3))
        at += 4
    return out


@pytest.mark.skipif(not os.path.exists(READELF), reason="no llvm-readelf")
def test_jumps_and_fills_keep_their_arrays_in_registers(tmp_path):
    found = kernels(tmp_path)
    names = [k for k in found if re.search(r"jump|fill_|philox_|tmt_(sm|il)", k)]
    assert sum("jump" in k for k in names) > 3 and len(names) > 100, len(found)
    # a few spilled scalars are no array
    assert not [(k, found[k]) for k in names if found[k] > (0 if "jump" in k else 16)]
