"""Vector registers that the built kernels keep in scratch memory.  The tile loops
of the prefill and decode kernels fit the register file; a reload in one waits for
every copy in flight, so a call slows down without any other sign."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2607_07740_amd import build

TOOLS = "/opt/rocm/llvm/bin"


@pytest.mark.skipif(not os.path.exists(TOOLS + "/llvm-readelf"), reason="no ELF reader")
def test_kernels_hold_their_registers(tmp_path):
    """At most a few values of a prologue, none of a loop (20 a visit)."""
    if not os.path.exists(build.LIB):
        build.build()
    lib = shutil.copy(build.LIB, str(tmp_path / "lib.so"))
    subprocess.run([TOOLS + "/llvm-objdump", "--offloading", lib], cwd=str(tmp_path), check=True,
                   capture_output=True, timeout=120)
    seen = 0
    for o in sorted(p for p in os.listdir(str(tmp_path)) if p.endswith("gfx950")):
        notes = subprocess.run([TOOLS + "/llvm-readelf", "--notes", o], cwd=str(tmp_path),
                               check=True, capture_output=True, text=True, timeout=120).stdout
        for name, spills in re.findall(r"\.name:\s+(_Z\w+).*?\.vgpr_spill_count:\s+(\d+)", notes,
                                       re.S):
            assert int(spills) <= 8, (name, int(spills))
            seen += 1
    assert seen > 20
