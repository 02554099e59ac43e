"""What the compiler reports of the built kernels: vector registers that went to scratch memory.
They are loads and stores in the middle of loops that are tuned by the requests they keep in flight,
and no result shows them."""
import os
import re
import subprocess

import pytest

from paper_2504_05638_amd import binding as B
from paper_2504_05638_amd import build

_TOOLS = "/opt/rocm/llvm/bin"


def test_no_vector_register_spills(tmp_path):
    if not os.path.exists(os.path.join(_TOOLS, "llvm-objdump")):
        pytest.skip("no LLVM tools here")
    B.lib()
    lib = tmp_path / "libtagc.so"
    lib.write_bytes(open(build.LIB, "rb").read())
    subprocess.run([os.path.join(_TOOLS, "llvm-objdump"), "--offloading", lib.name], cwd=tmp_path,
                   check=True, capture_output=True)
    spills = {}
    for f in tmp_path.glob("*gfx950"):
        notes = subprocess.run([os.path.join(_TOOLS, "llvm-readelf"), "--notes", str(f)], check=True,
                               capture_output=True, text=True).stdout
        name = None
        for line in notes.splitlines():
            m = re.match(r"\s*\.(symbol|vgpr_spill_count):\s+(\S+)", line)
            if m and m.group(1) == "symbol":
                name = m.group(2)
            elif m:
                spills[name] = int(m.group(2))
    assert len(spills) > 20 and any("place_kernel" in k for k in spills)
    assert any("peel_kernelILj12ELj8ELb1ELj4ELb1ELb0ELb0EE" in k for k in spills)
    over = {k: n for k, n in spills.items() if n}
    assert not over, over
