"""What the compiler reports of the built kernels: vector registers that went to scratch memory, which
are loads and stores in the middle of loops that are tuned by the requests they keep in flight, and the
local memory that decides which kernels share a compute unit.  No result shows either."""
import os
import re
import subprocess

import pytest

from paper_2504_05638_amd import binding as B
from paper_2504_05638_amd import build

_TOOLS = "/opt/rocm/llvm/bin"


def _kernels(tmp_path, field):
    """{kernel's symbol: value} of one number that the compiler notes for each."""
    if not os.path.exists(os.path.join(_TOOLS, "llvm-objdump")):
        pytest.skip("no LLVM tools here")
    B.lib()
    lib = tmp_path / "libtagc.so"
    lib.write_bytes(open(build.LIB, "rb").read())
    subprocess.run([os.path.join(_TOOLS, "llvm-objdump"), "--offloading", lib.name], cwd=tmp_path,
                   check=True, capture_output=True)
    found = {}
    for f in tmp_path.glob("*gfx950"):
        notes = subprocess.run([os.path.join(_TOOLS, "llvm-readelf"), "--notes", str(f)], check=True,
                               capture_output=True, text=True).stdout
        now = {}
        for line in notes.splitlines():
            m = re.match(r"\s*(?:- )?\s*\.(symbol|%s):\s+(\S+)" % field, line)
            if m:
                now[m.group(1)] = m.group(2)
            if len(now) == 2:  # (a kernel's fields come in the order of their names)
                found[now["symbol"]] = int(now[field])
                now = {}
    assert len(found) > 20 and any("place_kernel" in k for k in found)
    return found


def test_no_vector_register_spills(tmp_path):
    spills = _kernels(tmp_path, "vgpr_spill_count")
    assert any("peel_kernelILj12ELj8ELb1ELj4ELb1ELb0ELb0EE" in k for k in spills)
    over = {k: n for k, n in spills.items() if n}
    assert not over, over


def test_two_scans_leave_room_for_an_encoder(tmp_path):
    """The form of the scan for plans that have other buckets in flight (bf16): two of its workgroups
    and one of the encoder (a partition of the default size, 12288 cells) fit a compute unit."""
    lds = _kernels(tmp_path, "group_segment_fixed_size")
    scans = [n for k, n in lds.items() if re.search(r"scan_spill_kernelILi1ELb[01]ELb0EE", k)]
    assert len(scans) == 2 and 2 * max(scans) + 4 * 12288 <= 160 * 1024, scans
