"""Registers of the built collide kernels, read from the library's own code
object: no vector register is spilled, and at most 40 scalar ones.  (A spilled
scalar is written and read back by vector instructions; lanes outside the grid
that issue the collide's loads unconditionally cost up to 115 of them, and
FP32 grids a few per cent of their step.)"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2512_01027_amd import binding as B

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def notes(tmp_path_factory):
    if not os.path.exists(os.path.join(LLVM, "llvm-readelf")):
        pytest.skip("no llvm-readelf")
    if not os.path.exists(B.LIB_PATH):
        pytest.fail("libpulbm.so is not built (run __graft_entry__.build())")
    d = str(tmp_path_factory.mktemp("code"))
    shutil.copy(B.LIB_PATH, os.path.join(d, "lib.so"))
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", "lib.so"], cwd=d, check=True, capture_output=True)
    obj = [f for f in os.listdir(d) if "gfx950" in f]
    assert len(obj) == 1, obj
    out = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", os.path.join(d, obj[0])], check=True,
                         capture_output=True, text=True).stdout
    kernels = {}
    for block in out.split("  - .agpr_count")[1:]:
        name = re.search(r"\.name:\s+(\S+)", block).group(1)
        kernels[name] = {k: int(v) for k, v in re.findall(r"\.(\w+):\s+(\d+)\n", block)}
    return kernels


def test_collide_spills(notes):
    collide = {n: k for n, k in notes.items() if "k_collide" in n}
    assert len(collide) == 3 * 4 * 2 * 2  # lattice sets, storage widths, collisions, parities
    for name, k in collide.items():
        assert k["vgpr_spill_count"] == 0, name
        assert k["sgpr_spill_count"] <= 40, (name, k["sgpr_spill_count"])
