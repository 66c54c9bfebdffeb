"""Host side of the library on the CPU, against a stand-in HIP runtime
(tests/host_paths_driver.c, built here with gcc): what a GPU run cannot show,
such as pinned memory that runs out or a second device.

- coherent: the host widens a read-back's pieces only where the runtime
  guarantees that it sees what the GPU wrote (coherent pinned memory, or events
  that release to the system).
- device: a case is read from a thread whose current device is another one.
- nopinned, onepinned: no pinned memory, or one piece of it, is to be had.
- capture: the last case goes while a stream is under capture in global mode.
"""
import os
import shutil
import subprocess

import pytest

from paper_2512_01027_amd import binding as B

HERE = os.path.dirname(os.path.abspath(__file__))

pytestmark = pytest.mark.skipif(shutil.which("gcc") is None, reason="gcc is not installed")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not os.path.exists(B.LIB_PATH):
        pytest.fail("libpulbm.so is not built (run __graft_entry__.build())")
    exe = str(tmp_path_factory.mktemp("host_paths") / "host_paths")
    subprocess.run(["gcc", "-std=gnu11", "-O1", "-Wall", "-I", os.path.join(os.path.dirname(HERE), "include"), "-rdynamic",
                    "-o", exe, os.path.join(HERE, "host_paths_driver.c"), "-ldl"], check=True)
    return exe


def _run(driver, *args):
    r = subprocess.run([driver, B.LIB_PATH, *map(str, args)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
    return r.stdout


@pytest.mark.parametrize("scenario", ["coherent", "device", "nopinned", "onepinned", "capture"])
def test_read_back(driver, scenario):
    assert _run(driver, scenario).strip().endswith("ok")


@pytest.mark.parametrize("store", [0, 1, 2, 3])
def test_2d_collide_lds(driver, store):
    """LDS that the 2D collide's launch asks for: the rebuild's fields (P*, u* and
    phi of 700 cells, 544 of P) only where the case's collide rebuilds P and u, not
    for a case with a block; no more than the larger of them and h."""
    sb, ab = [8, 4, 2, 2][store], 8 if store == 0 else 4
    h = 0 if sb == 2 else 9 * 256 * sb
    case = lambda block: [int(v) for v in _run(driver, "lds", "k_collide", 2, 64, 40, 1, store, 0, block, 2).split()]  # noqa: E731
    assert case(1) == [h, h]
    fused = case(0)
    assert fused == fused[:1] * 2
    assert max(h, (5 * 700 + 544) * ab) <= fused[0] < max(h, (5 * 700 + 544) * ab) + 64


@pytest.mark.parametrize("store,bgk,wall,n,held", [
    (1, 0, 0, (64, 64, 64), False), (1, 0, 0, (100, 100, 100), True), (1, 0, 1, (100, 100, 100), False),
    (1, 0, 1, (128, 128, 128), False), (1, 0, 1, (192, 128, 128), True), (1, 1, 0, (128, 128, 128), False),
    (2, 0, 0, (192, 128, 128), False)])
def test_3d_collide_lds(driver, store, bgk, wall, n, held):
    """4 workgroups of the 4-byte D3Q27 collide to a CU (40,576 bytes each of its
    160 KiB), or 3 where its launch asks for 12 KiB more: the filter collision's
    from 128 MiB of populations, 512 MiB with walls."""
    lds = _run(driver, "lds", "k_collide", 3, *n, store, wall, 0, 2, bgk).split()
    assert [int(v) for v in lds] == [12288 if held else 0] * 2
