"""The planner's workgroup orders (CPU): complete, without repeats, and with
the XCDs' shares of work balanced (tests/native/tile_order.cpp)."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2510_16981_amd", "csrc")

SHAPES = {
    "one unit": [(2048, 6144, 1, 1, 1)],
    "fewer units than XCDs, ragged": [(999, 1333, 1, 1, 1), (650, 975, 1, 3, 1), (777, 1554, 3, 2, 1)],
    "two shapes of units": [(4096, 14336, 4, 2, 1), (14336, 4096, 4, 2, 1)],
    "one layer": [(4096, 4096, 1, 8, 1), (4096, 1024, 1, 8, 2), (4096, 4096, 8, 1, 1), (4096, 14336, 1, 8, 2),
                  (14336, 4096, 8, 1, 1)],
    "three layers": [(2048, 2048, 1, 8, 3), (2048, 8192, 1, 8, 2), (8192, 2048, 1, 8, 5)],
    "long and short": [(64, 6656, 1, 1, 9), (1024, 4096, 1, 4, 3), (131, 64, 1, 1, 11), (2048, 2048, 1, 1, 7)],
    # One row beside many small units (fp32 launches on 32 x 32 tiles): the
    # row's tile columns at that width would not fit the 16 bits of a tile.
    "widest": [(1, 2200000, 1, 1, 1), (8, 240000, 1, 30000, 1)],
    # More than 32768 tile rows of the pack.
    "tallest": [(2200000, 8, 1, 1, 1)],
}


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    out = tmp_path_factory.mktemp("order") / "tile_order"
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, os.path.join(ROOT, "tests", "native", "tile_order.cpp"),
                        os.path.join(CSRC, "plan.cpp"), "-o", str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return str(out)


@pytest.mark.parametrize("name", list(SHAPES))
def test_orders(exe, name):
    args = [str(v) for m in SHAPES[name] for v in m]
    r = subprocess.run([exe] + args, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
