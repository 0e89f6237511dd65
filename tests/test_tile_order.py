"""The planner's tile order: longest first and stable, whatever the number of
tiles (a comparison sort for few, a counting sort of the lengths for many) and
the tile size (one or two 12-bit digits), against a comparison sort."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PACKAGE = os.path.join(ROOT, "paper_1201_0398_amd")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    from paper_1201_0398_amd import aesgpu  # noqa: F401  (builds the library if there is none)

    gxx = shutil.which("g++")
    assert gxx, "g++ not found"
    exe = str(tmp_path_factory.mktemp("tile_order") / "tile_order")
    subprocess.run([gxx, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PACKAGE, "csrc"),
                    "-I", "/opt/rocm/include", os.path.join(ROOT, "tests", "native", "tile_order.cpp"),
                    os.path.join(PACKAGE, "libaesgpu.so"), "-Wl,-rpath," + PACKAGE, "-o", exe],
                   check=True)
    return exe


@pytest.mark.parametrize("messages,tile_blocks,longest", [
    (1, 256, 1), (500, 256, 256),            # few tiles: the comparison sort
    (2046, 64, 64), (2060, 4096, 4096),      # around 1024 tiles a set, one digit
    (3000, 4096, 20000), (3000, 4352, 4352),  # 4352: a second digit, of a few lengths
    (2500, 1 << 24, 1 << 24), (2500, 1 << 24, 3 << 24)])
def test_tile_order(driver, messages, tile_blocks, longest):
    subprocess.run([driver, str(messages), str(tile_blocks), str(longest)], check=True, timeout=60)
