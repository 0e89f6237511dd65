"""The tile size the planner chooses where the caller leaves it to the library:
two tiles a wave of the work that is cut into tiles.  CBC encryption is not (its
groups have a launch of their own), so it does not count, and a partial block
counts as one."""
import os
import shutil
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PACKAGE = os.path.join(ROOT, "paper_1201_0398_amd")


def test_default_tile_size(tmp_path):
    from paper_1201_0398_amd import aesgpu  # noqa: F401  (builds the library if there is none)

    exe = str(tmp_path / "default_tiles")
    subprocess.run([shutil.which("g++"), "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PACKAGE, "csrc"),
                    "-I", "/opt/rocm/include",
                    os.path.join(ROOT, "tests", "native", "default_tiles.cpp"),
                    os.path.join(PACKAGE, "libaesgpu.so"), "-Wl,-rpath," + PACKAGE, "-o", exe],
                   check=True)
    r = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
