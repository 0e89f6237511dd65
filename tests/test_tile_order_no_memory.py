"""The planner's sort of many tiles wants a second copy of them.  Where there is no
memory for it the plan is made all the same, in the same order, and no C++ exception
reaches the C entry (which would end the program)."""
import os
import shutil
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PACKAGE = os.path.join(ROOT, "paper_1201_0398_amd")


def test_plan_without_memory_for_a_second_copy(tmp_path):
    from paper_1201_0398_amd import aesgpu  # noqa: F401  (builds the library if there is none)

    exe = str(tmp_path / "no_memory")
    subprocess.run([shutil.which("g++"), "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PACKAGE, "csrc"),
                    "-I", "/opt/rocm/include",
                    os.path.join(ROOT, "tests", "native", "tile_order_no_memory.cpp"),
                    os.path.join(PACKAGE, "libaesgpu.so"), "-Wl,-rpath," + PACKAGE, "-o", exe],
                   check=True)
    r = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=60)
    assert r.returncode == 0, f"{r.returncode}: {r.stdout}"
