"""A batch's counters in device memory: each on a 128-byte line that holds
nothing else, in a plan as in the one-call batch's scratch, so that a pull or a
workgroup's exit never takes a descriptor's line away from the waves that read
it; and the parts of the layout neither overlap nor leave their alignment."""
import os
import shutil
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_counters_and_descriptors(tmp_path):
    exe = str(tmp_path / "batch_layout")
    subprocess.run([shutil.which("g++"), "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_1201_0398_amd", "csrc"),
                    "-I", "/opt/rocm/include",
                    os.path.join(ROOT, "tests", "native", "batch_layout.cpp"), "-o", exe],
                   check=True)
    subprocess.run([exe], check=True, timeout=60)
