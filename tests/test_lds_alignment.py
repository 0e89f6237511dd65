"""The staging writes the tables to the LDS as 16-byte words, so every LDS image
that it is given declares that alignment: the compiler happens to place the one
array of a kernel at offset 0, but promises no more than the array's own type."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1201_0398_amd", "csrc")


def test_every_lds_image_declares_16_byte_alignment():
    seen = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        if not os.path.isfile(path):
            continue
        with open(path) as f:
            for number, line in enumerate(f, 1):
                if not re.match(r"\s*__shared__\b", line):
                    continue
                seen += 1
                assert re.match(r"\s*__shared__\s+alignas\(16\)\s", line), \
                    f"{os.path.basename(path)}:{number}: {line.strip()}"
    assert seen >= 4      # the single-buffer, batch, resident and CBC-encryption kernels
