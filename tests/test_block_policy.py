"""Which single-buffer launches stream their blocks past the caches, and the
kernels on both sides of that choice.

A call streams from 128 MiB on, at 2 or 4 blocks per lane, on device memory.
Below that size a streamed call's output would be missing from the caches for
whoever reads it next, whatever the device's CU count or a forced number of
blocks per lane makes of the launch shape."""
import os
import re
import shutil
import subprocess

import pytest

import test_codegen as codegen
from gpu_common import log, requires_gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1201_0398_amd", "csrc")
MIB = 1 << 20
STREAM_BYTES = 128 * MIB

RULE = """
#include "aes_internal.h"
using aesgpu::streams;
constexpr uint64_t kMiB = 1 << 20;
static_assert(streams(4, 128 * kMiB, false) && streams(2, 128 * kMiB, false));
static_assert(!streams(4, 128 * kMiB - 16, false) && !streams(2, 4 * kMiB, false));
static_assert(!streams(1, 4096 * kMiB, false));
static_assert(!streams(4, 1024 * kMiB, true) && !streams(2, 1024 * kMiB, true));
int main() { return 0; }
"""


def test_streaming_goes_by_size_and_memory(tmp_path):
    src = tmp_path / "rule.cpp"
    src.write_text(RULE)
    subprocess.run([shutil.which("g++"), "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-fsyntax-only",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-I", "/opt/rocm/include",
                    str(src)], check=True)


def test_cached_kernels_of_2_and_4_blocks_per_lane(tmp_path):
    """Each exists, keeps its loop and its reads in flight as the streamed one
    does, and only the streamed ones have nontemporal accesses."""
    lines = codegen._asm("aes_kernels.hip", tmp_path)
    cached = 0
    for name, lo, hi in codegen._kernels(lines):
        m = re.search(r"aes_kernelILNS_2OpE(\d)ELi(\d+)ELi(\d+)ELb(\d)E", name)
        if not m:
            continue
        op, nr, shape = codegen.OPS[m.group(1)], int(m.group(2)), int(m.group(3))
        bpl = shape & 15
        blocks = [l for l in lines[lo:hi] if re.match(r"\s+buffer_(load|store)_dwordx4\s", l)]
        assert blocks
        streamed = sum(" nt" in l for l in blocks)
        if shape == 1 or shape > 16:
            assert streamed == 0, f"{op} Nr={nr} {bpl}/lane streams"
        else:
            assert streamed >= 2 * bpl, f"{op} Nr={nr} {bpl}/lane does not stream"
        if shape < 16:
            continue
        cached += 1
        loop = codegen._largest_loop(lines, lo, hi)
        body = lines[loop[0] + 1:loop[1]]
        assert not any(re.match(r"^\.LBB\d+_\d+:", l) for l in body), f"{op} Nr={nr} {bpl}/lane"
        got = codegen._in_flight(body)
        assert got >= codegen.MIN_IN_FLIGHT[bpl], f"{op} Nr={nr} {bpl}/lane: {got:.1f} in flight"
        assert codegen._scratch(lines, lo, hi) <= codegen.KNOWN_SPILLS.get((op, nr, bpl), 0)
    assert cached == 5 * 3 * 2


@pytest.mark.gpu
@requires_gpu
@pytest.mark.parametrize("bpl", [2, 4])
@pytest.mark.parametrize("n_bytes", [STREAM_BYTES - 16, STREAM_BYTES + 16 * 13])
def test_both_policies_agree_around_the_line(monkeypatch, bpl, n_bytes):
    """Every mode just below and just above the line, at a forced number of
    blocks per lane, against one block per lane (which is never streamed)."""
    import torch
    from paper_1201_0398_amd import aesgpu as A
    contexts = []
    for forced in (1, bpl):
        monkeypatch.setenv("AESGPU_FORCE_BPL", str(forced))
        contexts.append(A.aesgpu_create())
    try:
        g = torch.Generator(device="cuda")
        g.manual_seed(bpl)
        d_in = torch.randint(0, 256, (n_bytes,), dtype=torch.uint8, device="cuda", generator=g)
        want, got = torch.empty_like(d_in), torch.empty_like(d_in)
        for bits in (128, 192, 256):
            key = A.aesgpu_expand_key(bytes(range(bits // 8)))
            odd = n_bytes - 11                    # CTR takes any length
            calls = {
                "ecb_enc": lambda c, o: A.aesgpu_ecb_encrypt(c, key, d_in, o),
                "ecb_dec": lambda c, o: A.aesgpu_ecb_decrypt(c, key, d_in, o),
                "ctr": lambda c, o: A.aesgpu_ctr_xcrypt(c, key, bytes(12), 77, d_in, o, odd),
                "ctr_le128": lambda c, o: A.aesgpu_ctr_le128_xcrypt(c, key, bytes(range(16)), 0,
                                                                    d_in, o, odd),
                "cbc_dec": lambda c, o: A.aesgpu_cbc_decrypt(c, key, bytes(range(16)), d_in, o),
            }
            for name, call in calls.items():
                log(f"case: {name} AES-{bits} {n_bytes} B, {bpl} blocks per lane against 1")
                want.zero_()
                got.zero_()
                call(contexts[0], want)
                call(contexts[1], got)
                assert torch.equal(want, got), f"{name} AES-{bits}"
    finally:
        torch.cuda.synchronize()
        for c in contexts:
            A.aesgpu_destroy(c)
