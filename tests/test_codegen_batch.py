"""The batch and resident kernels' rounds keep many LDS table reads in flight, as
the single-buffer loops do: what a whole step costs rests on it.  Checked on the
CPU from hipcc's own assembly.  The rounds of whole steps are the straight pieces
of code with a round's reads (16 per block) of every block of a lane, two rounds at
least; the key expansion, which waits for one lookup after the other, and the
groups of one block per lane are not."""
import re

import test_codegen as codegen

# Two rounds at 2 blocks per lane (the decryption tiles of a plan at 4 run at 2 too).
LEAST_READS = 2 * 16 * 2
MIN_IN_FLIGHT = 10.0      # mean number of reads outstanding at a wait for them


def _straight_pieces(lines):
    piece = []
    for line in lines:
        if re.match(r"^\.LBB\d+_\d+:", line) or re.match(r"\s+s_(cbranch_\w+|branch)\s", line):
            yield piece
            piece = []
        piece.append(line)
    yield piece


def test_rounds_of_whole_steps_keep_reads_in_flight(tmp_path):
    lines = codegen._asm("aes_batch.hip", tmp_path)
    kernels = 0
    for name, lo, hi in codegen._kernels(lines):
        m = re.search(r"(batch|resident)_kernelILi([24])E", name)
        if not m:
            continue
        kernels += 1
        rounds = []
        for piece in _straight_pieces(lines[lo + 1:hi]):
            reads = sum(line.strip().startswith("ds_read") for line in piece)
            if reads >= LEAST_READS:
                rounds.append((reads, codegen._in_flight(piece)))
        # Both table sets, each with a piece per key size.
        assert len(rounds) >= 6, f"{name}: {rounds}"
        for reads, got in rounds:
            assert got >= MIN_IN_FLIGHT, f"{name}: {got:.1f} of {reads} reads in flight at a wait"
    assert kernels == 4
