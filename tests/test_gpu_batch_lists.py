"""GPU parity of how a batch is dealt out: batches of as many tiles as
workgroups, one fewer, one more, several rows of a workgroup's list and a row
begun, in both table sets at once, against the CPU oracle message by message;
and the call that plans and runs at once, whose own choice of small tiles must
not make a batch too large for its scratch."""
import numpy as np
import pytest

import oracle
from gpu_common import from_dev, log, requires_gpu, to_dev

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.fixture(scope="module")
def A():
    from paper_1201_0398_amd import aesgpu
    return aesgpu


@pytest.fixture(scope="module")
def ctx(A):
    c = A.aesgpu_create()
    yield c
    A.aesgpu_destroy(c)


# (rows, more): rows * CUs + more messages of one tile each.
@pytest.mark.parametrize("rows,more", [(0, 1), (0, 2), (1, -1), (1, 0), (1, 1), (2, 3), (16, 1),
                                       (33, -5)])
def test_lists_cover_every_tile(A, ctx, rows, more):
    import torch
    m = rows * A.aesgpu_ctx_num_cus(ctx) + more
    rng = np.random.default_rng(100 * rows + more + 7)
    modes = rng.integers(0, 3, size=m)                    # ECB, CTR, CBC
    dirs = np.where(modes == 2, 1, rng.integers(0, 2, size=m))
    lengths = 16 * rng.integers(1, 81, size=m)            # up to a group and a quarter
    lengths = np.where(modes == 1, lengths - rng.integers(0, 16, size=m), lengths)
    bits = np.array([128, 192, 256])[rng.integers(0, 3, size=m)]
    keys = rng.integers(0, 256, (m, 32), dtype=np.uint8)
    nonces = rng.integers(0, 256, (m, 12), dtype=np.uint8)
    ivs = rng.integers(0, 256, (m, 16), dtype=np.uint8)
    # (A CTR message is cut where its counter reaches a multiple of 256.)
    ctr0 = 256 * rng.integers(0, 1 << 23, size=m)
    span = 16 * ((lengths + 15) // 16) + 16 * rng.integers(0, 2, size=m)
    off = np.concatenate([[0], np.cumsum(span)[:-1]])
    total = int(span.sum())
    data = rng.integers(0, 256, total, dtype=np.uint8)
    log(f"case: {m} messages, {total} bytes")
    msgs = A.make_msgs(off, off, lengths, np.arange(m), bits, modes, dirs, nonces, ctr0, iv=ivs)
    d_keys, d_in = to_dev(keys.reshape(-1)), to_dev(data)
    plan = A.aesgpu_batch_plan(ctx, msgs)
    try:
        info = A.aesgpu_batch_info(plan)
        assert info.n_tiles_forward + info.n_tiles_inverse == m
        for _ in range(2):   # the second run finds the counters as the first left them
            d_out = torch.full((total,), 0x5A, dtype=torch.uint8, device="cuda")
            A.aesgpu_batch_run(plan, d_keys, m, d_in, d_out)
        out = from_dev(d_out)
    finally:
        A.aesgpu_batch_free(plan)
    want = np.full(total, 0x5A, dtype=np.uint8)
    for j in range(m):
        o, n = int(off[j]), int(lengths[j])
        key, src = keys[j, : bits[j] // 8], data[o:o + n]
        if modes[j] == 1:
            want[o:o + n] = oracle.ctr(key, nonces[j], int(ctr0[j]), src)
        elif modes[j] == 2:
            want[o:o + n] = oracle.cbc_decrypt(key, ivs[j], src)
        else:
            want[o:o + n] = oracle.ecb(key, src, decrypt=bool(dirs[j]))
    bad = np.flatnonzero(out != want)
    assert bad.size == 0, f"{bad.size} bytes differ, first at {bad[:1]}"


def test_chosen_tiles_do_not_outgrow_the_scratch(A, ctx):
    """100,000 one-block messages and one of 20,000 tiles of 8192 blocks: the
    descriptors fit the call's scratch with those tiles and not with smaller
    ones, which the library would choose by itself."""
    import torch
    small, big = 100_000, 20_000 * 8192 * 16
    n = np.concatenate([np.full(small, 16, dtype=np.int64), [big]])
    off = np.concatenate([[0], np.cumsum(n)[:-1]])
    m, total = small + 1, int(n.sum())
    log(f"case: {m} messages, {total} bytes")
    zero = np.zeros(m, dtype=np.int64)
    msgs = A.make_msgs(off, off, n, zero, np.full(m, 128), zero, zero)
    key = np.arange(32, dtype=np.uint8)
    d_keys = to_dev(key)
    d_in = torch.randint(0, 256, (total,), dtype=torch.uint8, device="cuda")
    d_out = torch.zeros_like(d_in)
    assert A.aesgpu_batch_run_noalloc(ctx, msgs, d_keys, 1, d_in, d_out, tile_blocks=4096,
                                      check=False) == A.AESGPU_ESCRATCH
    A.aesgpu_batch_run_noalloc(ctx, msgs, d_keys, 1, d_in, d_out)
    want = torch.empty_like(d_in)
    A.aesgpu_ecb_encrypt(ctx, A.aesgpu_expand_key(bytes(key[:16])), d_in, want)
    assert torch.equal(d_out, want)
