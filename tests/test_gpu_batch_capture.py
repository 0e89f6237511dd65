"""One plan run many times, in every way a program may: directly on buffers that
change from run to run, and captured into the caller's own graph whose replays see
new keys and messages in the captured buffers, with other work between them.  Every
run is checked message by message against the CPU oracle (both launches of a batch
with CBC encryption among them), so a run or a replay that finds the tile counters
or anything else as it should not be shows."""
import numpy as np
import pytest

import oracle
from gpu_common import from_dev, log, requires_gpu, to_dev

pytestmark = [pytest.mark.gpu, requires_gpu]

M = 300


@pytest.fixture(scope="module")
def A():
    from paper_1201_0398_amd import aesgpu
    return aesgpu


@pytest.fixture(scope="module")
def batch(A):
    """A plan over every mode, direction and key size, with odd CTR lengths."""
    rng = np.random.default_rng(77)
    b = {"modes": rng.integers(0, 3, size=M), "dirs": rng.integers(0, 2, size=M),
         "bits": np.array([128, 192, 256])[rng.integers(0, 3, size=M)],
         "nonces": rng.integers(0, 256, (M, 12), dtype=np.uint8),
         "ivs": rng.integers(0, 256, (M, 16), dtype=np.uint8),
         "ctr0": rng.integers(0, 1 << 30, size=M)}
    n = 16 * rng.integers(1, 700, size=M)
    b["n"] = np.where(b["modes"] == 1, n - rng.integers(0, 16, size=M), n)
    b["off"] = np.concatenate([[0], np.cumsum(n)[:-1]])
    b["total"] = int(n.sum())
    ctx = A.aesgpu_create()
    plan = A.aesgpu_batch_plan(ctx, A.make_msgs(b["off"], b["off"], b["n"], np.arange(M), b["bits"],
                                                b["modes"], b["dirs"], b["nonces"], b["ctr0"],
                                                iv=b["ivs"]))
    assert A.aesgpu_batch_info(plan).launches == 2
    yield plan, b
    A.aesgpu_batch_free(plan)
    A.aesgpu_destroy(ctx)


def _inputs(b, seed):
    rng = np.random.default_rng(seed)
    return (rng.integers(0, 256, (M, 32), dtype=np.uint8),
            rng.integers(0, 256, b["total"], dtype=np.uint8))


def _check(b, keys, data, out, what):
    want = np.full(b["total"], 0x5A, dtype=np.uint8)     # the gaps stay as they were
    for j in range(M):
        o, n = int(b["off"][j]), int(b["n"][j])
        key, src = keys[j, : b["bits"][j] // 8], data[o:o + n]
        if b["modes"][j] == 1:
            want[o:o + n] = oracle.ctr(key, b["nonces"][j], int(b["ctr0"][j]), src, threads=1)
        elif b["modes"][j] == 2:
            want[o:o + n] = (oracle.cbc_decrypt(key, b["ivs"][j], src, threads=1) if b["dirs"][j]
                             else oracle.cbc_encrypt(key, b["ivs"][j], src))
        else:
            want[o:o + n] = oracle.ecb(key, src, decrypt=bool(b["dirs"][j]), threads=1)
    bad = np.flatnonzero(out != want)
    assert bad.size == 0, f"{what}: {bad.size} bytes differ, first at {bad[:1]}"


def test_runs_on_changing_buffers(A, batch):
    import torch
    plan, b = batch
    for run in range(4):
        keys, data = _inputs(b, run)
        d_keys, d_in = to_dev(keys.reshape(-1)), to_dev(data)
        d_out = torch.full((b["total"],), 0x5A, dtype=torch.uint8, device="cuda")
        log(f"case: run {run} of one plan")
        A.aesgpu_batch_run(plan, d_keys, M, d_in, d_out)
        _check(b, keys, data, from_dev(d_out), f"run {run}")


def test_captured_into_the_callers_graph(A, batch):
    import torch
    plan, b = batch
    keys, data = _inputs(b, 100)
    d_keys, d_in = to_dev(keys.reshape(-1)), to_dev(data)
    d_out = torch.full((b["total"],), 0x5A, dtype=torch.uint8, device="cuda")
    A.aesgpu_batch_run(plan, d_keys, M, d_in, d_out)     # the kernels are loaded
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    log("case: capture of one run")
    with torch.cuda.graph(graph):
        A.aesgpu_batch_run(plan, d_keys, M, d_in, d_out)
    for replay in range(4):
        keys, data = _inputs(b, 200 + replay)
        d_keys.copy_(to_dev(keys.reshape(-1)))
        d_in.copy_(to_dev(data))
        d_out.fill_(0x5A)
        log(f"case: replay {replay}")
        graph.replay()
        torch.randint(0, 256, (1 << 20,), dtype=torch.uint8, device="cuda").sum()
        torch.cuda.synchronize()
        _check(b, keys, data, from_dev(d_out), f"replay {replay}")
        if replay == 1:                                  # an eager run between replays
            d_out.fill_(0x5A)
            A.aesgpu_batch_run(plan, d_keys, M, d_in, d_out)
            _check(b, keys, data, from_dev(d_out), "run between replays")
