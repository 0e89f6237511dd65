"""The calls that programs make of the library, as measured cases.

Each case is one pass through public entry points of
``paper_1201_0398_amd.aesgpu`` on inputs made from a seed: single-buffer calls
from 4 KiB to 4 GiB in every mode, both directions and all three key sizes,
batches of many messages with a key each (planned once, or planned and run in
one call), host buffers through the pipeline, and a burst of requests to the
server.  Every output is bytes, so two implementations either agree or one of
them is wrong.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_1201_0398_amd import aesgpu as A

KIB, MIB, GIB = 1 << 10, 1 << 20, 1 << 30
KEY_BITS = (128, 192, 256)
SINGLE = ("ecb_enc", "ecb_dec", "ctr", "ctr_le128", "cbc_dec")
HOST_OPS = {"ecb_enc": A.AESGPU_OP_ECB_ENCRYPT, "ecb_dec": A.AESGPU_OP_ECB_DECRYPT,
            "ctr": A.AESGPU_OP_CTR, "ctr_le128": A.AESGPU_OP_CTR_LE128,
            "cbc_dec": A.AESGPU_OP_CBC_DECRYPT}


def listed() -> list:
    return [
        # A short record of no round size, its counter in mid-stream: launch and latency
        # are all of it.
        {"name": "ctr_4k_odd", "kind": "single", "op": "ctr", "bits": 128, "bytes": 4 * KIB - 3},
        # A small buffer encrypted where it lies, one pass of the chip over it.
        {"name": "ecb_enc_4m", "kind": "single", "op": "ecb_enc", "bits": 256, "bytes": 4 * MIB},
        # A medium file decrypted in CBC, the mode most stored data is in.
        {"name": "cbc_dec_24m", "kind": "single", "op": "cbc_dec", "bits": 192,
         "bytes": 24 * MIB + 16 * 13},
        # A medium buffer decrypted with the longest key.
        {"name": "ecb_dec_64m", "kind": "single", "op": "ecb_dec", "bits": 256, "bytes": 64 * MIB},
        # The headline size: bulk encryption of 1 GiB.
        {"name": "ecb_enc_1g", "kind": "single", "op": "ecb_enc", "bits": 128, "bytes": GIB},
        # The paper's own counter mode on a large buffer of odd length.
        {"name": "ctr_le_200m_odd", "kind": "single", "op": "ctr_le128", "bits": 128,
         "bytes": 200_000_003},
        # The largest single call: 4 GiB of CTR with the longest key.
        {"name": "ctr_4g", "kind": "single", "op": "ctr", "bits": 256, "bytes": 4 * GIB},
        # A large batch, every message with its own key, key size and mode.
        {"name": "batch_65536", "kind": "batch", "modes": "ecb_ctr", "dir": 0, "messages": 65536,
         "longest": MIB},
        # Many short CBC messages encrypted, where the parallelism is across messages.
        {"name": "batch_cbc_enc_65536", "kind": "batch", "modes": "cbc", "dir": 0,
         "messages": 65536, "longest": 16 * KIB},
        # A batch seen once: planned and run in one call, both directions, odd CTR lengths.
        {"name": "batch_once_256", "kind": "once", "messages": 256, "longest": MIB},
        # A file in ordinary host memory, encrypted into ordinary host memory.
        {"name": "host_ctr_32m", "kind": "host", "op": "ctr", "bits": 128, "bytes": 32 * MIB + 5},
        # A burst of requests to the server, waited for.
        {"name": "serve_48", "kind": "serve", "requests": 48, "longest": 16 * MIB},
    ]


def _between(rng, lo: int, hi: int) -> int:
    """A whole number spread over the logarithm of lo..hi."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng) -> dict:
    kind = rng.choice(["single"] * 6 + ["batch"] * 3 + ["once", "host", "serve"])
    if kind in ("single", "host"):
        op = rng.choice(SINGLE)
        # (ECB from 4 MiB: smaller calls take what any launch takes.)
        least = 4 * MIB if op.startswith("ecb") else 4 * KIB
        n = _between(rng, least, 2 * GIB if kind == "single" else 128 * MIB)
        if not op.startswith("ctr"):
            n = n // 16 * 16          # ECB and CBC take whole blocks
        return {"kind": kind, "op": op, "bits": rng.choice(KEY_BITS), "bytes": n}
    if kind == "batch":
        modes = rng.choice(["ecb_ctr", "ecb_ctr", "cbc"])
        return {"kind": "batch", "modes": modes, "dir": rng.randrange(2),
                "messages": _between(rng, 64, 65536),
                "longest": 16 * KIB if modes == "cbc" else 16 * _between(rng, KIB, 64 * KIB)}
    if kind == "once":
        return {"kind": "once", "messages": _between(rng, 8, 4096),
                "longest": 16 * _between(rng, 64, 64 * KIB)}
    return {"kind": "serve", "requests": rng.randrange(4, 61),
            "longest": 16 * _between(rng, KIB, MIB)}


@functools.lru_cache(maxsize=None)
def _ctx():
    """A program creates its context once."""
    return A.aesgpu_create(torch.cuda.current_device())


class _Owned:
    """A handle that is given back with the state that holds it."""

    def __init__(self, handle, free):
        self.handle, self._free = handle, free

    def __del__(self):
        self._free(self.handle)


def _device_bytes(seed: int, n: int) -> torch.Tensor:
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    words = torch.empty((n + 7) // 8, dtype=torch.int64, device="cuda")
    words.random_(-(1 << 63), None, generator=g)
    return words.view(torch.uint8)[:n]


def _lengths(rng, m: int, longest: int) -> np.ndarray:
    """Message sizes: multiples of 16 B, log-uniform from 16 B to the longest."""
    u = rng.uniform(math.log(16), math.log(longest), size=m)
    return np.clip(16 * np.rint(np.exp(u) / 16).astype(np.int64), 16, longest)


def _packed(lengths: np.ndarray) -> np.ndarray:
    """Offsets of messages one behind the other, each 16-byte aligned."""
    room = (lengths + 15) // 16 * 16
    return np.concatenate([[0], np.cumsum(room)[:-1]])


def _keys(rng, m: int):
    """m keys of mixed size at a 32-byte stride, and their sizes in bits."""
    bits = np.asarray(KEY_BITS)[rng.integers(0, 3, size=m)]
    keys = rng.integers(0, 256, size=(m, 32), dtype=np.uint8)
    keys[np.arange(32)[None, :] >= (bits // 8)[:, None]] = 0
    return keys, bits


# ---- the messages of a batch, the requests of a burst ------------------------
# Sizes come from the case alone, so that every seed of a case is the same work.

def _batch_sizes(case: dict) -> np.ndarray:
    rng = np.random.default_rng(case["messages"])
    n = _lengths(rng, case["messages"], case["longest"])
    if case["kind"] == "once":
        odd = _once_modes(case)[0] == A.AESGPU_MODE_CTR
        n[odd] -= rng.integers(0, 16, size=int(odd.sum()))   # CTR takes any length
    return n


def _once_modes(case: dict):
    """Modes and directions of a mixed batch: ECB both ways, CTR, CBC decryption."""
    rng = np.random.default_rng(case["messages"] + 1)
    what = rng.integers(0, 4, size=case["messages"])
    modes = np.asarray([A.AESGPU_MODE_ECB, A.AESGPU_MODE_ECB, A.AESGPU_MODE_CTR,
                        A.AESGPU_MODE_CBC])[what]
    return modes, np.asarray([0, 1, 0, 1])[what]


def _request_sizes(case: dict) -> np.ndarray:
    rng = np.random.default_rng(case["requests"])
    return np.maximum(_lengths(rng, case["requests"], case["longest"]), 64)


def prepare(case: dict, seed: int) -> dict:
    rng = np.random.default_rng(seed)
    kind = case["kind"]
    if kind == "single":
        s = {"key": A.aesgpu_expand_key(rng.bytes(case["bits"] // 8)),
             "nonce": rng.bytes(12), "iv": rng.bytes(16), "ctr0": int(rng.integers(1, 1 << 20)),
             "in": _device_bytes(seed, case["bytes"])}
        s["out"] = torch.empty_like(s["in"])
    elif kind == "batch":
        m = case["messages"]
        n = _batch_sizes(case)
        at = _packed(n)
        keys, bits = _keys(rng, m)
        cbc = case["modes"] == "cbc"
        modes = np.full(m, A.AESGPU_MODE_CBC) if cbc else rng.integers(0, 2, size=m)
        msgs = A.make_msgs(at, at, n, np.arange(m), bits, modes, np.full(m, case["dir"]),
                           nonce=rng.integers(0, 256, size=(m, 12), dtype=np.uint8),
                           iv=rng.integers(0, 256, size=(m, 16), dtype=np.uint8))
        s = {"plan": _Owned(A.aesgpu_batch_plan(_ctx(), msgs), A.aesgpu_batch_free), "slots": m,
             "keys": torch.from_numpy(keys.reshape(-1)).cuda(),
             "in": _device_bytes(seed, int(n.sum()))}
        s["out"] = torch.empty_like(s["in"])
    elif kind == "once":
        m = case["messages"]
        n = _batch_sizes(case)
        at = _packed(n)
        keys, bits = _keys(rng, m)
        modes, dirs = _once_modes(case)
        s = {"msgs": A.make_msgs(at, at, n, np.arange(m), bits, modes, dirs,
                                 nonce=rng.integers(0, 256, size=(m, 12), dtype=np.uint8),
                                 iv=rng.integers(0, 256, size=(m, 16), dtype=np.uint8),
                                 ctr0=rng.integers(1, 1 << 20, size=m)),
             "slots": m, "keys": torch.from_numpy(keys.reshape(-1)).cuda(),
             "in": _device_bytes(seed, int(at[-1] + n[-1]))}
        s["out"] = torch.zeros_like(s["in"])   # the gaps behind odd lengths stay zero
    elif kind == "host":
        s = {"key": A.aesgpu_expand_key(rng.bytes(case["bits"] // 8)),
             "op": A.make_host_op(HOST_OPS[case["op"]], 1, rng.bytes(12), rng.bytes(16)),
             "in": rng.integers(0, 256, size=case["bytes"], dtype=np.uint8),
             "out": np.zeros(case["bytes"], dtype=np.uint8),
             "pipeline": _Owned(A.aesgpu_pipeline_create(_ctx()), A.aesgpu_pipeline_destroy)}
    else:
        n = _request_sizes(case)
        at = _packed(n)
        keys, bits = _keys(rng, 64)
        s = {"source": _device_bytes(seed, int(n.sum())), "views": {}, "held": []}
        s["requests"] = [(int(d), int(k), s["source"][int(a):int(a + b)], int(b)) for d, k, a, b in
                         zip(rng.integers(0, 2, size=n.size), rng.integers(0, 64, size=n.size),
                             at, n)]
        room = int(np.sum((n + 255) // 256 * 256)) + MIB
        s["server"] = _Owned(A.aesgpu_server_create(_ctx(), keys, bits, (room + 255) // 256 * 256),
                             A.aesgpu_server_destroy)
        torch.cuda.synchronize()       # the server reads the source on streams of its own
    s["kind"], s["what"] = kind, case.get("op")
    s["ctx"] = _ctx()
    return s


class _Range:
    """Device memory that the library owns, for torch to see."""

    def __init__(self, address: int, n: int):
        self.__cuda_array_interface__ = {"shape": (n,), "typestr": "|u1",
                                         "data": (address, False), "version": 2}


def _view(s: dict, address: int, n: int) -> torch.Tensor:
    if (address, n) not in s["views"]:
        view = torch.as_tensor(_Range(address, n), device="cuda")
        view.owner = s["server"]   # the memory is the server's: it lives as long as the view
        s["views"][address, n] = view
    return s["views"][address, n]


def _serve(s: dict) -> list:
    """Submits the burst, polls until all of it is done and returns the outputs
    where the server left them; they are given back before the next burst."""
    server = s["server"].handle
    for address, n in s["held"]:
        A.aesgpu_server_release(server, address, n)
    for i, (direction, key, data, n) in enumerate(s["requests"]):
        A.aesgpu_server_submit(server, i, direction, key, data, n)
    done = {}
    while len(done) < len(s["requests"]):
        for d in A.aesgpu_server_poll(server, 64):
            done[d.req_id] = (d.d_out, d.n_bytes)
    s["held"] = list(done.values())
    return [_view(s, *done[i]) for i in range(len(done))]


def run(state: dict):
    s = state
    kind, what, ctx = s["kind"], s["what"], s["ctx"]
    if kind == "single":
        if what == "ecb_enc":
            A.aesgpu_ecb_encrypt(ctx, s["key"], s["in"], s["out"])
        elif what == "ecb_dec":
            A.aesgpu_ecb_decrypt(ctx, s["key"], s["in"], s["out"])
        elif what == "ctr":
            A.aesgpu_ctr_xcrypt(ctx, s["key"], s["nonce"], s["ctr0"], s["in"], s["out"])
        elif what == "ctr_le128":
            A.aesgpu_ctr_le128_xcrypt(ctx, s["key"], s["iv"], 0, s["in"], s["out"])
        else:
            A.aesgpu_cbc_decrypt(ctx, s["key"], s["iv"], s["in"], s["out"])
    elif kind == "batch":
        A.aesgpu_batch_run(s["plan"].handle, s["keys"], s["slots"], s["in"], s["out"])
    elif kind == "once":
        A.aesgpu_batch_run_noalloc(ctx, s["msgs"], s["keys"], s["slots"], s["in"], s["out"])
    elif kind == "host":
        A.aesgpu_pipeline_run(s["pipeline"].handle, s["key"], s["op"], s["in"], s["out"])
    else:
        return _serve(s)
    return s["out"]


def work(case: dict) -> dict:
    """Each payload byte read once and written once, and a batch's or a burst's
    keys (32 bytes each).  The cipher has no floating-point operations."""
    if case["kind"] in ("single", "host"):
        n, keys = case["bytes"], 0
    elif case["kind"] == "serve":
        n, keys = int(_request_sizes(case).sum()), 0
    else:
        n, keys = int(_batch_sizes(case).sum()), 32 * case["messages"]
    return {"bytes": 2 * n + keys, "flops": 0}


def exact(case: dict, seed: int):
    """Outputs are bytes of a permutation or a key stream: there is one right
    answer, and nothing between it and a wrong one."""
    return None
