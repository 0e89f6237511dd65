"""The autotuner against the library's own choice of tile size: it is one of the
shapes timed, small tiles are too, and a cached shape is used only for the build
of the library that it was timed with and for a batch of the same kind."""
import numpy as np
import pytest

from gpu_common import log, requires_gpu, to_dev
from paper_1201_0398_amd import autotune


def test_candidates_cover_the_librarys_choices():
    for bpl in (1, 2, 4):
        tiles = {t for b, t in autotune.DEFAULT_CANDIDATES if b == bpl}
        assert {0, 256, 512, 4096} <= tiles       # 256 .. 4096: what the planner takes
        assert all(t % (64 * bpl) == 0 for t in tiles)


def test_key_tells_what_runs_on_which_tables():
    n = [4096, 4096]
    ecb = autotune.workload_key("gfx950", n, [0, 0], [0, 0])
    ecb_dec = autotune.workload_key("gfx950", n, [0, 0], [1, 1])
    cbc_dec = autotune.workload_key("gfx950", n, [2, 2], [1, 1])
    cbc_enc = autotune.workload_key("gfx950", n, [2, 2], [0, 0])
    ctr = autotune.workload_key("gfx950", n, [1, 1], [1, 1])
    assert cbc_dec == ecb_dec and "inv10" in cbc_dec       # one queue, the inverse tables
    assert ctr == ecb and "inv0" in ctr                    # CTR has one direction
    assert cbc_enc not in (ecb, ecb_dec)                   # no tiles at all


def test_cached_shapes_belong_to_a_build(tmp_path, monkeypatch):
    from paper_1201_0398_amd import aesgpu
    keys = []
    for content in (b"one build", b"another"):
        lib = tmp_path / content.decode().replace(" ", "_")
        lib.write_bytes(content)
        monkeypatch.setattr(aesgpu, "LIB_PATH", str(lib))
        keys.append(autotune.cache_key("gfx950", [4096], [0], [0]))
        assert keys[-1] == autotune.cache_key("gfx950", [4096], [0], [0])
        assert keys[-1].startswith(autotune.workload_key("gfx950", [4096], [0], [0]))
    assert keys[0] != keys[1]


@pytest.mark.gpu
@requires_gpu
def test_tuned_shape_is_no_slower_than_the_librarys(tmp_path):
    import torch
    from paper_1201_0398_amd import aesgpu as A
    ctx = A.aesgpu_create()
    try:
        rng = np.random.default_rng(5)
        m = 200
        lengths = 16 * rng.integers(1, 8192, size=m)
        at = np.concatenate([[0], np.cumsum(lengths)[:-1]])
        zero = np.zeros(m, dtype=np.int64)
        msgs = A.make_msgs(at, at, lengths, np.arange(m), np.full(m, 128), zero, zero)
        d_keys = to_dev(rng.integers(0, 256, 32 * m, dtype=np.uint8))
        d_in = to_dev(rng.integers(0, 256, int(lengths.sum()), dtype=np.uint8))
        d_out = torch.empty_like(d_in)
        plan = A.aesgpu_batch_plan(ctx, msgs)
        own = A.aesgpu_batch_info(plan)
        own = f"({int(own.blocks_per_lane)}, {int(own.tile_blocks)})"
        A.aesgpu_batch_free(plan)
        log("case: tuning 200 messages over the default candidates")
        choice = autotune.tune_batch(ctx, msgs, lengths, zero, zero, d_keys, m, d_in, d_out,
                                     path=str(tmp_path / "tune.json"))
        assert own in choice.timings
        assert choice.timings[f"({choice.blocks_per_lane}, {choice.tile_blocks})"] <= \
            choice.timings[own]
        assert choice.tile_blocks > 0
    finally:
        torch.cuda.synchronize()
        A.aesgpu_destroy(ctx)
