"""Default tiles (host code only; the workspace is never touched).

A thread keeps those it has looked for: making contexts for the same lattices
again costs far less than the first time.  FP32's split step keeps wide tiles
where rows do not start on 128 bytes.
"""
import time

import pytest

from paper_1805_08643_amd import binding
import lbm_inputs as li


def test_contexts_in_turn():
    params = [binding.make_params(li.params(200 + 2 * k, 190 + k, 180, storage="f64")) for k in range(40)]
    rounds = []
    for _ in range(4):
        t0 = time.perf_counter()
        for p in params:
            binding.lbm_destroy(binding.lbm_create(p, 4096, 1 << 40, 0))
        rounds.append(time.perf_counter() - t0)
    assert min(rounds[1:]) < rounds[0] / 3, rounds


def test_kept_tiles_are_the_same():
    shapes = [(8 * k, 5 + k, 9, st) for k in range(1, 60) for st in ("f64", "f32", "f16s", "f16n")]
    seen = {}
    for _ in range(3):
        for nx, ny, nz, st in shapes:
            ctx = binding.lbm_create(binding.make_params(li.params(nx, ny, nz, storage=st)), 4096, 1 << 40, 0)
            tile = binding.lbm_get_tile(ctx)
            binding.lbm_destroy(ctx)
            assert seen.setdefault((nx, ny, nz, st), tile) == tile


@pytest.mark.parametrize("shape,width", [((220, 220, 220), 128), ((250, 250, 250), 128), ((186, 184, 184), 128),
                                         ((252, 62, 240), 128), ((96, 96, 96), 96), ((256, 256, 256), 128)])
def test_fp32_split_rows(shape, width):
    ctx = binding.lbm_create(binding.make_params(li.params(*shape, storage="f32")), 4096, 1 << 40, 0)
    assert binding.lbm_get_step_mode(ctx)[0] == binding.STEP_MODES["split"]
    assert binding.lbm_get_tile(ctx)[0] == width
    binding.lbm_destroy(ctx)
