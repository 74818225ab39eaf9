"""The ways through a march that the tile decides: the same populations.

FP32's one-node march loads a plane ahead, or waits for its stores first (few
waves to a block and several blocks to a CU), by tile; runs of one plane, of
several with a ragged last one and of the whole height turn its registers and
the four LDS planes differently.  Each against a lattice in one run of small
blocks, bit for bit, after three steps.
"""
import pytest
import torch

import lbm_inputs as li

pytestmark = pytest.mark.gpu


def _lattice(shape, storage, op, wall, mode):
    from paper_1805_08643_amd.binding import Lattice
    cfg = li.params(*shape, storage=storage, op=op, wall_z=wall, T_over_Tc=0.8, theta_wall_deg=60.0, rho_ref=0.17,
                    f16_exp=0)
    lat = Lattice(cfg)
    lat.set_step_mode(mode)
    return lat


def _states(shape, storage, op, wall, mode, tiles):
    rho, u = li.random_fields(*shape, seed=6, rho_lo=0.15, rho_hi=0.2, umax=0.02)
    for tile in tiles:
        lat = _lattice(shape, storage, op, wall, mode)
        lat.set_tile(*tile)
        lat.init_fields(rho, u).step(3)
        yield lat.save_state()
        lat.close()


# 67 x 23 x 41: 630 and 1230 blocks of one wave (paced), 30 and 180 of one wave, 36
# and 4 of eight.
FP32_TILES = [(16, 4, 41), (16, 4, 2), (16, 4, 1), (16, 4, 7), (67, 7, 5), (67, 7, 41)]


@pytest.mark.parametrize("wall", [0, 1])
@pytest.mark.parametrize("op", ["nonorth", "orth"])
def test_fp32_march_by_tile(op, wall):
    states = list(_states((67, 23, 41), "f32", op, wall, "fused", FP32_TILES))
    for tile, s in zip(FP32_TILES, states):
        assert torch.equal(s, states[0]), tile


# 40 x 23 x 29: one plane, several with a ragged last run and the whole height;
# rows that leave lanes, and waves, of a role without a group.
SPLIT_TILES = [(40, 7, 29), (40, 6, 1), (16, 5, 4), (8, 9, 7), (40, 4, 10), (24, 23, 3)]


@pytest.mark.parametrize("wall", [0, 1])
@pytest.mark.parametrize("op", ["nonorth", "orth"])
@pytest.mark.parametrize("storage", ["f32", "f16s", "f16n"])
def test_split_step_by_tile(storage, op, wall):
    tiles = [t for t in SPLIT_TILES if storage != "f32" or t[0] * t[1] <= 512]
    states = list(_states((40, 23, 29), storage, op, wall, "split", tiles))
    for tile, s in zip(tiles, states):
        assert torch.equal(s, states[0]), tile


@pytest.mark.parametrize("op", ["nonorth", "orth"])
@pytest.mark.parametrize("shape,storage,mode", [((90, 80, 70), "f64", "fused"), ((96, 96, 96), "f32", "split"),
                                                ((98, 96, 90), "f16s", "pairs"), ((96, 96, 96), "f16n", "split")])
def test_default_runs_of_several_planes(shape, storage, mode, op):
    lat = _lattice(shape, storage, op, 0, mode)
    tile = lat.get_tile()
    lat.close()
    assert tile[2] > 2
    small = {"fused": 1, "pairs": 2, "split": 2 if storage == "f32" else 4}[mode]
    a, b = _states(shape, storage, op, 0, mode, [tile, (16 * small, 4, shape[2])])
    assert torch.equal(a, b)


@pytest.mark.parametrize("op", ["nonorth", "orth"])
@pytest.mark.parametrize("storage", ["f32", "f16s", "f16n"])
def test_batch_items_in_turn(storage, op):
    """Items with few rows (waves without a group) and more items than blocks."""
    from paper_1805_08643_amd.binding import Batch, Lattice
    cfgs = [li.params(*s, storage=storage, op=op, T_over_Tc=0.8, rho_ref=0.17, f16_exp=0)
            for s in [(12, 5, 9), (40, 23, 17), (8, 3, 30), (64, 33, 6)]]
    fields = [li.random_fields(c["nx"], c["ny"], c["nz"], seed=k, rho_lo=0.15, rho_hi=0.2, umax=0.02)
              for k, c in enumerate(cfgs)]
    b = Batch(cfgs)
    b.set_item_nodes(600)
    b.set_blocks(3)
    for k, (rho, u) in enumerate(fields):
        b.init_fields(k, rho, u)
    b.step(3)
    for k, (c, (rho, u)) in enumerate(zip(cfgs, fields)):
        lat = Lattice(c)
        lat.init_fields(rho, u).step(3)
        assert torch.equal(b.read_populations(k), lat.read_populations()), k
        lat.close()
    b.close()
