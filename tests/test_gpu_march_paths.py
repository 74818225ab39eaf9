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
