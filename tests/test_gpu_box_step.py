"""The step of runs with walls on x or y (k_single) where its grid can go wrong.

A block takes 256 consecutive nodes of one z-plane: planes of exactly one and
of several blocks, of one node more, rows and planes of a single node, and
every mix of walls and periodic axes.  One and three steps against the oracle
(FP64: 1e-12 of the node's density, the bound of the other parity tests), and
the store policies against each other byte for byte.
"""
import numpy as np
import pytest

import lbm_inputs as li
from oracle import ref

pytestmark = pytest.mark.gpu

SHAPES = [(16, 16, 5), (32, 16, 2), (257, 1, 3), (1, 7, 4), (5, 1, 2), (64, 9, 3), (3, 3, 3)]
WALLS = [(1, 1, 1), (1, 0, 1), (0, 1, 0), (1, 0, 0)]


def _run(cfg, rho, u, steps, policy):
    from paper_1805_08643_amd.binding import Lattice
    lat = Lattice(cfg)
    lat.set_store_policy(policy)
    lat.init_fields(rho, u).step(steps)
    f, raw = lat.read_populations().cpu().numpy(), lat.save_state().cpu().numpy()
    lat.close()
    return f, raw


@pytest.mark.parametrize("walls", WALLS)
@pytest.mark.parametrize("shape", SHAPES)
def test_box_step_grid_edges(shape, walls):
    nx, ny, nz = shape
    lid = (0.05, 0.0, -0.02) if walls[1] else (0.0, 0.0, 0.0)
    cfg = li.params(nx, ny, nz, storage="f64", psi_form="exp", G=0.0, sigma=0.0, tau_nu=0.8, wall_x=walls[0],
                    wall_y=walls[1], wall_z=walls[2], lid_u=lid, lid_rho=1.0, gravity=(0.0, 0.0, 1e-5))
    rho, u = li.random_fields(nx, ny, nz, seed=3, rho_lo=0.95, rho_hi=1.05, umax=0.02)
    p = ref.make_params(cfg)
    for steps in (1, 3):
        f, raw = _run(cfg, rho, u, steps, "cached")
        want = ref.step(p, ref.equilibrium(p, rho, u), steps)
        assert np.max(np.abs(f - want) / want.sum(0)) < 1e-12
        assert np.array_equal(raw, _run(cfg, rho, u, steps, "stream")[1])


@pytest.mark.parametrize("storage", ["f32", "f16s"])
def test_box_step_store_policies_other_formats(storage):
    cfg = li.params(33, 17, 5, storage=storage, psi_form="exp", G=0.0, sigma=0.0, tau_nu=0.8, wall_x=1, wall_y=1,
                    wall_z=1, lid_u=(0.05, 0.0, 0.0), lid_rho=1.0, rho_ref=1.0, f16_exp=12)
    rho, u = li.random_fields(33, 17, 5, seed=3, rho_lo=0.95, rho_hi=1.05, umax=0.02)
    assert np.array_equal(_run(cfg, rho, u, 3, "cached")[1], _run(cfg, rho, u, 3, "stream")[1])
