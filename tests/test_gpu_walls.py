"""The ghost layer of Eq. (57) at the edges of its kernel's 32 x 4 tiles.

Planes of one tile, of one node more or less, of a single row or column, and
the two-plane lattice whose second layers are each other's first: three FP64
steps against the oracle (1e-12 of the node's density, the bound of the other
parity tests), and FP32 within 5e-6 per step.
"""
import numpy as np
import pytest

import lbm_inputs as li
from oracle import ref

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("shape", [(32, 4, 3), (33, 5, 4), (31, 3, 2), (1, 1, 2), (64, 8, 2), (2, 9, 3), (1, 6, 3),
                                   (70, 1, 4)])
def test_ghost_layer_tiles(shape, storage):
    from paper_1805_08643_amd.binding import Lattice
    nx, ny, nz = shape
    cfg = li.params(nx, ny, nz, storage=storage, wall_z=1, T_over_Tc=0.8, theta_wall_deg=60.0, ghost_rho_min=0.02,
                    gravity=(0.0, 0.0, -1e-5))
    rho, u = li.random_fields(nx, ny, nz, seed=11, rho_lo=0.15, rho_hi=0.2, umax=0.02)
    lat = Lattice(cfg)
    lat.init_fields(rho, u).step(3)
    got = lat.read_populations().cpu().numpy()
    lat.close()
    p = ref.make_params(cfg)
    want = ref.step(p, ref.equilibrium(p, rho, u), 3)
    assert np.max(np.abs(got - want) / want.sum(0)) < (1e-12 if storage == "f64" else 1.5e-5)
