"""The ghost layer of Eq. (57) on narrow walls, whose kernel takes narrower tiles.

Walls longer than 1024 rows with widths on either side of each tile width,
the last tile full and not, against the oracle (three FP64 steps,
1e-12 of the node's density, the bound of the other parity tests), and a strip
of 2^26 rows, more than 32 x 4 tiles could cover in one launch: its fields
repeat every 64 rows, so it keeps the states of one period, bit for bit.
"""
import numpy as np
import pytest
import torch

import lbm_inputs as li
from oracle import ref

pytestmark = pytest.mark.gpu


def _config(nx, ny, nz, storage):
    return li.params(nx, ny, nz, storage=storage, wall_z=1, T_over_Tc=0.8, theta_wall_deg=60.0, ghost_rho_min=0.02,
                     rho_ref=0.17, f16_exp=0)


def _populations(cfg, rho, u, steps):
    from paper_1805_08643_amd.binding import Lattice
    lat = Lattice(cfg)
    lat.init_fields(rho, u).step(steps)
    f = lat.read_populations()
    lat.close()
    return f


@pytest.mark.parametrize("shape", [(1, 1079, 2), (1, 1025, 2), (2, 1055, 3), (3, 1057, 3), (4, 1056, 2), (5, 1041, 3),
                                   (8, 1040, 3), (9, 1033, 2), (16, 1032, 2), (17, 1030, 2)])
def test_narrow_walls(shape):
    nx, ny, nz = shape
    cfg = _config(nx, ny, nz, "f64")
    rho, u = li.random_fields(nx, ny, nz, seed=4, rho_lo=0.15, rho_hi=0.2, umax=0.02)
    got = _populations(cfg, rho, u, 3).cpu().numpy()
    p = ref.make_params(cfg)
    want = ref.step(p, ref.equilibrium(p, rho, u), 3)
    assert np.max(np.abs(got - want) / want.sum(0)) < 1e-12


@pytest.mark.parametrize("shape,storage", [((1, 2 ** 26, 2), "f16s"), ((6, 64 * 300, 3), "f64")])
def test_strip_repeats_its_period(shape, storage):
    nx, ny, nz = shape
    gen = torch.Generator().manual_seed(9)
    rho = 0.17 + 0.02 * torch.rand((nz, 64, nx), generator=gen, dtype=torch.float64)
    u = 0.02 * (torch.rand((3, nz, 64, nx), generator=gen, dtype=torch.float64) - 0.5)
    want = _populations(_config(nx, 64, nz, storage), rho, u, 2).view(19, nz, 64 * nx)
    k = ny // 64
    got = _populations(_config(nx, ny, nz, storage), rho.cuda().repeat(1, k, 1), u.cuda().repeat(1, 1, k, 1), 2)
    got = got.view(19, nz, k, 64 * nx)
    assert bool(torch.isfinite(want).all())
    assert all(bool((got[a] == want[a, :, None]).all()) for a in range(19))
