"""The step of runs with walls on x or y (k_single) on long thin ducts.

A duct whose fields repeat every 64 planes keeps the states of one period, bit
for bit.  The longest has more planes than a launch has threads for at one
256-thread block each (2^24 such blocks would be 2^32 threads).
"""
import pytest
import torch

import lbm_inputs as li

pytestmark = pytest.mark.gpu


def _populations(nx, ny, nz, storage, rho, u):
    from paper_1805_08643_amd.binding import Lattice
    cfg = li.params(nx, ny, nz, storage=storage, psi_form="exp", G=0.0, sigma=0.0, tau_nu=0.8, wall_x=1, wall_y=1,
                    wall_z=0, lid_u=(0.0, 0.0, 0.02), lid_rho=1.0, rho_ref=1.0, f16_exp=12)
    lat = Lattice(cfg)
    lat.init_fields(rho, u).step(2)
    f = lat.read_populations()
    lat.close()
    return f


@pytest.mark.parametrize("shape,storage", [((1, 1, 2 ** 24 + 64), "f32"), ((3, 5, 6400), "f64"), ((17, 16, 640), "f16s"),
                                           ((16, 16, 640), "f32")])
def test_duct_repeats_its_period(shape, storage):
    nx, ny, nz = shape
    gen = torch.Generator().manual_seed(9)
    rho = 1.0 + 0.05 * torch.rand((64, ny * nx), generator=gen, dtype=torch.float64)
    u = 0.02 * (torch.rand((3, 64, ny * nx), generator=gen, dtype=torch.float64) - 0.5)
    want = _populations(nx, ny, 64, storage, rho, u)
    k = nz // 64
    got = _populations(nx, ny, nz, storage, rho.cuda().repeat(k, 1), u.cuda().repeat(1, k, 1))
    assert bool((got.view(19, k, -1) == want.view(19, 1, -1)).all())
    assert bool(torch.isfinite(want).all())
