"""The tile a new lattice steps with, at the edges of the search for it.

Single nodes, rows, columns and stacks, rows beyond the widest tile, columns
beyond the tallest, cubes either side of one residency of the chip: the tile
lies in the lattice, the step accepts it, and the populations are the ones of
the smallest tile, bit for bit.
"""
import numpy as np
import pytest

import lbm_inputs as li

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1), (1, 1, 700), (1, 600, 2), (600, 1, 2), (4, 4, 4), (8, 520, 3), (516, 3, 5), (254, 2, 3),
          (23, 19, 17), (25, 24, 23), (64, 64, 3), (100, 36, 20), (128, 72, 24)]


@pytest.mark.parametrize("storage", ["f64", "f32", "f16s", "f16n"])
@pytest.mark.parametrize("shape", SHAPES)
def test_default_tile(shape, storage):
    from paper_1805_08643_amd.binding import Lattice
    nx, ny, nz = shape
    if storage == "f16n":
        nx = max(4, nx // 4 * 4)
    cfg = li.params(nx, ny, nz, storage=storage, T_over_Tc=0.8, rho_ref=0.17, f16_exp=0)
    rho, u = li.random_fields(nx, ny, nz, seed=5, rho_lo=0.15, rho_hi=0.2, umax=0.02)
    states = []
    for smallest in (False, True):
        lat = Lattice(cfg)
        tx, ty, cz = lat.get_tile()[:3]
        assert 1 <= tx <= nx and 1 <= ty <= ny and 1 <= cz <= nz
        if smallest:
            npt = {"fused": 1, "pairs": 2, "split": 2 if storage == "f32" else 4}[lat.step_mode()]
            lat.set_tile(npt, 1, 1)
        else:
            lat.set_tile(tx, ty, cz)  # what the search gives, the setter accepts
        lat.init_fields(rho, u).step(2)
        states.append(lat.read_populations().cpu().numpy())
        lat.close()
    assert np.array_equal(states[0], states[1])


@pytest.mark.parametrize("storage,count", [("f16s", 2), ("f16s", 40), ("f32", 40)])
def test_default_batch_items(storage, count):
    """Few runs and many: the item size a batch chooses gives the states of
    another one; a mode change chooses anew unless the caller had chosen."""
    from paper_1805_08643_amd.binding import Batch
    runs = li.c5_batch(n_runs=count, seed=3, sizes=(32, 48))
    batches = []
    for chosen in (False, True):
        b = Batch([dict(p, storage=storage, rho_ref=0.17, f16_exp=0) for p, _ in runs])
        if chosen:
            b.set_item_nodes(5000)
        for k, (_, init) in enumerate(runs):
            b.init_droplets(k, init["droplets"], init["rho_L"], init["rho_V"], init["W"])
        b.step(2)
        batches.append(b)
    a, b = batches
    assert a.tuning()[1] in (4096, 8192, 12288, 16384, 24576, 32768) and b.tuning()[1] == 5000
    for k in range(count):
        assert bool((a.read_populations(k) == b.read_populations(k)).all()), k
    a.set_step_mode("fused")
    b.set_step_mode("fused")
    assert a.tuning()[1] == 8192 and b.tuning()[1] == 5000
    a.close()
    b.close()
