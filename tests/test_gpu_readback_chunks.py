"""Fields and diagnostics where their chunks of 256 nodes, taken in groups of
eight from the end, are one, a group, one more, or end in a part of either.

Densities against the sums of the populations (the order of 19 FP64 terms:
1e-14), and the mass against their sum (1e-13: at most 2^13 terms, added in
parts).
"""
import pytest
import torch

import lbm_inputs as li

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nodes", [1, 255, 256, 257, 1793, 2047, 2048, 2049, 2304, 8191])
def test_every_node_once(nodes):
    from paper_1805_08643_amd.binding import Lattice
    lat = Lattice(li.params(nodes, 1, 1, storage="f64", T_over_Tc=0.8))
    rho, u = li.random_fields(nodes, 1, 1, seed=2, rho_lo=0.15, rho_hi=0.2, umax=0.02)
    lat.init_fields(rho, u).step(2)
    want = lat.read_populations().sum(0)
    out = lat.read_fields()
    assert float(((out["rho"] - want).abs() / want).max()) < 1e-14
    assert all(bool(torch.isfinite(v).all()) for v in out.values())
    d = lat.diagnostics()
    assert abs(d["mass"] - float(want.sum())) < 1e-13 * float(want.sum())
    assert d["nonfinite"] == 0
    lat.close()
