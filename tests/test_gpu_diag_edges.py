"""The FP64 diagnostics and solute totals where their summation changes: up to 3072
blocks of 256 cells one launch sums a lattice's partials, more take a launch over
chunks of 1024 first.  Sums against numpy within 2 n u sum|terms|, as the two
orders of n terms may differ."""
import numpy as np
import pytest

from test_gpu_diag_sums import _close, _problem

from paper_0912_4230_amd.sim import Simulation

pytestmark = pytest.mark.gpu

# 3072 blocks exactly, and one more that holds three cells (the last chunk a single row)
SHAPES = [(64, 64, 192), (5, 157287, 1)]


@pytest.mark.parametrize("shape", SHAPES)
def test_sums_on_both_sides(shape):
    assert (int(np.prod(shape)) + 255) // 256 == (3072 if shape == SHAPES[0] else 3073)
    p = _problem(shape, nspecies=2)
    sim = Simulation(p, storage="f64")
    sim.step(2)
    rho, vel, conc, d = sim.moments()
    rho, vel, conc = rho.cpu().numpy(), vel.cpu().numpy(), conc.cpu().numpy()
    _close(d[0], rho)
    for a in range(3):
        _close(d[1 + a], rho * vel[a])
    _close(d[4], p.eps * conc[0])
    assert d[7] == 0.0
    for k, total in enumerate(sim.solute_totals()):
        _close(total, p.eps * conc[k])
    sim.close()
