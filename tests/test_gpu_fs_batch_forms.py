"""A free-surface lattice without surface tension has the same bits alone and in a batch with one that has
it, which sends both through the surface-tension form of the step: every storage form rounds the populations
alike in the two (FP16 did not while the compiler fused one form's last operation with its conversion)."""
import dataclasses

import numpy as np
import pytest

from paper_0912_4230_amd import inputs as I
from paper_0912_4230_amd.sim import Simulation, step_batch

pytestmark = pytest.mark.gpu


def _state(sim):
    cls, mass, fill, lost = sim.free_surface(fill=True)
    rho, vel, _, diag = sim.moments()
    return [t.cpu().numpy() for t in (cls, mass, fill, rho, vel, sim.populations(0))] + [diag]


@pytest.mark.parametrize("storage", ["f64", "f32", "bf16", "f16", "bf16s", "f16s"])
@pytest.mark.parametrize("shape", [(24, 20, 22), (48, 40, 44)])
def test_plain_lattice_beside_one_with_surface_tension(storage, shape):
    p = I.penetration(shape=shape, seed=3)
    alone = Simulation(p, storage=storage)
    alone.step(30)
    ref = _state(alone)
    assert (ref[0] == 1).any()
    alone.close()
    a = Simulation(p, storage=storage)
    b = Simulation(dataclasses.replace(I.penetration(shape=(20, 24, 18), seed=4), A=0.01), storage=storage)
    step_batch([a, b], [30, 30])
    for x, y in zip(_state(a), ref):
        assert np.array_equal(x, y)
    a.close()
    b.close()
