"""The free-surface step under both of its cache policies (lbm.hip: cache_policy)
gives the same bits: a small lattice steps alone (streaming) and in a batch
whose populations it pays to keep in the memory-side cache."""
import numpy as np
import pytest

from paper_0912_4230_amd import inputs as I
from paper_0912_4230_amd.sim import Simulation, step_batch

pytestmark = pytest.mark.gpu

STORED = {"f64": 8, "f32": 4, "bf16": 2, "f16": 2, "bf16s": 2, "f16s": 2}


def _problem(shape, option, seed):
    p = I.penetration(shape=shape, seed=seed, ring_angle=30.0 if option == "tensor" else None)
    if option == "tension":
        p.A = 1e-3
    return p


def _state(sim):
    rho, vel, conc, diag = sim.moments()
    cls, mass, lam, lost = sim.free_surface(fill=True)
    return [t.cpu().numpy() for t in (rho, vel, conc, sim.populations(), cls, mass, lam)] + [diag, np.array(lost)]


@pytest.mark.parametrize("storage,option", [(s, "") for s in STORED] +
                         [("f64", "tension"), ("f32", "tensor"), ("f16s", "tension")])
def test_policies_give_the_same_bits(storage, option):
    small = _problem((21, 18, 25), option, 1)
    alone = Simulation(small, storage=storage)
    alone.step(30)
    ref = _state(alone)
    alone.close()
    n = int(70e6 / (2 * 19 * STORED[storage]) / (64 * 61)) + 1
    big, sim = Simulation(_problem((64, 61, n), option, 2), storage=storage), Simulation(small, storage=storage)
    step_batch([sim, big], [30, 30])
    for a, b in zip(_state(sim), ref):
        assert np.array_equal(a, b, equal_nan=True)
    sim.close()
    big.close()
