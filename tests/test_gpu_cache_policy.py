"""The cache policies of the step (lbm.hip: cache_policy) give the same bits.

A small lattice steps alone with its populations kept in the caches; in a
batch whose populations exceed the memory-side cache it steps streaming
(rows of whole lines in the large lattice beside it) or with plain loads (rows
that are not).  Moments, populations and diagnostics agree bitwise."""
import numpy as np
import pytest

from paper_0912_4230_amd import inputs as I
from paper_0912_4230_amd.sim import Simulation, step_batch

pytestmark = pytest.mark.gpu

STORED = {"f64": 8, "f32": 4, "bf16": 2, "f16": 2, "bf16s": 2, "f16s": 2}
CASES = [("single", "f64", ""), ("single", "bf16", ""), ("miscible", "f32", ""), ("miscible", "f16", ""),
         ("miscible", "f16s", ""), ("immiscible", "f32", ""), ("immiscible", "bf16s", ""),
         ("miscible", "f32", "tensor"), ("miscible", "f32", "solid"), ("miscible", "bf16", "solid"),
         ("miscible", "bf16s", "species")]


def _problem(physics, shape, option, seed):
    nx, ny, nz = shape
    if physics == "single":
        p = I.poiseuille(shape=shape)
    elif physics == "immiscible":
        p = I.drop(shape=shape, radius=min(shape) / 4.0)
    else:
        p = I.miscible(shape=shape, seed=seed, ring_angle=30.0 if option == "tensor" else None)
        if option == "solid":
            p.solid = I.block_obstacles(shape, seed=seed, solid_fraction=0.2)
        elif option == "species":
            p.species_tau_d = (0.8,)
            p.c0 = np.zeros((2, nz, ny, nx))
            p.faces[0].conc_x, p.faces[1].conc_x = (0.5,), (0.0,)
    return p


def _state(sim):
    rho, vel, conc, diag = sim.moments()
    pops = [sim.populations(k) for k in range(1 if sim.problem.physics == I.SINGLE else 1 + sim.problem.nspecies)]
    return [t.cpu().numpy() for t in [rho, vel, conc] + pops] + [diag]


@pytest.mark.parametrize("physics,storage,option", CASES)
def test_policies_give_the_same_bits(physics, storage, option):
    small = _problem(physics, (21, 18, 15), option, 1)
    alone = Simulation(small, storage=storage)
    alone.step(4)
    ref = _state(alone)
    alone.close()
    per_cell = 2 * 19 * STORED[storage] * (1 if physics == "single" else 2)
    for nx in (128, 101):          # rows of whole lines, and not
        big = Simulation(_problem(physics, (nx, 96, int(280e6 / per_cell / (nx * 96)) + 1), option, 2), storage=storage)
        sim = Simulation(small, storage=storage)
        assert big.nbytes + sim.nbytes > 256e6
        step_batch([sim, big], [4, 4])
        for a, b in zip(_state(sim), ref):
            assert np.array_equal(a, b)
        sim.close()
        big.close()
