"""The class passes of the free surface at the sizes where one launch (a block
with the classes in LDS) takes over from three: 57,344 cells for lattices one
cell thick, 36,864 else.  Against the oracle in FP64, classes exact and fields
at the bound of the parity tests; and steps in which more cells convert than
the block lists at once (3,072)."""
import numpy as np
import pytest

from gpu_util import rel_l2
from paper_0912_4230_amd import inputs as I
from paper_0912_4230_amd.sim import Simulation, step_batch

pytestmark = pytest.mark.gpu


def _compare(p, steps, sim=None):
    from oracle import oracle as O
    own = sim is None
    if own:
        sim = Simulation(p, storage="f64")
        sim.step(steps)
    o = O.Oracle(p)
    o.step(steps)
    cls, mass, _ = sim.free_surface()
    oc, om, _ = o.fs_state()
    fluid = o.cell_types() == 0
    cls, mass = cls.cpu().numpy(), mass.cpu().numpy()
    assert np.array_equal(cls[fluid], oc[fluid])
    assert rel_l2(mass, om, fluid) < 1e-10
    rho, vel, conc, _ = sim.moments()
    r, v, c = o.moments()
    live = fluid & (oc > 0)
    assert rel_l2(rho.cpu().numpy(), r, live) < 1e-10
    assert rel_l2(vel.cpu().numpy(), v, live) < 1e-10
    assert rel_l2(conc.cpu().numpy(), c, live) < 1e-10
    o.close()
    if own:
        sim.close()
    return oc


def _drop(shape):
    return I.falling_drop(shape=shape, radius=8.3, centre=(shape[0] / 2 + 0.3, 10.4, 0.0), tau=0.7, speed=0.05)


@pytest.mark.parametrize("shape", [(16, 40, 1), (239, 239, 1), (256, 224, 1), (239, 240, 1)])
def test_drop_at_the_edges(shape):
    start = Simulation(_drop(shape), storage="f64")
    before = start.free_surface()[0].cpu().numpy()
    start.close()
    assert (_compare(_drop(shape), 60) != np.minimum(before, 2)).sum() > 20   # cells did convert


@pytest.mark.parametrize("shape", [(33, 33, 33), (36, 32, 32), (37, 32, 32), (13, 7, 5)])
def test_penetration_at_the_edges(shape):
    _compare(I.penetration(shape=shape, seed=2), 40)


@pytest.mark.parametrize("shape", [(33, 33, 33), (230, 200, 1)])
def test_more_conversions_than_the_list_holds(shape):
    nx, ny, nz = shape
    rng = np.random.default_rng(5)
    # nearly full interface cells everywhere in a strongly varying flow, some gas among them
    c0 = np.where(rng.random((nz, ny, nx)) < 0.05, 0.0, 0.9995)
    p = I.Problem(shape=shape, physics=I.FREESURF, nu0=0.2, c0=c0, vel0=0.05 * (rng.random((3, nz, ny, nx)) - 0.5))
    a = _compare(p, 1)
    assert (a == 2).sum() > 3072        # filled in one step
    _compare(p, 3)


def test_small_and_large_lattices_in_a_batch():
    shapes = [(239, 239, 1), (239, 240, 1), (16, 40, 1)]
    sims = [Simulation(_drop(s), storage="f64") for s in shapes]
    step_batch(sims, [30] * 3)
    for s, sim in zip(shapes, sims):
        _compare(_drop(s), 30, sim)
        sim.close()
