"""Waves that hold fluid, reservoir and solid cells (and lanes beyond the last
cell) in the step forms that run the update in all lanes of a wave: the
single-fluid and two-fluid models against the oracle at the bounds of the
parity tests, and several solutes in 16 bits, where a second solute with the
first one's parameters has to reproduce it bit for bit."""
import numpy as np
import pytest

from gpu_util import rel_l2, run_pair
from paper_0912_4230_amd import inputs as I
from paper_0912_4230_amd.sim import Simulation

pytestmark = pytest.mark.gpu

# one cell more and one less than whole waves, a row inside a wave, a row over two
SHAPES = [(13, 5, 11), (7, 9, 3), (67, 5, 3), (129, 3, 4)]


def _mixed(shape, physics):
    nx, ny, nz = shape
    rng = np.random.default_rng(nx)
    p = I.Problem(shape=shape, physics=physics, forchheimer=physics != I.IMMISCIBLE, A=0.0)
    p.faces[0] = I.Face(kind=I.RESERVOIR, rho=1.02, conc=0.8)
    p.faces[1] = I.Face(kind=I.RESERVOIR, rho=1.0, conc=0.1)
    p.eps = 0.5 + 0.4 * rng.random((nz, ny, nx))
    p.kinv = 20.0 * rng.random((3, nz, ny, nx))
    p.c0 = 0.1 + 0.8 * rng.random((nz, ny, nx))
    p.solid = (rng.random((nz, ny, nx)) < 0.2).astype(np.uint8)
    return p


@pytest.mark.parametrize("physics", [I.SINGLE, I.IMMISCIBLE])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("storage,tol", [("f64", 1e-10), ("f32", 1e-5)])
def test_mixed_waves_match_the_oracle(physics, shape, storage, tol):
    g, r, mask, _, _ = run_pair(_mixed(shape, physics), 12, storage)
    for a, b in zip(g[:2 if physics == I.SINGLE else 3], r):
        assert rel_l2(a, b, mask) < tol


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("storage", ["bf16", "f16"])
def test_identical_solutes_in_mixed_waves(shape, storage):
    p = _mixed(shape, I.MISCIBLE)
    p.species_tau_d = (0.8, 0.8)
    p.faces[0].conc_x, p.faces[1].conc_x = (0.8, 0.8), (0.1, 0.1)
    p.c0 = np.stack([p.c0] * 3)
    sim = Simulation(p, storage=storage)
    sim.step(12)
    a, b = sim.populations(2).cpu().numpy(), sim.populations(3).cpu().numpy()
    assert np.isfinite(a).all() and np.array_equal(a, b)
    conc = sim.moments()[2].cpu().numpy()
    assert np.array_equal(conc[1], conc[2])
    # reservoir cells keep their state, solid cells none
    w = np.array([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12)
    res = np.zeros(p.solid.shape, dtype=bool)
    res[:, :, [0, -1]] = True
    res &= p.solid == 0
    c = np.where(np.arange(shape[0]) == 0, 0.8, 0.1)[None, None, :] * p.eps
    bound = 2.0 ** (-8 if storage == "bf16" else -11)       # rounding to 8 and 11 bits
    for q in range(19):
        assert np.all(np.abs(a[q][res] - w[q] * c[res]) <= bound * w[q] * c[res])
        assert not a[q][p.solid != 0].any()
    sim.close()
