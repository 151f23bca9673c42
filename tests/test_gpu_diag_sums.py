"""The FP64 diagnostics against sums of the same moments taken in numpy, at the
sizes where the summation changes: 1024 blocks of 256 cells is the largest
lattice whose partials one block sums, more take a launch over chunks of 1024
first, the last chunk ragged.

Both sides add the same n FP64 terms in different orders, so they differ by at
most 2 n u sum|terms| (u = 2^-53; Higham, Accuracy and Stability of Numerical
Algorithms, Sec. 4.2): the tolerance.  Maxima and counts are exact."""
import numpy as np
import pytest

from paper_0912_4230_amd import inputs as I
from paper_0912_4230_amd.sim import Simulation, step_batch

pytestmark = pytest.mark.gpu

# cells: one block, 1024 blocks exactly, one block more with a single cell, 1027
# (ragged), 8256 (chunks of 1024 and a last of 64)
SHAPES = [(16, 4, 4), (64, 64, 64), (5, 52429, 1), (37, 64, 111), (128, 128, 129)]


def _problem(shape, nspecies=1):
    nx, ny, nz = shape
    rng = np.random.default_rng(nx * 7 + nz)
    p = I.Problem(shape=shape, physics=I.MISCIBLE, tau_d=0.65, nu0=0.1)
    p.eps = 0.4 + 0.4 * rng.random((nz, ny, nx))
    p.kinv = 50.0 * rng.random((3, nz, ny, nx))
    p.rho0 = 1.0 + 0.01 * rng.random((nz, ny, nx))
    p.vel0 = 0.02 * (rng.random((3, nz, ny, nx)) - 0.5)
    if nspecies > 1:
        p.species_tau_d = (0.8, 0.7)[:nspecies - 1]
    p.c0 = rng.random((nspecies, nz, ny, nx) if nspecies > 1 else (nz, ny, nx))
    return p


def _close(got, terms):
    """got against the sum of the terms"""
    t = np.asarray(terms, dtype=np.float64).reshape(-1)
    tol = 2.0 * t.size * 2.0 ** -53 * np.abs(t).sum()
    assert abs(got - t.sum()) <= tol, (got, t.sum(), tol)


@pytest.mark.parametrize("shape", SHAPES)
def test_diagnostics_are_the_sums_of_the_moments(shape):
    p = _problem(shape)
    sim = Simulation(p, storage="f64")
    sim.step(2)
    before = sim.moments()[1].cpu().numpy()
    sim.step(1)
    rho, vel, conc, d = sim.moments()
    rho, vel, conc = rho.cpu().numpy(), vel.cpu().numpy(), conc.cpu().numpy()
    _close(d[0], rho)
    for a in range(3):
        _close(d[1 + a], rho * vel[a])
    _close(d[4], p.eps * conc)
    uu = (vel * vel).sum(axis=0)
    du = ((vel - before) ** 2).sum(axis=0)
    # a quotient of two such sums of positive terms, and the rounding of its terms
    assert abs(d[5] - du.sum() / uu.sum()) <= d[5] * (4.0 * uu.size + 16.0) * 2.0 ** -53
    assert abs(d[6] - np.sqrt(uu.max())) <= 4.0 * 2.0 ** -53 * d[6]
    assert d[7] == 0.0
    sim.close()


@pytest.mark.parametrize("shape", SHAPES[1:4])
def test_solute_totals_are_the_sums_of_the_moments(shape):
    p = _problem(shape, nspecies=3)
    sim = Simulation(p, storage="f64")
    sim.step(2)
    conc = sim.moments()[2].cpu().numpy()
    for k, total in enumerate(sim.solute_totals()):
        _close(total, p.eps * conc[k])
    sim.close()


def test_diagnostics_do_not_depend_on_the_batch():
    # lattices summed in one launch and in two, together and alone
    alone, sims = [], []
    for shape in SHAPES[:4]:
        s = Simulation(_problem(shape), storage="f32")
        s.step(3)
        alone.append(s.diag())
        s.close()
        sims.append(Simulation(_problem(shape), storage="f32"))
    step_batch(sims, [3] * len(sims))
    for s, d in zip(sims, alone):
        assert np.array_equal(s.diag(), d)
        s.close()
