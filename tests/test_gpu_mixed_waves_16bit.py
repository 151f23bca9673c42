"""Waves that hold fluid, reservoir and solid cells, and lanes beyond the last
cell, in the 16-bit step forms that run the update in all lanes: single-fluid,
two-fluid and several-solute steps against the FP64 oracle, and a second solute
with the first one's parameters against the first.

Bounds.  A store rounds every population's deviation (or, in the second lattice,
population) by a factor 1 + d, |d| <= u = 2^-9 (BF16) or 2^-12 (FP16); the split
forms round smaller remainders.  The sums over a cell's populations that the
moments are change by at most u S a step, S = the largest sum of their magnitudes
in a cell, and N steps of one sign by N u S; collision and drag return a part of
such an error, of either sign.  The bounds are 4 N u S, and twice that in the
two-fluid model, whose recolouring moves populations along a normalised gradient.
A lane that pulled from a wrong cell is off by the differences between the random
cells, of the order of S itself."""
import numpy as np
import pytest

from test_gpu_mixed_waves import SHAPES, _mixed

from paper_0912_4230_amd import inputs as I
from paper_0912_4230_amd.sim import Simulation

pytestmark = pytest.mark.gpu

N = 12
U = {"bf16": 2.0 ** -9, "bf16s": 2.0 ** -9, "f16": 2.0 ** -12, "f16s": 2.0 ** -12}


def _oracle(p):
    from oracle import oracle as O
    o = O.Oracle(p)
    o.step(N)
    r, v, c = o.moments()
    conc = [o.species_conc(k) for k in range(p.nspecies)] if p.nspecies > 1 else [c]
    mask = o.cell_types() == 0
    o.close()
    return r, v, conc, mask


def _magnitudes(p):
    """The largest sums of |f - w| (first lattice) and |h| (the others) in a cell of the FP64 lattice, of steps 1..N."""
    sim = Simulation(p, storage="f64")
    s = [0.0] * (1 if p.physics == I.SINGLE else 1 + p.nspecies)
    for _ in range(N):
        sim.step(1)
        for k in range(len(s)):
            s[k] = max(s[k], float(sim.populations(k).abs().sum(dim=0).max()))
    sim.close()
    return s


def _check(p, storage):
    r, v, c, mask = _oracle(p)
    s = _magnitudes(p)
    sim = Simulation(p, storage=storage)
    sim.step(N)
    rho, vel, conc, _ = sim.moments()
    rho, vel, conc = [t.double().cpu().numpy() for t in (rho, vel, conc)]
    unit = (8.0 if p.physics == I.IMMISCIBLE else 4.0) * N * U[storage]
    err = [float(np.abs(rho - r)[mask].max()), float(np.abs(vel - v)[:, mask].max())]
    bound = [unit * s[0], unit * s[0] / float(r[mask].min())]
    for k in range(len(s) - 1):
        g = conc[k] if p.nspecies > 1 else conc
        # eps C is the sum of the solute's populations, rho C that of fluid 1's
        scale = float(p.eps[mask].min() if p.physics == I.MISCIBLE else r[mask].min())
        err.append(float(np.abs(g - c[k])[mask].max()))
        bound.append(unit * s[1 + k] / scale)
    print(f"[mixed waves] {p.physics} {p.shape} {storage}: errors {err}, bounds {bound}", flush=True)
    assert all(e <= b for e, b in zip(err, bound)), (err, bound)
    return sim


@pytest.mark.parametrize("physics", [I.SINGLE, I.IMMISCIBLE])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("storage", list(U))
def test_mixed_waves_16bit(physics, shape, storage):
    _check(_mixed(shape, physics), storage).close()


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("storage", list(U))
def test_further_solute_equals_the_first(shape, storage):
    p = _mixed(shape, I.MISCIBLE)
    p.species_tau_d = (p.tau_d,)
    p.faces[0].conc_x, p.faces[1].conc_x = (0.8,), (0.1,)
    p.c0 = np.stack([p.c0] * 2)
    sim = _check(p, storage)
    a, b = sim.populations(1).cpu().numpy(), sim.populations(2).cpu().numpy()
    assert np.isfinite(a).all() and np.array_equal(a, b)
    sim.close()
