"""The step forms of the cache policies that only larger lattices take: plain loads
in the split forms and in the FP32 tensor step with rows of whole lines, and
streaming with obstacles.  Which policy a launch takes is looked up
(policy_util), so that a line that moves cannot make a test compare a form with
itself.  A small lattice steps alone and in the launch of a large one; moments,
populations and diagnostics agree bitwise."""
import numpy as np
import pytest

from policy_util import KEEP, REUSE, STREAM, lattice, policies

from paper_0912_4230_amd import inputs as I
from paper_0912_4230_amd.sim import Simulation, step_batch

pytestmark = pytest.mark.gpu

TINY, MID = (21, 18, 15), (41, 36, 30)
# storage, option, the small lattice and its policy alone, the large one and the policy of their launch
CASES = [("f16s", "", TINY, KEEP, (213, 203, 204), REUSE), ("bf16s", "", TINY, KEEP, (213, 203, 204), REUSE),
         ("f16s", "solid", TINY, KEEP, (183, 181, 184), REUSE), ("bf16s", "species", TINY, KEEP, (183, 181, 184), REUSE),
         ("f16s", "tensor", TINY, KEEP, (183, 181, 184), REUSE), ("bf16s", "solid", TINY, KEEP, (128, 120, 110), STREAM),
         ("f32", "tensor", TINY, KEEP, (256, 224, 192), REUSE), ("f32", "tensor", TINY, KEEP, (128, 96, 80), STREAM),
         ("bf16", "tensor", TINY, KEEP, (161, 132, 175), STREAM), ("f64", "tensor", TINY, KEEP, (171, 114, 128), STREAM),
         ("f32", "solid", MID, STREAM, (101, 96, 95), REUSE), ("bf16", "solid", (45, 44, 60), STREAM, (131, 124, 112), REUSE),
         ("f16", "", (45, 44, 60), STREAM, (151, 124, 112), REUSE)]


def _problem(shape, option, seed):
    nx, ny, nz = shape
    rng = np.random.default_rng(seed)
    p = I.Problem(shape=shape, physics=I.MISCIBLE, forchheimer=True, nu0=0.1, tau_d=0.65)
    p.faces[0] = I.Face(kind=I.RESERVOIR, rho=1.02, conc=0.8, conc_x=(0.5,))
    p.faces[1] = I.Face(kind=I.RESERVOIR, rho=1.0, conc=0.1, conc_x=(0.2,))
    p.eps = 0.5 + 0.4 * rng.random((nz, ny, nx), dtype=np.float32)
    p.kinv = 20.0 * rng.random((6 if option == "tensor" else 3, nz, ny, nx), dtype=np.float32)
    if option == "tensor":          # positive definite: the diagonal outweighs the rest
        p.kinv[:3] += 21.0
        p.kinv[3:] -= 10.0
    elif option == "solid":
        p.solid = (rng.random((nz, ny, nx), dtype=np.float32) < 0.2).astype(np.uint8)
    elif option == "species":
        p.species_tau_d = (0.8,)
    p.c0 = rng.random((p.nspecies, nz, ny, nx) if p.nspecies > 1 else (nz, ny, nx), dtype=np.float32)
    return p


def _state(sim):
    rho, vel, conc, diag = sim.moments()
    return [t.cpu().numpy() for t in [rho, vel, conc] + [sim.populations(k) for k in range(1 + sim.problem.nspecies)]] + [diag]


@pytest.mark.parametrize("storage,option,small,alone,large,together", CASES)
def test_forms_give_the_same_bits(storage, option, small, alone, large, together):
    opts = {"links": option == "solid", "tensor": option == "tensor", "species": 2 if option == "species" else 1}
    a, b = [lattice("miscible", storage, s, **opts) for s in (small, large)]
    assert policies([[a]]) == [alone] and policies([[a, b]]) == [together]
    p = _problem(small, option, 1)
    sim = Simulation(p, storage=storage)
    sim.step(4)
    ref = _state(sim)
    assert np.isfinite(ref[0]).all()
    sim.close()
    big, sim = Simulation(_problem(large, option, 2), storage=storage), Simulation(p, storage=storage)
    step_batch([sim, big], [4, 4])
    for x, y in zip(_state(sim), ref):
        assert np.array_equal(x, y)
    sim.close()
    big.close()
