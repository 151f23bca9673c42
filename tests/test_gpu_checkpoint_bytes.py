"""What a checkpoint holds is the lattice's: set up in workspaces that held
different bytes before, two lattices give checkpoints that differ only where no
call ever writes (the padding of the planes and fields; free surface: the share
and velocity planes, 32 bytes per cell, and the row lists), before the first
step, when the step has not written its copy of the populations yet, and after
it.

The bytes 0x00 and 0xa5 differ, so the differing bytes count the unset ones.  A
population plane is followed by at most 768 bytes of padding, a field by at most
255; there are fewer than 32 fields."""
import numpy as np
import pytest

from gpu_util import ensure_built, need_gpu

from paper_0912_4230_amd import inputs as I
from paper_0912_4230_amd.sim import Simulation

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _setup():
    need_gpu()
    ensure_built()


def _problem(physics):
    shape = (24, 22, 20)
    if physics == "single":
        return I.poiseuille(shape=shape)
    if physics == "two-fluid":
        return I.drop(shape=shape, radius=5.0)
    if physics == "free surface":
        return I.penetration(shape=shape, seed=1)
    p = I.miscible(shape=shape, seed=0)
    if physics == "two solutes":
        p.species_tau_d = (0.8,)
        p.c0 = np.zeros((2,) + shape[::-1])
        p.faces[0].conc_x, p.faces[1].conc_x = (0.5,), (0.0,)
    return p


LATTICES = {"single": 1, "miscible": 2, "two-fluid": 2, "free surface": 1, "two solutes": 3}


@pytest.mark.parametrize("physics,storage", [("single", "f64"), ("miscible", "f32"), ("miscible", "bf16"),
                                             ("miscible", "f16s"), ("two-fluid", "bf16s"), ("two solutes", "bf16s"),
                                             ("two solutes", "f16"), ("free surface", "f32"), ("free surface", "f16s")])
def test_checkpoints_hold_no_unset_state(physics, storage):
    p = _problem(physics)
    cells = int(np.prod(p.shape))
    allowed = 38 * LATTICES[physics] * 768 + 32 * 256
    if physics == "free surface":
        allowed += 32 * cells + 8 * (cells // 256 + 64)
    sim = Simulation(p, storage=storage)
    for steps in (0, 1):
        saved = []
        for byte in (0x00, 0xa5):
            sim.ws.fill_(byte)
            sim._set_medium(p, False)
            sim.step(steps)
            saved.append(sim.save_state())
        unset = int((saved[0] != saved[1]).sum())
        print(f"[checkpoint] {physics} {storage}: {unset} of {saved[0].nbytes} bytes unset after {steps} steps", flush=True)
        assert unset <= allowed, (steps, unset, allowed)
    sim.close()


def test_resume_before_the_first_step():
    """A checkpoint taken before the first step, loaded into a lattice that has stepped."""
    p = _problem("free surface")
    a = Simulation(p, storage="bf16s")
    buf = a.save_state()
    a.step(20)
    b = Simulation(p, storage="bf16s")
    b.step(9)
    b.load_state(buf).step(20)
    for x, y in zip(a.moments()[:3] + a.free_surface(fill=True)[:3], b.moments()[:3] + b.free_surface(fill=True)[:3]):
        assert np.array_equal(x.cpu().numpy(), y.cpu().numpy(), equal_nan=True)
    a.close()
    b.close()
