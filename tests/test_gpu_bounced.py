"""The count of cells with a link cut by the obstacle mask, which the cache policy goes by: made at set-up
in every stride-th block of 256 cells, and again when a state is loaded."""
import numpy as np
import pytest

from paper_0912_4230_amd import binding as B
from paper_0912_4230_amd import inputs as I
from paper_0912_4230_amd.sim import Simulation

pytestmark = pytest.mark.gpu


def _count_at(ck):
    """The place of the count in a checkpoint: the second word behind the header, whose fifth 8 bytes are
    the payload's size."""
    return len(ck) - int(ck[32:40].view(np.uint64)[0]) + 4


def _expected(p, solid):
    nx, ny, nz = p.shape
    cut = np.zeros(solid.shape, dtype=bool)
    for d in np.ndindex(3, 3, 3):
        if 0 < sum(v != 1 for v in d) < 3:
            cut |= np.roll(solid, [v - 1 for v in d], (0, 1, 2))
    cut &= ~solid
    for axis, n in ((0, nx), (1, ny), (2, nz)):
        for side in (0, 1):
            kind, a = p.faces[2 * axis + side].kind, 2 - axis
            take = lambda i: tuple(i if k == a else slice(None) for k in range(3))
            if kind != I.PERIODIC:                      # cells on the face's plane are never fluid
                cut[take(0 if side == 0 else n - 1)] = False
            if kind == I.WALL:                          # those next to it have links cut by the face
                cut[take(1 if side == 0 else n - 2)] = False
    cut = cut.reshape(-1)
    stride = -(-cut.size // 256) // 64 | 1
    return int(sum(cut[b:b + 256].sum() for b in range(0, cut.size, 256 * stride)))


@pytest.mark.parametrize("shape,physics,fraction", [
    ((19, 17, 15), I.MISCIBLE, 0.1), ((64, 4, 1), I.SINGLE, 0.3), ((33, 20, 40), I.FREESURF, 0.0), ((150, 61, 47), I.IMMISCIBLE, 0.02)])
def test_count_of_bounced_cells(shape, physics, fraction):
    nx, ny, nz = shape
    rng = np.random.default_rng(5)
    p = I.Problem(shape=shape, physics=physics, nu0=0.1, tau_d=0.65)
    if physics == I.MISCIBLE:
        p.faces[0], p.faces[1] = I.Face(kind=I.RESERVOIR, rho=1.01), I.Face(kind=I.RESERVOIR, rho=1.0)
    if nz > 2:
        p.faces[4], p.faces[5] = I.Face(kind=I.WALL), I.Face(kind=I.WALL)
    p.solid = (rng.random((nz, ny, nx)) < fraction).astype(np.uint8)
    p.c0 = rng.random((nz, ny, nx))
    sim = Simulation(p, storage="f32")
    ck = sim.save_state()
    at = _count_at(ck)
    want = _expected(p, p.solid.astype(bool))
    assert int(ck[at:at + 4].view(np.int32)[0]) == want
    ck[at:at + 4] = 0x55      # a state of a build that left the word unset
    sim.load_state(ck)
    assert int(sim.save_state()[at:at + 4].view(np.int32)[0]) == want
    sim.close()
