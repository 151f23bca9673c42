"""Batches of as many lattices as a launch takes (64) and more: every block finds its
lattice, the last one of a full launch among them.  Lattices of different sizes
step together and alone with the same bits."""
import numpy as np
import pytest

from paper_0912_4230_amd import inputs as I
from paper_0912_4230_amd.sim import Simulation, step_batch

pytestmark = pytest.mark.gpu


def _problem(kind, i):
    shape = (5 + i % 7, 4 + i % 11, 5 + i % 13)
    if kind == "miscible":
        return I.miscible(shape=shape, seed=i)
    if kind == "two-fluid":
        return I.drop(shape=shape, radius=2.0, speed=0.02)
    return I.penetration(shape=shape, seed=i)


@pytest.mark.parametrize("kind,n", [("miscible", 63), ("miscible", 64), ("miscible", 65), ("miscible", 130),
                                    ("two-fluid", 66), ("free surface", 67)])
def test_full_batches(kind, n):
    alone = []
    for i in range(n):
        s = Simulation(_problem(kind, i), storage="f32")
        s.step(3)
        alone.append([t.cpu().numpy() for t in s.moments()[:3]] + [s.populations().cpu().numpy(), s.diag()])
        s.close()
    sims = [Simulation(_problem(kind, i), storage="f32") for i in range(n)]
    step_batch(sims, [3] * n)
    for s, want in zip(sims, alone):
        got = [t.cpu().numpy() for t in s.moments()[:3]] + [s.populations().cpu().numpy(), s.diag()]
        for a, b in zip(got, want):
            assert np.array_equal(a, b)
        s.close()
