"""Which cache policy a step takes (csrc/cache_policy.hpp, compiled for the host):
groups of a batch keep their populations in the memory-side cache only where they
fit there together."""
import pytest

from policy_util import KEEP, REUSE, STREAM, lattice, policies


def _pair(a, b, storage="f32"):
    return [[lattice("miscible", storage, (e,) * 3) for e in a], [lattice("immiscible", storage, (e,) * 3) for e in b]]


@pytest.mark.parametrize("groups,want", [
    # alone, each fits
    (_pair((94,), ())[:1], [KEEP]), (_pair((), (94,))[1:], [KEEP]),
    # two that do not fit together
    (_pair((64, 64), (94,)), [STREAM, REUSE]), (_pair((80,), (80,)), [REUSE, REUSE]),
    (_pair((90,), (64,)), [REUSE, STREAM]), (_pair((110,), (110,), "bf16"), [REUSE, REUSE]),
    # two that do
    (_pair((61,), (61,)), [KEEP, KEEP]), (_pair((72,), (72,)), [KEEP, KEEP]),
    # only one would keep: what streams beside it does not count
    (_pair((64,), (90,)), [STREAM, KEEP]), (_pair((96,), (80,)), [STREAM, KEEP]), (_pair((192,), (60,)), [STREAM, KEEP]),
])
def test_groups_keep_only_what_fits_together(groups, want):
    assert policies(groups) == want


def test_storage_forms_are_groups_of_their_own():
    forms = ("f64", "f32", "bf16", "f16s")
    one = [[lattice("miscible", s, (81, 80, 80))] for s in forms]
    assert [policies([g])[0] for g in one][1:] == [KEEP] * 3
    assert KEEP not in policies(one)


def test_free_surface_counts():
    fs, tank = [lattice("freesurf", "f32", (100, 100, 90))], [lattice("single", "f32", (100, 100, 90))]
    assert policies([fs]) == [KEEP] and policies([tank]) == [KEEP]
    assert policies([fs, tank]) == [STREAM, REUSE]
