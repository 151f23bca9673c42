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


# (storage, shape, options, policy): alone, on both sides of every line of the rule
LINES = [
    # 16-bit miscible forms keep from 40 MB on
    ("bf16", (65, 63, 64), {}, STREAM), ("bf16", (67, 64, 72), {}, KEEP), ("f16", (46, 105, 64), {}, KEEP),
    ("f16", (67, 64, 72), {"links": True}, KEEP), ("bf16", (61, 58, 76), {"tensor": True}, KEEP),
    # up to what fits with the medium
    ("bf16", (151, 106, 96), {}, KEEP), ("bf16", (79, 106, 199), {}, REUSE), ("bf16", (115, 115, 115), {"uniform": True}, KEEP),
    ("bf16", (164, 82, 106), {"tensor": True}, KEEP), ("f16", (109, 88, 162), {"tensor": True}, REUSE),
    ("bf16", (154, 133, 71), {"links": True}, KEEP), ("bf16", (138, 125, 94), {"links": True}, REUSE),
    ("f16s", (142, 118, 86), {}, KEEP), ("f16s", (122, 94, 132), {}, STREAM),
    ("f16s", (135, 94, 102), {"tensor": True}, KEEP), ("bf16s", (74, 145, 139), {"tensor": True}, STREAM),
    ("f32", (94, 94, 94), {}, KEEP), ("f32", (98, 98, 98), {}, REUSE), ("f32", (85, 122, 76), {"tensor": True}, KEEP),
    ("f32", (97, 108, 79), {"tensor": True, "links": True}, REUSE), ("f64", (82, 51, 94), {"tensor": True}, KEEP),
    ("f64", (55, 83, 92), {"tensor": True}, REUSE),
    ("f32", (59, 58, 59), {}, STREAM), ("f32", (61, 61, 61), {}, KEEP), ("f32", (64, 64, 64), {}, STREAM),
    # deviations: plain loads up to 600 MB and from planes of 35 MB on
    ("f16", (177, 133, 154), {}, REUSE), ("f16", (212, 169, 122), {}, STREAM), ("f16", (243, 97, 228), {}, STREAM),
    ("bf16", (187, 199, 213), {}, STREAM), ("bf16", (217, 208, 208), {}, REUSE), ("bf16", (200, 200, 200), {}, STREAM),
    ("bf16", (212, 169, 122), {"species": 2}, REUSE), ("f16", (243, 97, 228), {"links": True}, REUSE),
    # with a tensor up to 400 MB; with obstacles too from planes of 30 MB on
    ("bf16", (147, 114, 150), {"tensor": True}, REUSE), ("f16", (133, 135, 202), {"tensor": True}, STREAM),
    ("bf16", (187, 199, 213), {"tensor": True}, STREAM), ("bf16", (243, 251, 238), {"tensor": True}, REUSE),
    ("f16", (122, 275, 167), {"tensor": True, "links": True}, STREAM),
    ("f16", (201, 211, 166), {"tensor": True, "links": True}, STREAM),
    ("bf16", (165, 241, 203), {"tensor": True, "links": True}, REUSE),
    # split forms from planes of 35 MB on, 24 MB with more arithmetic
    ("bf16s", (189, 233, 150), {}, STREAM), ("bf16s", (187, 199, 213), {}, STREAM), ("f16s", (101, 310, 299), {}, REUSE),
    ("bf16s", (187, 199, 213), {"tensor": True}, REUSE), ("f16s", (155, 151, 140), {"tensor": True}, STREAM),
    ("f16s", (200, 200, 200), {"links": True}, REUSE), ("f16s", (160, 160, 160), {"links": True}, STREAM),
    ("bf16s", (183, 129, 172), {"species": 2}, STREAM), ("f16s", (230, 212, 214), {"species": 2}, REUSE),
    # FP32 and FP64: always, but with a tensor and no obstacles not between 600 MB (FP64 500)
    # and planes of 29 MB
    ("f32", (163, 207, 181), {}, REUSE), ("f32", (256, 256, 256), {}, STREAM), ("f32", (256, 256, 256), {"links": True}, REUSE),
    ("f32", (123, 125, 127), {"tensor": True}, REUSE), ("f32", (49, 293, 160), {"tensor": True}, STREAM),
    ("f32", (95, 226, 184), {"tensor": True}, STREAM),
    ("f32", (243, 251, 238), {"tensor": True}, REUSE), ("f32", (95, 226, 184), {"tensor": True, "links": True}, REUSE), ("f32", (193, 228, 119), {"tensor": True}, STREAM),
    ("f64", (130, 94, 62), {"tensor": True}, REUSE), ("f64", (75, 111, 105), {"tensor": True}, STREAM),
    ("f64", (171, 114, 128), {"tensor": True}, STREAM),
    ("f64", (111, 191, 214), {"tensor": True}, REUSE),
    ("f32", (192, 203, 224), {"tensor": True}, STREAM), ("f32", (256, 224, 192), {"tensor": True}, REUSE),
]


@pytest.mark.parametrize("storage,shape,options,want", LINES)
def test_lines_of_the_miscible_step(storage, shape, options, want):
    assert policies([[lattice("miscible", storage, shape, **options)]]) == [want]


@pytest.mark.parametrize("physics,storage,shape,line,options", [
    ("miscible", "f32", (160, 160, 160), 0.08, {}), ("miscible", "f32", (192, 200, 120), 0.08, {}),
    ("miscible", "f32", (128, 100, 100), 0.015, {}), ("miscible", "f32", (192, 128, 200), 0.12, {"tensor": True}),
    ("miscible", "f64", (128, 128, 128), 0.15, {}), ("miscible", "f64", (96, 80, 90), 0.05, {}),
    ("miscible", "f64", (128, 128, 128), 0.25, {"tensor": True}), ("miscible", "f64", (128, 128, 128), 0.05, {"species": 2}),
    ("miscible", "f32", (160, 160, 160), 0.03, {"species": 2}), ("miscible", "bf16", (160, 160, 160), 0.09, {}),
    ("miscible", "f16", (200, 200, 200), 0.09, {}), ("miscible", "f16", (212, 169, 122), 0.09, {}),
    ("miscible", "bf16s", (200, 190, 180), 0.12, {}), ("miscible", "f16s", (200, 200, 200), 0.05, {}),
    ("single", "f32", (256, 256, 256), 0.004, {}), ("immiscible", "f32", (128, 128, 128), 0.004, {}),
])
def test_obstacles_count_by_their_bounced_links(physics, storage, shape, line, options):
    at = [policies([[lattice(physics, storage, shape, links=True, bounced=b, **options)]])[0]
          for b in (0.0, 0.9 * line, 1.1 * line)]
    assert at == [STREAM, STREAM, REUSE]


@pytest.mark.parametrize("storage,shape,options", [
    ("f32", (256, 256, 256), {}), ("f64", (256, 256, 120), {}), ("bf16", (256, 256, 256), {}), ("bf16", (128, 120, 130), {"species": 2}),
    ("bf16", (128, 120, 130), {}), ("f16s", (256, 256, 256), {}), ("f16s", (256, 200, 140), {"species": 2}),
    ("f32", (243, 251, 238), {}), ("f16", (151, 124, 112), {})])
def test_plain_loads_pay_whatever_the_mask_holds(storage, shape, options):
    assert policies([[lattice("miscible", storage, shape, links=True, bounced=0.0, **options)]]) == [REUSE]


def test_planes_of_a_launch_add_up():
    a, b = lattice("miscible", "bf16", (187, 187, 187)), lattice("miscible", "bf16", (162, 162, 162))
    assert policies([[a]]) == policies([[b]]) == [STREAM] and policies([[a, b]]) == [REUSE]


@pytest.mark.parametrize("a,b,storage,want", [
    # the others stream beside what is kept
    ((50, 71, 54), (125,), "f32", [KEEP, STREAM]), ((100,), (161,), "bf16", [KEEP, STREAM]),
    ((98, 56, 106), (95, 60), "bf16", [STREAM, KEEP]),
    # with more than 4.5 times its bytes nothing is kept
    ((49, 52), (161,), "f32", [REUSE, REUSE]), ((83,), (178,), "f32", [REUSE, REUSE]),
    ((121, 117, 63, 143, 65), (77, 96), "bf16", [REUSE, REUSE]),
])
def test_plain_loads_beside_kept_groups(a, b, storage, want):
    groups = _pair(a, b, storage)
    for g in groups:
        for c in g:         # the two-fluid lattices lie in a medium too
            c.medium = c.cells * (16 + 4 * (g is groups[1]))
    assert policies(groups) == want


@pytest.mark.parametrize("physics,storage,shape,want", [
    ("single", "f64", (47, 31, 29), KEEP), ("single", "f64", (39, 34, 48), STREAM), ("single", "f64", (46, 33, 47), STREAM),
    ("single", "f32", (58, 61, 41), KEEP), ("single", "bf16", (84, 80, 43), KEEP), ("single", "f32", (51, 64, 50), STREAM),
    ("immiscible", "f64", (24, 32, 23), KEEP), ("immiscible", "f64", (41, 30, 32), STREAM),
    ("miscible", "f32", (34, 33, 33), KEEP), ("miscible", "f32", (40, 40, 40), STREAM),
])
def test_smallest_lattices(physics, storage, shape, want):
    assert policies([[lattice(physics, storage, shape)]]) == [want]
