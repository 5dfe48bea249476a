"""How many additions in a row stand behind an element of C (host only): the
price of gathers may move a plan to another kernel, never to longer chains than
those of the reference, the cheapest plan without that price."""
import json
import random

import pytest

import paper_1607_00145_amd as g


def describe(pattern, ext, dtype=g.GETT_FLOAT32):
    shape = lambda m: [ext[x] for x in m]
    C, A, B = pattern.split("-")
    st, h = g.gett_plan(dtype, ",".join(C), shape(C), None, ",".join(A), shape(A), None,
                        ",".join(B), shape(B), None, 0)
    assert st == 0
    try:
        return json.loads(g.gett_plan_describe(h))
    finally:
        g.gett_destroy(h)


def chain(d):
    """Additions in a row behind an element of C: positions summed in one
    accumulator and partial tiles, on average over C."""
    K, n, t, P = d["size_k"], d["kbox"]["steps"], d["tail"], d["kslices"]
    if P > 1:   # slots on the direct-load kernel are added up eight at a time
        return K / P + (min(P, 8) + P // 8 if d["kernel"] == "direct" else P)
    if d["kernel"] == "tail":
        tiles, full, run = d["grid"]["workgroups"], t["full_tiles"], t["boxes"]
        # the boxes of the other tiles one after the other, cut into runs and at tiles' ends
        cuts = sorted({*range(0, (tiles - full) * n, n), *range(0, (tiles - full) * n, run),
                       (tiles - full) * n})
        square = sum((b - a) ** 2 for a, b in zip(cuts, cuts[1:]))
        return (full * K + square / n * K / n) / tiles
    return K


# contracted sets that are summed in slices: (pattern, extents, chain before the price of gathers)
SLICED = [
    ("abij-iejf-faeb", {"i": 37, "j": 38, "a": 44, "b": 48, "e": 51, "f": 53}, 690),
    ("abcd-aebf-fdec", {"a": 48, "b": 49, "c": 42, "d": 48, "e": 48, "f": 50}, 608),
    ("abij-iejf-faeb", {"i": 43, "j": 40, "a": 48, "b": 56, "e": 51, "f": 56}, 735),
    ("abij-iejf-faeb", {"i": 32, "j": 32, "a": 48, "b": 48, "e": 48, "f": 51}, 384),
    ("abcd-aebf-fdec", {"a": 40, "b": 40, "c": 40, "d": 35, "e": 38, "f": 42}, 410),
    ("abcd-eafb-fdec", {"a": 52, "b": 40, "c": 48, "d": 48, "e": 48, "f": 48}, 580),
    ("mnop-mkoq-qnkp", {"m": 32, "n": 33, "o": 31, "p": 32, "k": 31, "q": 40}, 192),
    ("ab-acd-dbc", {"a": 384, "b": 376, "c": 376, "d": 384}, 2320),
]


@pytest.mark.parametrize("pattern,ext,most", SLICED, ids=lambda v: v if isinstance(v, str) else None)
def test_sliced_sets_stay_sliced(pattern, ext, most):
    d = describe(pattern, ext)
    assert chain(d) <= most, (d["kernel"], d["tile"]["id"], d["kslices"], chain(d))


def test_no_longer_than_the_reference():
    """Drawn contractions, most with odd extents: the description's own figure
    for the plan is not above the reference's, and agrees with the plan."""
    rng = random.Random(4)
    families = [("abij-iejf-faeb", 60), ("abcd-aebf-fdec", 56), ("abcd-eafb-fdec", 60),
                ("mnop-mkoq-qnkp", 56), ("ab-acd-dbc", 380), ("abc-bda-dc", 380),
                ("ab-ka-bk", 3000), ("abcdef-degb-gfac", 24)]
    for i in range(400):
        pattern, top = families[i % len(families)]
        ext = {m: rng.randint(max(4, top // 6), top) for m in sorted(set(pattern) - {"-"})}
        for dtype in (g.GETT_FLOAT32, g.GETT_FLOAT64):
            d = describe(pattern, ext, dtype)
            assert d["chain"] <= d["reference_chain"] * (1 + 1e-6), (pattern, ext, dtype)
            # (a tail's figure averages over where its runs end)
            rel = 0.1 if d["kernel"] == "tail" else 1e-4
            assert d["chain"] == pytest.approx(chain(d), rel=rel), (pattern, ext)
