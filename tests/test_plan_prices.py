"""The plans' picks against measured times (host only).  For contractions
whose kernel the price of set-up, gathers and C's order decides, the times of
the candidates on an MI355X (us, fp32, beta = 0, median of three): (kernel, tile,
K slices).  The plan's pick has to be listed and within a tenth of the best.
Of the 28 contractions timed this holds for the 24 below; three picks are 13 to
32 % behind, and one (1487 us against 852) is taken for its shorter sums."""
import json

import pytest

import paper_1607_00145_amd as g

# pattern, extents, unused elements behind each first mode, times
MEASURED = [
    ("abcdef-degb-gfac", {"a": 28, "b": 20, "c": 20, "d": 24, "e": 20, "f": 20, "g": 24}, 0,
     {("macro", 3, 1): 138.1, ("macro", 9, 1): 145.0, ("macro", 2, 1): 150.1,
      ("macro", 0, 1): 185.1, ("macro", 4, 1): 197.3, ("macro", 1, 1): 197.9}),
    ("abcdef-degb-gfac", {"a": 28, "b": 20, "c": 20, "d": 24, "e": 20, "f": 20, "g": 48}, 0,
     {("macro", 3, 1): 170.8, ("macro", 9, 1): 180.5, ("macro", 2, 1): 189.5,
      ("macro", 0, 1): 226.2, ("macro", 1, 1): 241.2}),
    ("abcdef-degb-gfac", {"a": 28, "b": 20, "c": 20, "d": 24, "e": 20, "f": 20, "g": 64}, 0,
     {("macro", 3, 1): 203.8, ("macro", 9, 1): 215.1, ("macro", 2, 1): 226.5,
      ("macro", 0, 1): 262.7, ("macro", 4, 1): 277.9, ("macro", 1, 1): 283.9}),
    ("abcdef-degb-gfac", {"a": 28, "b": 20, "c": 20, "d": 24, "e": 20, "f": 20, "g": 96}, 0,
     {("macro", 3, 1): 270.8, ("macro", 9, 1): 288.2, ("macro", 2, 1): 301.4,
      ("macro", 0, 1): 336.7, ("macro", 4, 1): 353.7, ("macro", 1, 1): 377.3}),
    ("abcdef-degb-gfac", {"a": 28, "b": 20, "c": 20, "d": 24, "e": 20, "f": 20, "g": 128}, 0,
     {("macro", 3, 1): 335.6, ("macro", 9, 1): 358.0, ("macro", 2, 1): 374.4,
      ("macro", 0, 1): 411.1, ("macro", 4, 1): 432.7, ("macro", 1, 1): 459.3,
      ("direct", 8, 1): 469.3}),
    ("abcdef-degb-gfac", {"a": 28, "b": 20, "c": 20, "d": 24, "e": 20, "f": 20, "g": 192}, 0,
     {("direct", 7, 1): 454.7, ("macro", 3, 1): 468.5, ("direct", 8, 1): 473.7}),
    ("abcdef-degb-gfac", {"a": 28, "b": 20, "c": 20, "d": 24, "e": 20, "f": 20, "g": 256}, 0,
     {("direct", 7, 1): 530.8, ("direct", 8, 1): 538.4, ("macro", 7, 1): 568.8,
      ("macro", 8, 1): 580.4, ("tail", 2, 1): 591.5, ("macro", 3, 1): 597.1,
      ("macro", 9, 1): 648.1}),
    ("ab-ak-kb", {"a": 4096, "b": 4096, "k": 64}, 0,
     {("direct", 4, 1): 27.7, ("macro", 9, 1): 28.2, ("macro", 4, 1): 29.5,
      ("direct", 8, 1): 30.0, ("macro", 0, 1): 30.2, ("macro", 2, 1): 30.2,
      ("macro", 3, 1): 30.8}),
    ("ab-ak-kb", {"a": 4096, "b": 4096, "k": 128}, 0,
     {("direct", 4, 1): 41.3, ("direct", 8, 1): 44.8, ("macro", 4, 1): 45.6,
      ("macro", 9, 1): 46.4, ("macro", 0, 1): 46.7, ("direct", 7, 1): 48.2,
      ("macro", 8, 1): 48.7}),
    ("ab-ak-kb", {"a": 4096, "b": 4096, "k": 256}, 0,
     {("direct", 4, 1): 71.1, ("direct", 8, 1): 74.7, ("macro", 4, 1): 78.2,
      ("direct", 7, 1): 78.5, ("macro", 0, 1): 80.1, ("macro", 8, 1): 81.9,
      ("macro", 9, 1): 84.1}),
    ("ab-ak-kb", {"a": 8192, "b": 8192, "k": 32}, 0,
     {("macro", 2, 1): 61.2, ("macro", 3, 1): 61.9, ("direct", 4, 1): 63.9,
      ("macro", 0, 1): 66.2, ("macro", 9, 1): 66.5, ("macro", 4, 1): 68.4, ("macro", 1, 1): 69.4}),
    ("ab-ak-kb", {"a": 8192, "b": 8192, "k": 64}, 0,
     {("macro", 2, 1): 91.0, ("direct", 4, 1): 92.4, ("macro", 3, 1): 92.7,
      ("direct", 8, 1): 100.3, ("macro", 9, 1): 101.0, ("macro", 0, 1): 101.2,
      ("macro", 4, 1): 102.2}),
    ("ab-ak-kb", {"a": 8192, "b": 8192, "k": 128}, 0,
     {("direct", 4, 1): 153.6, ("macro", 2, 1): 154.7, ("macro", 3, 1): 162.0,
      ("direct", 8, 1): 165.0, ("macro", 4, 1): 168.1, ("macro", 0, 1): 170.0,
      ("macro", 9, 1): 171.7}),
    ("ab-ak-kb", {"a": 8192, "b": 8192, "k": 256}, 0,
     {("direct", 4, 1): 271.4, ("direct", 8, 1): 283.2, ("macro", 2, 1): 283.9,
      ("direct", 7, 1): 293.1, ("macro", 3, 1): 297.4, ("macro", 4, 1): 301.5,
      ("macro", 0, 1): 305.2}),
    ("ab-ak-kb", {"a": 16384, "b": 16384, "k": 64}, 0,
     {("macro", 2, 1): 349.9, ("direct", 4, 1): 351.0, ("macro", 3, 1): 355.1,
      ("macro", 0, 1): 376.2, ("macro", 4, 1): 388.1, ("macro", 9, 1): 398.3,
      ("direct", 7, 1): 400.0}),
    ("ab-ak-kb", {"a": 16384, "b": 16384, "k": 128}, 0,
     {("direct", 4, 1): 592.4, ("macro", 2, 1): 596.8, ("macro", 3, 1): 616.6,
      ("direct", 7, 1): 627.2, ("direct", 8, 1): 629.3, ("macro", 4, 1): 649.5,
      ("macro", 0, 1): 653.5}),
    ("abc-bda-dc", {"a": 136, "b": 197, "c": 56, "d": 176}, 0,
     {("macro", 5, 1): 31.6, ("macro", 1, 1): 33.9, ("macro", 2, 1): 36.3, ("macro", 0, 1): 36.5,
      ("direct-element", 4, 1): 40.2, ("macro", 4, 1): 40.5, ("macro", 9, 1): 41.3}),
    ("abc-bda-dc", {"a": 296, "b": 272, "c": 16, "d": 256}, 8,
     {("macro", 6, 1): 23.7, ("macro", 9, 2): 31.3}),
    ("abc-bda-dc", {"a": 196, "b": 148, "c": 161, "d": 53}, 0,
     {("direct-element", 7, 1): 20.3, ("macro", 7, 1): 21.5, ("macro", 0, 1): 23.8,
      ("macro", 2, 1): 24.1, ("direct-element", 8, 1): 24.6, ("macro", 8, 1): 24.9,
      ("direct-element", 4, 1): 25.2}),
    ("ab-ka-bk", {"a": 10784, "b": 1771, "k": 54}, 0,
     {("direct-element", 4, 1): 38.1, ("direct-element", 7, 1): 45.7, ("macro", 4, 1): 45.7,
      ("direct-element", 8, 1): 46.0, ("macro", 2, 1): 50.0, ("macro", 7, 1): 52.2,
      ("macro", 8, 1): 53.6}),
    ("abcd-aeb-edc", {"a": 80, "b": 88, "c": 40, "d": 56, "e": 55}, 0,
     {("direct-element", 4, 1): 31.4, ("macro", 3, 1): 33.2, ("direct-element", 7, 1): 33.5,
      ("macro", 4, 1): 33.6, ("direct-element", 8, 1): 33.8, ("macro", 9, 1): 33.9,
      ("macro", 8, 1): 34.2}),
    ("abcijk-dabi-cdjk", {"a": 22, "b": 16, "c": 16, "d": 81, "i": 24, "j": 18, "k": 14}, 0,
     {("direct-element", 4, 1): 82.7, ("macro", 4, 1): 89.2, ("direct-element", 8, 1): 92.9,
      ("direct-element", 7, 1): 94.4, ("macro", 7, 1): 96.6, ("macro", 5, 1): 102.0,
      ("macro", 8, 1): 103.6}),
    ("abcd-aebf-fdec", {"a": 53, "b": 51, "c": 50, "d": 49, "e": 47, "f": 45}, 0,
     {("direct-element", 8, 1): 301.8, ("direct-element", 7, 1): 302.4,
      ("direct-element", 4, 1): 319.8, ("tail", 2, 1): 346.0, ("macro", 0, 1): 368.2,
      ("macro", 2, 1): 373.9, ("macro", 0, 2): 379.5}),
    ("abij-iejf-faeb", {"a": 61, "b": 61, "e": 61, "f": 61, "i": 23, "j": 23}, 0,
     {("macro", 9, 2): 222.9, ("macro", 6, 1): 244.2, ("macro", 2, 4): 254.5,
      ("macro", 0, 4): 271.8, ("direct-element", 4, 1): 303.9, ("macro", 8, 2): 313.3,
      ("macro", 9, 1): 315.6}),
]

# fp64, beta = 0.5: tiles that leave CUs idle, Y gathered in single elements
MEASURED_F64 = [
    ("abc-bda-dc", {"a": 120, "b": 109, "c": 7, "d": 128}, 0,
     {("macro", 12, 1): 13.3, ("macro", 13, 1): 22.9}),
    ("abc-bda-dc", {"a": 121, "b": 112, "c": 8, "d": 128}, 3,
     {("macro", 12, 1): 14.4, ("macro", 13, 1): 24.3}),
    ("abc-bda-dc", {"a": 90, "b": 99, "c": 6, "d": 88}, 0,
     {("macro", 12, 1): 10.3, ("macro", 13, 1): 15.5}),
    ("abc-bda-dc", {"a": 77, "b": 92, "c": 5, "d": 74}, 8,
     {("macro", 12, 1): 8.3, ("macro", 13, 1): 12.2}),
]


def describe(pattern, ext, pad, dtype=g.GETT_FLOAT32):
    C, A, B = pattern.split("-")
    args = []
    for m in (C, A, B):
        shape = [ext[x] for x in m]
        stride, acc = [], 1
        for i, e in enumerate(shape):
            stride.append(acc)
            acc *= e + (pad if i == 0 else 0)
        args += [",".join(m), shape, stride]
    st, h = g.gett_plan(dtype, *args, 0)
    assert st == 0
    try:
        return json.loads(g.gett_plan_describe(h))
    finally:
        g.gett_destroy(h)


def check(d, times):
    pick = (d["kernel"], d["tile"]["id"], d["kslices"])
    assert pick in times, (pick, sorted(times.items(), key=lambda t: t[1])[:3])
    assert times[pick] <= 1.10 * min(times.values()), (pick, times[pick], min(times.values()))


def names(table):
    return [p + "-" + "x".join(str(e) for e in x.values()) for p, x, _, _ in table]


@pytest.mark.parametrize("pattern,ext,pad,times", MEASURED, ids=names(MEASURED))
def test_pick_is_near_the_best(pattern, ext, pad, times):
    check(describe(pattern, ext, pad), times)


@pytest.mark.parametrize("pattern,ext,pad,times", MEASURED_F64, ids=names(MEASURED_F64))
def test_pick_is_near_the_best_f64(pattern, ext, pad, times):
    check(describe(pattern, ext, pad, g.GETT_FLOAT64), times)


def test_a_short_run_of_c_is_no_longer_stream():
    """The price counts the partial lines of a short run of C several times over,
    the walk does not: this C is no bound of its 128 x 256 tiles (474 us, 533
    with the tiles and the rows in the order of a stream)."""
    d = describe("abcdef-degb-gfac",
                 {"a": 28, "b": 20, "c": 20, "d": 24, "e": 20, "f": 20, "g": 192}, 0)
    assert d["kernel"] == "direct" and not d["streaming"]
