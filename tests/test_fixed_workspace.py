"""Plans that gett_contract_noalloc takes (host only): its fixed workspace holds
64 MiB of partial tiles and 65536 counters, and the price of gathers does not
move a plan beyond them where the model without that price stays within."""
import random

import pytest

import paper_1607_00145_amd as g
from test_sum_chains import describe

LIMIT = (64 << 20, 65536)

# (pattern, extents, dtype): taken by the plans of the model without gathers
TAKEN = [
    ("abcd-eafb-fdec", {"a": 56, "b": 40, "c": 40, "d": 48, "e": 60, "f": 47}, g.GETT_FLOAT64),
    ("mnop-mkoq-qnkp", {"m": 35, "n": 40, "o": 40, "p": 40, "k": 37, "q": 30}, g.GETT_FLOAT64),
    ("abij-iejf-faeb", {"i": 31, "j": 32, "a": 47, "b": 45, "e": 49, "f": 50}, g.GETT_FLOAT64),
    ("abcd-aebf-fdec", {"a": 35, "b": 40, "c": 40, "d": 39, "e": 33, "f": 40}, g.GETT_FLOAT64),
    ("ab-ka-bk", {"a": 5392, "b": 8600, "k": 579}, g.GETT_FLOAT64),
    ("abcd-eafb-fdec", {"a": 48, "b": 44, "c": 44, "d": 48, "e": 49, "f": 48}, g.GETT_FLOAT32),
    ("mnop-mkoq-qnkp", {"m": 50, "n": 44, "o": 48, "p": 51, "k": 46, "q": 48}, g.GETT_FLOAT32),
]


def within(d):
    return d["workspace_bytes"] <= LIMIT[0] and d["workspace_counters"] <= LIMIT[1]


@pytest.mark.parametrize("pattern,ext,dtype", TAKEN,
                         ids=[f"{p}-{'f64' if t else 'f32'}" for p, _, t in TAKEN])
def test_accepted_plans_stay_accepted(pattern, ext, dtype):
    d = describe(pattern, ext, dtype)
    assert within(d), (d["kernel"], d["tile"]["id"], d["kslices"], d["workspace_bytes"] >> 20)


def test_within_where_the_reference_is():
    """Drawn contractions, most with odd extents, around the sizes whose
    partial tiles reach the limit."""
    rng = random.Random(9)
    families = [("abij-iejf-faeb", 60), ("abcd-aebf-fdec", 60), ("abcd-eafb-fdec", 60),
                ("mnop-mkoq-qnkp", 56), ("ab-acd-dbc", 380)]
    refused = 0
    for i in range(400):
        pattern, top = families[i % len(families)]
        ext = {m: rng.randint(2 * top // 3, top) for m in sorted(set(pattern) - {"-"})}
        for dtype in (g.GETT_FLOAT32, g.GETT_FLOAT64):
            d = describe(pattern, ext, dtype)
            assert within(d) or not d["reference_fits"], (pattern, ext, dtype)
            refused += not within(d)
    assert 0 < refused < 400   # the draws lie on both sides of the limit
