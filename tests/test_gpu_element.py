"""GPU parity of the element-wise direct-load kernel (fp32: operands that do
not both gather in 16-byte vectors), against the oracle: lanes along the
free or the contracted index of each operand, ragged tiles, one to many boxes
of the linearised contracted set with the last one partial or whole, several
contracted indices of odd extents in one box, operands off the 16-byte grid,
gapped and permuted layouts, integer inputs exact, alpha = 0."""
import numpy as np
import pytest

from test_gpu_direct import DIRECT_TILES, IDS, describe, shapes
from test_gpu_parity import check_case

pytestmark = pytest.mark.gpu

CASES = {
    # both [k][row], one [row][k], both [row][k]
    "ab-ak-bk": (("a,b", "a,k", "b,k"), {"a": 131, "b": 257, "k": 64}),
    "ab-ak-kb": (("a,b", "a,k", "k,b"), {"a": 257, "b": 130, "k": 33}),
    "ab-ka-kb": (("a,b", "k,a", "k,b"), {"a": 129, "b": 263, "k": 31}),
    "ba-ka-bk": (("b,a", "k,a", "b,k"), {"a": 255, "b": 127, "k": 97}),
    # boxes across contracted indices
    "abij-iejf-faeb": (("a,b,i,j", "i,e,j,f", "f,a,e,b"),
                       {"a": 13, "b": 11, "i": 9, "j": 15, "e": 7, "f": 5}),
    "abcd-kalb-cldk": (("a,b,c,d", "k,a,l,b", "c,l,d,k"),
                       {"a": 17, "b": 9, "c": 21, "d": 7, "k": 23, "l": 23}),
    # an empty free set
    "a-ak-k": (("a,", "a,k", "k,"), {"a": 301, "k": 201}),
    # one position
    "ab-a-b": (("a,b", "a,", "b,"), {"a": 133, "b": 139}),
}


def force(monkeypatch, tile):
    monkeypatch.setenv("GETT_FORCE_TILE", tile)
    monkeypatch.setenv("GETT_FORCE_KIND", "6")


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("dtype,tile", DIRECT_TILES, ids=IDS)
def test_element(gpu, monkeypatch, dtype, tile, name):
    force(monkeypatch, tile)
    modes, ext = CASES[name]
    assert describe(modes, ext, dtype)["kernel"] == "direct-element"
    rng = np.random.default_rng(70 + len(name) + int(tile))
    for alpha, beta in [(1.0, 0.0), (-0.5, 1.5), (0.0, -1.0)]:
        check_case(gpu, rng, modes, shapes(modes, ext), dtype, alpha, beta)
    check_case(gpu, rng, modes, shapes(modes, ext), dtype, 1.0, 0.5, offsets=(0, 1, 3))
    check_case(gpu, rng, modes, shapes(modes, ext), dtype, 1.0, 0.5,
               kinds=("gapped", "permuted", "gapped"))
    got, ref = check_case(gpu, rng, modes, shapes(modes, ext), dtype, 1.0, 1.0, dist="int")
    np.testing.assert_array_equal(got.astype(np.float64), ref.out64)


def test_vector_operands_keep_the_vector_kernel(monkeypatch):
    force(monkeypatch, "8")
    modes = ("a,b", "a,k", "k,b")
    assert describe(modes, {"a": 512, "b": 512, "k": 64})["kernel"] == "macro"
