"""GPU parity of the direct-load kernel on a split K box (X in vectors along
the block of its stride-one contracted index, Y in vectors along its own,
strided in the box), against the oracle: every fp32 tile that carries it,
whole and ragged tiles, whole and partial boxes, the boxes walked by cache
line (v divides into whole blocks) and in plain order (it does not), integer
inputs exact, and the aligned-only fall-back."""

import numpy as np
import pytest

import paper_1607_00145_amd as g
from test_gpu_direct import DIRECT_TILES, IDS, describe, force_direct, shapes
from test_gpu_parity import check_case

pytestmark = pytest.mark.gpu

MODES = ("a,b,c,d", "e,a,f,b", "f,d,e,c")
# name: extents, boxes, walked by line
CASES = {
    "whole": ({"a": 32, "b": 16, "c": 8, "d": 32, "e": 16, "f": 12}, 6, True),
    "ragged": ({"a": 36, "b": 9, "c": 7, "d": 20, "e": 64, "f": 20}, 40, True),
    "one_box": ({"a": 16, "b": 5, "c": 3, "d": 12, "e": 8, "f": 4}, 1, True),
    "partial": ({"a": 20, "b": 11, "c": 6, "d": 28, "e": 20, "f": 24}, 18, False),
    "f16": ({"a": 32, "b": 6, "c": 5, "d": 32, "e": 24, "f": 48}, 36, True),
}


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("dtype,tile", DIRECT_TILES, ids=IDS)
def test_direct_ksplit(gpu, monkeypatch, dtype, tile, name):
    force_direct(monkeypatch, tile)
    ext, boxes, lines = CASES[name]
    d = describe(MODES, ext, dtype)
    assert d["kernel"] == "direct" and d["gather_y"] == "k-vector-strided"
    assert d["kbox"]["steps"] == boxes
    assert any("|" in k or k.startswith("e<") for k in d["k_order"]) == lines
    rng = np.random.default_rng(40 + len(name) + int(tile))
    for alpha, beta in [(1.0, 0.0), (-0.5, 1.5)]:
        check_case(gpu, rng, MODES, shapes(MODES, ext), dtype, alpha, beta)
    got, ref = check_case(gpu, rng, MODES, shapes(MODES, ext), dtype, 1.0, 1.0, dist="int")
    np.testing.assert_array_equal(got.astype(np.float64), ref.out64)
    # operands off the 16-byte grid: the tile's macro-kernel, element-wise,
    # over the same order of boxes
    check_case(gpu, rng, MODES, shapes(MODES, ext), dtype, 1.0, 0.5, offsets=(0, 1, 3))


@pytest.mark.parametrize("dtype,tile", DIRECT_TILES, ids=IDS)
def test_rows_past_a_ragged_tile_do_not_leak(gpu, monkeypatch, dtype, tile):
    """Rows past the last load the tile's first row; an infinity there stays
    in its own row (and column) of C."""
    import torch

    force_direct(monkeypatch, tile)
    a, b, k = 140, 132, 64
    A = torch.ones((k, a), device=gpu).t()
    B = torch.ones((b, k), device=gpu).t()
    A[128, 3] = float("inf")   # the first row (or column) of the second tile
    B[5, 128] = float("nan")
    C = torch.zeros((b, a), device=gpu).t()
    p = g.Plan(("a,b", "a,k", "k,b"), C, A, B)
    assert p.describe()["kernel"] == "direct"
    p(A, B, C)
    want = torch.full((a, b), float(k), device=gpu)
    want[128, :] = float("inf")
    want[:, 128] = float("nan")
    assert torch.equal(torch.nan_to_num(C, nan=-1.0), torch.nan_to_num(want, nan=-1.0))
