"""GPU parity of C stored off the 16-byte grid: a lane's columns go as one
vector where they follow one another in C and element by element where a run
or C ends inside the group.  Every tile of both types, runs of every length
modulo the vector, a C base off the grid, gapped C, every beta path; and the
fp32 tile of 32 rows over its gather modes."""
import numpy as np
import pytest

from test_gpu_parity import TILES, check_case

pytestmark = pytest.mark.gpu


def shapes(modes, ext):
    return tuple([ext[x] for x in m.split(",") if x] for m in modes)


@pytest.mark.parametrize("dtype,tile", [(dt, t) for dt in (np.float32, np.float64)
                                        for t in range(TILES[dt])])
def test_unaligned_c(gpu, monkeypatch, dtype, tile):
    monkeypatch.setenv("GETT_FORCE_TILE", str(tile))
    monkeypatch.setenv("GETT_FORCE_KIND", "0")
    rng = np.random.default_rng(900 + tile)
    modes = ("a,b,c", "a,k,c", "k,b")
    for a in (13, 14, 15, 16):
        sh = shapes(modes, {"a": a, "b": 37, "c": 11, "k": 9})
        for alpha, beta in [(1.0, 0.0), (-0.5, 1.5)]:
            check_case(gpu, rng, modes, sh, dtype, alpha, beta)
        check_case(gpu, rng, modes, sh, dtype, 1.0, 0.5, offsets=(1, 0, 0))
        check_case(gpu, rng, modes, sh, dtype, 1.0, 0.5, kinds=("gapped", "dense", "dense"))
        check_case(gpu, rng, modes, sh, dtype, 1.0, 1.0, kinds=("permuted", "gapped", "dense"))


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_y_walks_its_own_index(gpu, dtype):
    """A Y that is stride-one along a late index of C, of odd extents: the
    index moves up behind C's first one."""
    rng = np.random.default_rng(7)
    modes = ("a,b,c,d,e", "e,f,b,a,d", "c,f")
    sh = shapes(modes, {"a": 13, "b": 7, "c": 9, "d": 5, "e": 15, "f": 11})
    for alpha, beta in [(1.0, 0.0), (-0.5, 1.5)]:
        check_case(gpu, rng, modes, sh, dtype, alpha, beta)
    check_case(gpu, rng, modes, sh, dtype, 1.0, 1.0, kinds=("gapped", "permuted", "gapped"))


@pytest.mark.parametrize("ext", [{"a": 48, "b": 20, "c": 24, "e": 16, "f": 36},
                                 {"a": 33, "b": 21, "c": 31, "e": 15, "f": 17}])
@pytest.mark.parametrize("modes", [("a,b,c,e", "e,f,b,a", "c,f"), ("a,b,c,e", "a,f,b,e", "f,c"),
                                   ("a,b,c,e", "f,a,b,e", "c,f")])
def test_few_rows_tile(gpu, monkeypatch, modes, ext):
    monkeypatch.setenv("GETT_FORCE_TILE", "9")
    rng = np.random.default_rng(9)
    for alpha, beta in [(1.0, 0.0), (-0.5, 1.5), (0.0, 1.0)]:
        check_case(gpu, rng, modes, shapes(modes, ext), np.float32, alpha, beta)
