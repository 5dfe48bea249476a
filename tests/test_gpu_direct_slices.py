"""GPU parity of K slices on the direct-load kernel (the fp32 tiles that carry
it, both operands in vectors): the slots summed in slice order by a second
launch.  Whole and ragged tiles and boxes, slices that start inside a later
contracted index, more slices than boxes, every beta path, integer inputs
exact, identical bits from call to call, the no-allocation entry's workspace,
and the macro-kernel's slices for operands off the 16-byte grid."""
import numpy as np
import pytest

import paper_1607_00145_amd as g
from test_gpu_direct import DIRECT_TILES, IDS, describe, shapes
from test_gpu_parity import check_case

pytestmark = pytest.mark.gpu

CASES = {
    "ab-acd-dbc": (("a,b", "a,c,d", "d,b,c"), {"a": 132, "b": 140, "c": 11, "d": 40}),
    "ab-cda-cdb": (("a,b", "c,d,a", "c,d,b"), {"a": 256, "b": 256, "c": 32, "d": 9}),
    "abc-dac-db": (("a,b,c", "d,a,c", "d,b"), {"a": 20, "b": 300, "c": 13, "d": 100}),
}


@pytest.mark.parametrize("slices", [2, 5, 50])
@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("dtype,tile", DIRECT_TILES, ids=IDS)
def test_direct_slices(gpu, monkeypatch, dtype, tile, name, slices):
    monkeypatch.setenv("GETT_FORCE_TILE", tile)
    monkeypatch.setenv("GETT_FORCE_KSLICES", str(slices))
    modes, ext = CASES[name]
    d = describe(modes, ext, dtype)
    assert d["kslices"] == slices and d["gather_x"] in ("row-vector", "k-vector")
    assert d["kernel"] == "direct"
    assert d["gather_y"] in ("row-vector", "k-vector")
    rng = np.random.default_rng(slices + len(name) + int(tile))
    for alpha, beta in [(1.0, 0.0), (-0.5, 1.5), (0.0, 2.0)]:
        check_case(gpu, rng, modes, shapes(modes, ext), dtype, alpha, beta)
    check_case(gpu, rng, modes, shapes(modes, ext), dtype, 1.0, 0.5, offsets=(1, 0, 0))
    check_case(gpu, rng, modes, shapes(modes, ext), dtype, 1.0, 0.5, offsets=(0, 1, 0))
    got, ref = check_case(gpu, rng, modes, shapes(modes, ext), dtype, 1.0, 1.0, dist="int")
    np.testing.assert_array_equal(got.astype(np.float64), ref.out64)


SPLIT = {   # operands stride-one along different contracted indices
    "ab-kla-lkb": (("a,b", "k,l,a", "l,k,b"), {"a": 132, "b": 260, "k": 48, "l": 40}),
    "ab-klma-lmkb": (("a,b", "k,l,m,a", "l,m,k,b"), {"a": 256, "b": 140, "k": 24, "l": 20, "m": 5}),
}


@pytest.mark.parametrize("slices", [2, 7])
@pytest.mark.parametrize("name", list(SPLIT))
@pytest.mark.parametrize("dtype,tile", DIRECT_TILES, ids=IDS)
def test_slices_after_a_k_split(gpu, monkeypatch, dtype, tile, name, slices):
    """Strided vectors of Y: the same tiles' slices on the macro-kernel, which
    start inside the split indices and end in partial blocks (l = 20 or 40
    against boxes of 8 by 4)."""
    monkeypatch.setenv("GETT_FORCE_TILE", tile)
    monkeypatch.setenv("GETT_FORCE_KSLICES", str(slices))
    modes, ext = SPLIT[name]
    d = describe(modes, ext, dtype)
    assert d["kslices"] == slices and d["gather_y"] == "k-vector-strided"
    assert d["y_vector_stride"] > 1 and d["kernel"] == "macro"
    rng = np.random.default_rng(slices + 17 * int(tile))
    for alpha, beta in [(1.0, 0.0), (-0.5, 1.5)]:
        check_case(gpu, rng, modes, shapes(modes, ext), dtype, alpha, beta)
    got, ref = check_case(gpu, rng, modes, shapes(modes, ext), dtype, 1.0, 1.0, dist="int")
    np.testing.assert_array_equal(got.astype(np.float64), ref.out64)


def test_same_bits_and_no_alloc(gpu, monkeypatch):
    """A small C over a long contracted set: one result bit for bit from
    repeated calls, another stream and the fixed workspace."""
    import torch

    monkeypatch.setenv("GETT_FORCE_TILE", "4")
    monkeypatch.setenv("GETT_FORCE_KSLICES", "31")

    gen = torch.Generator(device=gpu).manual_seed(5)
    A = torch.rand((96, 94, 384), generator=gen, device=gpu).permute(2, 1, 0)
    B = torch.rand((94, 376, 96), generator=gen, device=gpu).permute(2, 1, 0)
    outs = [torch.zeros((376, 384), device=gpu).t() for _ in range(4)]
    p = g.Plan(("a,b", "a,c,d", "d,b,c"), outs[0], A, B)
    assert p.describe()["kslices"] == 31 and p.describe()["tile"]["id"] == 4
    p(A, B, outs[0])
    p(A, B, outs[1])
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        p(A, B, outs[2])
    torch.cuda.current_stream().wait_stream(s)
    st = g.gett_contract_noalloc(p._h, 1.0, A.data_ptr(), B.data_ptr(), 0.0, outs[3].data_ptr(),
                                 torch.cuda.current_stream().cuda_stream)
    assert st == 0
    torch.cuda.synchronize()
    for o in outs[1:]:
        assert torch.equal(o, outs[0])


def test_threads_on_one_stream(gpu, monkeypatch):
    """Four host threads call one plan on one stream, each with its own inputs
    and C: every C has the bits of the same call made alone.  (The two launches
    of a call share the stream's slots, so they have to be enqueued together.)"""
    import threading

    import torch

    monkeypatch.setenv("GETT_FORCE_TILE", "4")
    monkeypatch.setenv("GETT_FORCE_KSLICES", "14")
    gen = torch.Generator(device=gpu).manual_seed(6)
    new = lambda *s: torch.rand(s, generator=gen, device=gpu).permute(*reversed(range(len(s))))
    sets = [(new(24, 94, 384), new(94, 376, 24)) for _ in range(4)]
    ref = [torch.zeros((376, 384), device=gpu).t() for _ in sets]
    p = g.Plan(("a,b", "a,c,d", "d,b,c"), ref[0], *sets[0])
    assert p.describe()["kslices"] == 14 and p.describe()["tile"]["id"] == 4
    for (A, B), C in zip(sets, ref):
        p(A, B, C)
    outs = [[torch.zeros((376, 384), device=gpu).t() for _ in range(40)] for _ in sets]
    torch.cuda.synchronize()
    stream = torch.cuda.current_stream()
    start = threading.Barrier(len(sets))

    def work(i):
        start.wait()
        for C in outs[i]:
            p(*sets[i], C, stream=stream)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(sets))]
    [t.start() for t in threads]
    [t.join() for t in threads]
    torch.cuda.synchronize()
    for i in range(len(sets)):
        assert all(torch.equal(C, ref[i]) for C in outs[i]), i
