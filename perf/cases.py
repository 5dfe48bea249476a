"""Performance cases of the tensor-contraction library: what its users run.

A case is one contraction C = alpha A B + beta C through `Plan` (planned once,
called many times, as a program that contracts the same shapes again and again
does), or one transposition through `gett_transpose`.  All tensors are
column-major (the first mode is stride-one), the library's default layout;
`pad` leaves that many unused elements behind each run of the first mode (a
view into a larger tensor).

The listed cases are the five workloads of the benchmark, members of the
48-contraction benchmark's families at its own extents, one point of its
contracted-extent sweep, a coupled-cluster contraction whose extents are odd,
and the transposition.  `draw` gives other members of the same families with
other extents: half of them multiples of eight, the rest as they fall.
"""
from __future__ import annotations

import math

import torch

import paper_1607_00145_amd as gett

ITEM = {"f32": 4, "f64": 8}
TORCH = {"f32": torch.float32, "f64": torch.float64}


def _contract(name, dtype, pattern, ext, alpha=1.0, beta=0.0, pad=0, normal=False):
    c, a, b = pattern.split("-")
    case = {"op": "contract", "dtype": dtype, "C": c, "A": a, "B": b,
            "ext": ",".join(f"{m}={e}" for m, e in ext.items()), "alpha": alpha, "beta": beta,
            "pad": pad, "normal": normal}
    return dict(case, name=name) if name else case


def _transpose(name, dtype, pattern, ext, alpha=1.0, beta=0.0):
    out, inp = pattern.split("-")
    case = {"op": "transpose", "dtype": dtype, "C": out, "A": inp, "B": "",
            "ext": ",".join(f"{m}={e}" for m, e in ext.items()), "alpha": alpha, "beta": beta,
            "pad": 0, "normal": False}
    return dict(case, name=name) if name else case


def _all(modes, e):
    return {m: e for m in modes}


def listed():
    return [
        # the smallest call: a 32^3 tensor times a 32 x 32 matrix, all launch and latency
        _contract("ttm3_f32_32", "f32", "abc-akc-kb", _all("abck", 32)),
        # a small C (1152 x 1152) and a contracted extent of 64: one point of the
        # sweep between bandwidth- and compute-bound
        _contract("sweep_f32_k64", "f32", "apb-akb-kp", {"a": 32, "p": 1152, "b": 36, "k": 64}),
        # tensor times matrix that reads a large 5D tensor and writes a small one
        # (an index transformation to a smaller basis)
        _contract("ttm5_f32", "f32", "abcde-efbad-cf",
                  {"a": 48, "b": 36, "c": 24, "d": 36, "e": 48, "f": 36}),
        # small contracted extent, C read and written: bound by C's stream
        _contract("bw4x3_f32", "f32", "abcd-aeb-edc", dict(_all("abcd", 112), e=16), 1.5, 1.0),
        # CCSD(T) triples: 6D output, one small contracted index, single precision ...
        _contract("triples_f32", "f32", "abcdef-degb-gfac",
                  {"a": 24, "b": 20, "c": 20, "d": 24, "e": 20, "f": 20, "g": 24}),
        # ... and double precision
        _contract("triples_f64", "f64", "abcijk-dabi-cdjk", _all("abcdijk", 24)),
        # a small matrix contracted over two long indices
        _contract("deepk_f32", "f32", "ab-acd-dbc", {"a": 384, "b": 376, "c": 376, "d": 384}),
        # coupled-cluster doubles: 4D x 4D, compute-bound, double precision, accumulating
        _contract("doubles_f64", "f64", "abij-iejf-faeb", _all("abijef", 48), 1.0, 1.0,
                  normal=True),
        # the same contraction at extents as molecules have them: 23 occupied, 61 virtual
        _contract("doubles_odd_f64", "f64", "abij-iejf-faeb",
                  {"i": 23, "j": 23, "a": 61, "b": 61, "e": 61, "f": 61}, 1.0, 1.0, normal=True),
        # 4D x 4D shaped like a 4096^3 matrix product
        _contract("gemm4_f32", "f32", "mnop-mkoq-qnkp", _all("mnopkq", 64)),
        # 4D x 4D whose operands are stride-one along different contracted indices;
        # the largest call
        _contract("ksplit_f32", "f32", "abcd-eafb-fdec",
                  {"a": 96, "b": 84, "c": 84, "d": 84, "e": 96, "f": 96}),
        # reordering a 4D tensor for another program: every index reversed
        _transpose("reverse4_f32", "f32", "dcba-abcd", _all("abcd", 112)),
    ]


# Families that draw() takes its cases from: patterns, extents of the largest
# case, the factor the extents may shrink by, alpha / beta.
_FAMILIES = [
    # tensor times matrix, 3D to 5D
    ("abc-akc-kb", {"a": 320, "k": 128, "c": 320, "b": 128}, 10.0),
    ("abc-bda-dc", {"a": 384, "b": 384, "c": 24, "d": 384}, 4.0),
    ("abc-adc-bd", {"a": 384, "b": 384, "c": 376, "d": 376}, 6.0),
    ("abcd-ebad-ce", {"a": 96, "b": 84, "c": 24, "d": 84, "e": 96}, 4.0),
    ("abcde-efbad-cf", {"a": 48, "b": 36, "c": 24, "d": 36, "e": 48, "f": 36}, 3.0),
    # small contracted extent
    ("abcd-aeb-edc", {"a": 112, "b": 112, "c": 112, "d": 112, "e": 24}, 4.0),
    # contracted-extent sweep on a small C
    ("apb-akb-kp", {"a": 32, "p": 1152, "b": 36, "k": 1024}, 8.0),
    ("apbq-akb-pkq", {"a": 32, "p": 32, "b": 36, "q": 36, "k": 1024}, 6.0),
    # triples
    ("abcijk-dabi-cdjk", dict(_all("abcdijk", 22)), 2.5),
    ("abcdef-degb-gfac", {"a": 24, "b": 20, "c": 20, "d": 24, "e": 20, "f": 20, "g": 24}, 2.5),
    ("abcdef-gdab-efgc", {"a": 24, "b": 20, "c": 20, "d": 20, "e": 24, "f": 20, "g": 24}, 2.5),
    # a small matrix over two long indices
    ("ab-acd-dbc", {"a": 384, "b": 376, "c": 376, "d": 384}, 6.0),
    # 4D x 4D
    ("abij-iejf-faeb", {"i": 48, "j": 48, "a": 64, "b": 64, "e": 64, "f": 64}, 4.0),
    ("mnop-mkoq-qnkp", _all("mnopkq", 64), 4.0),
    ("abcd-aebf-fdec", {"a": 64, "b": 56, "c": 56, "d": 56, "e": 56, "f": 64}, 4.0),
    ("abcd-eafb-fdec", {"a": 64, "b": 56, "c": 56, "d": 56, "e": 64, "f": 64}, 4.0),
]
_PERMS = [("ba", 8192, 8.0), ("cba", 448, 6.0), ("bac", 448, 6.0), ("acb", 448, 6.0),
          ("dcba", 112, 4.0), ("cdab", 112, 4.0), ("badc", 112, 4.0), ("adcb", 112, 4.0),
          ("fedcba", 22, 2.5), ("abcfed", 22, 2.5)]


def _extent(rng, top, scale):
    e = max(3, round(top / scale * rng.uniform(0.75, 1.0)))
    return 8 * max(1, round(e / 8)) if rng.random() < 0.5 else e


def draw(rng):
    dtype = rng.choice(("f32", "f64"))
    if rng.random() < 1 / 6:
        out, top, shrink = rng.choice(_PERMS)
        inp = "".join(sorted(out))
        scale = math.exp(rng.uniform(0.0, math.log(shrink)))
        ext = {m: _extent(rng, top, scale) for m in inp}
        return _transpose(None, dtype, f"{out}-{inp}", ext, beta=rng.choice((0.0, 0.0, 1.0)))
    pattern, top, shrink = rng.choice(_FAMILIES)
    scale = math.exp(rng.uniform(0.0, math.log(shrink)))
    ext = {}
    for m, e in top.items():
        small = e <= 24 and len(top) < 7 and m not in pattern.split("-")[0]
        ext[m] = _extent(rng, e, min(scale, 2.0) if small else scale)
    alpha, beta = rng.choice(((1.0, 0.0), (1.0, 0.0), (1.0, 1.0), (1.5, 0.5)))
    return _contract(None, dtype, pattern, ext, alpha, beta, pad=rng.choice((0, 0, 0, 0, 8, 3)))


def _ext(case):
    return {m: int(e) for m, e in (x.split("=") for x in case["ext"].split(","))}


def _column_major(shape, pad, dtype):
    """An uninitialised column-major tensor (strides of a tensor whose first
    extent is `pad` longer)."""
    full = list(shape)
    full[0] += pad
    t = torch.empty(full[::-1], dtype=dtype, device="cuda").permute(*range(len(full) - 1, -1, -1))
    return t[: shape[0]]


def _draw_into(t, gen, normal):
    """Fill t, in its storage order, with U[-1,1] or N(0,1) values."""
    s = t.permute(*range(t.dim() - 1, -1, -1))
    if normal:
        s.copy_(torch.randn(s.shape, generator=gen, dtype=t.dtype, device=t.device))
    else:
        s.copy_(torch.rand(s.shape, generator=gen, dtype=t.dtype, device=t.device)).mul_(2).sub_(1)
    return t


def _inputs(case, seed):
    ext, dt = _ext(case), TORCH[case["dtype"]]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    shape = lambda k: [ext[m] for m in case[k]]
    A = _draw_into(_column_major(shape("A"), case["pad"], dt), gen, case["normal"])
    B = None
    if case["op"] == "contract":
        B = _draw_into(_column_major(shape("B"), case["pad"], dt), gen, case["normal"])
    C = _column_major(shape("C"), case["pad"], dt)
    if case["beta"] != 0.0:
        _draw_into(C, gen, False)
    return A, B, C


def prepare(case, seed):
    A, B, C = _inputs(case, seed)
    state = {"case": case, "A": A, "B": B, "C": C}
    if case["op"] == "contract":
        state["plan"] = gett.Plan(tuple(",".join(case[k]) for k in ("C", "A", "B")), C, A, B)
    else:
        ext = _ext(case)
        state["dtype"] = gett.GETT_FLOAT32 if case["dtype"] == "f32" else gett.GETT_FLOAT64
        state["extent"] = [ext[m] for m in case["A"]]
        state["stride_in"] = list(A.stride())
        state["stride_out"] = [C.stride(case["C"].index(m)) for m in case["A"]]
    return state


def run(state):
    case, A, C = state["case"], state["A"], state["C"]
    if case["op"] == "contract":
        return state["plan"](A, state["B"], C, alpha=case["alpha"], beta=case["beta"])
    st = gett.gett_transpose(state["dtype"], state["extent"], state["stride_in"],
                             state["stride_out"], case["alpha"], A.data_ptr(), case["beta"],
                             C.data_ptr(), torch.cuda.current_stream().cuda_stream)
    if st != 0:
        raise gett.GettError(st, "gett_transpose")
    return C


def _contracted(case):
    return [m for m in case["A"] if m not in case["C"]] if case["op"] == "contract" else []


def work(case):
    ext = _ext(case)
    size = lambda modes: math.prod(ext[m] for m in modes)
    n = size(case["A"]) + size(case["B"] or "") * (case["op"] == "contract")
    n += size(case["C"]) * (2 if case["beta"] != 0.0 else 1)
    flops = 2 * size(case["C"]) * size(_contracted(case)) if case["op"] == "contract" else 0
    return {"bytes": ITEM[case["dtype"]] * n, "flops": flops}


def tolerance(case):
    """A transposition that neither scales nor accumulates moves values
    unchanged.  Otherwise: the rounding of sums of K products in any order --
    the error of a sum of K random terms, relative to the sum's own size,
    grows as sqrt(K) unit round-offs (the partial sums grow as sqrt(k)).
    Measured against 64-bit (fp32) and another library's (fp64) sums: 8e-8 at
    K = 16, 1.4e-7 at 64, 1.1e-6 at 4096 (fp32), 1.2e-15 at 2304 (fp64);
    the bound is about four times that."""
    if case["op"] == "transpose" and case["alpha"] == 1.0 and case["beta"] == 0.0:
        return "exact"
    u = 2.0 ** -24 if case["dtype"] == "f32" else 2.0 ** -53
    ext = _ext(case)
    k = math.prod(ext[m] for m in _contracted(case))
    return {"rel": u * (2.0 + math.sqrt(k))}


def exact(case, seed):
    A, B, C = _inputs(case, seed)
    A, ext = A.double(), _ext(case)
    if case["op"] == "transpose":
        out = A.permute(*[case["A"].index(m) for m in case["C"]]) * case["alpha"]
    else:
        k = _contracted(case)
        m = [x for x in case["A"] if x not in k]
        n = [x for x in case["B"] if x not in k]
        size = lambda modes: math.prod(ext[x] for x in modes)
        a = A.permute(*[case["A"].index(x) for x in m + k]).reshape(size(m), size(k)).contiguous()
        b = B.double().permute(*[case["B"].index(x) for x in k + n]).reshape(size(k), size(n)).contiguous()
        out = (a @ b).reshape([ext[x] for x in m + n])
        out = out.permute(*[(m + n).index(x) for x in case["C"]]) * case["alpha"]
    if case["beta"] != 0.0:
        out = out + case["beta"] * C.double()
    return out
