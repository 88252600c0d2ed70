"""The performance cases of the library: matrix products through the torch
entry points of paper_2608_06812_amd.ozfp4, over the sizes that they are
called with.

A case names its entry point ("path"), the product's m, n and k, the moduli
or limb count ("count", 0: the entry point's default), the spread phi of the
entry law (U - 0.5) exp(phi N), how the caller holds the operands ("layout":
"col", column-major as in BLAS, or "row", contiguous torch tensors) and an
opt-in mode of the library ("mode": "", "heads" or "wide").

Paths and their ranges:
  dgemm    FP64 product, 1 to 32768 lines a side, 14 to 20 moduli (18 is the fewest
           that is FP64-accurate, 19 the default); with mode "heads" the list
           with five one-limb moduli first (21 moduli, the 18 greedy moduli's
           result), with mode "wide" capacities up to 63 bits (23 moduli) for
           wide exponent ranges
  noalloc  the same product on the library's fixed scratch memory
  split    FP64 product of wide-range inputs by the two-term split
  ozi      FP64 product by scheme I (15 limbs)
  sgemm    FP32 product
  igemm    INT8 x INT8 -> INT32 product
"""

import math

import torch

from paper_2608_06812_amd import ozfp4

MODE_HEADS = 5
MODE_WIDE_BITS = 63


def _case(name, path, m, n, k, count, phi=0.5, layout="col", mode=""):
    return {"name": name, "path": path, "m": m, "n": n, "k": k, "count": count, "phi": phi,
            "layout": layout, "mode": mode}


def listed():
    return [
        # the smallest product of the repository's workloads: launches and
        # the wait for the non-finite check count
        _case("dgemm_256", "dgemm", 256, 256, 256, 14),
        # a block of a blocked algorithm, from contiguous torch tensors
        _case("dgemm_1024_row", "dgemm", 1024, 1024, 1024, 18, layout="row"),
        # the size at which accuracy and throughput are traced
        _case("dgemm_4096", "dgemm", 4096, 4096, 4096, 18),
        # the headline size
        _case("dgemm_16384", "dgemm", 16384, 16384, 16384, 18),
        # sizes that no tile divides, from contiguous torch tensors
        _case("dgemm_ragged_row", "dgemm", 1500, 777, 3001, 19, layout="row"),
        # a tall matrix times a block of vectors (block Krylov, projections)
        _case("dgemm_tall", "dgemm", 20000, 48, 2000, 19),
        # the trailing update of a blocked factorisation
        _case("dgemm_update", "dgemm", 6000, 6000, 384, 18),
        # a small product in a program that may not allocate
        _case("noalloc_512", "noalloc", 512, 384, 640, 18),
        # wide exponent ranges at full accuracy
        _case("split_1536", "split", 1536, 1536, 4096, 19, phi=4.0),
        # scheme I, the cross-check of scheme II
        _case("ozi_1024", "ozi", 1024, 1024, 1024, 15),
        # FP32 emulation with the default moduli count, contiguous tensors
        _case("sgemm_2048_row", "sgemm", 2048, 2048, 2048, 0, layout="row"),
        # the INT8 workload
        _case("igemm_8192", "igemm", 8192, 8192, 8192, 0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _shape(rng, top):
    """A product's m, n, k: near-square, a tall or wide one, a long inner
    dimension or a low-rank update; multiples of 128 among odd sizes."""
    kind = rng.choice(("square", "square", "square", "skinny", "long", "update"))
    base = _log(rng, 64, top)
    if kind == "square":
        dims = [base if rng.random() < 0.5 else max(1, int(base * rng.uniform(0.6, 1.2)))
                for _ in range(3)]
    elif kind == "skinny":
        dims = [_log(rng, 1000, 8 * top), _log(rng, 1, 200), _log(rng, 64, 2 * top)]
        if rng.random() < 0.5:
            dims[0], dims[1] = dims[1], dims[0]
    elif kind == "long":
        dims = [_log(rng, 64, max(128, top // 8)), _log(rng, 64, max(128, top // 8)),
                _log(rng, 4096, 16 * top)]
    else:
        dims = [_log(rng, 512, 2 * top), _log(rng, 512, 2 * top), _log(rng, 64, 512)]
    if rng.random() < 0.4:
        dims = [max(128, d // 128 * 128) if d >= 128 else d for d in dims]
    return dims


def draw(rng):
    path = rng.choice(("dgemm",) * 6 + ("noalloc", "split", "ozi", "sgemm", "sgemm", "igemm",
                                        "igemm"))
    layout = rng.choice(("col", "col", "row"))
    phi, mode, count = 0.5, "", 0
    if path == "dgemm":
        m, n, k = _shape(rng, 4096)
        mode = rng.choice(("", "", "", "heads", "wide"))
        count = {"": rng.choice((14, 16, 18, 18, 19, 20)), "heads": 21, "wide": 23}[mode]
        phi = 4.0 if mode == "wide" else 0.5
    elif path == "noalloc":
        # the planes and residues of 18 moduli have to fit the scratch memory
        m, n, k = (_log(rng, 16, 1000) for _ in range(3))
        count = 18
    elif path == "split":
        m, n, k = _shape(rng, 1536)
        phi, count = 4.0, 19
    elif path == "ozi":
        m, n, k = _shape(rng, 1536)
        count = 15
    elif path == "sgemm":
        m, n, k = _shape(rng, 4096)
        count = rng.choice((0, 0, 10))
    else:
        m, n, k = _shape(rng, 6144)
    case = _case("", path, m, n, k, count, phi, layout, mode)
    del case["name"]
    return case


def _dtype(case):
    return {"sgemm": torch.float32, "igemm": torch.int8}.get(case["path"], torch.float64)


def _matrix(case, rows, cols, along_rows, gen):
    """A rows x cols matrix of the entry law; a line along k holds random
    values whatever the layout. along_rows: rows are adjacent in memory."""
    shape = (cols, rows) if along_rows else (rows, cols)
    if _dtype(case) == torch.int8:
        X = torch.randint(-128, 128, shape, dtype=torch.int8, device="cuda", generator=gen)
    else:
        X = torch.randn(shape, dtype=torch.float64, device="cuda", generator=gen)
        X.mul_(case["phi"]).exp_()
        X.mul_(torch.rand(shape, dtype=torch.float64, device="cuda", generator=gen).sub_(0.5))
        X = X.to(_dtype(case))
    return X.t() if along_rows else X


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    col = case["layout"] == "col"
    A = _matrix(case, case["m"], case["k"], col, gen)
    B = _matrix(case, case["k"], case["n"], col, gen)
    return A, B


def prepare(case, seed):
    ozfp4.load()
    ozfp4.ozfp4_init()
    A, B = _inputs(case, seed)
    state = {"case": dict(case), "A": A, "B": B}
    if case["path"] == "noalloc":
        state["out"] = torch.empty((case["n"], case["m"]), dtype=torch.float64, device="cuda").t()
    return state


def run(state):
    case, A, B = state["case"], state["A"], state["B"]
    path, count = case["path"], case["count"]
    if path == "dgemm":
        if case["mode"] == "heads":
            ozfp4.ozfp4_set_one_limb_moduli(MODE_HEADS)
        elif case["mode"] == "wide":
            ozfp4.ozfp4_set_max_capacity(MODE_WIDE_BITS)
        try:
            return ozfp4.dgemm(A, B, count)
        finally:
            ozfp4.ozfp4_set_one_limb_moduli(0)
            ozfp4.ozfp4_set_max_capacity(53)
    if path == "noalloc":
        return ozfp4.dgemm_noalloc(A, B, state["out"], count)
    if path == "split":
        return ozfp4.dgemm_split(A, B, count)
    if path == "ozi":
        return ozfp4.dgemm_ozi(A, B, count)
    if path == "sgemm":
        return ozfp4.sgemm(A, B, count or None)
    return ozfp4.igemm_s8(A, B)


def work(case):
    """Operands read once and C written once; the limb products of the
    method: four per two-limb modulus (three for 169, the first of the greedy
    list), one per one-limb modulus, four times all of them for the two-term
    split, limbs squared for scheme I, nine for INT8. FP32 emulation takes 10
    moduli where its default is asked for."""
    m, n, k, path, L = case["m"], case["n"], case["k"], case["path"], case["count"]
    if path == "ozi":
        products = L * L
    elif path == "igemm":
        products = 9
    elif path == "sgemm":
        products = 4 * (L or 10) - 1
    elif case["mode"] == "heads":
        products = 4 * (L - MODE_HEADS) - 1 + MODE_HEADS
    else:
        products = (4 * L - 1) * (4 if path == "split" else 1)
    size = {"sgemm": 4, "igemm": 1}.get(path, 8)
    csize = {"sgemm": 4, "igemm": 4}.get(path, 8)
    return {"bytes": float(size * (m * k + k * n) + csize * m * n),
            "flops": 2.0 * products * m * n * k}


def tolerance(case):
    """Every path defines its result bit for bit: the product of the converted
    operands is exact and rounded once, and the INT8 product is exact."""
    return "exact"


def exact(case, seed):
    """A B in 64 bits. The INT8 product's sums stay below 2^53, so the FP64
    product is exact."""
    A, B = _inputs(case, seed)
    C = torch.matmul(A.double(), B.double())
    if case["path"] == "igemm":
        C = C.to(torch.int64).to(torch.int32)   # wraps modulo 2^32, as the path does
    return C.t().contiguous().t()
