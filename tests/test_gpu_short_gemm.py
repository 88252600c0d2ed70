"""GPU parity of the residue GEMM for short products (128 x 128 tiles, k in
64-wide stages through a 4-slot ring): every residue against (A~ B~) mod m
from the oracle's converted integers, exactly. The sizes sit at the edges of
the ring's fill (1 to 6 stages), of the tile (127 to 129 lines) and of the
residue composition's first border (1280 / 1281 k in one range). Constant
operands keep the sums from cancelling: every product of a modulus then has
the same sign and limbs. Long inner dimensions over few tiles run in several
k ranges, whose lengths stay below the composition's other borders;
test_gpu_exactness_limits.py takes those in one range, with the largest
limbs."""

import numpy as np
import pytest

import oracle as o
from gpu_util import announce, dev_cm, to_np
from paper_2608_06812_amd.workloads import dgemm_inputs

pytestmark = pytest.mark.gpu

SEED = 20261204

CASES = [
    (1, 1, 1, 18, "random"),
    (127, 129, 63, 18, "random"),
    (128, 128, 64, 14, "random"),
    (129, 127, 65, 18, "random"),
    (257, 100, 130, 27, "random"),
    (100, 257, 200, 19, "random"),
    (130, 60, 256, 18, "random"),
    (60, 130, 257, 18, "constant"),
    (300, 300, 321, 18, "random"),
    (96, 80, 1280, 18, "constant"),
    (96, 80, 1281, 18, "constant"),
    (200, 140, 1337, 27, "random"),
    (129, 257, 2049, 27, "random"),
    (300, 290, 3000, 18, "constant"),
    (500, 400, 9000, 16, "random"),
    (1030, 900, 700, 18, "random"),
]

# k cut into ranges whose residues are added modulo m, and how many
RANGES = [
    (129, 257, 3000, 18, "random", 2),
    (300, 290, 9000, 18, "constant", 3),
    (100, 129, 2049, 18, "random", 4),
    (500, 400, 20000, 18, "random", 5),
    (64, 64, 17472, 18, "constant", 13),
    (64, 64, 17473, 18, "constant", 14),
    (40, 150, 70000, 19, "constant", 13),
]

# outputs of enough tiles that a block runs several moduli (k up to 512):
# whole and short last groups, 1 to 8 stages a modulus
GROUPED = [(2600, 2500, 30, 18), (2560, 2700, 64, 19), (3000, 2300, 130, 23), (2500, 2600, 257, 18),
           (2300, 3100, 512, 18), (5000, 4900, 200, 18)]


def _inputs(m, n, k, kind):
    if kind == "random":
        return dgemm_inputs(m, n, k, 0.5, SEED + m + 3 * n + 7 * k)
    # a line of one value per row / column: the sums over k do not cancel
    rng = np.random.default_rng(SEED + k)
    A = np.repeat(1.0 + rng.random((m, 1)), k, axis=1)
    B = np.repeat(1.0 + rng.random((1, n)), k, axis=0)
    return A, B


@pytest.mark.parametrize("m,n,k,L,kind", CASES + [c[:-1] for c in RANGES])
def test_residues_of_short_products(gpu_lib, m, n, k, L, kind):
    A, B = _inputs(m, n, k, kind)
    moduli = o.select_moduli(L)
    cA, cB = o.capacity_bits(k, moduli)
    Ai = o.to_integers(A, o.shift_exponents(A, axis=1, c=cA), axis=1)
    Bi = o.to_integers(B, o.shift_exponents(B, axis=0, c=cB), axis=0)
    announce(f"short GEMM m={m} n={n} k={k} L={L} {kind}")
    R = to_np(gpu_lib.residues(dev_cm(A), dev_cm(B), L))
    assert 168.0 ** 2 * k < 2.0 ** 53
    for l, q in enumerate(moduli):
        ra = o.residues(Ai, q).astype(np.float64)
        rb = o.residues(Bi, q).astype(np.float64)
        want = np.mod(np.rint(ra @ rb).astype(np.int64), q)
        assert np.array_equal(R[l].T.astype(np.int64), want), f"modulus {q}"


@pytest.mark.parametrize("m,n,k,L", GROUPED)
def test_residues_of_several_moduli_a_block(gpu_lib, m, n, k, L):
    import torch
    A, B = dgemm_inputs(m, n, k, 0.5, SEED + m + k)
    moduli = o.select_moduli(L)
    cA, cB = o.capacity_bits(k, moduli)
    Ai = o.to_integers(A, o.shift_exponents(A, axis=1, c=cA), axis=1)
    Bi = o.to_integers(B, o.shift_exponents(B, axis=0, c=cB), axis=0)
    announce(f"several moduli a block m={m} n={n} k={k} L={L}")
    R = gpu_lib.residues(dev_cm(A), dev_cm(B), L)
    for l, q in enumerate(moduli):   # the vendor's FP64 product is exact here
        ra = torch.from_numpy(o.residues(Ai, q).astype(np.float64)).cuda()
        rb = torch.from_numpy(o.residues(Bi, q).astype(np.float64)).cuda()
        want = torch.remainder(torch.round(ra @ rb).to(torch.int64), q).to(torch.uint8)
        assert torch.equal(R[l].t(), want), f"modulus {q}"


def test_split_route_in_k_ranges(gpu_lib):
    """The four products of the two-term split in one launch, k in ranges,
    with and without one-limb heads: entries of few bits, whose product FP64
    holds exactly."""
    rng = np.random.default_rng(SEED)
    m, n, k = 130, 100, 5000
    A = rng.integers(-1000, 1001, size=(m, k)).astype(np.float64)
    B = rng.integers(-1000, 1001, size=(k, n)).astype(np.float64)
    want = A @ B
    announce("split in k ranges")
    try:
        for heads, L in ((0, 19), (4, 21)):
            gpu_lib.ozfp4_set_one_limb_moduli(heads)
            C = to_np(gpu_lib.dgemm_split(dev_cm(A), dev_cm(B), L))
            assert np.array_equal(C, want)
            assert np.array_equal(to_np(gpu_lib.dgemm(dev_cm(A), dev_cm(B), L)), want)
    finally:
        gpu_lib.ozfp4_set_one_limb_moduli(0)


def test_noalloc_without_room_for_the_ranges(gpu_lib):
    """A call whose planes and residues just fit the scratch array runs with
    one k range (its other ranges' residues would not fit), with the
    workspace call's bits."""
    import torch
    m, n, k, L = 200, 180, 28928, 18
    assert gpu_lib.ozfp4_init() == gpu_lib.OZFP4_OK
    A, B = dgemm_inputs(m, n, k, 0.5, SEED)
    Ad, Bd = dev_cm(A), dev_cm(B)
    out = torch.zeros((n, m), dtype=torch.float64, device="cuda").t()
    announce("noalloc at the scratch limit")
    gpu_lib.dgemm_noalloc(Ad, Bd, out, L)
    assert torch.equal(out, gpu_lib.dgemm(Ad, Bd, L))
    Ad = dev_cm(np.ones((m, k + 256)))
    Bd = dev_cm(np.ones((k + 256, n)))
    with pytest.raises(gpu_lib.OzFP4Error) as e:
        gpu_lib.dgemm_noalloc(Ad, Bd, out, L)
    assert e.value.code == gpu_lib.OZFP4_ESCRATCH
