"""GPU parity of the residue GEMM for short products (128 x 128 tiles, k in
64-wide stages through a 4-slot ring): every residue against (A~ B~) mod m
from the oracle's converted integers, exactly. The sizes sit at the edges of
the ring's fill (1 to 6 stages), of the tile (127 to 129 lines) and of the
residue composition's ranges of k (1280 / 1281 and 17472 / 17473, where the
sums of 4 (acc0 + 13 acc1 + 169 acc2) and of 4 (acc1 + 13 acc2) reach 2^24
at most). Constant operands drive the sums towards those bounds: every
product of a modulus then has the same sign and limbs."""

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
    (64, 64, 17472, 18, "constant"),
    (64, 64, 17473, 18, "constant"),
    (40, 150, 70000, 19, "constant"),
]


def _inputs(m, n, k, kind):
    if kind == "random":
        return dgemm_inputs(m, n, k, 0.5, SEED + m + 3 * n + 7 * k)
    # a line of one value per row / column: the sums over k do not cancel
    rng = np.random.default_rng(SEED + k)
    A = np.repeat(1.0 + rng.random((m, 1)), k, axis=1)
    B = np.repeat(1.0 + rng.random((1, n)), k, axis=0)
    return A, B


@pytest.mark.parametrize("m,n,k,L,kind", CASES)
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
