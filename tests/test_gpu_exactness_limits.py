"""GPU parity of the GEMMs at the ends of the ranges in which one accumulation
and its composition are exact, each case at a size that the dispatch rules
leave to one kernel in one k range (test_routes_host.py holds them to that):

* residues: k at which the composition changes from one reduction to two
  (1280 / 1281) and from two to FP64 (short: 17472 / 17473, long, whose k is
  padded to 128: 17408 / 17409), and the largest k, 131072;
* INT8: the longest range of the short GEMM, 40960 k of the largest limb
  sums, and several of the long one's accumulations (81920 k at most);
* scheme I: the longest k of its short GEMM, 8192, of the largest limbs.

Residue operands: lines of one integer that is, modulo each of about six
moduli, the class whose limbs make the largest products (57 = -8 - 8 13
modulo 169, whose cross term then reaches 2^22 in units of the stored values
at k = 131072, the FP32 limit), so that the sums of those moduli do not
cancel over k; each line starts with a power of two that makes its conversion
exact and ends in ones, whose limb products (a quarter) an inexact
accumulation would drop."""

import numpy as np
import pytest

import oracle as o
from gpu_util import announce, bits_equal, dev_cm, to_np

# (m, n, k, moduli, kernel)
RESIDUES = [(1024, 1024, k, 18, "short") for k in (1280, 1281, 17472, 17473, 20000, 131072)] + \
           [(1536, 1152, k, 19, "long") for k in (17408, 17409, 131072)]
INT8 = [(3200, 3072, 40960, "short"), (40, 24, 700000, "long")]
OZI = (40, 24, 8192)


def _largest_class(m):
    """The residue of m whose limbs (c0, c1) make the largest 2 c0 c1 + 13 c1^2,
    the terms of a square that the composition's second bound counts."""
    def size(r):
        c0, c1 = o.two_limb_split(r, m)
        return 2 * c0 * c1 + 13 * c1 * c1
    return max(range(m), key=size)


def _extreme_integers(moduli, below):
    """Integers below `below`, each in the largest class of as many moduli in
    turn as fit (CRT), until every modulus has had its turn."""
    out, x, M = [], 0, 1
    for m in moduli:
        if M * m >= below:
            out.append(x)
            x, M = 0, 1
        x += M * ((_largest_class(m) - x) * pow(M, -1, m) % m)
        M *= m
    return out + [x]


def extreme_lines(k, moduli):
    """Distinct rows of A and columns of B (as rows), exact under conversion."""
    cA, cB = o.capacity_bits(k, moduli)
    values = _extreme_integers(moduli, 2 ** (cB - 1))
    for m in moduli:
        assert any(x % m == _largest_class(m) for x in values)
    lines = []
    for c in (cA, cB):
        X = np.empty((2 * len(values) + 1, k))
        for g, x in enumerate(values):
            X[2 * g], X[2 * g + 1] = x, -x
        X[-1] = values[0]
        X[-1, k // 2:] = -values[-1]               # a line that turns half way
        X[:, 0] = 2.0 ** (c - 1)
        X[:, -3:] = 1.0
        lines.append(X)
    return lines


def test_extreme_lines_on_host():
    """The lines convert exactly, and modulo 169 every limb is +-8."""
    assert o.two_limb_split(57, 169) == (-8, -8) and _largest_class(169) == 57
    for L, k in ((18, 1280), (19, 17408), (18, 131072), (19, 131072)):
        moduli = o.select_moduli(L)
        lines = extreme_lines(k, moduli)
        for X, c in zip(lines, o.capacity_bits(k, moduli)):
            Xi = o.to_integers(X, o.shift_exponents(X, axis=1, c=c), axis=1)
            assert np.array_equal(Xi, X.astype(np.int64))
            assert set(np.unique(np.abs(np.stack(o.limb_planes(Xi[:1, 1:-3], 169))))) == {8}


def _repeat(X, lines):
    """Column-major device operand (lines x k) that repeats the rows of X."""
    import torch
    idx = torch.arange(lines, device="cuda") % X.shape[0]
    return torch.from_numpy(np.ascontiguousarray(X.T)).cuda()[:, idx].contiguous().t()


def _spread(want, m, n):
    """The m x n matrix whose element (i, j) is want[i % rows, j % columns]."""
    return want[np.arange(m) % want.shape[0]][:, np.arange(n) % want.shape[1]]


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k,L,kernel", RESIDUES)
def test_residues_of_one_long_accumulation(gpu_lib, m, n, k, L, kernel):
    import torch
    moduli = o.select_moduli(L)
    Ad, Bd = extreme_lines(k, moduli)
    A = _repeat(Ad, m)
    B = gpu_lib.colmajor(_repeat(Bd, n).t())
    announce(f"{kernel} residue GEMM at its limit m={m} n={n} k={k} L={L}")
    R = gpu_lib.residues(A, B, L)
    Ai, Bi = Ad.astype(np.int64), Bd.astype(np.int64)
    assert 168.0 ** 2 * k < 2.0 ** 53
    for l, q in enumerate(moduli):
        ra, rb = o.residues(Ai, q).astype(np.float64), o.residues(Bi, q).astype(np.float64)
        want = np.mod(np.rint(ra @ rb.T).astype(np.int64), q).astype(np.uint8)
        assert torch.equal(R[l].t().cpu(), torch.from_numpy(_spread(want, m, n))), f"modulus {q}"
    if k == 131072:
        announce(f"dgemm m={m} n={n} k={k} L={L}")
        C = to_np(gpu_lib.dgemm(A, B, L))
        assert bits_equal(C, _spread(o.dgemm(Ad, np.ascontiguousarray(Bd.T), L)["C"], m, n))


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k,kernel", INT8)
def test_int8_longest_range(gpu_lib, m, n, k, kernel):
    """The values whose limb products make the largest sums:
    -112 = -8 - 8 13 (128 a k in the second accumulator), 73 = 8 - 8 13 + 169
    (80 in the third), beside -128, the largest product of the values, with
    signs that turn along some lines and a last k of small products."""
    import torch
    assert o.limb_decompose(-112, 3) == [-8, -8, 0] and o.limb_decompose(73, 3) == [8, -8, 1]
    rows = np.repeat(np.array([[-112], [73], [-112], [-128], [112]], dtype=np.int8), k, axis=1)
    cols = np.repeat(np.array([[-112], [73], [-57], [-128]], dtype=np.int8), k, axis=1)
    rows[2, ::2] = 112
    rows[4, k // 2:] = -57
    rows[:, -1] = 1
    want = (rows.astype(np.int64) @ cols.astype(np.int64).T).astype(np.int32)   # wraps
    announce(f"int8 {kernel} GEMM at its limit m={m} n={n} k={k}")
    C = gpu_lib.igemm_s8(_repeat(rows, m), gpu_lib.colmajor(_repeat(cols, n).t()))
    assert torch.equal(C.cpu(), torch.from_numpy(_spread(want, m, n)))


@pytest.mark.gpu
def test_scheme_one_longest_short_product(gpu_lib):
    """k = 8192 of fourteen limbs of 8 and one of 1: the largest partial sums
    of scheme I's short GEMM, recomposed to the exact integer product."""
    x = sum(8 * 13 ** i for i in range(14)) + 13 ** 14
    assert o.limb_decompose(x, 15) == [8] * 14 + [1]
    m, n, k = OZI
    A = np.full((m, k), float(x))
    B = np.full((k, n), float(x))
    A[1, :] = -float(x)
    B[:, 2] = -float(x)
    A[3, 1::2] = -float(x)
    res = o.dgemm_ozi(A, B, 15)
    announce(f"scheme I short GEMM at its limit m={m} n={n} k={k}")
    H = to_np(gpu_lib.ozi_partials(dev_cm(A), dev_cm(B), 15))
    total = np.zeros((m, n), dtype=object)
    for h in range(H.shape[0]):
        total = total + H[h].T.astype(object) * 2197 ** h
    assert np.all(total == res["x"])
    assert bits_equal(to_np(gpu_lib.dgemm_ozi(dev_cm(A), dev_cm(B), 15)), res["C"])
