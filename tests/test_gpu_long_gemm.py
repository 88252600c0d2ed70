"""GPU parity of the residue GEMM for long products (256 x 128 tiles, blocks
of one XCD started in step), at the smallest sizes that take it (k above
6144 and at least 1024 blocks): a tile grid that divides by the 8 XCDs and
one that does not (its last arrival groups are short), three moduli's worth of
blocks, the four GEMMs of the two-term split sharing one call's counters,
and a second stream that holds part of the GPU, so that groups stay short
and the wait ends by its bound. Residues against (A~ B~) mod m with the
oracle's converted integers and the vendor's FP64 product (exact below
2^53)."""

import numpy as np
import pytest

import oracle as o
from gpu_util import announce, bits_equal, dev_cm, to_np
from paper_2608_06812_amd.workloads import dgemm_inputs

pytestmark = pytest.mark.gpu

SEED = 20261205


def _want_residues(A, B, k, L):
    import torch
    moduli = o.select_moduli(L)
    cA, cB = o.capacity_bits(k, moduli)
    Ai = o.to_integers(A, o.shift_exponents(A, axis=1, c=cA), axis=1)
    Bi = o.to_integers(B, o.shift_exponents(B, axis=0, c=cB), axis=0)
    assert 168.0 ** 2 * k < 2.0 ** 53
    for q in moduli:
        ra = torch.from_numpy(o.residues(Ai, q).astype(np.float64)).cuda()
        rb = torch.from_numpy(o.residues(Bi, q).astype(np.float64)).cuda()
        yield q, torch.remainder(torch.round(ra @ rb).to(torch.int64), q).to(torch.uint8)


CASES = [(1024, 2048, 6145, 18), (1100, 1900, 6272, 16), (8000, 2050, 6200, 3)]


@pytest.mark.parametrize("m,n,k,L", CASES)
def test_residues_of_long_products(gpu_lib, m, n, k, L):
    import torch
    A, B = dgemm_inputs(m, n, k, 0.5, SEED + m)
    announce(f"long GEMM m={m} n={n} k={k} L={L}")
    R = gpu_lib.residues(dev_cm(A), dev_cm(B), L)
    for l, (q, want) in enumerate(_want_residues(A, B, k, L)):
        assert torch.equal(R[l].t(), want), f"modulus {q}"


def test_split_runs_four_long_gemms(gpu_lib):
    """The split route equals scheme I's exact product wherever its operands
    hold the inputs exactly: entries of few bits."""
    rng = np.random.default_rng(SEED)
    m, n, k, L = 1100, 1900, 6272, 19
    A = rng.integers(-1000, 1001, size=(m, k)).astype(np.float64)
    B = rng.integers(-1000, 1001, size=(k, n)).astype(np.float64)
    announce("split with four long GEMMs")
    C = to_np(gpu_lib.dgemm_split(dev_cm(A), dev_cm(B), L))
    assert bits_equal(C, A @ B)      # integer sums below 2^53: exact in FP64


def test_long_product_beside_another_stream(gpu_lib):
    import torch
    m, n, k, L = 1100, 1900, 6272, 18
    A, B = dgemm_inputs(m, n, k, 0.5, SEED + 1)
    Ad, Bd = dev_cm(A), dev_cm(B)
    want = gpu_lib.dgemm(Ad, Bd, L).clone()
    X = torch.randn(4096, 4096, device="cuda")
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    announce("long GEMM beside FP32 products on another stream")
    with torch.cuda.stream(side):
        for _ in range(20):
            Y = X @ X
    C = gpu_lib.dgemm(Ad, Bd, L)
    torch.cuda.synchronize()
    assert torch.equal(C, want) and bool(torch.isfinite(Y).all())
