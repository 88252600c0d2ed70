"""GPU parity of the INT8 path at the edges of its splits, exact against
numpy's integer product modulo 2^32: the encoder's blocks of 128 lines x 64
k with whole and partial words, leading dimensions that leave rows and
columns unaligned, the short GEMM's ring fill (1 to 6 stages of 64), tile
remainders, k ranges (with sums that wrap) and the rule's borders to the long
GEMM (k = 1024, a full round of tiles, more than 16 ranges). The ranges here
are short of the longest one that is exact, which
test_gpu_exactness_limits.py takes."""

import numpy as np
import pytest

from gpu_util import announce

pytestmark = pytest.mark.gpu

SEED = 20261207

# (m, n, k, extra rows of A's, B's and C's leading dimensions, extreme values)
CASES = [
    (1, 1, 1, 0, 0, 0, False), (1, 5, 33, 0, 3, 1, False), (3, 130, 63, 1, 2, 3, False),
    (127, 63, 64, 0, 0, 0, False), (128, 64, 65, 0, 1, 0, False), (129, 65, 128, 3, 0, 5, False),
    (130, 200, 191, 2, 5, 2, True), (257, 129, 256, 0, 0, 0, False), (255, 70, 321, 1, 1, 1, False),
    (300, 260, 385, 4, 16, 0, False), (700, 500, 1024, 0, 0, 0, False),
    (700, 500, 1025, 1, 0, 0, False), (60, 50, 5000, 0, 7, 0, True),
    (129, 65, 41000, 0, 0, 1, True), (40, 30, 200001, 1, 1, 0, True),
    (2048, 2040, 1100, 0, 0, 0, False), (1000, 3000, 1500, 1, 2, 3, False),
    (5, 3, 700000, 0, 0, 0, True),
]


def _device(X, extra):
    import torch
    P = np.full((X.shape[0] + extra, X.shape[1]), 99, dtype=np.int8)
    P[:X.shape[0]] = X
    return torch.from_numpy(np.ascontiguousarray(P.T)).cuda().t()[:X.shape[0]]


@pytest.mark.parametrize("m,n,k,ea,eb,ec,extreme", CASES)
def test_igemm_at_the_edges(gpu_lib, m, n, k, ea, eb, ec, extreme):
    import torch
    rng = np.random.default_rng(SEED + m + 5 * n + 11 * k)
    if extreme:   # no cancellation: sums reach 2^31 and wrap where k allows
        A = rng.integers(-128, -119, size=(m, k)).astype(np.int8)
        B = rng.integers(-128, -119, size=(k, n)).astype(np.int8)
    else:
        A = rng.integers(-128, 128, size=(m, k)).astype(np.int8)
        B = rng.integers(-128, 128, size=(k, n)).astype(np.int8)
    # |sums| < 2^14 k < 2^53: exact in FP64
    want = np.rint(A.astype(np.float64) @ B.astype(np.float64)).astype(np.int64).astype(np.int32)
    full = torch.full((n, m + ec), 7, dtype=torch.int32, device="cuda").t()
    announce(f"igemm m={m} n={n} k={k} ld extra {ea} {eb} {ec}")
    C = gpu_lib.igemm_s8(_device(A, ea), _device(B, eb), out=full[:m])
    assert np.array_equal(C.cpu().numpy(), want)
    assert bool((full[m:] == 7).all())
