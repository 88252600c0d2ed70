"""GPU parity of scheme I's GEMMs at the edges of their rule and of the short
one's ring and tiles: partial sums H against the oracle's limbs, multiplied
exactly in FP64 on the CPU. 1 to 6 stages per pair, one to five limb blocks,
tile remainders, tile counts that 8 divides and does not, k at the border of
the short GEMM's rule (8192) with operands whose sums do not cancel, and the
long GEMM just beyond. (The largest limbs at 8192 are
test_gpu_exactness_limits.py's.)"""

import numpy as np
import pytest

import oracle as o
from gpu_util import announce, dev_cm, to_np
from paper_2608_06812_amd.workloads import dgemm_inputs

pytestmark = pytest.mark.gpu

SEED = 20261210

CASES = [
    (1, 1, 1, 15, False), (128, 64, 64, 15, False), (129, 65, 65, 13, False), (60, 200, 192, 1, False),
    (257, 130, 256, 4, False), (130, 300, 321, 9, False), (300, 260, 384, 15, False),
    (1500, 700, 100, 12, False), (100, 90, 8192, 15, True), (100, 90, 8193, 15, True),
    (40, 30, 20000, 7, True),
]


def _blocks(Xi, p):
    """Values of the blocks of three greedy limbs."""
    limbs = o.ozi_limbs(Xi, p)
    limbs += [np.zeros_like(limbs[0])] * (-p % 3)
    return [(limbs[i] + 13 * limbs[i + 1] + 169 * limbs[i + 2]).astype(np.float64)
            for i in range(0, len(limbs), 3)]


@pytest.mark.parametrize("m,n,k,p,same", CASES)
def test_dgemm_ozi_at_the_edges(gpu_lib, m, n, k, p, same):
    """Every partial sum H against the oracle's limbs, and sampled outputs C
    against the product of the converted integers (exact integers), correctly
    rounded."""
    if same:   # one value per line: no cancellation over k
        rng = np.random.default_rng(SEED + k)
        A = np.repeat(1.0 + rng.random((m, 1)), k, axis=1)
        B = np.repeat(1.0 + rng.random((1, n)), k, axis=0)
    else:
        A, B = dgemm_inputs(m, n, k, 0.5, SEED + m + n + k)
    announce(f"ozi m={m} n={n} k={k} p={p}")
    C = to_np(gpu_lib.dgemm_ozi(dev_cm(A), dev_cm(B), p))
    cap, _, _ = gpu_lib.ozfp4_ozi_config(p)
    s = np.asarray(o.shift_exponents(A, axis=1, c=cap), dtype=np.int64)
    t = np.asarray(o.shift_exponents(B, axis=0, c=cap), dtype=np.int64)
    H = to_np(gpu_lib.ozi_partials(dev_cm(A), dev_cm(B), p))
    # block values below 8 (1 + 13 + 169): sums below 2^53, exact in FP64
    D = _blocks(o.to_integers(A, s, axis=1), p)
    E = _blocks(o.to_integers(B, t, axis=0), p)
    nblk = len(D)
    assert H.shape[0] == 2 * nblk - 1 and nblk * 1464.0 ** 2 * k < 2.0 ** 53
    for h in range(2 * nblk - 1):
        want = sum(D[I] @ E[h - I] for I in range(nblk) if 0 <= h - I < nblk)
        assert np.array_equal(H[h].T, want.astype(np.int64)), h
    rows = sorted({0, m // 2, m - 1})
    cols = sorted({0, 31 % n, n // 2, n - 1})
    Ai = o.to_integers(A[rows], s[rows], axis=1)
    Bi = o.to_integers(B[:, cols], t[cols], axis=0)
    for a, i in enumerate(rows):
        for b, j in enumerate(cols):
            x = sum(int(u) * int(v) for u, v in zip(Ai[a], Bi[:, b]))
            e = int(s[i] + t[j])
            want = float(x / 2 ** e) if e >= 0 else float(x * 2 ** -e)   # correctly rounded
            assert C[i, j] == want, (i, j)


@pytest.mark.parametrize("m,n,k", [(1500, 700, 300), (300, 260, 700), (520, 500, 3000)])
def test_ozi_equals_scheme_two_on_whole_outputs(gpu_lib, m, n, k):
    """At 53-bit capacities both schemes round the same exact product."""
    import torch
    A, B = dgemm_inputs(m, n, k, 0.5, SEED + k)
    Ad, Bd = dev_cm(A), dev_cm(B)
    assert gpu_lib.ozfp4_capacity(k, 20) == (53, 53)
    announce(f"ozi against scheme II m={m} n={n} k={k}")
    assert torch.equal(gpu_lib.dgemm_ozi(Ad, Bd, 15), gpu_lib.dgemm(Ad, Bd, 20))
