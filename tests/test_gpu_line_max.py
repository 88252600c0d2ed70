"""GPU line maxima at the edges of their split: line counts around the 4, 16
and 64 lines of a block where lines are adjacent (A) and the four of a block
where they are contiguous (B), k around the chunks, leading dimensions above
the line count; the largest element sits at a random place of each line.
Shifts against the oracle's. A NaN or infinity anywhere is reported by that
call and by no other."""

import numpy as np
import pytest

import oracle as o
from gpu_util import announce, dev_cm, to_np

pytestmark = pytest.mark.gpu

SEED = 20261206


def _peaked(rng, lines, k):
    """lines x k, one large element per line, its exponent per line."""
    X = rng.random((lines, k)) - 0.5
    X[np.arange(lines), rng.integers(0, k, size=lines)] = np.ldexp(1.5, rng.integers(1, 200, size=lines))
    return X


def _padded(X, extra):
    """Column-major device copy with leading dimension rows + extra."""
    import torch
    P = np.full((X.shape[0] + extra, X.shape[1]), np.nan)
    P[:X.shape[0]] = X
    return dev_cm(P)[:X.shape[0]]


SHAPES = [(1, 1, 1), (3, 2, 255), (4, 5, 2049), (5, 4, 257), (16, 17, 4097), (17, 16, 513),
          (64, 65, 1025), (65, 64, 8200), (130, 3, 20001), (2, 300, 131072), (700, 900, 96)]


@pytest.mark.parametrize("m,n,k", SHAPES)
def test_shifts_at_the_edges_of_the_split(gpu_lib, m, n, k):
    rng = np.random.default_rng(SEED + m + k)
    A, B = _peaked(rng, m, k), _peaked(rng, n, k).T
    cA, cB = o.capacity_bits(k, o.select_moduli(19))
    announce(f"shifts m={m} n={n} k={k}")
    s, t = gpu_lib.scales(_padded(A, 3), _padded(B, 5), 19)
    assert np.array_equal(to_np(s), np.asarray(o.shift_exponents(A, axis=1, c=cA), dtype=np.int64))
    assert np.array_equal(to_np(t), np.asarray(o.shift_exponents(B, axis=0, c=cB), dtype=np.int64))


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("m,n,k", [(5, 4, 2049), (70, 65, 700)])
def test_non_finite_is_reported_by_its_call_alone(gpu_lib, m, n, k, bad):
    import torch
    rng = np.random.default_rng(SEED)
    A, B = _peaked(rng, m, k), _peaked(rng, n, k).T
    good = gpu_lib.dgemm(dev_cm(A), dev_cm(B), 18).clone()
    A2, B2 = A.copy(), B.copy()
    A2[m - 1, k - 1] = bad
    B2[k - 1, 0] = bad
    announce(f"non-finite {bad} m={m} n={n} k={k}")
    for X, Y in ((A2, B), (A, B2)):
        with pytest.raises(gpu_lib.OzFP4Error) as e:
            gpu_lib.dgemm(dev_cm(X), dev_cm(Y), 18)
        assert e.value.code == gpu_lib.OZFP4_ENONFINITE
        with pytest.raises(gpu_lib.OzFP4Error) as e:
            gpu_lib.sgemm(dev_cm(X).float(), dev_cm(Y).float(), 10)
        assert e.value.code == gpu_lib.OZFP4_ENONFINITE
        assert torch.equal(gpu_lib.dgemm(dev_cm(A), dev_cm(B), 18), good)
