"""GPU parity of every product, the opt-in modes of the FP64 one included, over
the storage orders that the torch helpers accept: row-major operands are read
in place, every other layout through a column-major copy, and each gives the
bits of the same matrix in column-major order. Odd sizes and leading
dimensions leave lines unaligned; a single row, a single column, step slices,
expanded rows and transposed views are among the forms."""

import numpy as np
import pytest

from gpu_util import announce

pytestmark = pytest.mark.gpu

SEED = 20261208


def _with(setter, on, off, call):
    """call with an opt-in mode of the library set around it."""
    def run(g, A, B):
        getattr(g, setter)(on)
        try:
            return call(g, A, B)
        finally:
            getattr(g, setter)(off)
    return run


PRODUCTS = {
    "dgemm": ("float64", lambda g, A, B: g.dgemm(A, B, 18)),
    "noalloc": ("float64", lambda g, A, B: g.dgemm_noalloc(
        A, B, A.new_zeros((B.shape[1], A.shape[0])).t(), 18)),
    "split": ("float64", lambda g, A, B: g.dgemm_split(A, B, 19)),
    "ozi": ("float64", lambda g, A, B: g.dgemm_ozi(A, B, 15)),
    "sgemm": ("float32", lambda g, A, B: g.sgemm(A, B)),
    "igemm": ("int8", lambda g, A, B: g.igemm_s8(A, B)),
    "wide": ("float64", _with("ozfp4_set_max_capacity", 63, 53, lambda g, A, B: g.dgemm(A, B, 23))),
    "heads": ("float64", _with("ozfp4_set_one_limb_moduli", 5, 0, lambda g, A, B: g.dgemm(A, B, 21))),
    "karatsuba": ("float64", _with("ozfp4_set_karatsuba", True, False,
                                   lambda g, A, B: g.dgemm(A, B, 18))),
}


def _forms(X):
    """The matrix X (column-major) in other layouts."""
    import torch
    rows, cols = X.shape
    yield "row", X.contiguous()
    P = torch.zeros((rows, cols + 3), dtype=X.dtype, device=X.device)
    P[:, 1:cols + 1] = X
    yield "row, padded, off by one", P[:, 1:cols + 1]
    Q = torch.zeros((rows, 2 * cols), dtype=X.dtype, device=X.device)
    Q[:, ::2] = X
    yield "every second column", Q[:, ::2]
    Q = torch.zeros((2 * rows, cols), dtype=X.dtype, device=X.device)
    Q[::2] = X
    yield "every second row", Q[::2]
    C = torch.zeros((cols, rows + 5), dtype=X.dtype, device=X.device)
    C[:, 2:rows + 2] = X.t()
    yield "column, padded", C[:, 2:rows + 2].t()


@pytest.mark.parametrize("name", PRODUCTS)
@pytest.mark.parametrize("m,n,k", [(130, 67, 201), (64, 96, 256), (1, 33, 70), (45, 1, 129), (33, 50, 1),
                                   (300, 4, 1500)])
def test_storage_orders_give_the_same_bits(gpu_lib, name, m, n, k):
    import torch
    dtype, call = PRODUCTS[name]
    dtype = getattr(torch, dtype)
    assert gpu_lib.ozfp4_init() == gpu_lib.OZFP4_OK
    gen = torch.Generator().manual_seed(SEED + m + n + k)
    def draw(r, c):
        if dtype == torch.int8:
            return torch.randint(-128, 128, (r, c), generator=gen, dtype=dtype)
        return (torch.rand((r, c), generator=gen, dtype=torch.float64) - 0.5).to(dtype)
    A = gpu_lib.colmajor(draw(m, k).cuda())
    B = gpu_lib.colmajor(draw(k, n).cuda())
    announce(f"layouts {name} m={m} n={n} k={k}")
    want = call(gpu_lib, A, B).clone()
    for label, X in _forms(A):
        assert torch.equal(X, A)
        assert torch.equal(call(gpu_lib, X, B), want), ("A", label)
    for label, Y in _forms(B):
        assert torch.equal(call(gpu_lib, A, Y), want), ("B", label)
    assert torch.equal(call(gpu_lib, A.contiguous(), B.contiguous()), want)
    if m > 1:   # one row repeated: stride 0 along the rows
        E = A[:1].contiguous().expand(m, k)
        assert torch.equal(call(gpu_lib, E, B), call(gpu_lib, gpu_lib.colmajor(E), B))


def test_product_refuses_other_strides(gpu_lib):
    """Refused on the host: the pointers are never read."""
    import torch
    x = torch.zeros(64, dtype=torch.float64, device="cuda")
    p = x.data_ptr()
    f = gpu_lib.ozfp4_product
    for a, b in (((2, 9), (1, 8)), ((1, 3), (1, 8)), ((3, 1), (1, 8)), ((1, 4), (2, 9)), ((1, 4), (0, 1))):
        assert f(0, 4, 4, 8, p, *a, p, *b, p, 4, 18) == gpu_lib.OZFP4_EINVAL, (a, b)
    assert f(6, 4, 4, 8, p, 1, 4, p, 1, 8, p, 4, 18) == gpu_lib.OZFP4_EINVAL
    assert f(0, 4, 4, 8, p, 1, 4, p, 1, 8, p, 3, 18) == gpu_lib.OZFP4_EINVAL
    assert f(0, 4, 4, 8, p, 1, 4, p, 1, 8, p, 4, 0) == gpu_lib.OZFP4_EMODULI
    with pytest.raises(gpu_lib.OzFP4Error) as e:
        gpu_lib.sgemm(x[:16].view(4, 4).float(), x[:16].view(4, 4).float(), 0)
    assert e.value.code == gpu_lib.OZFP4_EMODULI
