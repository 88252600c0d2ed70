"""GPU limb planes at the values where the encoder's quotient is least exact:
integers next to multiples and half-multiples of every modulus, of every
size up to the capacity and both signs, through each encoder (greedy list,
one-limb heads, Karatsuba mode, capacities above 53 bits). Codes against the
oracle's planes."""

import numpy as np
import pytest

import oracle as o
from gpu_util import announce, dev_cm, oracle_plane_codes, to_np, unpack_planes

pytestmark = pytest.mark.gpu

SEED = 20261209


def _values(moduli, bits, count, rng):
    """`count` exact doubles, integers below 2^bits in magnitude (multiples of
    2^(bits - 53) above 2^53): q m + r around multiples and half-multiples."""
    out = [2 ** bits - 2 ** max(0, bits - 53), 0, 1, -1]
    while len(out) < count:
        m = int(rng.choice(moduli))
        size = int(rng.integers(8, bits))
        q = int(rng.integers(0, 1 << 62)) % max(1, (1 << size) // m)
        v = q * m + int(rng.choice([-1, 0, 1, m // 2, m // 2 + 1, (m + 1) // 2 - 1]))
        v = int(float(v))                      # rounded to a double above 2^53
        if abs(v) < 2 ** bits:
            out.append(v if rng.random() < 0.5 else -v)
    return np.array([float(v) for v in out[:count]])


@pytest.mark.parametrize("mode,L,k", [("greedy", 19, 96), ("greedy", 27, 96), ("heads", 21, 96),
                                      ("karatsuba", 19, 96), ("wide", 24, 96)])
def test_planes_at_extreme_values(gpu_lib, mode, L, k):
    rng = np.random.default_rng(SEED)
    lines = 70
    try:
        if mode == "heads":
            gpu_lib.ozfp4_set_one_limb_moduli(5)
        elif mode == "karatsuba":
            gpu_lib.ozfp4_set_karatsuba(True)
        elif mode == "wide":
            gpu_lib.ozfp4_set_max_capacity(63)
        moduli = gpu_lib.ozfp4_moduli(L)
        cA, cB = gpu_lib.ozfp4_capacity(k, L)
        assert min(cA, cB) >= 53 and (mode != "wide" or cB > 53)
        # a line's first value is its largest, below 2^c, so its shift is 0
        A = np.stack([_values(moduli, cA, k, rng) for _ in range(lines)])
        B = np.stack([_values(moduli, cB, k, rng) for _ in range(lines)]).T
        announce(f"extreme values {mode} L={L}")
        pa, pb = gpu_lib.limb_planes(dev_cm(A), dev_cm(B), L)
        rows_pad, k_pad, _ = gpu_lib.ozfp4_plane_layout(lines, k)
        got_a, got_b = (unpack_planes(to_np(p), rows_pad, k_pad) for p in (pa, pb))
    finally:
        gpu_lib.ozfp4_set_one_limb_moduli(0)
        gpu_lib.ozfp4_set_karatsuba(False)
        gpu_lib.ozfp4_set_max_capacity(53)
    Ai = np.array([[int(v) for v in row] for row in A], dtype=object)
    Bi = np.array([[int(v) for v in row] for row in B.T], dtype=object)
    if mode == "heads":
        tables = [_table(gpu_lib, l) for l in range(L)]
        for got, Xi in ((got_a, Ai), (got_b, Bi)):
            for l, m in enumerate(moduli):
                r = np.array([[int(v) % m for v in row] for row in Xi])
                code = np.asarray(tables[l])[r]
                assert np.array_equal(got[2 * l][:lines, :k], code & 0xF), m
                assert np.array_equal(got[2 * l + 1][:lines, :k], code >> 4), m
    else:
        for got, Xi in ((got_a, Ai), (got_b, Bi)):
            want = oracle_plane_codes(Xi, moduli, rows_pad, k_pad, karatsuba=mode == "karatsuba")
            assert np.array_equal(got, want)


def _table(lib, l):
    """Codes of every residue of modulus l (c0 in the low nibble), from the
    library's table, which the host tests check against the oracle."""
    lib.ozfp4_set_one_limb_moduli(5)
    try:
        m, codes = lib.ozfp4_two_limb_table(l)
    finally:
        lib.ozfp4_set_one_limb_moduli(0)
    assert len(codes) == m
    return np.frombuffer(codes, dtype=np.uint8)
