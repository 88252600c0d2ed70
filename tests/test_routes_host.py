"""The dispatch rules on the host: the bounds that the kernels' exactness and
launches rest on, over random sizes, and that the GPU tests written for one
route still take it."""

import random

import test_gpu_exactness_limits as limits
import test_gpu_long_gemm as long_gemm
import test_gpu_short_gemm as short_gemm
from route_util import longest_range, routes


def _sizes(rng, count, top):
    log = lambda hi: int(round(2 ** rng.uniform(0, hi)))
    return [(log(15.3), log(15.3), log(top)) for _ in range(count)]


def test_ranges_stay_within_their_bounds():
    rng = random.Random(20261211)
    sizes = _sizes(rng, 4000, 17)
    mods = [(rng.randint(1, 27), rng.choice((1, 4))) for _ in sizes]
    for (m, n, k), (nmod, nprod), (kernel, ranges, group) in zip(
            sizes, mods, routes([("res", *s, *q) for s, q in zip(sizes, mods)])):
        assert 1 <= ranges <= 16                  # byte sums of residues: 16 * 255 < 2^16
        assert 1 <= group <= nmod
        assert ranges == 1 or k // 64 + 1 >= 8 * ranges
        if kernel == "long":                      # the long GEMM has no ranges
            assert k > 6144 and ranges == 1
    sizes = _sizes(rng, 4000, 24)
    for (m, n, k), (kernel, ranges) in zip(sizes, routes([("s8", *s) for s in sizes])):
        assert 1 <= ranges <= 16
        if kernel == "short":                     # 192 k < 2^23
            assert longest_range(k, ranges) <= 40960
    sizes = _sizes(rng, 4000, 17)
    for (m, n, k), (kernel,) in zip(sizes, routes([("ozi", *s, 9) for s in sizes])):
        assert kernel == "long" or k <= 8192      # 960 k < 2^23


def test_limit_cases_reach_their_kernel_in_one_range():
    want = [kernel for *_, kernel in limits.RESIDUES]
    got = routes([("res", m, n, k, L, 1) for m, n, k, L, _ in limits.RESIDUES])
    assert got == [(kernel, 1, 1) for kernel in want]
    assert routes([("s8", m, n, k) for m, n, k, _ in limits.INT8]) == \
        [(kernel, 1) for *_, kernel in limits.INT8]
    assert routes([("ozi", *limits.OZI, 9)]) == [("short",)]


def test_cases_of_the_residue_gemms_take_their_route():
    ask = lambda cases: routes([("res", *c[:4], 1) for c in cases])
    assert ask(short_gemm.RANGES) == [("short", c[5], 1) for c in short_gemm.RANGES]
    assert {r[:2] for r in ask(short_gemm.CASES)} == {("short", 1)}
    assert all(kernel == "short" and group > 1 for kernel, _, group in ask(short_gemm.GROUPED))
    assert {r[0] for r in ask(long_gemm.CASES)} == {"long"}
