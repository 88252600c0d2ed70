"""The dispatch rules on the host: the bounds that the kernels' exactness and
launches rest on, over random sizes, and that the GPU tests written for one
route still take it."""

import random

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
