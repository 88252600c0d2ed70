"""The library's dispatch rules (paper_2608_06812_amd/csrc/routes.hpp) on the
host: which GEMM a product takes and in how many k ranges, for the tests whose
sizes are chosen to reach one of them."""

import os
import shutil
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
_exe = None


def _binary():
    global _exe
    if _exe is None:
        gxx = shutil.which("g++")
        if gxx is None:
            pytest.skip("no host C++ compiler")
        out = os.path.join(tempfile.mkdtemp(prefix="routes"), "routes_host")
        subprocess.run([gxx, "-O1", "-std=c++17", "-Wall", "-Wextra", "-Werror",
                        "-I", os.path.join(ROOT, "paper_2608_06812_amd", "csrc"),
                        os.path.join(ROOT, "tests", "routes_host.cpp"), "-o", out], check=True)
        _exe = out
    return _exe


def routes(queries):
    """One answer per query tuple: ("res", m, n, k, nmod, nprod) -> (kernel,
    ranges, moduli a block), ("s8", m, n, k) -> (kernel, ranges), ("ozi", m,
    n, k, nh) -> (kernel,)."""
    text = "\n".join(" ".join(str(v) for v in q) for q in queries) + "\n"
    run = subprocess.run([_binary()], input=text, capture_output=True, text=True, check=True)
    out = []
    for line in run.stdout.splitlines():
        kernel, *counts = line.split()
        out.append((kernel, *(int(c) for c in counts)))
    assert len(out) == len(queries)
    return out


def longest_range(k, ranges):
    """k of the longest of `ranges` ranges, in whole 64-wide stages."""
    nst = (k + 63) // 64
    return 64 * max(nst * (p + 1) // ranges - nst * p // ranges for p in range(ranges))
