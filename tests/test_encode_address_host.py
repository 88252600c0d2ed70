"""Host build of the scheme-II encoder's table addresses
(paper_2608_06812_amd/csrc/encode_address.hpp) under UBSan: every 16-bit
quotient and every table remainder of every modulus has to give the entry's
address, with no undefined operation on the way."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "encode_address_host.cpp")
INC = os.path.join(ROOT, "paper_2608_06812_amd", "csrc")


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    # clang: g++ narrows the arithmetic before its sanitizer looks at it
    clang = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "clang++")
    if not os.path.exists(clang):
        clang = shutil.which("clang++")
    if clang is None:
        pytest.skip("no clang")
    out = str(tmp_path_factory.mktemp("addr") / "encode_address_host")
    subprocess.run([clang, "-O2", "-std=c++17", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                    "-I", INC, SRC, "-o", out], check=True)
    return subprocess.run([out], capture_output=True, text=True)


def test_every_address_is_its_entry(run):
    assert run.returncode == 0, run.stdout + run.stderr
    assert int(run.stdout) > 4 * 27 * 65536 * 7      # every quotient of every modulus and list
