"""Calls whose kernel launches fail, on the CPU with a stand-in for the HIP
runtime (tests/launch_errors_host.cpp): a call that ends early with its line
maxima still queued must not hand its non-finite flag to the next call, at
any entry point and whichever launch fails, and calls that end normally wait
for their stream only."""

import os
import shutil
import subprocess

import pytest

from paper_2608_06812_amd import ozfp4

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def test_a_failed_call_leaves_no_flag_behind(tmp_path):
    if not os.path.exists(ozfp4.LIB_PATH):
        from paper_2608_06812_amd import build
        build.build()
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    exe, libdir = str(tmp_path / "launch_errors_host"), os.path.dirname(ozfp4.LIB_PATH)
    subprocess.run([gxx, "-O1", "-std=c++17", "-rdynamic", "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "launch_errors_host.cpp"), "-L", libdir, "-lozfp4",
                    f"-Wl,-rpath,{libdir}", f"-Wl,-rpath,{os.path.join(ROCM, 'lib')}",
                    "-Wl,--allow-shlib-undefined", "-o", exe], check=True, timeout=120)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout + run.stderr
    assert int(run.stdout) >= 30       # every launch of ten entry points failed once
