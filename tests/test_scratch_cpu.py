"""The scratch kept between calls (tx_scratch.cpp), compiled for the host over a
simulated runtime (scratch_host/): which buffers are handed out again, and what
happens where memory, events or slots run out.  No GPU is needed."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SOURCE = os.path.join(HERE, "..", "paper_2401_13834_amd", "csrc", "tx_scratch.cpp")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if not cxx:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path_factory.mktemp("scratch") / "driver")
    stub = os.path.join(HERE, "scratch_host")
    subprocess.run([cxx, "-std=c++17", "-O1", "-g", "-Wall", "-pthread", "-I", stub, os.path.join(stub, "driver.cpp"), SOURCE,
                    "-o", exe], check=True, timeout=120)
    return exe


@pytest.mark.parametrize("check", ["reuse", "lost", "memory", "room", "locks", "error"])
def test_kept_scratch(driver, check):
    r = subprocess.run([driver, check], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
