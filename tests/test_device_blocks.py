"""Device blocks that contexts keep between calls, on a stand-in for the HIP runtime
(device_blocks.cpp): CPU only."""

import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(os.path.dirname(HERE), "paper_2303_05883_amd")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("blocks") / "device_blocks")
    subprocess.run(["g++", "-std=c++17", "-O1", "-rdynamic", os.path.join(HERE, "device_blocks.cpp"), "-o", exe,
                    os.path.join(PKG, "liblqcd.so"), "-Wl,-rpath," + PKG, "-Wl,--allow-shlib-undefined"], check=True)
    return exe


@pytest.mark.parametrize("case", ["no_heap", "failed_copy", "reclaim", "bound"])
def test_case(program, case):
    r = subprocess.run([program, case], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
