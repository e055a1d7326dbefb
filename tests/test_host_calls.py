"""Whole calls of the C ABI without a GPU: the library's host code on a HIP
runtime that launches nothing (tests/fake_hip.cpp), which shows what each call
waits for and how much scratch it asks for."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(os.path.dirname(HERE), "paper_2310_15235_amd")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("host_calls") / "host_calls")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-rdynamic",
                           os.path.join(HERE, "host_calls_main.cpp"),
                           os.path.join(HERE, "fake_hip.cpp"), "-L", PKG, "-ltrevr2",
                           "-Wl,-rpath," + PKG, "-Wl,--allow-shlib-undefined", "-o", exe])
    return exe


@pytest.mark.parametrize("case", ["stream_order", "kept_depths", "adjoint_room", "adjoint_estimate"])
def test_host_calls(program, case):
    r = subprocess.run([program, case], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
