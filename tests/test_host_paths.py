"""The library's host code on a fake HIP runtime over host memory
(native/fake_hip.hpp): paths that a healthy device does not take, and what
happens to results, blocks and errors there.  No kernel runs."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2403_08692_amd", "libvsh.so")
NATIVE = os.path.join(ROOT, "tests", "native")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not os.path.exists(LIB):
        pytest.skip("libvsh.so is not built (run __graft_entry__.build())")
    exe = str(tmp_path_factory.mktemp("host") / "host_paths")
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"), "-I" + NATIVE, os.path.join(NATIVE, "host_paths.cpp"),
                    "-o", exe, "-rdynamic", "-pthread", LIB, "-Wl,-rpath," + os.path.dirname(LIB),
                    "-Wl,--allow-shlib-undefined"], check=True)
    return exe


@pytest.mark.parametrize("scenario", ["forked child", "serving, little memory", "failing calls", "no device address",
                                      "result beyond the pool", "no host memory", "waves of small launches"])
def test_host_path(program, scenario):
    r = subprocess.run([program, scenario], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
