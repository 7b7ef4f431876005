"""The library's host code -- scratch, pools, launches -- against a stand-in for
the HIP runtime (tests/host), where no kernel runs and memory that has been freed
is known.  Runs on the CPU."""
import os
import re
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
PKG = os.path.join(ROOT, "paper_1705_09905_amd")
SRC = os.path.join(HERE, "host", "checks.cpp")
NAMES = re.findall(r'^ +\{"(\w+)", \[\]', open(SRC).read(), re.M)


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "checks")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(PKG, "csrc"), "-I", "/opt/rocm/include", SRC, "-o", exe, "-rdynamic",
                    os.path.join(PKG, "libfcoo.so"), "-Wl,-rpath," + PKG, "-L/opt/rocm/lib",
                    "-Wl,-rpath-link,/opt/rocm/lib", "-Wl,-rpath,/opt/rocm/lib"], check=True)
    return exe


@pytest.mark.parametrize("name", NAMES)
def test_host(program, name):
    r = subprocess.run([program, name], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr
