"""The host runtime on a device made of host memory (tests/c_abi/host_fake.cpp): what a handle's
options do to the tables that its launches read."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host_fake") / "host_fake")
    pkg = os.path.join(ROOT, "paper_2208_14228_amd", "csrc")
    subprocess.check_call(["g++", "-O1", "-g", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"),
                           "-I", pkg, "-I", "/opt/rocm/include", os.path.join(HERE, "c_abi", "host_fake.cpp"),
                           os.path.join(pkg, "es_api.cpp"), "-o", exe])
    return exe


@pytest.mark.parametrize("what", ["options", "auto", "host slots", "rule", "masks", "norms", "many", "no memory"])
def test_handle(program, what):
    out = subprocess.run([program, what], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and f"{what}: passed" in out.stdout, out.stdout + out.stderr
