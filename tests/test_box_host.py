"""The box object (csrc/box.hip) when the runtime reports errors, on a stand-in
for the HIP runtime and the kernels' launchers (fake_hip.hpp, box_cases.cpp)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_1601_03815_amd", "csrc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("box") / "cases")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    # the launchers that no case calls stay unresolved
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-D__align__(n)=", "-DHIP_SYMBOL(x)=(x)",
                    "-I" + os.path.join(rocm, "include"), "-x", "c++", os.path.join(HERE, "box_cases.cpp"),
                    os.path.join(CSRC, "box.hip"), "-o", exe, "-lpthread", "-Wl,--unresolved-symbols=ignore-all"],
                   check=True)
    return exe


@pytest.mark.parametrize("case", ["failing_launch", "failing_mesh"])
def test_box_on_errors(program, case):
    r = subprocess.run([program, case], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stderr)
