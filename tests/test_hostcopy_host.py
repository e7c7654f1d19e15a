"""The copies of results to the host (csrc/hostcopy.hip) on a stand-in for the
HIP runtime (fake_hip.hpp): what one GPU cannot show, and what it must not."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_1601_03815_amd", "csrc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("hostcopy") / "cases")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(rocm, "include"), "-x", "c++",
                    os.path.join(HERE, "hostcopy_cases.cpp"), os.path.join(CSRC, "hostcopy.hip"), "-o", exe, "-lpthread"],
                   check=True)
    return exe


@pytest.mark.parametrize("case", ["two_devices", "known_destinations", "per_thread_stream", "out_of_memory", "box_at_exit", "phases"])
def test_copies_to_the_host(program, case):
    r = subprocess.run([program, case], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stderr)
