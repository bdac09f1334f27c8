"""Host: an adjoint run whose graphs cannot be instantiated falls back to launches
and reads the same tape.

The host side of the library is compiled with the host compiler against a device
made of host memory (tests/host/stub_device.cc), in which no captured graph
instantiates.  The adjoint steps then have to read the tape entries of the states
T - 1, T - 2, ..., 0, whatever number of launches a segment takes.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1008_2865_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    exe = str(tmp_path_factory.mktemp("host") / "stub_device")
    subprocess.run([cxx, "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-x", "c++", os.path.join(CSRC, "lb_api.hip"),
                    os.path.join(ROOT, "tests", "host", "stub_device.cc"),
                    # What the adjoint does not call stays undefined.
                    "-Wl,--unresolved-symbols=ignore-all", "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("every", [3, 4, 5, 6, 10, 15, 25])
def test_backward_reads_the_tape_of_every_state(program, every):
    T = 3 * every + 1
    run = subprocess.run([program, "32", str(T), str(every)], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0, run.stderr
    tried, *levels = [float(v) for v in run.stdout.split()]
    assert tried == 1  # one attempt, launches from then on
    assert levels == list(range(T - 1, -1, -1))
