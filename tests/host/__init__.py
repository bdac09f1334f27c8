"""The library's host side on a device made of host memory, as a program."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
CSRC = os.path.join(ROOT, "paper_1008_2865_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def build(folder):
    """The program of stub_device.cc, built with the host compiler."""
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    exe = os.path.join(str(folder), "stub_device")
    subprocess.run([cxx, "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-x", "c++", os.path.join(CSRC, "lb_api.hip"),
                    os.path.join(ROOT, "tests", "host", "stub_device.cc"),
                    # What the program does not call stays undefined.
                    "-Wl,--unresolved-symbols=ignore-all", "-o", exe], check=True)
    return exe


def run(exe, *args):
    """The program's output lines."""
    done = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=60)
    assert done.returncode == 0, done.stderr
    return done.stdout.splitlines()
