"""Host code of the library without a GPU: each tests/host/test_*.cpp is a program that links
libsparc_hip.so under a stand-in for the HIP runtime (tests/host/fake_hip.hpp), which records
launches, streams and allocations and runs no kernel.  A program ends with status 0, or prints
the line of the check that failed."""
import glob
import os
import subprocess

import pytest

from paper_1603_04339_amd import sparc as sp

HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "host")
ROOT = os.path.dirname(os.path.dirname(HERE))
PKG = os.path.join(ROOT, "paper_1603_04339_amd")
PROGRAMS = sorted(os.path.basename(p)[5:-4] for p in glob.glob(os.path.join(HERE, "test_*.cpp")))


@pytest.mark.parametrize("name", PROGRAMS)
def test_host_code(name, tmp_path):
    sp.load()   # says how to build it where none is built
    exe = str(tmp_path / name)
    cmd = ["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
           "-I" + os.path.join(ROOT, "include"), os.path.join(HERE, f"test_{name}.cpp"), "-o", exe,
           "-L" + PKG, "-l:libsparc_hip.so", "-Wl,-rpath," + PKG, "-Wl,-rpath,/opt/rocm/lib",
           "-L/opt/rocm/lib", "-lamdhip64", "-rdynamic"]
    built = subprocess.run(cmd, capture_output=True, text=True)
    assert built.returncode == 0, built.stderr
    ran = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert ran.returncode == 0, ran.stdout + ran.stderr
