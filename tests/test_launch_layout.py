"""What the query entry points launch, without a GPU: tests/launch_layout.cpp stands in for the HIP runtime and records the kernels, grids and arguments of
random batches.  A merge reads exactly the partial results that the kernel in front of it writes, and they lie in the workspace that the call asks for."""
import os
import shutil
import subprocess

import pytest

from paper_2502_05431_amd import build as BUILD

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs a host C++ compiler")
    if not os.path.exists(BUILD.LIB):
        BUILD.build(verbose=False)
    exe = str(tmp_path_factory.mktemp("launch") / "launch_layout")
    subprocess.run(["g++", "-O1", "-std=c++17", "-rdynamic", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", os.path.join(BUILD.ROOT, "include"), "-I", BUILD.CSRC,
                    "-o", exe, os.path.join(HERE, "launch_layout.cpp"), "-L", BUILD.PKG, "-lape_hip", "-Wl,-rpath," + BUILD.PKG, "-L/opt/rocm/lib", "-Wl,-rpath,/opt/rocm/lib"], check=True)
    return exe


def test_partial_results_of_random_batches(recorder):
    out = subprocess.run([recorder], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout + out.stderr
    assert int(out.stdout.split(",")[1].split()[0]) > 100     # a call's last launch of one request that is dealt out: reached
