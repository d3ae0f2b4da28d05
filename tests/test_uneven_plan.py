"""The split plans of uneven batches (csrc/ape_plan.h) compile for the host, and tests/plan_deal.cpp drives them: every request is covered by
splits of its own within the even plan's workspace, and a decode step goes out in more launches than its requests need only where each of
them is dealt out."""
import os
import shutil
import subprocess

import pytest

from paper_2502_05431_amd import build as BUILD

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host C++ compiler")
def test_plans(tmp_path):
    exe = str(tmp_path / "plan_deal")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-I", BUILD.CSRC,
                    "-o", exe, os.path.join(HERE, "plan_deal.cpp")], check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout + out.stderr
