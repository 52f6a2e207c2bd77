"""Host checks of the pipelined W4A4 kernel's plain C++ parts.  Its LDS stage layout (tests/host/pipe_stage_map.cpp): every
byte that is read has one writer among a workgroup's threads, and the reader finds the channels that it expects.  Its
split of the tokens between two tile sizes (tests/host/pipe_plan_walk.cpp): the plan of the walk over every split."""
import os
import shutil
import subprocess

import pytest

from paper_2605_16732_amd import build as BLD

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("name", ["pipe_stage_map", "pipe_plan_walk"])
def test_host_check(name, tmp_path):
    cxx = shutil.which("g++") or shutil.which("clang++") or "/opt/rocm/lib/llvm/bin/clang++"
    if not os.path.exists(cxx):
        pytest.skip("no host compiler")
    exe = str(tmp_path / name)
    subprocess.run([cxx, "-O2", "-std=c++17", "-I", BLD.CSRC, os.path.join(ROOT, "tests", "host", name + ".cpp"), "-o", exe],
                   check=True, capture_output=True)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0 and run.stdout.startswith("0 failure(s)"), run.stdout
