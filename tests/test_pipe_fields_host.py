"""Host check of the pipelined W4A4 kernel's stores for activations in field form (tests/host/pipe_fields_map.cpp)."""
import os
import shutil
import subprocess

import pytest

from paper_2605_16732_amd import build as BLD

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_stage_of_field_form(tmp_path):
    cxx = shutil.which("g++") or shutil.which("clang++") or "/opt/rocm/lib/llvm/bin/clang++"
    if not os.path.exists(cxx):
        pytest.skip("no host compiler")
    exe = str(tmp_path / "map")
    subprocess.run([cxx, "-O2", "-std=c++17", "-I", BLD.CSRC, os.path.join(ROOT, "tests", "host", "pipe_fields_map.cpp"), "-o", exe],
                   check=True, capture_output=True)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0 and run.stdout.startswith("0 failure(s)"), run.stdout
