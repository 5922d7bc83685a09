"""The sweep's host-side plan (paper_2502_20610_amd/csrc/sweep_plan.cpp) under
the address and undefined-behaviour sanitizers: tiles cover the grid, and the
progress marks held cover every block of every pass in every coefficient mode."""
import os
import shutil
import subprocess

import pytest

from tests.test_sanitizers_cpu import ROOT, SAN, _run

CSRC = os.path.join(ROOT, "paper_2502_20610_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_sweep_plan_under_address_and_undefined_sanitizers(tmp_path):
    exe = str(tmp_path / "sweep_check")
    subprocess.run(["g++", "-std=c++17"] + SAN + ["-I" + CSRC, os.path.join(CSRC, "sweep_plan.cpp"),
                    os.path.join(ROOT, "tests", "sanitize", "sweep_check.cpp"), "-o", exe], check=True)
    assert "sweep plan checks passed" in _run(exe)


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_ring_distance_bound_under_address_and_undefined_sanitizers(tmp_path):
    exe = str(tmp_path / "ring_check")
    subprocess.run(["g++", "-std=c++17"] + SAN + ["-I" + CSRC, os.path.join(CSRC, "plan.cpp"),
                    os.path.join(ROOT, "tests", "sanitize", "ring_check.cpp"), "-o", exe], check=True)
    assert "ring checks passed" in _run(exe)


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_array_ranges_under_address_and_undefined_sanitizers(tmp_path):
    exe = str(tmp_path / "ranges_check")
    subprocess.run(["g++", "-std=c++17"] + SAN + ["-I" + CSRC, os.path.join(ROOT, "tests", "sanitize", "ranges_check.cpp"),
                    "-o", exe], check=True)
    assert "range checks passed" in _run(exe)
