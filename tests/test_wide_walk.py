"""Slab parameters of the four-wide walk on the CPU: no rounding of the box tests
enters a box late or leaves it early."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = "/opt/rocm/bin/hipcc"


def _run(tmp_path, driver):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "driver")
    # -ffp-contract=off: the chain's own fused multiply-adds are written out
    b = subprocess.run([HIPCC, "--offload-host-only", "-std=c++17", "-O2", "-ffp-contract=off", "-x", "hip", "-o", exe,
                        os.path.join(HERE, driver)], capture_output=True, text=True, timeout=300)
    assert b.returncode == 0, b.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:]


def test_slabs_are_conservative(tmp_path):
    _run(tmp_path, "wide_walk_driver.cpp")


def test_units_contain_and_are_conservative(tmp_path):
    _run(tmp_path, "wide_units_driver.cpp")


def test_hierarchy_checks_refuse_planted_mistakes(tmp_path):
    _run(tmp_path, "hierarchy_check_driver.cpp")
