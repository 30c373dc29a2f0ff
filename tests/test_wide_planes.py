"""The four-wide nodes' FP16 planes on the CPU: outward rounding over every
FP16 value and random FP32 ones, containment of the FP32 boxes."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = "/opt/rocm/bin/hipcc"


def test_planes_round_outwards(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "planes")
    b = subprocess.run([HIPCC, "--offload-host-only", "-std=c++17", "-O2", "-x", "hip", "-o", exe,
                        os.path.join(HERE, "wide_planes_driver.cpp")], capture_output=True, text=True, timeout=300)
    assert b.returncode == 0, b.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:]
