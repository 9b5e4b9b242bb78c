"""The halo protocol of the split SAP phase kernel with the copies on a wave of their own
(tests/host/parts_protocol_wave.cpp): updates of single sites and copies of single words of a step
in any order, bit for bit against the unsplit sweeps (no GPU)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_parts_protocol_wave(tmp_path):
    exe = tmp_path / "parts_protocol_wave"
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-o", str(exe), os.path.join(HERE, "host", "parts_protocol_wave.cpp")])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout + out.stderr
    assert "all protocol cases agree" in out.stdout
