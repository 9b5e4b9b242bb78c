"""Host logic of the choice between two and four lanes per site (tests/host/alone_rule.cpp; no GPU)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_alone_rule(tmp_path):
    exe = tmp_path / "alone_rule"
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-o", str(exe), os.path.join(HERE, "host", "alone_rule.cpp")])
    assert subprocess.run([str(exe)], timeout=60).returncode == 0
