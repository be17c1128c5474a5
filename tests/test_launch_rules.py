"""Rules by which a launch's sizes select its kernel, checked on the host over their whole range (check_launch_rules.cpp)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_launch_rules(tmp_path):
    exe = tmp_path / "check_launch_rules"
    subprocess.run(["g++", "-std=c++17", "-O1", "-o", str(exe), os.path.join(HERE, "check_launch_rules.cpp")], check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout + run.stderr
    assert "launch rules ok" in run.stdout
