"""A call with splits whose second launch fails (check_split_failure.cpp): on the CPU, with stand-ins for the runtime."""
import os
import subprocess

import pytest

from paper_2509_22622_amd import binding as B

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no ROCm toolchain")
def test_slots_are_given_back_when_the_merge_is_not_launched(tmp_path):
    assert os.path.exists(B.LIB_PATH)
    exe = tmp_path / "check_split_failure"
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-rdynamic", "-Wno-unused-command-line-argument",
                    os.path.join(HERE, "check_split_failure.cpp"), "-ldl", "-o", str(exe)], check=True, capture_output=True, text=True)
    run = subprocess.run([str(exe), B.LIB_PATH], capture_output=True, text=True)
    assert run.returncode == 0 and "slots given back" in run.stdout, run.stdout + run.stderr
