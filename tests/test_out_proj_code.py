"""Generated code of the output projection: it issues its LDS reads by hand, a k-step ahead, so a spilled fragment register
would store stale data."""
import os
import re
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_projection_kernels_do_not_spill():
    src = os.path.join(ROOT, "paper_2509_22622_amd", "csrc", "out_proj.hip")
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "out_proj.s")
        subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang",
                        "-target-feature", "-Xclang", "-packed-fp32-ops", "-S", "--cuda-device-only", src, "-o", out],
                       check=True, capture_output=True, text=True)
        text = open(out).read()
    spills = dict(re.findall(r"\.name:\s+(\S+)[\s\S]*?\.vgpr_spill_count:\s+(\d+)", text))
    ours = {k: int(v) for k, v in spills.items() if "ll_out_proj_kernel" in k}
    assert len(ours) == 4 and all(v == 0 for v in ours.values()), f"spills: {ours}"
