"""Generated code of the narrow backward kernels: like the wide ones they issue LDS reads by hand with counted waits, so
a spilled fragment register would store stale data."""
import os
import re
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_narrow_backward_kernels_do_not_spill():
    src = os.path.join(ROOT, "paper_2509_22622_amd", "csrc", "attn_bwd.hip")
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "attn_bwd.s")
        subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang",
                        "-target-feature", "-Xclang", "-packed-fp32-ops", "-S", "--cuda-device-only", src, "-o", out],
                       check=True, capture_output=True)
        text = open(out).read()
    spills = dict(re.findall(r"\.name:\s+(\S+)[\s\S]*?\.vgpr_spill_count:\s+(\d+)", text))
    narrow = {k: int(v) for k, v in spills.items() if "_narrow_kernel" in k}
    assert len(narrow) == 2 and all(v == 0 for v in narrow.values()), f"spills: {narrow}"
