"""Generated code of the attention kernels for narrow (8-bit cache) and for split tiles: like the others they issue LDS reads by hand
with counted waits, so a spilled fragment register would store stale data."""
import os
import re
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _spills(source):
    src = os.path.join(ROOT, "paper_2509_22622_amd", "csrc", source)
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "kernels.s")
        subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang",
                        "-target-feature", "-Xclang", "-packed-fp32-ops", "-S", "--cuda-device-only", src, "-o", out],
                       check=True, capture_output=True, text=True)
        text = open(out).read()
    return {k: int(v) for k, v in re.findall(r"\.name:\s+(\S+)[\s\S]*?\.vgpr_spill_count:\s+(\d+)", text)}


def test_narrow_and_split_kernels_do_not_spill():
    ours = {k: v for k, v in _spills("attn_fp8.hip").items() if "ll_attn_fp8_kernel" in k and any(f"ELi{m}E" in k for m in (3, 4, 5, 6))}
    assert len(ours) == 8 and all(v == 0 for v in ours.values()), f"spills: {ours}"


def test_bf16_split_kernels_do_not_spill():
    """The merges' too, with their loop over a tile's shares."""
    ours = {k: v for k, v in _spills("attn_stream16.hip").items() if "ll_attn_split16_kernel" in k or "ll_attn_merge16_kernel" in k}
    assert len(ours) == 42 and all(v == 0 for v in ours.values()), f"spills: {ours}"


def test_key_group_kernels_do_not_spill():
    """The 8-bit kernels whose tiles' keys are dealt to groups of waves."""
    ours = {k: v for k, v in _spills("attn_fp8.hip").items() if "ll_attn_fp8_kernel" in k and "ELi7E" in k}
    assert len(ours) == 2 and all(v == 0 for v in ours.values()), f"spills: {ours}"
