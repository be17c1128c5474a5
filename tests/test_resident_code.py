"""Generated code of the resident-key attention kernels: their keys and values go to LDS by loads that the compiler does not
count as writes of it, so every wave has to wait for its own (vmcnt(0)) before the barrier behind which all waves read."""
import os
import re
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_direct_to_lds_loads_have_landed_at_the_barrier():
    src = os.path.join(ROOT, "paper_2509_22622_amd", "csrc", "attn_resident.hip")
    assert re.search(r"s_waitcnt\([^;]*;[^\n]*\n\s*__syncthreads", open(src).read()), "the wait is the compiler's choice"
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "attn_resident.s")
        subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang",
                        "-target-feature", "-Xclang", "-packed-fp32-ops", "-S", "--cuda-device-only", src, "-o", out],
                       check=True, capture_output=True)
        text = open(out).read()
    kernels = re.findall(r"^(_ZN2ll\d+ll_attn_resident_kernel\S+):(.*?)^\s*s_endpgm", text, re.M | re.S)
    assert len(kernels) == 4
    for name, body in kernels:
        code = [line.split(";")[0].strip() for line in body.splitlines()]
        to_lds = [i for i, line in enumerate(code) if line.startswith("global_load_lds")]
        barrier = next(i for i in range(to_lds[-1], len(code)) if code[i].startswith("s_barrier"))
        between = code[to_lds[-1]:barrier]
        assert any(re.match(r"s_waitcnt (.*\s)?vmcnt\(0\)", line) for line in between), name
        assert not any(line.startswith("ds_read") for line in between), name


def test_resident_kernels_do_not_spill():
    """They issue LDS reads by hand, ahead of their MFMAs: a spilled fragment register would store stale data, and a scalar load among
    them would be counted with them."""
    src = os.path.join(ROOT, "paper_2509_22622_amd", "csrc", "attn_resident.hip")
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "attn_resident.s")
        subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang",
                        "-target-feature", "-Xclang", "-packed-fp32-ops", "-S", "--cuda-device-only", src, "-o", out],
                       check=True, capture_output=True)
        text = open(out).read()
    spills = dict(re.findall(r"\.name:\s+(\S+)[\s\S]*?\.vgpr_spill_count:\s+(\d+)", text))
    ours = {k: int(v) for k, v in spills.items() if "ll_attn_resident_kernel" in k}
    assert len(ours) == 4 and all(v == 0 for v in ours.values()), f"spills: {ours}"
    for body in re.findall(r"^_ZN2ll\d+ll_attn_resident_kernel\S+:(.*?)^\s*s_endpgm", text, re.M | re.S):
        steps = [block for block in re.split(r"^\.LBB", body, flags=re.M) if "lgkmcnt(3)" in block]
        assert steps and not any("s_load" in block for block in steps)
