"""Generated code of the attention kernels for narrow (8-bit cache) and for split tiles: like the others they issue LDS reads by hand
with counted waits, so a spilled fragment register would store stale data."""
import functools
import os
import re
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@functools.lru_cache(None)
def _assembly(source):
    src = os.path.join(ROOT, "paper_2509_22622_amd", "csrc", source)
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "kernels.s")
        subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang",
                        "-target-feature", "-Xclang", "-packed-fp32-ops", "-S", "--cuda-device-only", src, "-o", out],
                       check=True, capture_output=True, text=True)
        return open(out).read()


def _spills(source):
    return {k: int(v) for k, v in re.findall(r"\.name:\s+(\S+)[\s\S]*?\.vgpr_spill_count:\s+(\d+)", _assembly(source))}


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


def test_a_touch_is_the_last_load_before_the_wait_that_leaves_it_out():
    """Kblocks brought into L2 ahead: a hand-over's wait leaves the touch (the kernels' only 4-byte load to LDS) in flight and counts
    loads in the order of their issue, so it must be the wave's last one.  Both stand in the source behind a statement that
    no load may be moved across; the generated code has nothing but address arithmetic between them, in one block."""
    kernels = re.findall(r"^(_ZN2ll\d+ll_attn_\S+):(.*?)^\s*s_endpgm", _assembly("attn_stream16.hip"), re.M | re.S)
    touching = {name: body for name, body in kernels if re.search(r"global_load_lds_dword\s", body)}
    assert len(touching) == 3
    for name, body in touching.items():
        lines = [line.strip() for line in body.splitlines()]
        waits = [i for i, line in enumerate(lines) if line == "s_waitcnt vmcnt(1)" and lines[i - 1].endswith("ASMSTART")]
        assert len(waits) == len(re.findall(r"global_load_lds_dword\s", body)) - 1, name       # but for the one in front of the first step
        for i in waits:
            last = next(j for j in range(i - 1, 0, -1) if re.match(r"(global|buffer|flat|scratch)_|\.L", lines[j]))
            assert lines[last].startswith("global_load_lds_dword "), (name, lines[last])
            fence = max(j for j in range(last) if lines[j].endswith("ASMEND"))
            assert lines[fence - 1].endswith("ASMSTART"), (name, lines[fence - 1])               # the empty statement
            assert not any(re.match(r"(global|buffer|flat|scratch|ds)_|\.L", line) for line in lines[fence:last]), name
