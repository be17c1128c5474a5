"""Rules by which a launch's sizes select its kernel, checked on the host over their whole range (check_launch_rules.cpp, and through
the library's host calls)."""
import ctypes as C
import os
import random
import shutil
import subprocess

import pytest

from paper_2509_22622_amd import binding as B

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_launch_rules(tmp_path):
    exe = tmp_path / "check_launch_rules"
    subprocess.run(["g++", "-std=c++17", "-O1", "-o", str(exe), os.path.join(HERE, "check_launch_rules.cpp")], check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout + run.stderr
    assert "launch rules ok" in run.stdout


def test_rules_of_launches_of_several_chunks():
    """Four key groups of an 8-bit re-prefill: one round of 64-row tiles, key sets of 7 to 64 kblocks.  A clip's split last round: equal
    chunks only, no more tiles than leave the full rounds full, all shares in one round.  Over seeded random launches, and at the edges."""
    rng = random.Random(11)
    dealt = split = 0
    for _ in range(3000):
        heads, head_dim, n = rng.randint(1, 24), rng.choice([64, 128]), rng.randint(1, 24)
        rows = rng.choice([rng.randint(1, 300), rng.randint(1, 5000)])
        longest = rng.choice([6, 7, 64, 65, rng.randint(1, 80)])
        chunks = [(rows, max(1, longest - i * rng.randint(0, 3))) for i in range(n)]
        if B.attn_key_groups_fp8(head_dim, heads, chunks) == 4:
            dealt += 1
            assert sum(-(-r // 64) for r, _ in chunks) * heads <= 256 and 7 <= max(k for _, k in chunks) <= 64
        base = rng.randint(16, 800)
        chunks = [(rows, base + rng.randint(0, 2 if rng.random() < 0.8 else 3)) for _ in range(n)]
        tiles, splits = B.attn_clip_tail(head_dim, heads, chunks)
        if tiles == 0:
            assert splits == 1
            continue
        split += 1
        per_head = sum(-(-r // 256) for r, _ in chunks)
        assert splits > 1 and tiles < per_head and tiles * heads * splits <= 256
        assert (per_head - tiles) * heads <= per_head * heads // 256 * 256 < (per_head - tiles + 1) * heads
        assert all(abs(k - chunks[0][1]) <= 2 for _, k in chunks)
    assert dealt > 100 and split > 100
    ragged = [(780, 172)] * 7
    assert B.attn_clip_tail(128, 10, ragged) == (3, 8) and B.attn_clip_tail(128, 10, [(390, 160)] + ragged) == (0, 1)


@pytest.mark.parametrize("call, outputs", [("ll_attn_key_groups", 1), ("ll_attn_key_groups_fp8", 1), ("ll_attn_clip_tail", 2)])
def test_host_calls_refuse_what_is_no_launch(call, outputs):
    fn, out = getattr(B.lib(), call), [C.byref(C.c_int()) for _ in range(outputs)]
    ints = lambda *x: (C.c_int * len(x))(*x)
    assert fn(128, 4, 2, ints(100, 100), ints(20, 20), *out) == B.LL_OK
    for args in [(96, 4, 1, ints(100), ints(20)), (128, 0, 1, ints(100), ints(20)), (128, 1025, 1, ints(100), ints(20)),
                 (128, 4, 0, ints(100), ints(20)), (128, 4, 25, ints(*[100] * 25), ints(*[20] * 25)), (128, 4, 1, ints(0), ints(20)),
                 (128, 4, 2, ints(100, 100), ints(20, 0)), (128, 4, 1, None, ints(20)), (128, 4, 1, ints(100), None)]:
        assert fn(*args, *out) != B.LL_OK, args
    for i in range(outputs):
        assert fn(128, 4, 1, ints(100), ints(20), *(None if j == i else o for j, o in enumerate(out))) != B.LL_OK
