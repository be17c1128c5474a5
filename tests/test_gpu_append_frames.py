"""One cache write of many frames (append_kernel.hip, append_fp8.hip): up to 8 in the short argument block, up to 16 in the long
one, more in further launches.  Every frame gets the bits it has when it is written alone."""
import pytest
import torch

from paper_2509_22622_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kv_format", ["bf16", "fp8_e4m3"])
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("n", [8, 9, 16, 17])
def test_frames_written_together_and_one_by_one(kv_format, head_dim, n):
    heads, gh, gw = 3, 5, 9                          # ragged frames of 45 tokens
    P = gh * gw
    g = torch.Generator(device="cuda").manual_seed(n)
    q, k, v = (torch.empty((n * P, heads, head_dim), dtype=torch.bfloat16, device="cuda").normal_(generator=g) for _ in range(3))
    together, alone = (B.Cache(1, heads, head_dim, gh, gw, 1, 0, 20, kv_format=kv_format) for _ in range(2))
    together.recache_prefill(0, True, 0, n, q, k, v, torch.empty_like(q))
    kind = torch.uint8 if kv_format == "fp8_e4m3" else torch.bfloat16
    q_out = torch.empty((P, heads, head_dim), dtype=kind, device="cuda")
    for f in range(n):
        rows = slice(f * P, (f + 1) * P)
        alone.chunk_append(0, f, 1, q[rows].contiguous(), k[rows].contiguous(), v[rows].contiguous(), q_out)
    assert together.live_frames(0) == alone.live_frames(0) == list(range(n))
    for f in range(n):
        got, want = ([torch.empty((P, heads, head_dim), dtype=kind, device="cuda") for _ in range(2)] for _ in range(2))
        together.read_frame(0, f, *got)
        alone.read_frame(0, f, *want)
        torch.cuda.synchronize()
        for a, b in zip(got, want):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), f
    together.close()
    alone.close()
