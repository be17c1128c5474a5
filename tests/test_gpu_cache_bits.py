"""The cache write's arithmetic bit for bit, written out in numpy: each rotary pair is one rounded fp32 product and one
fused multiply-add per component, in an order fixed in kernels.h, and one rounding to the stored type.  A kernel whose
compiler picks another order stores a neighbouring value for some keys.

The fused multiply-add in 64 bits: a bf16 number times an fp32 one is exact there, and so is the sum but for operands more
than 2^20 apart, whose last bit is far below a rounding to bf16 or E4M3."""
import math

import numpy as np
import pytest
import torch

from paper_2509_22622_amd import binding as B

pytestmark = pytest.mark.gpu

GRID, CHUNK, FIRST, HEADS = (30, 52), 2, 46, 12      # enough keys for some to lie next to a rounding boundary


def _cos_sin(D):
    """[frames * tokens, 1, D / 2] in fp32, frames FIRST and FIRST + 1."""
    n = D // 6
    n_t = D // 2 - 2 * n
    tok = np.tile(np.arange(GRID[0] * GRID[1]), CHUNK)
    frame = np.repeat(np.arange(FIRST, FIRST + CHUNK), GRID[0] * GRID[1])
    angle = np.concatenate([pos[:, None] * 10000.0 ** (-np.arange(m) / m)
                            for pos, m in ((frame, n_t), (tok // GRID[1], n), (tok % GRID[1], n))], 1)[:, None, :]
    return np.cos(angle).astype(np.float32), np.sin(angle).astype(np.float32)


def _fma(a, b, c):
    return (a.astype(np.float64) * b + c.astype(np.float64)).astype(np.float32)


def _turned(x, scaled):
    c, s = _cos_sin(x.shape[-1])
    x = x.float().cpu().numpy()
    re, im = x[..., 0::2], x[..., 1::2]
    o_re = _fma(re, c, -(im * s))
    o_im = _fma(re, s, im * c) if scaled else _fma(im, c, re * s)
    return np.stack([o_re, o_im], -1).reshape(x.shape)


def _inputs(D):
    g = torch.Generator(device="cuda").manual_seed(D)
    shape = (CHUNK * GRID[0] * GRID[1], HEADS, D)
    return [torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=g) for _ in range(3)]


def _written(cache, shape, dtype):
    P = shape[0] // CHUNK
    k, v = torch.empty(shape, dtype=dtype, device="cuda"), torch.empty(shape, dtype=dtype, device="cuda")
    for i in range(CHUNK):
        cache.read_frame(0, FIRST + i, k[i * P:(i + 1) * P], v[i * P:(i + 1) * P])
    torch.cuda.synchronize()
    return k.cpu(), v.cpu()


def _cache(D, **kw):
    cache = B.Cache(1, HEADS, D, *GRID, CHUNK, 0, 3, **kw)
    rows = 3 * GRID[0] * GRID[1]
    x = torch.zeros((rows, HEADS, D), dtype=torch.bfloat16, device="cuda")
    cache.recache_prefill(0, True, FIRST - 3, 3, x, x, x, torch.empty_like(x))      # the video so far: FIRST comes next
    return cache


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("with_queries", [True, False])
def test_bf16_cache(D, with_queries):
    q, k, v = _inputs(D)
    q_out = torch.empty_like(q)
    cache = _cache(D)
    cache.chunk_append(0, FIRST, CHUNK, *((q, k, v, q_out) if with_queries else (None, k, v, None)))
    got_k, got_v = _written(cache, k.shape, torch.bfloat16)
    cache.close()
    as_bits = lambda x: torch.as_tensor(x).to(torch.bfloat16).cpu().view(torch.int16)
    assert torch.equal(as_bits(got_k), as_bits(_turned(k, False)))
    assert torch.equal(as_bits(got_v), as_bits(v))
    if with_queries:
        scale = np.float32(math.log2(math.e) / math.sqrt(D))
        assert torch.equal(as_bits(q_out), as_bits(_turned(q, True) * scale))


@pytest.mark.parametrize("D", [64, 128])
def test_8_bit_cache(D):
    q, k, v = _inputs(D)
    q_out = torch.empty(q.shape, dtype=torch.uint8, device="cuda")
    cache = _cache(D, kv_format="fp8_e4m3")
    cache.chunk_append(0, FIRST, CHUNK, q, k, v, q_out)
    got_k, got_v = _written(cache, k.shape, torch.uint8)
    cache.close()
    codes = lambda x: torch.as_tensor(x).float().to(torch.float8_e4m3fn).view(torch.uint8).cpu()
    scale = np.float32(math.log2(math.e) / math.sqrt(D))
    assert torch.equal(got_k, codes(_turned(k, True)))
    assert torch.equal(got_v, codes(v))
    assert torch.equal(q_out.cpu(), codes(_turned(q, True) * scale))
