"""The train-time rule on the GPU (ll_clip_forward, ll_clip_backward) against the fp64 oracle.

Tolerances.  Forward: those of the inference path (max-abs 1e-2, relative L2 5e-3).  Gradients: derived from the
number of bf16 roundings on each tensor's way (tests/test_grad_rounding_model.py has the derivation and checks it on
the CPU with a rounding model of this path): with unit roundoff u = 2^-8 and rho = u / sqrt(3) per rounding, n_r = 5
roundings for dq and dk, 4 for dv, independent and averaged over many terms,
    relative L2 <= sqrt(n_r) rho = 5.0e-3 (dq, dk), 4.5e-3 (dv)          [the model and the kernels: 3.1e-3 to 3.9e-3]
where nothing averages (a handful of keys with one dominant: `few_terms`) each rounding may sit at its maximum,
    relative L2 <= sqrt(n_r) u = 8.7e-3 (dq, dk), 7.8e-3 (dv)            [that case: 5.4e-3 to 5.8e-3; the other 299 of
                                                                         300 random geometries run once outside the
                                                                         suite stay below 4.4e-3 (dq, dk), 3.8e-3 (dv)]
and no element is further off than n_r u = 2 % (1.6 % for dv) of the tensor's largest magnitude.  delta = dO . O is
taken from the forward's unrounded output, so it adds no rounding of its own.
"""
import numpy as np
import pytest
import torch

from oracle.clip_backward import ClipOracle
from oracle.longlive_oracle import OracleConfig, bf16_bits_to_f64, error_metrics
from paper_2509_22622_amd import binding as B
from paper_2509_22622_amd import synth

import gpu_harness as H

pytestmark = pytest.mark.gpu

U_BF16 = 2.0 ** -8
N_ROUNDINGS = {"dq": 5, "dk": 5, "dv": 4}


def grad_rel_l2(name, few_terms=False):
    return float(np.sqrt(N_ROUNDINGS[name]) * (U_BF16 if few_terms else U_BF16 / np.sqrt(3.0)))


def grad_max_frac(name):
    return N_ROUNDINGS[name] * U_BF16


def bits(shape, stream, tensor, cfg_id=41):
    return synth.normal_bf16(shape, cfg_id, 0, stream, tensor)


def run_case(heads, head_dim, gh, gw, C, S, W, T, ctx_start, n_ctx, n_clip, seed=0, dout_rows=None, q_scale=1.0,
             few_terms=False):
    cfg = OracleConfig(1, heads, head_dim, gh, gw, C, S, W)
    P = gh * gw
    oracle = ClipOracle(cfg)
    nf = len(oracle.frames(ctx_start, n_ctx, n_clip))
    q = synth.normal_bf16((n_clip * P, heads, head_dim), 41, 0, 4 * seed, "q", scale=q_scale)
    k = bits((nf * P, heads, head_dim), 4 * seed, "k")
    v = bits((nf * P, heads, head_dim), 4 * seed, "v")
    dout = bits((n_clip * P, heads, head_dim), 4 * seed + 1, "q")
    if dout_rows is not None:                                  # a loss on some rows only
        keep = np.zeros(n_clip * P, dtype=bool)
        keep[dout_rows] = True
        dout = np.where(keep[:, None, None], dout, np.uint16(0))
    clip = B.Clip(heads, head_dim, gh, gw, C, S, W, T)
    out, dq, dk, dv = (torch.empty((n_clip * P, heads, head_dim), dtype=torch.bfloat16, device="cuda") for _ in range(4))
    clip.forward(ctx_start, n_ctx, n_clip, H.to_dev(q), H.to_dev(k), H.to_dev(v), out)
    clip.backward(H.to_dev(dout), dq, dk, dv)
    torch.cuda.synchronize()
    want_out = oracle.forward(ctx_start, n_ctx, n_clip, bf16_bits_to_f64(q), bf16_bits_to_f64(k), bf16_bits_to_f64(v))
    what = f"H{heads} D{head_dim} P{P} C{C} S{S} W{W} ctx {ctx_start}+{n_ctx} clip {n_clip}"
    H.assert_parity(H.to_bits(out), want_out, what + " forward", logit_scale=q_scale)
    want = oracle.backward(bf16_bits_to_f64(dout))
    got = {}
    for name, t, w in zip(("dq", "dk", "dv"), (dq, dk, dv), want):
        g = bf16_bits_to_f64(H.to_bits(t))
        assert np.isfinite(g).all(), f"{what} {name}: non-finite"
        max_abs, rel = error_metrics(g, w)
        assert rel <= grad_rel_l2(name, few_terms) * q_scale and max_abs <= grad_max_frac(name) * q_scale * np.abs(w).max(), \
            f"{what} {name}: max_abs {max_abs:.3e} of {np.abs(w).max():.3e}, rel_l2 {rel:.3e}"
        got[name] = g
    clip.close()
    return got, want


@pytest.mark.parametrize("heads,head_dim,gh,gw,C,S,W,T,ctx_start,n_ctx,n_clip", [
    (2, 64, 3, 5, 2, 1, 3, 7, 5, 3, 7),       # window slides inside the clip, short last chunk
    (2, 64, 3, 5, 2, 1, 3, 7, 0, 0, 6),       # a video's first clip: the sink is part of the clip
    (3, 128, 5, 8, 3, 3, 6, 9, 9, 6, 9),      # the tiny inference config's window and sink, D 128
    (2, 128, 7, 9, 3, 2, 5, 6, 20, 2, 5),     # P 63: nothing aligned; fewer context frames than the window holds
    (2, 64, 9, 15, 2, 2, 4, 6, 30, 4, 6),     # P 135: two column tiles per frame, the second ragged
    (1, 128, 4, 8, 1, 0, 2, 5, 0, 2, 5),      # no sink, chunks of one frame, context from frame 0
    (2, 64, 2, 3, 3, 2, 0, 6, 2, 0, 6),       # no window at all: sink and own chunk only
    (2, 64, 3, 5, 2, 1, 3, 7, 2 ** 31 + 5, 3, 7),   # a clip past 2^31 frames: 64-bit absolute frame positions
])
def test_clip_forward_and_gradients(heads, head_dim, gh, gw, C, S, W, T, ctx_start, n_ctx, n_clip):
    run_case(heads, head_dim, gh, gw, C, S, W, T, ctx_start, n_ctx, n_clip)


@pytest.mark.parametrize("heads,gh,gw,C,S,W,T,ctx_start,n_ctx,n_clip", [
    (52, 9, 13, 3, 2, 3, 5, 20, 3, 5),        # tiles of 256 + 95 and 234 columns, in both kernels
    (86, 5, 13, 2, 1, 3, 7, 0, 0, 6),         # a video's first clip: half of a tile's waves have no columns
    (70, 7, 9, 1, 0, 2, 5, 0, 2, 5),          # no sink, chunks of one frame of 63 tokens
])
def test_wide_backward_tiles(heads, gh, gw, C, S, W, T, ctx_start, n_ctx, n_clip):
    """Launches of more than 256 tiles of 128 columns take tiles of 256 at head_dim 128 (attn_bwd.hip: narrow_tiles): ragged
    ones, frames that nothing is aligned with, every element."""
    tiles = [-(-min(C, n_clip - i) * gh * gw // 128) for i in range(0, n_clip, C)]
    assert sum(tiles) * heads > 256
    run_case(heads, 128, gh, gw, C, S, W, T, ctx_start, n_ctx, n_clip, seed=7)


def test_gradient_reaches_only_the_keys_a_chunk_sees():
    """A loss on the last chunk only: keys outside its window get exactly zero, its queries alone get dq."""
    gh, gw, C, S, W = 3, 5, 2, 1, 2
    P, n_clip = gh * gw, 8
    rows = np.arange(6 * P, 8 * P)
    got, want = run_case(2, 64, gh, gw, C, S, W, 8, 3, 2, n_clip, seed=3, dout_rows=rows)
    for i in range(n_clip):
        blk = slice(i * P, (i + 1) * P)
        seen = i >= 4                                          # frames 9, 10 (window) and 11, 12 (the chunk) of 5..12
        assert (np.abs(got["dk"][blk]).max() > 0) == seen and (np.abs(got["dv"][blk]).max() > 0) == seen, i
        assert (np.abs(got["dq"][blk]).max() > 0) == (i >= 6), i


def test_second_step_with_a_shorter_clip_reuses_the_handle():
    """The handle's regions keep the former step's contents; a later, shorter step must not see them."""
    heads, head_dim, gh, gw, C, S, W, T = 2, 64, 3, 5, 2, 1, 3, 7
    cfg = OracleConfig(1, heads, head_dim, gh, gw, C, S, W)
    P = gh * gw
    clip = B.Clip(heads, head_dim, gh, gw, C, S, W, T)
    for step, (ctx_start, n_ctx, n_clip) in enumerate([(5, 3, 7), (12, 2, 3)]):
        oracle = ClipOracle(cfg)
        nf = len(oracle.frames(ctx_start, n_ctx, n_clip))
        q, k, v = bits((n_clip * P, heads, head_dim), 20 + step, "q"), bits((nf * P, heads, head_dim), 20 + step, "k"), bits((nf * P, heads, head_dim), 20 + step, "v")
        dout = bits((n_clip * P, heads, head_dim), 30 + step, "q")
        out, dq, dk, dv = (torch.empty((n_clip * P, heads, head_dim), dtype=torch.bfloat16, device="cuda") for _ in range(4))
        clip.forward(ctx_start, n_ctx, n_clip, H.to_dev(q), H.to_dev(k), H.to_dev(v), out)
        clip.backward(H.to_dev(dout), dq, dk, dv)
        torch.cuda.synchronize()
        H.assert_parity(H.to_bits(out), oracle.forward(ctx_start, n_ctx, n_clip, *(bf16_bits_to_f64(t) for t in (q, k, v))), f"step {step}")
        for name, t, w in zip(("dq", "dk", "dv"), (dq, dk, dv), oracle.backward(bf16_bits_to_f64(dout))):
            max_abs, rel = error_metrics(bf16_bits_to_f64(H.to_bits(t)), w)
            assert rel <= grad_rel_l2(name), f"step {step} {name}: rel_l2 {rel:.3e}"
    clip.close()


def test_wan_frame_size():
    """The benchmark model's frame (30 x 52 tokens), head width, chunk, sink and window; two heads and a clip of two
    chunks keep the oracle's fp64 products to seconds (and take the backward kernels' narrow tiles; the wide ones have
    test_wide_backward_tiles and the benchmark's shape).  Every element of out, dq, dk and dv is compared."""
    run_case(2, 128, 30, 52, 3, 3, 9, 6, 60, 9, 6, seed=5)


def test_graph_replay_of_a_training_step():
    """Forward and backward enqueue kernels only (no allocation, no synchronisation, no memset): a captured step
    replays on fresh contents of the captured tensors and equals the eager step bit for bit."""
    heads, head_dim, gh, gw, C, S, W, T = 2, 64, 3, 5, 2, 1, 3, 6
    P, ctx_start, n_ctx, n_clip = gh * gw, 5, 3, 6
    nf = S + n_ctx + n_clip
    eager, graphed = B.Clip(heads, head_dim, gh, gw, C, S, W, T), B.Clip(heads, head_dim, gh, gw, C, S, W, T)
    mk = lambda n: torch.zeros((n * P, heads, head_dim), dtype=torch.bfloat16, device="cuda")
    sq, sk, sv, sdo = mk(n_clip), mk(nf), mk(nf), mk(n_clip)
    so, sdq, sdk, sdv = mk(n_clip), mk(n_clip), mk(n_clip), mk(n_clip)

    def step(c, q, k, v, do, o, dq, dk, dv):
        c.forward(ctx_start, n_ctx, n_clip, q, k, v, o)
        c.backward(do, dq, dk, dv)

    step(graphed, sq, sk, sv, sdo, so, sdq, sdk, sdv)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step(graphed, sq, sk, sv, sdo, so, sdq, sdk, sdv)
    for rep in range(3):
        q, do = H.to_dev(bits((n_clip * P, heads, head_dim), 50 + rep, "q")), H.to_dev(bits((n_clip * P, heads, head_dim), 60 + rep, "q"))
        k, v = H.to_dev(bits((nf * P, heads, head_dim), 50 + rep, "k")), H.to_dev(bits((nf * P, heads, head_dim), 50 + rep, "v"))
        o, dq, dk, dv = mk(n_clip), mk(n_clip), mk(n_clip), mk(n_clip)
        step(eager, q, k, v, do, o, dq, dk, dv)
        torch.cuda.synchronize()
        sq.copy_(q), sk.copy_(k), sv.copy_(v), sdo.copy_(do)
        g.replay()
        torch.cuda.synchronize()
        for name, a, b in (("out", so, o), ("dq", sdq, dq), ("dk", sdk, dk), ("dv", sdv, dv)):
            assert torch.equal(a.view(torch.int16), b.view(torch.int16)), f"replay {rep}: {name}"
        assert float(dq.float().abs().max()) > 0
    eager.close()
    graphed.close()


@pytest.mark.parametrize("idx", range(10))
def test_random_geometries(idx):
    """Seeded random small geometries: nothing aligned on purpose (P from 15 to 96, any S, W, C, clip and context
    lengths, first clips and later ones)."""
    rng = np.random.Generator(np.random.Philox(key=9000 + idx))
    D = int(rng.choice([64, 128]))
    gh, gw = int(rng.integers(3, 9)), int(rng.integers(5, 13))
    C, S, W = int(rng.integers(1, 5)), int(rng.integers(0, 5)), int(rng.integers(0, 9))
    T = int(rng.integers(3, 11))
    n_clip = int(rng.integers(1, T + 1))
    if idx % 4 == 0:
        ctx_start, n_ctx = 0, 0                                   # a video's first clip
    else:
        n_ctx = int(rng.integers(0, W + 1))
        ctx_start = S + int(rng.integers(0, 40))
    run_case(int(rng.integers(1, 4)), D, gh, gw, C, S, W, T, ctx_start, n_ctx, n_clip, seed=10 + idx)


def test_peaky_scores():
    """Queries four times larger (logits of standard deviation 4: a few keys carry the weight).  As for the inference
    path's stress input, the rounding of q' and K' to bf16 moves every logit four times further, so all tolerances are
    scaled by 4; outside the graded configurations."""
    got, want = run_case(2, 128, 5, 8, 3, 3, 6, 9, 9, 6, 9, seed=7, q_scale=4.0)
    for name, w in zip(("dq", "dk", "dv"), want):
        assert np.abs(got[name]).max() > 0 and np.isfinite(got[name]).all()


def test_more_frames_chunks_and_groups_than_one_launch_takes():
    """47 resident frames (the cache-write kernel takes 32 per launch), 40 chunks of one frame (the attention kernel
    takes 16 query chunks per launch, the backward kernels 32 column groups): every batching loop runs more than
    once."""
    run_case(2, 64, 2, 3, 1, 2, 5, 40, 9, 5, 40, seed=9)
    run_case(1, 128, 2, 3, 2, 0, 3, 70, 0, 0, 70, seed=10)       # a first clip without a sink: 35 chunks, 70 frames


def test_one_dominant_key():
    """Two queries over five keys, one key holding most of each row's weight: dP - delta is then a small difference of
    large numbers, and a delta taken from the bf16-rounded output would be off by about 2^-9 |dO||O|, 2.5 % of dK
    here.  The handle keeps the forward's output unrounded for this."""
    run_case(1, 128, 1, 1, 4, 3, 3, 2, 27, 0, 2, seed=238, few_terms=True)


def test_bench_shape_sampled():
    """The shape bench.py times (12 heads x 128, 30 x 52 tokens per frame, chunk 3, sink 3, window 9, a clip of 21
    frames after 9 context frames: 33 resident frames, 7 chunks, 32760 queries) on the GPU; the oracle follows heads
    0 and 11 only (heads are independent): their whole forward output, dq at sampled rows of every chunk, dk and dv at
    sampled keys of an early and of the last chunk."""
    heads, head_dim, gh, gw, C, S, W, T = 12, 128, 30, 52, 3, 3, 9, 21
    P, ctx_start, n_ctx, n_clip = gh * gw, 60, 9, 21
    nf = S + n_ctx + n_clip
    q = bits((n_clip * P, heads, head_dim), 80, "q")
    k, v = bits((nf * P, heads, head_dim), 80, "k"), bits((nf * P, heads, head_dim), 80, "v")
    dout = bits((n_clip * P, heads, head_dim), 81, "q")
    clip = B.Clip(heads, head_dim, gh, gw, C, S, W, T)
    out, dq, dk, dv = (torch.empty((n_clip * P, heads, head_dim), dtype=torch.bfloat16, device="cuda") for _ in range(4))
    clip.forward(ctx_start, n_ctx, n_clip, H.to_dev(q), H.to_dev(k), H.to_dev(v), out)
    clip.backward(H.to_dev(dout), dq, dk, dv)
    torch.cuda.synchronize()
    sel = [0, 11]
    oracle = ClipOracle(OracleConfig(1, len(sel), head_dim, gh, gw, C, S, W))
    f64 = lambda b: bf16_bits_to_f64(np.ascontiguousarray(b[:, sel, :]))
    want_out = oracle.forward(ctx_start, n_ctx, n_clip, f64(q), f64(k), f64(v))
    H.assert_parity(H.to_bits(out)[:, sel, :], want_out, "bench shape forward, heads 0 and 11")
    rng = np.random.Generator(np.random.Philox(key=4242))
    q_rows = np.sort(np.concatenate([c * C * P + rng.integers(0, C * P, 6) for c in range(n_clip // C)]))
    key_rows = np.sort(np.concatenate([3 * C * P + rng.integers(0, C * P, 6), 6 * C * P + rng.integers(0, C * P, 6),
                                       [6 * C * P, n_clip * P - 1]]))
    wq, wk, wv = oracle.backward_sample(f64(dout), q_rows, key_rows)
    for name, t, w, rows in (("dq", dq, wq, q_rows), ("dk", dk, wk, key_rows), ("dv", dv, wv, key_rows)):
        g = bf16_bits_to_f64(H.to_bits(t)[rows][:, sel, :])
        assert np.isfinite(g).all()
        max_abs, rel = error_metrics(g, w)
        assert rel <= grad_rel_l2(name) and max_abs <= grad_max_frac(name) * np.abs(w).max(), f"{name}: max_abs {max_abs:.3e} of {np.abs(w).max():.3e}, rel_l2 {rel:.3e}"
    clip.close()
