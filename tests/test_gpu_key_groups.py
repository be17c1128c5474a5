"""Kernels that a launch's size selects, at the edges of what they take.

Launches of few rows and heads deal a tile's keys to 2, 4 or 8 groups of the workgroup's waves (attn_stream16.hip);
the groups' results meet in LDS.  Where that can go wrong: shares of unequal length, fewer kblocks than groups, a last
kblock of one key, a last tile of one row, a score far above its own group's reference, periods of the groups' rings that
wrap.  The small shapes here take the largest grouping a head_dim has, 8 groups at 64 and 4 at 128, from five kblocks on,
and 2 (4 at 64 with three or four) below; every other grouping with long shares has its shapes below, which ask
attn_key_groups what they get.
Cross-attention over a prompt that fits into LDS whole (256 tokens at head_dim 128, 512 at 64) runs in a kernel of its
own (attn_resident.hip) unless a variant is forced: both run here on the same inputs."""
import pytest
import torch

from paper_2509_22622_amd import binding as B
from perf import cases

pytestmark = pytest.mark.gpu


def _reference(q, k, v):
    """[rows, H, D] in 64 bits."""
    q, k, v = (x.double().transpose(0, 1) for x in (q, k, v))
    w = torch.softmax(torch.stack([a @ b.T.contiguous() for a, b in zip(q, k)]) * q.shape[-1] ** -0.5, -1)
    return torch.stack([a @ b for a, b in zip(w, v)]).transpose(0, 1)


def _check(heads, head_dim, n_q, n_keys, seed, spoil=None, streamed=True):
    g = torch.Generator(device="cuda").manual_seed(seed)
    q, k, v = (torch.empty((n, heads, head_dim), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
               for n in (n_q, n_keys, n_keys))
    if spoil is not None:
        spoil(q, k)
    prompt = B.Prompt(1, heads, head_dim, n_keys)
    prompt.recache(0, k, v)
    out = torch.full_like(q, 7.0)
    if streamed:
        B.set_attn_variant({n: v for v, n in B.attn_variant_names().items()}[f"d{head_dim}_stream16_qscale"])
    try:
        prompt.cross_attn(0, q, out)
    finally:
        B.set_attn_variant(0)
    torch.cuda.synchronize()
    prompt.close()
    want = _reference(q, k, v)
    err = (out.double() - want).norm() / want.norm()
    return out, want, float(err)


@pytest.mark.parametrize("streamed", [True, False])
@pytest.mark.parametrize("heads, head_dim", [(2, 64), (3, 128)])
@pytest.mark.parametrize("n_keys", [1, 31, 33, 64, 97, 128, 225, 256, 257, 289, 511, 1000])
@pytest.mark.parametrize("n_q", [1, 33, 64, 95])
def test_shares_of_every_length(heads, head_dim, n_q, n_keys, streamed):
    """bf16 operands and weights: half a unit in the last place (2^-9) on q', on the weights and on the result, in
    quadrature about 2.9e-3; up to 5e-3 where few keys leave nothing to average over."""
    _, _, err = _check(heads, head_dim, n_q, n_keys, 1000 * n_q + n_keys, streamed=streamed)
    assert err <= 5e-3


@pytest.mark.parametrize("n_keys", [65, 384, 399])
def test_two_groups(n_keys):
    _, _, err = _check(24, 128, 1170, n_keys, n_keys)
    assert err <= 5e-3


@pytest.mark.parametrize("streamed", [True, False])
@pytest.mark.parametrize("heads, head_dim, n_q", [(2, 64, 70), (3, 128, 70), (24, 128, 1170)])
@pytest.mark.parametrize("at", [3, 200, 300, 511])
def test_a_score_far_above_one_groups_reference(heads, head_dim, n_q, at, streamed):
    """Key `at` is 40 times query 5: its logit exceeds every other of that row by some 40 sqrt(D), beyond what a fixed
    reference holds, and the whole weight of the row lies in one group."""
    def spoil(q, k):
        k[at] = 40 * q[5]

    n_keys = 512 if streamed or head_dim == 64 or at > 255 else 256
    out, want, _ = _check(heads, head_dim, n_q, n_keys, at, spoil, streamed)
    assert bool(torch.isfinite(out).all())
    row = want[5]
    assert float((out[5].double() - row).norm() / row.norm()) <= 2.0 ** -8


@pytest.mark.parametrize("heads, head_dim, n_q, n_keys", [(2, 64, 70, 1000), (3, 128, 70, 1000), (24, 128, 1170, 700)])
@pytest.mark.parametrize("lo, hi", [(128, 160), (256, 600), (480, 640)])
def test_keys_without_weight_where_a_share_begins(heads, head_dim, n_q, n_keys, lo, hi):
    """Keys [lo, hi) score minus infinity (feature 0 of every query is positive, theirs is -inf): a share of the keys may
    begin with, or consist of, such keys, and the row is the softmax over the others.  Those score 300 to 500 (log2) below
    zero, so a share that begins with weightless keys cannot fall back to a reference near zero either."""
    def spoil(q, k):
        q[..., :2] = 1
        k[..., 1] = -3000
        k[lo:hi, :, 0] = float("-inf")

    out, want, err = _check(heads, head_dim, n_q, n_keys, lo, spoil)
    assert bool(torch.isfinite(out).all())
    assert err <= 5e-3


LONG_SHARES = [(64, 24, 1560, 1), (64, 24, 1170, 2), (64, 12, 1170, 4), (64, 12, 300, 8),
               (128, 24, 1560, 1), (128, 24, 1170, 2), (128, 12, 1170, 4)]


@pytest.mark.parametrize("head_dim, heads, n_q, groups", LONG_SHARES)
@pytest.mark.parametrize("n_keys, at", [(300, None), (641, 640), (1000, 700)])
def test_long_shares(head_dim, heads, n_q, groups, n_keys, at):
    """Every grouping with shares of several steps, odd and even, unlike ones beside each other; with one score far above
    the reference of its own share."""
    def spoil(q, k):
        if at is not None:
            k[at] = 40 * q[5]

    assert B.attn_key_groups(head_dim, heads, [(n_q, -(-n_keys // 32))]) == groups
    out, want, err = _check(heads, head_dim, n_q, n_keys, n_keys, spoil)
    assert bool(torch.isfinite(out).all())
    assert err <= 5e-3


def _rel(got, want):
    return float((got.double() - want).norm() / want.norm())


@pytest.mark.parametrize("head_dim, heads, grid, groups", [
    (64, 24, (20, 26), 1), (64, 24, (15, 26), 2), (64, 12, (15, 26), 4), (64, 12, (9, 11), 8),
    (128, 24, (20, 26), 1), (128, 24, (15, 26), 2), (128, 12, (15, 26), 4)])
def test_long_shares_in_the_cache(head_dim, heads, grid, groups):
    """A streamed chunk of every grouping against the pass in 64 bits, to the benchmark's relative tolerance; the kernels
    that turn the queries themselves give the bits of those that take them turned."""
    case = {"kind": "stream", "cache": "bf16", "layers": 1, "heads": heads, "head_dim": head_dim, "grid_h": grid[0],
            "grid_w": grid[1], "chunk": 3, "sink": 3, "window": 6, "frames": 3, "first_frame": 47, "video_chunks": 0, "q_std": 2.0}
    P = grid[0] * grid[1]
    assert B.attn_key_groups(head_dim, heads, [(3 * P, -(-12 * P // 32))]) == groups
    outs = []
    for form in ("two_call", "unrotated"):
        state = cases.prepare({**case, "form": form}, 5)
        outs += cases.run(state)
        torch.cuda.synchronize()
        state["cache"].close()
    assert torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16))
    assert _rel(outs[0], cases.exact(case, 5)[0]) <= 5e-3 * case["q_std"]


@pytest.mark.parametrize("head_dim, heads, grid, clip_frames, groups", [
    (64, 24, (7, 19), 8, 1), (64, 16, (7, 19), 8, 2), (64, 12, (7, 19), 5, 4), (64, 1, (11, 17), 5, 8),
    (128, 24, (7, 19), 8, 1), (128, 16, (7, 19), 8, 2), (128, 1, (7, 19), 5, 4)])
def test_long_shares_in_a_clip(head_dim, heads, grid, clip_frames, groups):
    """The form that also writes the row sums, of every grouping: output and gradients against 64 bits.  Gradients to the five
    bf16 roundings on their way (test_narrow_backward_tiles)."""
    case = {"kind": "clip", "heads": heads, "head_dim": head_dim, "grid_h": grid[0], "grid_w": grid[1], "chunk": 3, "sink": 2,
            "window": 4, "ctx_start": 20, "n_ctx": 4, "clip_frames": clip_frames, "q_std": 1.0}
    state = cases.prepare(case, 6)
    got = cases.run(state)
    torch.cuda.synchronize()
    chunks = []
    for i in range(-(-clip_frames // 3)):
        kblocks = sum(-(-end // 32) - begin // 32 for begin, end in state["clip"].chunk_key_ranges(i))
        chunks.append((min(3, clip_frames - 3 * i) * grid[0] * grid[1], kblocks))
    assert B.attn_key_groups(head_dim, heads, chunks) == groups
    for name, a, b in zip(("out", "dq", "dk", "dv"), got, cases.exact(case, 6)):
        assert _rel(a, b) <= 5e-3, name
    state["clip"].close()


@pytest.mark.parametrize("heads, head_dim, n_keys", [(12, 128, 200), (300, 64, 33), (300, 64, 97), (400, 64, 97), (7, 64, 512)])
def test_resident_keys_over_many_rows(heads, head_dim, n_keys):
    """Several blocks of rows per wave, and more heads than CUs (at 97 keys 400 fill two rounds to three
    quarters, 300 do not and stream)."""
    _, _, err = _check(heads, head_dim, 9001, n_keys, n_keys, streamed=False)
    assert err <= 5e-3


@pytest.mark.parametrize("head_dim, n_keys", [(128, 256), (64, 400)])
def test_resident_keys_ignore_a_longer_prompt_before(head_dim, n_keys):
    """NaN keys and values of an earlier, longer prompt lie behind the last key of this one; in place."""
    heads, n_q = 3, 100
    prompt = B.Prompt(1, heads, head_dim, 512)
    bad = torch.full((512, heads, head_dim), float("nan"), dtype=torch.bfloat16, device="cuda")
    prompt.recache(0, bad, bad)
    g = torch.Generator(device="cuda").manual_seed(n_keys)
    q, k, v = (torch.empty((n, heads, head_dim), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
               for n in (n_q, n_keys - 7, n_keys - 7))
    prompt.recache(0, k, v)
    want = _reference(q, k, v)
    prompt.cross_attn(0, q, q)
    torch.cuda.synchronize()
    prompt.close()
    assert float((q.double() - want).norm() / want.norm()) <= 5e-3


@pytest.mark.parametrize("heads, head_dim, n_q", [(1, 64, 1), (3, 64, 65), (1, 128, 4160), (12, 128, 63), (12, 128, 700),
                                                  (12, 128, 2500), (5, 128, 9100), (5, 64, 25000)])
def test_projection_tiles(heads, head_dim, n_q):
    """The projection's tile shapes (64 x 64, 128 x 64, 128 x 128, 256 x 128, by rows and features), ragged in both
    directions: an identity weight returns the attention output bit for bit, a random one the product in 64 bits to
    one bf16 rounding (2^-9 relative)."""
    g = torch.Generator(device="cuda").manual_seed(n_q)
    n = heads * head_dim
    prompt = B.Prompt(1, heads, head_dim, 64)
    k, v, q = (torch.empty((m, heads, head_dim), dtype=torch.bfloat16, device="cuda").normal_(generator=g) for m in (50, 50, n_q))
    prompt.recache(0, k, v)
    attn = torch.empty_like(q)
    prompt.cross_attn(0, q, attn)
    workspace = torch.empty(prompt.cross_attn_out_workspace_bytes(n_q), dtype=torch.uint8, device="cuda")
    y = torch.full((n_q, n), 7.0, dtype=torch.bfloat16, device="cuda")
    eye = torch.eye(n, dtype=torch.bfloat16, device="cuda")
    w = torch.empty((n, n), dtype=torch.bfloat16, device="cuda").normal_(0, n ** -0.5, generator=g)
    packed = torch.empty_like(w)
    for weight in (eye, w):
        prompt.pack_out_weight(weight, packed)
        prompt.cross_attn_out(0, q, packed, workspace, y)
        torch.cuda.synchronize()
        want = attn.view(n_q, n).double() @ weight.double().T
        if weight is eye:
            assert torch.equal(y.view(torch.int16), attn.view(n_q, n).view(torch.int16))
        else:
            assert float((y.double() - want).norm() / want.norm()) <= 2.0 ** -9
    prompt.close()


@pytest.mark.parametrize("heads, grid, n_clip", [(1, (5, 13), 5), (3, (9, 13), 4)])
def test_narrow_backward_tiles(heads, grid, n_clip):
    """Small clips at head_dim 128 take backward tiles of 128 columns: key sets and rows that are no multiple of 32 or 128,
    several chunks, against the gradients in 64 bits.  Five bf16 roundings on a gradient's way (2^-9 / sqrt(3) x 2 each in
    relative 2-norm): sqrt(5) x 2.26e-3 = 5.0e-3."""
    D, C, S, W, ctx = 128, 2, 2, 3, 7
    P = grid[0] * grid[1]
    g = torch.Generator(device="cuda").manual_seed(heads)
    make = lambda n: torch.empty((n * P, heads, D), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    q, dout, k, v = make(n_clip), make(n_clip), make(S + W + n_clip), make(S + W + n_clip)
    clip = B.Clip(heads, D, *grid, C, S, W, n_clip)
    out, dq, dk, dv = (torch.empty_like(q) for _ in range(4))
    clip.forward(ctx, W, n_clip, q, k, v, out)
    clip.backward(dout, dq, dk, dv)
    torch.cuda.synchronize()
    clip.close()

    from oracle.clip_backward import ClipOracle
    from oracle.longlive_oracle import OracleConfig
    oracle = ClipOracle(OracleConfig(1, heads, D, *grid, C, S, W))
    host = lambda t: t.double().cpu().numpy()
    want = (oracle.forward(ctx, W, n_clip, host(q), host(k), host(v)), *oracle.backward(host(dout)))
    for name, got, ref in zip(("out", "dq", "dk", "dv"), (out, dq, dk, dv), want):
        ref = torch.from_numpy(ref).cuda()
        assert float((got.double() - ref).norm() / ref.norm()) <= 5.0e-3, name


@pytest.mark.parametrize("heads, head_dim, grid, chunk, sink, window, n_win", [
    (12, 128, (15, 26), 3, 3, 9, 12), (12, 64, (16, 19), 2, 2, 4, 6), (21, 128, (6, 19), 1, 2, 5, 6),
    (16, 64, (10, 16), 3, 3, 6, 9), (10, 64, (17, 23), 3, 2, 5, 7), (12, 128, (19, 33), 2, 2, 6, 8)])
def test_prefill_equals_streaming_where_a_chunk_takes_key_groups(heads, head_dim, grid, chunk, sink, window, n_win):
    """Streamed chunk by chunk or rebuilt in one call, the outputs of a chunk whose keys no call deals to several workgroups are the
    same bits: into how many key groups its tiles are dealt depends on the chunk, not on the launch it is part of."""
    P, nf = grid[0] * grid[1], sink + n_win
    g = torch.Generator(device="cuda").manual_seed(P)
    q, k, v = (torch.empty((nf * P, heads, head_dim), dtype=torch.bfloat16, device="cuda").normal_(generator=g) for _ in range(3))
    streamed, rebuilt = (B.Cache(1, heads, head_dim, *grid, chunk, sink, window) for _ in range(2))
    want, got = torch.empty_like(q), torch.empty_like(q)
    starts = [*range(0, sink, chunk), *range(sink, nf, chunk)]
    assert B.attn_key_groups(head_dim, heads, [(chunk * P, -(-(sink + window + chunk) * P // 32))]) > 1
    for n in {end - f0 for f0, end in zip(starts, starts[1:] + [nf])}:
        assert B.attn_split(head_dim, heads, n * P, -(-(sink + window + n) * P // 32))[1] == 1
    for f0, end in zip(starts, starts[1:] + [nf]):
        rows = slice(f0 * P, end * P)
        streamed.chunk_append(0, f0, end - f0, None, k[rows], v[rows], None)
        streamed.sink_window_attn_unrotated(0, q[rows], want[rows])
    rebuilt.recache_prefill(0, True, sink, n_win, q, k, v, got)
    torch.cuda.synchronize()
    streamed.close()
    rebuilt.close()
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("kind, heads, grid, chunk, sink, window", [
    ("stream", 12, (15, 26), 3, 3, 9),            # 228 tiles, a head's on one XCD or two
    ("stream", 16, (10, 20), 4, 0, 16),           # a last tile of 32 rows
    ("stream", 40, (8, 8), 1, 1, 20),             # one tile a head: no one to take turns with
    ("stream", 48, (10, 13), 1, 1, 20),           # three
    ("stream", 40, (13, 20), 1, 1, 20),           # five, the last of four rows
    ("prefill", 12, (15, 26), 3, 3, 9)])          # placed by groups
@pytest.mark.parametrize("q_std", [1.0, 5.0])
def test_four_groups_over_many_keys(kind, heads, grid, chunk, sink, window, q_std):
    """From 16 MB of keys and values on, a head's tiles on one XCD bring kblocks into L2 ahead of their steps by turns: shares that
    end within the distance, launches placed by groups, and peaky logits, whose pass that follows the maximum leaves it.  Twice
    the same bits.  5e-3 as everywhere, times the logits' standard deviation (gpu_harness.assert_parity)."""
    P = grid[0] * grid[1]
    full = (sink + window + chunk) * P
    assert B.attn_key_groups(128, heads, [(chunk * P, -(-full // 32))]) == 4 and full * heads * 512 >= 16 << 20
    assert B.attn_split(128, heads, chunk * P, -(-full // 32)) == (4, 1)
    case = {"kind": kind, "cache": "bf16", "layers": 1, "heads": heads, "head_dim": 128, "grid_h": grid[0], "grid_w": grid[1],
            "chunk": chunk, "sink": sink, "window": window, "q_std": q_std}
    case.update({"form": "unrotated", "frames": chunk, "first_frame": sink + window + 5, "video_chunks": 0, "sink_relative": False}
                if kind == "stream" else {"win_start": sink + 7, "n_win": window})
    state = cases.prepare(case, 3)
    out = cases.run(state)[0].clone()
    want = cases.exact(case, 3)[0]
    assert float((out.double() - want).norm() / want.norm()) <= 5e-3 * q_std
    again = cases.run(state)[0]
    assert torch.equal(again.view(torch.int16), out.view(torch.int16))
    state["cache"].close()
