"""Streamed chunks whose tiles' keys are dealt to several workgroups, merged by a second launch (split.h).

Where that can go wrong: shares of unequal length, warm-up chunks of fewer kblocks than splits, tiles and slices of the merge
of few rows, a score far above one share's reference, shares without weight, output in place of the queries, a call replayed in
a HIP graph, calls on several streams over one pool of slots, and workgroups that find no slot.  Every shape asks for what
it gets.  References are in 64 bits, tolerances those of the unsplit path (bf16 operands, weights and results: up to 5e-3 of the
2-norm, times the spread of the logits)."""
import pytest
import torch

from paper_2509_22622_amd import binding as B
from perf import cases

pytestmark = pytest.mark.gpu

# heads, head_dim, grid, chunk, sink, window, frames, (groups, splits)
SHAPES = [
    (4, 128, (10, 19), 1, 3, 20, 1, (4, 9)),    # three tiles of 64 rows, the last of 62
    (1, 128, (6, 8), 2, 4, 26, 2, (4, 6)),    # shares of one and two kblocks
    (5, 128, (12, 20), 3, 2, 14, 3, (4, 4)),
    (3, 128, (9, 13), 3, 0, 21, 1, (4, 7)),    # a short chunk: 117 of 351 rows
    (3, 128, (20, 39), 3, 3, 4, 3, (2, 4)),
    (4, 128, (26, 41), 2, 3, 9, 2, (1, 7)),
    (3, 64, (5, 19), 2, 3, 50, 2, (8, 7)),
    (3, 64, (16, 45), 1, 3, 16, 1, (4, 7)),
    (1, 64, (30, 52), 3, 3, 9, 3, (2, 6)),
]


def _case(heads, head_dim, grid, chunk, sink, window, frames, **kw):
    return {"kind": "stream", "cache": "bf16", "layers": 1, "heads": heads, "head_dim": head_dim, "grid_h": grid[0],
            "grid_w": grid[1], "chunk": chunk, "sink": sink, "window": window, "frames": frames, "first_frame": sink + window + 4,
            "video_chunks": 0, "q_std": 2.0, "form": "two_call", **kw}


def _split(heads, head_dim, grid, chunk, sink, window, frames):
    P = grid[0] * grid[1]
    return B.attn_split(head_dim, heads, frames * P, -(-(sink + window + frames) * P // 32))


def _rel(got, want):
    return float((got.double() - want).norm() / want.norm())


def _bits(t):
    return t.view(torch.int16)


@pytest.mark.parametrize("shape", SHAPES)
def test_split_tiles(shape):
    """Both forms of the call give the same bits; so does a second pass, one that writes over its queries, and one without free slots
    (none, or some of a tile's), where the merge takes a tile's shares one after another."""
    *geo, split = shape
    assert _split(*geo) == split
    case = _case(*geo)
    want = cases.exact(case, 5)[0]
    state = cases.prepare({**case, "form": "unrotated"}, 5)
    unrotated = cases.run(state)[0].clone()
    torch.cuda.synchronize()
    state["cache"].close()
    state = cases.prepare(case, 5)
    out = cases.run(state)[0]
    layer, _, _, _, _, q_out, _ = state["passes"][0]
    assert _rel(out, want) <= 5e-3 * case["q_std"]
    assert torch.equal(_bits(out), _bits(unrotated))
    again = torch.full_like(out, 7.0)
    state["cache"].sink_window_attn(layer, q_out, again)
    assert torch.equal(_bits(again), _bits(out))
    for first, n in ((0, 512), (0, 2), (1, 511)):
        B.hold_split_slots(first, n, True)
        try:
            again.fill_(7.0)
            state["cache"].sink_window_attn(layer, q_out, again)
            in_place = q_out.clone()
            state["cache"].sink_window_attn(layer, in_place, in_place)
        finally:
            B.hold_split_slots(first, n, False)
        assert torch.equal(_bits(again), _bits(out)), (first, n)
        assert torch.equal(_bits(in_place), _bits(out)), (first, n)
    state["cache"].sink_window_attn(layer, q_out, q_out)
    assert torch.equal(_bits(q_out), _bits(out))
    state["cache"].close()


@pytest.mark.parametrize("shape", [SHAPES[1], SHAPES[2], SHAPES[5], SHAPES[6]])
def test_a_video_from_its_first_frame(shape):
    """Warm-up chunks have fewer kblocks than the full window's splits; with a sink at a fixed rotary distance as well."""
    *geo, _ = shape
    for sink_relative in (False, True):
        case = _case(*geo, video_chunks=1 + -(-(geo[4] + geo[5] + 4) // geo[3]), sink_relative=sink_relative)
        state = cases.prepare(case, 7)
        got = cases.run(state)
        for i, (a, b) in enumerate(zip(got, cases.exact(case, 7))):
            # (a re-indexed sink's queries are rounded once more)
            assert _rel(a, b) <= (7e-3 if sink_relative else 5e-3) * case["q_std"], i
        state["cache"].close()


@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[1], SHAPES[6]])
def test_first_chunks_written_over_their_queries(shape):
    """The first chunks have fewer than two kblocks a key group: one share, whose workgroup stores the finished rows.  With the output
    in place of the queries the merge must not compute them again."""
    *geo, (groups, _) = shape
    first = -(-geo[6] * geo[2][0] * geo[2][1] // 32)
    assert first // groups <= 1
    case = _case(*geo, video_chunks=1 + -(-(geo[4] + geo[5] + 4) // geo[3]))
    state = cases.prepare(case, 13)
    want = cases.run(state)
    exact = cases.exact(case, 13)
    cache = state["cache"]
    cache.reset()
    for (layer, start, q, k, v, q_out, _), apart, ref in zip(state["passes"], want, exact):
        cache.chunk_append(layer, start, case["frames"], q, k, v, q_out)
        cache.sink_window_attn(layer, q_out, q_out)
        assert torch.equal(_bits(q_out), _bits(apart)), start
        assert _rel(q_out, ref) <= 5e-3 * case["q_std"], start
    cache.close()


@pytest.mark.parametrize("heads, head_dim, grid, chunk, sink, window, n_win", [
    (2, 128, (14, 14), 1, 3, 8, 6), (1, 128, (8, 19), 1, 2, 16, 8), (1, 128, (4, 19), 2, 4, 24, 22), (1, 128, (6, 42), 3, 2, 5, 5)])
def test_split_re_prefill_with_a_re_indexed_sink(heads, head_dim, grid, chunk, sink, window, n_win):
    """The rotated queries wait in `out`; the first chunks have fewer than two kblocks a key group, so their tiles do not split."""
    P = grid[0] * grid[1]
    assert B.attn_split(head_dim, heads, chunk * P, -(-(sink + window + chunk) * P // 32))[1] > 1
    case = {"kind": "prefill", "cache": "bf16", "layers": 1, "heads": heads, "head_dim": head_dim, "grid_h": grid[0], "grid_w": grid[1],
            "chunk": chunk, "sink": sink, "window": window, "win_start": sink + window + 9, "n_win": n_win, "q_std": 2.0, "sink_relative": True}
    state = cases.prepare(case, 3)
    out = cases.run(state)[0]
    for i, (a, b) in enumerate(zip(out.split(P), cases.exact(case, 3)[0].split(P))):
        assert _rel(a, b) <= 7e-3 * case["q_std"], i     # a re-indexed sink's queries are rounded once more
    state["cache"].close()


def _cached(cache, P, heads, D):
    """Rotated keys and values of the live frames, oldest first."""
    kv = [tuple(torch.empty((P, heads, D), dtype=torch.bfloat16, device="cuda") for _ in range(2)) for _ in cache.live_frames(0)]
    for f, (k, v) in zip(cache.live_frames(0), kv):
        cache.read_frame(0, f, k, v)
    return (torch.cat(x) for x in zip(*kv))


@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[4], SHAPES[5], SHAPES[7]])
@pytest.mark.parametrize("spoil", ["far", "weightless"])
def test_unlike_shares(shape, spoil):
    """A key along a query takes that row's whole weight, far above every other share's reference; or the keys of several frames
    score minus infinity and fill whole shares and the beginnings of others."""
    heads, D, grid, chunk, sink, window, frames, split = shape
    P, f0 = grid[0] * grid[1], sink + window + 4
    g = torch.Generator(device="cuda").manual_seed(P)
    make = lambda n: torch.empty((n * P, heads, D), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    k, v, kc, vc, q = make(sink + window), make(sink + window), make(frames), make(frames), make(frames)
    pair = (D - 4 * (D // 6)) // 2 - 1               # the frame axis's slowest pair: a positive angle below pi / 2 at frames 1 .. f0
    if spoil == "weightless":
        for x in (k, kc):
            x[..., 2 * pair:2 * pair + 2] = 0
        for first, last in ((1, 2), (sink + 1, sink + 4), (sink + window - 1, sink + window)):
            k[first * P:last * P, :, 2 * pair] = float("-inf")
    cache = B.Cache(1, heads, D, *grid, chunk, sink, window)
    cache.recache_prefill(0, True, f0 - window, window, k, k, v, torch.empty_like(k))
    cache.chunk_append(0, f0, frames, q, kc, vc, torch.empty_like(q))
    keys, values = _cached(cache, P, heads, D)
    q = make(frames) * 0.25                           # as the cache write would leave them: scores in the log2 domain
    if spoil == "far":
        q[5] = 2 * keys[len(keys) // 2]
    else:
        q[..., 2 * pair:2 * pair + 2] = 0.5
    out = torch.empty_like(q)
    cache.sink_window_attn(0, q, out)
    torch.cuda.synchronize()
    cache.close()
    want = torch.empty(out.shape, dtype=torch.float64, device="cuda")
    for h in range(heads):
        scores = q[:, h].double() @ keys[:, h].double().T.contiguous()
        assert not bool(scores.isnan().any())
        want[:, h] = torch.softmax(scores * 0.6931471805599453, 1) @ values[:, h].double()
    assert bool(torch.isfinite(out).all())
    assert _rel(out, want) <= 5e-3


def test_replays_of_a_captured_call():
    heads, D, grid, chunk, sink, window, frames, split = SHAPES[2]
    state = cases.prepare(_case(*SHAPES[2][:-1], form="unrotated"), 9)
    layer, start, q, k, v, _, out = state["passes"][0]
    cases.run(state)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        cases.run(state)
    for seed in range(4):
        fresh = cases.prepare(_case(*SHAPES[2][:-1], form="unrotated"), 20 + seed)
        want = cases.run(fresh)[0]
        for mine, theirs in zip((q, k, v), fresh["passes"][0][2:5]):
            mine.copy_(theirs)
        cache, same = state["cache"], fresh["cache"]
        same.sink_window_attn_unrotated(0, q, want)       # the program's own work between replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        eager = torch.empty_like(out)
        cache.sink_window_attn_unrotated(0, q, eager)
        assert torch.equal(_bits(out), _bits(eager)), seed
        same.close()
    state["cache"].close()


@pytest.mark.parametrize("cache", ["bf16", "fp8_e4m3"])
def test_calls_on_several_streams(cache):
    """Eight streams over one pool, several of them on one layer: each call's output has the bits of the call alone, whatever slots the
    others leave it, and no slot stays taken."""
    case = _case(*(SHAPES[2] if cache == "bf16" else SHAPES8[0])[:-1], cache=cache)
    state = cases.prepare(case, 11)
    want = cases.run(state)[0].clone()
    handle, q = state["cache"], state["passes"][0][5]
    streams = [torch.cuda.Stream() for _ in range(8)]
    outs = [[torch.empty_like(want) for _ in range(10)] for _ in streams]
    torch.cuda.synchronize()
    for i in range(10):
        for s, o in zip(streams, outs):
            with torch.cuda.stream(s):
                handle.sink_window_attn(0, q, o[i])
    torch.cuda.synchronize()
    for o in [x for y in outs for x in y]:
        assert torch.equal(_bits(o), _bits(want))
    assert B.split_slots_taken() == 0
    handle.close()


# the 8-bit cache: heads, head_dim, grid, chunk, sink, window, frames, (groups, splits): 256 / groups rows a tile
SHAPES8 = [(2, 128, (5, 49), 4, 0, 9, 4, (2, 10)), (4, 128, (10, 19), 1, 3, 20, 1, (2, 9)), (3, 64, (20, 26), 3, 1, 9, 3, (2, 12)),
           (2, 128, (30, 52), 3, 3, 9, 3, (1, 6)), (2, 64, (9, 39), 4, 0, 21, 3, (2, 15))]


def _split8(heads, head_dim, grid, chunk, sink, window, frames):
    P = grid[0] * grid[1]
    return B.attn_split(head_dim, heads, frames * P, -(-(sink + window + frames) * P // 64), "fp8_e4m3")


def _two_terms(out, want):
    """Weights rounded once, to 3 mantissa bits, are off by 2.6 % of the 2-norm; the two terms of a split tile's by some 2^-9, beside
    the rounding of the result (2^-9 / sqrt(3) x 2): 6e-3 is what both can add up to where few keys leave nothing to average."""
    return _rel(out, want) <= 6e-3


@pytest.mark.parametrize("shape", SHAPES8)
def test_split_tiles_of_the_8_bit_cache(shape):
    """Against 64 bits with the operands as the cache holds them; again with slots taken; the same video from its first frame."""
    *geo, split = shape
    assert _split8(*geo) == split
    case = _case(*geo, cache="fp8_e4m3")
    want = cases.exact(case, 5)[0]
    state = cases.prepare(case, 5)
    out = cases.run(state)[0]
    layer, _, _, _, _, q_out, _ = state["passes"][0]
    assert _two_terms(out, want)
    again = torch.full_like(out, 7.0)
    state["cache"].sink_window_attn(layer, q_out, again)
    assert torch.equal(_bits(again), _bits(out))
    for first, n in ((0, 512), (0, 2), (1, 511)):
        B.hold_split_slots(first, n, True)
        try:
            again.fill_(7.0)
            state["cache"].sink_window_attn(layer, q_out, again)
        finally:
            B.hold_split_slots(first, n, False)
        assert torch.equal(_bits(again), _bits(out)), (first, n)
    state["cache"].sink_window_attn(layer, q_out, again)
    assert torch.equal(_bits(again), _bits(out))
    state["cache"].close()
    case = _case(*geo[:6], geo[3], cache="fp8_e4m3", video_chunks=1 + -(-(geo[4] + geo[5] + 4) // geo[3]))
    state = cases.prepare(case, 7)
    for i, (a, b) in enumerate(zip(cases.run(state), cases.exact(case, 7))):
        assert _two_terms(a, b), i
    state["cache"].close()


@pytest.mark.parametrize("kv_format, shape", [("bf16", (21, 128, (15, 45), 3, 4, 14, 3)), ("fp8_e4m3", (8, 64, (30, 25), 3, 0, 14, 3))])
def test_more_tiles_without_slots_than_spaces(kv_format, shape):
    """168 and 144 tiles that their merge has to compute, in 128 spaces: the last ones wait for the first."""
    heads, head_dim, grid, chunk, sink, window, frames = shape
    groups, splits = _split(*shape) if kv_format == "bf16" else _split8(*shape)
    rows = 256 // groups
    assert splits > 1 and heads * -(-frames * grid[0] * grid[1] // rows) > 128
    state = cases.prepare(_case(*shape, cache=kv_format), 3)
    out = cases.run(state)[0].clone()
    torch.cuda.synchronize()
    B.hold_split_slots(0, 512, True)
    try:
        again = cases.run(state)[0]
        torch.cuda.synchronize()
    finally:
        B.hold_split_slots(0, 512, False)
    assert torch.equal(_bits(again), _bits(out))
    assert B.split_slots_taken() == 0
    state["cache"].close()


@pytest.mark.parametrize("heads, head_dim, grid, sink, n_win", [(2, 128, (13, 23), 2, 8), (2, 64, (11, 33), 3, 9)])
def test_split_re_prefill_of_the_8_bit_cache(heads, head_dim, grid, sink, n_win):
    """Chunks of unlike key sets in one launch with splits."""
    case = {"kind": "prefill", "cache": "fp8_e4m3", "layers": 1, "heads": heads, "head_dim": head_dim, "grid_h": grid[0],
            "grid_w": grid[1], "chunk": 3, "sink": sink, "window": 7, "win_start": 20, "n_win": n_win, "q_std": 2.0}
    state = cases.prepare(case, 3)
    out = cases.run(state)[0].clone()
    torch.cuda.synchronize()
    want = cases.exact(case, 3)[0]
    assert _two_terms(out, want)
    for first, n in ((0, 512), (1, 300)):
        B.hold_split_slots(first, n, True)
        try:
            again = cases.run(state)[0]
        finally:
            B.hold_split_slots(first, n, False)
        assert torch.equal(_bits(again), _bits(out)), (first, n)
    state["cache"].close()


@pytest.mark.parametrize("head_dim, heads, groups, grid, chunk, sink, window, frames", [
    (128, 16, 2, (15, 26), 3, 2, 8, 3), (128, 24, 4, (10, 10), 3, 2, 20, 3), (128, 1, 4, (8, 9), 4, 0, 18, 3), (64, 6, 4, (9, 15), 2, 2, 6, 2)])
def test_narrow_tiles_of_the_8_bit_cache(head_dim, heads, groups, grid, chunk, sink, window, frames):
    """Tiles of 128 and 64 rows give every row the bits it has in a wider one, which a launch of many heads takes."""
    P, f0 = grid[0] * grid[1], sink + window + 4
    many = -(-240 // -(-frames * P // 256))
    assert _split8(heads, head_dim, grid, chunk, sink, window, frames) == (groups, 1)
    wider = _split8(many, head_dim, grid, chunk, sink, window, frames)
    assert wider[0] < groups and wider[1] == 1
    g = torch.Generator(device="cuda").manual_seed(P)
    make = lambda n: torch.empty((n * P, many, head_dim), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    past, new = [make(sink + window) for _ in range(2)], [make(frames) for _ in range(3)]
    outs = []
    for h in (many, heads):
        k, v = (x[:, :h].contiguous() for x in past)
        q, kc, vc = (x[:, :h].contiguous() for x in new)
        cache = B.Cache(1, h, head_dim, *grid, chunk, sink, window, kv_format="fp8_e4m3")
        cache.recache_prefill(0, True, f0 - window, window, k, k, v, torch.empty_like(k))
        q_out, out = torch.empty(q.shape, dtype=torch.uint8, device="cuda"), torch.full_like(q, 7.0)
        cache.chunk_append(0, f0, frames, q, kc, vc, q_out)
        cache.sink_window_attn(0, q_out, out)
        torch.cuda.synchronize()
        cache.close()
        outs.append(out)
    assert torch.equal(_bits(outs[0][:, :heads].contiguous()), _bits(outs[1]))


@pytest.mark.parametrize("heads, head_dim, grid, chunk, sink, n_win", [(1, 128, (6, 42), 3, 2, 5), (3, 128, (10, 19), 1, 3, 20), (1, 64, (30, 52), 3, 3, 9)])
def test_re_prefill_whose_chunks_all_split(heads, head_dim, grid, chunk, sink, n_win):
    """Groups and splits chosen for the launch (up to 23 chunks); slots taken: the same bits."""
    case = {"kind": "prefill", "cache": "bf16", "layers": 1, "heads": heads, "head_dim": head_dim, "grid_h": grid[0], "grid_w": grid[1],
            "chunk": chunk, "sink": sink, "window": n_win, "win_start": 24, "n_win": n_win, "q_std": 2.0}
    P = grid[0] * grid[1]
    assert B.attn_split(head_dim, heads, chunk * P, -(-(sink + n_win + chunk) * P // 32))[1] > 1
    state = cases.prepare(case, 3)
    out = cases.run(state)[0].clone()
    torch.cuda.synchronize()
    want = cases.exact(case, 3)[0]
    assert _rel(out, want) <= 1e-2                   # logits of standard deviation 2: twice 5e-3
    for first, n in ((0, 512), (1, 300)):
        B.hold_split_slots(first, n, True)
        try:
            again = cases.run(state)[0].clone()
            torch.cuda.synchronize()
        finally:
            B.hold_split_slots(first, n, False)
        assert torch.equal(_bits(again), _bits(out)), (first, n)
    state["cache"].close()


@pytest.mark.parametrize("kv_format, heads, head_dim, grid, chunk, sink, window, n_win", [
    ("bf16", 4, 128, (10, 19), 1, 3, 20, 12), ("bf16", 3, 64, (16, 45), 1, 3, 16, 6), ("fp8_e4m3", 2, 128, (13, 23), 3, 2, 7, 8)])
def test_re_prefill_beside_streaming_of_chunks_that_split(kv_format, heads, head_dim, grid, chunk, sink, window, n_win):
    """Where a streamed chunk's tiles split, the re-prefill's rows have other roundings, and no more than that."""
    P, nf = grid[0] * grid[1], sink + n_win
    assert B.attn_split(head_dim, heads, chunk * P, -(-(sink + window + chunk) * P // (32 if kv_format == "bf16" else 64)), kv_format)[1] > 1
    g = torch.Generator(device="cuda").manual_seed(P)
    q, k, v = (torch.empty((nf * P, heads, head_dim), dtype=torch.bfloat16, device="cuda").normal_(generator=g) for _ in range(3))
    streamed, rebuilt = (B.Cache(1, heads, head_dim, *grid, chunk, sink, window, kv_format=kv_format) for _ in range(2))
    want, got = torch.empty_like(q), torch.empty_like(q)
    starts = [*range(0, sink, chunk), *range(sink, nf, chunk)]
    for f0, end in zip(starts, starts[1:] + [nf]):
        rows = slice(f0 * P, end * P)
        q_out = torch.empty(q[rows].shape, dtype=torch.bfloat16 if kv_format == "bf16" else torch.uint8, device="cuda")
        streamed.chunk_append(0, f0, end - f0, q[rows], k[rows], v[rows], q_out)
        streamed.sink_window_attn(0, q_out, want[rows])
    rebuilt.recache_prefill(0, True, sink, n_win, q, k, v, got)
    torch.cuda.synchronize()
    streamed.close()
    rebuilt.close()
    # twice a path's 5e-3 (bf16), or one path's weights of 3 mantissa bits, 2.6 % of the 2-norm each, and the other's
    assert _rel(got, want.double()) <= (1e-2 if kv_format == "bf16" else 3e-2)


@pytest.mark.parametrize("heads, head_dim, grid, chunk, clip_frames, tail", [
    (8, 128, (15, 26), 3, 21, (3, 10)),       # 280 tiles: three of the five of every head's first chunk
    (15, 128, (10, 20), 1, 20, (3, 5)),       # 300 tiles, one a chunk: the first three chunks
    (5, 128, (15, 26), 2, 28, (5, 8)),        # 280 tiles, four a chunk: the first chunk and a tile of the next
    (9, 128, (15, 26), 2, 15, (0, 1)),        # 270 tiles, but the last chunk is a frame shorter: one launch
    (15, 64, (15, 26), 3, 21, (1, 11))])      # 525 tiles, one a head
def test_clip_whose_last_round_is_split(heads, head_dim, grid, chunk, clip_frames, tail):
    """The tiles of a clip's forward pass that do not fill a round of workgroups have their keys dealt to several: output and, by
    way of the row sums, gradients against 64 bits (test_gpu_clip.py: 5e-3 each); with slots taken the same bits."""
    case = {"kind": "clip", "heads": heads, "head_dim": head_dim, "grid_h": grid[0], "grid_w": grid[1], "chunk": chunk, "sink": 3,
            "window": 9, "ctx_start": 40, "n_ctx": 9, "clip_frames": clip_frames, "q_std": 1.0}
    rows, n_chunks = grid[0] * grid[1], -(-clip_frames // chunk)
    index = B.Clip(heads, head_dim, *grid, chunk, 3, 9, clip_frames, device=None)
    index.forward(40, 9, clip_frames)
    kblocks = [sum(-(-end // 32) - begin // 32 for begin, end in index.chunk_key_ranges(c)) for c in range(n_chunks)]
    assert n_chunks <= 24 and B.attn_clip_tail(head_dim, heads, [(min(chunk, clip_frames - c * chunk) * rows, kblocks[c])
                                                                 for c in reversed(range(n_chunks))]) == tail
    state = cases.prepare(case, 3)
    got = [x.clone() for x in cases.run(state)]
    torch.cuda.synchronize()
    for a, b in zip(got, cases.exact(case, 3)):
        assert _rel(a, b) <= 5e-3
    for first, n in ((0, 512), (1, 300)):
        B.hold_split_slots(first, n, True)
        try:
            again = [x.clone() for x in cases.run(state)]
            torch.cuda.synchronize()
        finally:
            B.hold_split_slots(first, n, False)
        for a, b in zip(again, got):
            assert torch.equal(_bits(a), _bits(b)), (first, n)
    assert B.split_slots_taken() == 0
    state["clip"].close()
