"""The operands of a training step laid out in one launch, and its gradients in one launch (clip_layout.hip, attn_bwd.hip).

Where the layout can go wrong: kblocks of many frames (fewer than 32 tokens a frame), grid rows that wrap once or often inside a
kblock, a last kblock of few rows, queries that begin inside a kblock, a clip that contains the sink.  Where the launch of both
gradients can: tiles of both kinds on the chip at once, dealt out evenly or placed by work, and clips of more groups of columns
than one launch holds.  Output and gradients against 64 bits, to the five bf16 roundings on a gradient's way (5.0e-3, twice that
where a few keys leave nothing to average)."""
import pytest
import torch

from paper_2509_22622_amd import binding as B
from perf import cases

pytestmark = pytest.mark.gpu


def _check(tol, heads, head_dim, grid, chunk, sink, window, n_ctx, clip_frames, ctx_start=9):
    case = {"kind": "clip", "heads": heads, "head_dim": head_dim, "grid_h": grid[0], "grid_w": grid[1], "chunk": chunk, "sink": sink,
            "window": window, "ctx_start": ctx_start, "n_ctx": n_ctx, "clip_frames": clip_frames, "q_std": 1.0}
    state = cases.prepare(case, 4)
    got = [x.clone() for x in cases.run(state)]
    again = cases.run(state)                         # a used handle
    torch.cuda.synchronize()
    for name, a, b, c in zip(("out", "dq", "dk", "dv"), got, cases.exact(case, 4), again):
        assert float((a.double() - b).norm() / b.norm()) <= tol, name
        assert torch.equal(a.view(torch.int16), c.view(torch.int16)), name
    state["clip"].close()


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("grid", [(1, 1), (1, 3), (2, 5), (1, 31), (1, 33), (3, 40), (11, 3), (4, 32)])
def test_frames_and_grid_rows_inside_a_kblock(head_dim, grid):
    _check(1e-2, 2, head_dim, grid, 2, 3, 4, 3, 5)


@pytest.mark.parametrize("head_dim", [64, 128])
def test_no_sink_no_context(head_dim):
    _check(1e-2, 1, head_dim, (3, 7), 3, 0, 2, 0, 7)


@pytest.mark.parametrize("heads, head_dim, grid, chunk, clip_frames", [
    (3, 128, (3, 5), 1, 40), (2, 64, (2, 9), 1, 33),             # more groups than one launch takes
    (16, 128, (13, 20), 1, 9), (24, 64, (13, 20), 1, 9),         # several rounds: placed by work
    (5, 128, (13, 20), 3, 9), (1, 128, (5, 13), 3, 5), (9, 64, (9, 13), 2, 6)])
def test_both_gradients_in_one_launch(heads, head_dim, grid, chunk, clip_frames):
    _check(5.0e-3, heads, head_dim, grid, chunk, 2, 4, 4, clip_frames)


@pytest.mark.parametrize("heads, head_dim, grid, chunk, clip_frames", [
    (1, 128, (18, 10), 3, 8), (2, 128, (5, 13), 1, 20), (1, 64, (11, 30), 2, 5), (1, 128, (13, 20), 1, 24)])
def test_a_small_clip_whose_chunks_split(heads, head_dim, grid, chunk, clip_frames):
    _check(5.0e-3, heads, head_dim, grid, chunk, 3, 5, 5, clip_frames)


@pytest.mark.parametrize("heads, head_dim, grid, chunk, clip_frames", [
    (16, 128, (13, 20), 1, 9), (2, 128, (5, 13), 3, 5), (12, 64, (13, 20), 2, 8), (2, 64, (2, 9), 1, 33)])
def test_gradients_written_over_dout(heads, head_dim, grid, chunk, clip_frames):
    """Each gradient in place of dout: the bits of tensors apart.  (Both kinds of tiles run in one launch, or, past 32 chunks, in
    several: none may read dout, which dV is written over.)"""
    case = {"kind": "clip", "heads": heads, "head_dim": head_dim, "grid_h": grid[0], "grid_w": grid[1], "chunk": chunk, "sink": 2,
            "window": 4, "ctx_start": 9, "n_ctx": 4, "clip_frames": clip_frames, "q_std": 1.0}
    state = cases.prepare(case, 6)
    want = [x.clone() for x in cases.run(state)[1:]]
    dout = state["in"][3]
    for i in range(3):
        got = [torch.full_like(dout, 7.0) for _ in range(3)]
        got[i] = dout.clone()
        state["clip"].backward(got[i], *got)
        torch.cuda.synchronize()
        for name, a, b in zip(("dq", "dk", "dv"), got, want):
            assert torch.equal(a.view(torch.int16), b.view(torch.int16)), (name, i)
    state["clip"].close()
